"""Turn ops (angles other than eighths) of fused runs: the register-plane pass
against the LDS-plane pass, bitwise, and against the phase formed on the host,
at the entry counts and op counts where the tables' loops and the capture
planes end."""
import numpy as np
import pytest

from paper_2105_01533_amd import workloads as W

pytestmark = pytest.mark.gpu

COUNTS = [1, 64, 65, 256, 257, 320, 321, 1024, 1025, 1280, 1281, 2047, 2048, 2049, 2304, 6000]


@pytest.fixture(scope="module")
def sim():
    from paper_2105_01533_amd import sim as S
    return S


def _run(sim, n, state, ops, flags):
    s = sim.Simulator(n, 8192, 1e-15, flags=flags, tuned=False)
    try:
        s.import_state(*state)
        s.apply_ops(ops)
        return s.export(sort=False)
    finally:
        s.close()


# Planes left for captured conditions: 64, 64, 24, 8 and none.
@pytest.mark.parametrize("n", [14, 60, 100, 115, 125])
@pytest.mark.parametrize("turns", [1, 8, 9, 24, 25, 64, 65, 130])
def test_turns_match_lds_planes(sim, n, turns):
    rng = W.SplitMix64(100 * n + turns)
    c, bare = W.Circuit(), W.Circuit()
    for _ in range(16):
        c.x(rng.randint(n))
    angle = np.zeros(n)
    for k in range(turns):
        q, t = rng.randint(n), rng.uniform() * 6.0
        ctrl = rng.distinct(n, 1 + rng.randint(3))
        ctrl = tuple(x for x in ctrl if x != q) if k % 3 == 1 else ()
        c.gate(W.K_RZ, q, ctrl, param=t)
        bare.gate(W.K_RZ, q, (), param=t)
        angle[q] += t
        if k % 4 == 2:
            a, b = rng.distinct(n, 2)
            c.x(a, (b,))
    for _ in range(16):
        bare.gate(W.K_S, 0)                      # (16 gates: no phase; the run takes the bit planes)
    for m in COUNTS:
        state = W.random_state(m + n, m, n)
        got = _run(sim, n, state, c.array(), 0)
        want = _run(sim, n, state, c.array(), sim.SIM_FLAG_BS_LDS)
        assert all(x.tobytes() == y.tobytes() for x, y in zip(got, want)), (m, "LDS planes")
        lo, hi, amp = _run(sim, n, state, bare.array(), 0)
        bits = [((lo if q < 64 else hi) >> np.uint64(q & 63)) & np.uint64(1) for q in range(n)]
        phase = sum(0.5 * angle[q] * (2.0 * bits[q] - 1.0) for q in range(n))
        ref = state[2] * np.exp(1j * phase)
        # An angle of up to 130 x 3 turns on the host: rounding of its sum, 4e2 eps.
        assert np.abs(amp - ref).max() < 1e-12, m
