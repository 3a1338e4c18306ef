"""Branching gates through the prepared single pass -- the gate's write applies
the short run after it and indexes its outputs for the next gate, partners
next to each other are found without the index, gates known apart build none,
gates that may not fit are found out later -- against the separate count, scan
and write passes, which do none of this: bitwise the same state, in the same
order, with the same counters."""
import numpy as np
import pytest

from helpers import assert_same_state
from oracle import Oracle
from paper_2105_01533_amd import workloads as W

pytestmark = pytest.mark.gpu
COUNTERS = ("gates_applied", "updates", "u2_applied", "u2_skipped", "u2_split", "measures", "pruned", "peak_nnz",
            "mono_passes")


@pytest.fixture(scope="module")
def sim():
    from paper_2105_01533_amd import sim as S
    return S


def _chain(n, seed, gates=24, measure=False):
    """Branching gates with runs of 0..20 gates between them: H pairs on one
    qubit around flips of it (partners next to each other), controlled and
    rotated gates, qubits never touched before (no partners)."""
    rng = W.SplitMix64(seed)
    c = W.Circuit()
    for g in range(gates):
        q = rng.randint(min(n, 16))
        kind = rng.randint(4)
        if kind == 0:
            c.h(q)
            c.x(q, ((q + 1) % n,))
            c.h(q)
        elif kind == 1:
            c.gate(W.K_RY, q, controls=((q + 3) % n,), param=0.3 + 0.1 * g)
        elif kind == 2:
            c.gate(W.K_RX, n - 1 - (g % 3), param=0.2)
            c.gate(W.K_RX, n - 1 - (g % 3), param=-0.2)
        else:
            c.h(q)
        for _ in range(rng.randint(21) if g % 2 else 0):
            W._random_mono(rng, c, n, 0.7, 0.3, 0)
        if measure and g % 6 == 5:
            c.measure(rng.randint(n), rng.uniform())
    return c.array()


def _run(S, n, cap, eps, ops, state, flags, **kw):
    s = S.Simulator(n, cap, eps, flags=flags, tuned=False, **kw)
    try:
        s.import_state(*state)
        rc, outs, st = s.apply_ops(ops, raise_on_error=False)
        return rc, list(outs), st, s.export(sort=False)
    finally:
        s.close()


def _same(a, b):
    assert a[0] == b[0] and a[1] == b[1]
    for k in COUNTERS:
        assert a[2][k] == b[2][k], k
    for x, y in zip(a[3], b[3]):
        assert x.tobytes() == y.tobytes()


@pytest.mark.parametrize("n", [20, 64, 65, 128])
@pytest.mark.parametrize("entries", [1, 63, 1025, 9000])
@pytest.mark.parametrize("mono_mode", [0, 1])
def test_prepared_chain_matches_two_pass(sim, n, entries, mono_mode):
    state = W.random_state(100 + entries + n, entries, n)
    ops = _chain(n, 7 * entries + n, gates=14, measure=True)
    flags = sim.SIM_FLAG_U2_GLOBAL_INDEX
    a = _run(sim, n, 1 << 18, 1e-9, ops, state, flags, mono_mode=mono_mode)
    b = _run(sim, n, 1 << 18, 1e-9, ops, state, flags | sim.SIM_FLAG_U2_TWO_PASS, mono_mode=mono_mode)
    _same(a, b)


@pytest.mark.parametrize("n", [40, 100])
@pytest.mark.parametrize("entries", [(1 << 18) - 1, (1 << 18) + 1, (1 << 19) + 1, (1 << 20) + 4097])
def test_tile_sizes_match_two_pass(sim, n, entries):
    state = W.random_state(entries, entries, n)
    c = W.Circuit()
    c.gate(W.K_RY, 3, controls=(5,), param=0.7)
    c.x(2, (3,))
    c.gate(W.K_RY, 3, controls=(5,), param=-0.4)
    c.h(n - 1)
    out = [_run(sim, n, 1 << 23, 1e-12, c.array(), state, f) for f in (0, sim.SIM_FLAG_U2_TWO_PASS)]
    _same(*out)


@pytest.mark.parametrize("n", [30, 90])
@pytest.mark.parametrize("after", [0, 1, 5])
def test_gate_that_does_not_fit(sim, n, after):
    """The call ends with the state, counters and outcomes of before the gate
    that did not fit, however many ops were launched after it; the handle goes
    on from there."""
    entries = 9000
    lo, hi, amp = W.random_state(31, entries, n)
    c = W.Circuit()
    c.x(1, (2,))
    c.h(3)                                     # 18,000 entries: fits
    c.gate(W.K_T, 3)
    c.h(4)                                     # 36,000: does not
    for k in range(after):
        c.x(6, (4,))
        c.gate(W.K_RX, 5 + k, param=0.3)
        c.measure(2, 0.4)
    out = [_run(sim, n, 30_000, 0.0, c.array(), (lo, hi, amp), f) for f in (0, sim.SIM_FLAG_U2_TWO_PASS)]
    assert out[0][0] == sim.SIM_E_CAPACITY and out[0][2]["gates_applied"] == 3
    for k in COUNTERS:
        assert out[0][2][k] == out[1][2][k], k
    for x, y in zip(out[0][3], out[1][3]):
        assert x.tobytes() == y.tobytes()
    s = sim.Simulator(n, 30_000, 0.0, tuned=False)
    try:
        s.import_state(lo, hi, amp)
        s.apply_ops(c.array(), raise_on_error=False)
        more = W.Circuit()
        more.gate(W.K_H, 3)                    # pairs every entry; the T between keeps both outputs: 18,000 still
        more.x(7, (1,))
        more.h(8)                              # 36,000: does not fit either
        rc, _, st = s.apply_ops(more.array(), raise_on_error=False)
        assert rc == sim.SIM_E_CAPACITY and st["gates_applied"] == 2
        o = Oracle(n, 0.0)
        o.import_state(lo, hi, amp)
        o.run(np.concatenate([c.array()[:3], more.array()[:2]]))
        assert_same_state(s.export(), o.export(), what="after a gate that did not fit")
    finally:
        s.close()


def test_near_capacity_fits(sim):
    """Gates at the capacity whose outputs do fit (H pairs folding back) run on
    without the host reading the count, and match the two-pass form."""
    n, entries = 50, 20_000
    state = W.random_state(77, entries, n)
    c = W.Circuit()
    for q in (3, 9, 30):
        c.h(q)
        c.gate(W.K_S, q)
        c.gate(W.K_SDG, q)
        c.h(q)
    out = [_run(sim, n, 2 * entries, 1e-20, c.array(), state, f) for f in (0, sim.SIM_FLAG_U2_TWO_PASS)]
    _same(*out)
    assert out[0][2]["u2_applied"] == 6 and len(out[0][3][0]) == entries
