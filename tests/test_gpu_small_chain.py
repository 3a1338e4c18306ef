"""Chains of branching gates on small states in one launch (the LDS index),
against the global index gate by gate: bitwise the same state, outcomes and
counters, at the counts where the chain's paths and its end change."""
import numpy as np
import pytest

from paper_2105_01533_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    from paper_2105_01533_amd import sim as S
    return S


@pytest.mark.parametrize("n", [24, 70, 128])
@pytest.mark.parametrize("entries", [1, 2, 511, 512, 513, 1025, 4096, 8191])
def test_chain_matches_global_index(sim, n, entries):
    """Gates with runs of 0, 1, 15 and 16 ops between them (16 are a pass of
    their own), folding gates, a capped gate, a trailing run, more gates than a
    launch takes, and a measurement between chains."""
    rng = W.SplitMix64(9 * entries + n)
    c = W.Circuit()
    for g in range(20):
        q = rng.randint(n)
        for _ in range((0, 1, 15, 16)[g % 4]):
            W._random_mono(rng, c, n, 0.6, 0.4, 0)
        if g % 5 == 4:
            c.h(q, cap=3000 if g % 2 else 20)
        elif g % 5 == 3:
            c.gate(W.K_RY, q, controls=((q + 1) % n,), param=0.4)
        else:                                    # out and back
            c.gate(W.K_RX, q, param=0.3)
            c.gate(W.K_T, (q + 2) % n)
            c.gate(W.K_RX, q, param=-0.3)
        if g == 9:
            c.measure(rng.randint(n), rng.uniform())
    c.gate(W.K_S, 1)
    state = W.random_state(55 + entries, entries, n)
    out = []
    for flags in (0, sim.SIM_FLAG_U2_GLOBAL_INDEX, sim.SIM_FLAG_U2_GLOBAL_INDEX | sim.SIM_FLAG_U2_TWO_PASS):
        s = sim.Simulator(n, 1 << 17, 1e-12, flags=flags, tuned=False)
        try:
            s.import_state(*state)
            rc, outs, st = s.apply_ops(c.array(), raise_on_error=False)
            out.append((rc, list(outs), st, s.export(sort=False)))
        finally:
            s.close()
    for o in out[1:]:
        assert o[0] == out[0][0] and o[1] == out[0][1]
        for k in ("gates_applied", "updates", "u2_applied", "u2_skipped", "u2_split", "pruned", "peak_nnz", "mono_passes"):
            assert o[2][k] == out[0][2][k], k
        for x, y in zip(o[3], out[0][3]):
            assert x.tobytes() == y.tobytes()


@pytest.mark.parametrize("n", [24, 64, 65, 128])
@pytest.mark.parametrize("entries", [1024, 1026, 2047, 2048, 2049, 3072, 4095, 4096, 4097, 8192])
def test_gates_over_several_blocks_match_global_index(sim, n, entries):
    """One gate at each bound on the count: runs of 0, 7, 8, 9 and 15 ops
    before it, half the partners present, controls, and a folding gate."""
    for g, ops in enumerate((0, 7, 8, 9, 15)):
        rng = W.SplitMix64(entries + 100 * n + g)
        lo, hi, amp = W.random_state(entries + g, entries, n)
        q = rng.randint(n)
        half = entries // 2
        for x, w in ((lo, q < 64), (hi, q >= 64)):   # the second half: partners of every other entry
            flip = (np.uint64(1) << np.uint64(q & 63)) if w else np.uint64(0)
            x[half:half + half // 2] = x[:half:2][:half // 2] ^ flip
        keep = np.unique(np.stack([hi, lo]), axis=1, return_index=True)[1]
        keep = keep[np.argsort(W.splitmix64_array(g, 0, len(keep)))]
        state = lo[keep], hi[keep], amp[keep]
        c = W.Circuit()
        for _ in range(ops):
            W._random_mono(rng, c, n, 0.6, 0.4, 0)
        c.gate(W.K_RX, q, controls=((q + 3) % n,) if g % 2 else (), param=0.7)
        c.h(q)
        out = []
        for flags in (0, sim.SIM_FLAG_U2_GLOBAL_INDEX):
            s = sim.Simulator(n, 1 << 16, 1e-12, flags=flags, tuned=False)
            try:
                s.import_state(*state)
                _, _, st = s.apply_ops(c.array())
                out.append((st, s.export(sort=False)))
            finally:
                s.close()
        for k in ("gates_applied", "updates", "u2_applied", "pruned", "peak_nnz", "mono_passes"):
            assert out[0][0][k] == out[1][0][k], (ops, k)
        for x, y in zip(out[0][1], out[1][1]):
            assert x.tobytes() == y.tobytes(), ops
