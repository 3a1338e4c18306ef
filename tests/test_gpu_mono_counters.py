"""The mono_pass class counts its own launches' work: a short run that a
branching gate's kernels apply on their way moves no bytes of its own."""
import itertools

import pytest

from paper_2105_01533_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [40, 90])
@pytest.mark.parametrize("entries, launches", [
    (500, 0),        # one chain
    (2000, 1),       # a chain, then the LDS index over several blocks
    (4000, 1),       # the latter twice
    (20_000, 1),     # the global index
])
def test_mono_pass_counts_its_own_launches(entries, launches, n):
    from paper_2105_01533_amd import sim
    c = W.Circuit()
    c.x(1, (2,))
    c.gate(W.K_T, 3)
    for q in (5, 7):               # (no entry has its partner: each doubles the entries)
        c.h(q)
        c.x(2, (1,))
        c.gate(W.K_S, 4)
        c.gate(W.K_RZ, 8, param=0.3)
    runs = [(2, entries), (3, 2 * entries), (3, 4 * entries)]     # gates, entries
    s = sim.Simulator(n, 8 * entries, 0.0, tuned=False, mono_mode=sim.SIM_MONO_DIRECT)
    try:
        s.import_state(*W.random_state(64, entries, n))
        sim.sim_kernel_stats_reset(s.h)
        _, _, st = s.apply_ops(c.array())
        ks = sim.sim_kernel_stats(s.h)["mono_pass"]
        assert st["updates"] == sum(g * e for g, e in runs) + 3 * entries and st["mono_passes"] == 3
        assert ks["launches"] == launches
        per = 2 * (16 if n > 64 else 8) + 32
        own = [(sum(g * e for g, e in some), per * sum(e for _, e in some))
               for some in itertools.combinations(runs, launches)]
        assert (ks["updates"], ks["alg_bytes"]) in own
    finally:
        s.close()
