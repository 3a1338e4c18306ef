"""Measurements at the entry counts where the blocks' ranges change (256
entries a block, then 512 blocks, then longer ranges): single and in chains,
against numpy."""
import numpy as np
import pytest

from paper_2105_01533_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    from paper_2105_01533_amd import sim as S
    return S


@pytest.mark.parametrize("n", [50, 100])
@pytest.mark.parametrize("entries", [1, 2, 255, 256, 257, 513, 4096, 131071, 131072, 131073, 262145, 300001])
def test_measure_chain(sim, n, entries):
    lo, hi, amp = W.random_state(31 + entries, entries, n)
    rng = W.SplitMix64(entries + n)
    qubits = [rng.randint(n) for _ in range(3)]
    us = [rng.uniform() for _ in range(3)]
    c = W.Circuit()
    for q, u in zip(qubits, us):
        c.measure(q, u)
    for capacity in (entries, 1 << 20):          # the grid follows the bound, the ranges the count
        s = sim.Simulator(n, capacity, 1e-30)
        try:
            s.import_state(lo, hi, amp)
            _, outs, _ = s.apply_ops(c.array())
            got = s.export(sort=False)
        finally:
            s.close()
        l, h, a, want = lo, hi, amp, []
        for q, u in zip(qubits, us):
            bit = (((l if q < 64 else h) >> np.uint64(q & 63)) & np.uint64(1)).astype(bool)
            w = np.abs(a) ** 2
            p0, p1 = w[~bit].sum(), w[bit].sum()
            assert abs(u - p0 / (p0 + p1)) > 1e-9    # (no draw is decided by rounding)
            o = int(not u < p0 / (p0 + p1))
            want.append(o)
            keep = bit == bool(o)
            l, h, a = l[keep], h[keep], a[keep] / np.sqrt(p1 if o else p0)
        assert list(outs) == want
        assert np.array_equal(got[0], l) and np.array_equal(got[1], h)
        # Sums of up to 3e5 terms in some order, a square root and a product, three times.
        assert np.abs(got[2] - a).max() < 1e-12
