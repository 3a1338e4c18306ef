"""State import's duplicate check and sorted export, against numpy, at the
counts where the tiles of the sort and its merge passes change."""
import numpy as np
import pytest

from paper_2105_01533_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    from paper_2105_01533_amd import sim as S
    return S


def _labels(kind, m, n):
    """Distinct labels below 2^n in no order."""
    lo, hi, amp = W.random_state(7 * m + n, m, n)
    top = (1 << n) - 1
    if kind == "dense" and m <= top:          # 0 .. m - 1, or down from the largest label
        v = [top - i if n > 64 and i & 1 else i for i in range(m)]
        p = np.argsort(W.splitmix64_array(3, 0, m))
        lo = np.array([x & (2**64 - 1) for x in v], np.uint64)[p]
        hi = np.array([x >> 64 for x in v], np.uint64)[p]
    elif kind == "descending":
        o = np.lexsort((lo, hi))[::-1]
        lo, hi = lo[o], hi[o]
    elif kind == "one low word" and n >= 100:   # only the high words differ
        hi = np.argsort(W.splitmix64_array(5, 0, m)).astype(np.uint64)
        lo = np.full(m, (1 << 64) - 1, np.uint64)
    return lo, hi, amp


@pytest.mark.parametrize("n", [30, 64, 65, 128])
@pytest.mark.parametrize("m", [0, 1, 2, 3, 63, 1025, 4095, 4096, 4097, 8192, 8193, 12289, 40000, 300001])
def test_sorted_export(sim, n, m):
    for kind in ("random", "dense", "descending", "one low word"):
        lo, hi, amp = _labels(kind, m, n)
        s = sim.Simulator(n, max(m, 1), 1e-12)
        try:
            s.import_state(lo, hi, amp)
            o = np.lexsort((lo, hi))
            for _ in range(2):                 # (the stored order is not touched)
                a = s.export()
                b = s.export(sort=False)
                for x, y, z in zip(a, b, (lo, hi, amp)):
                    assert np.array_equal(x, z[o]), (kind, "sorted")
                    assert np.array_equal(y, z), (kind, "stored")
        finally:
            s.close()


@pytest.mark.parametrize("n", [50, 100])
def test_import_takes_any_label_arrays(sim, n):
    """Contiguous and strided words, Python integers, one value for all."""
    lo, hi, amp = W.random_state(9, 3000, n)
    s = sim.Simulator(n, 3000, 1e-12)
    try:
        for l, h in ((lo, hi), (np.repeat(lo, 2)[::2], np.repeat(hi, 3)[::3]), (lo[::-1][::-1], hi), (lo, hi.tolist())):
            s.import_state(l, h, amp)
            assert all(np.array_equal(x, y) for x, y in zip(s.export(sort=False), (lo, hi, amp)))
        if n <= 64:
            s.import_state(lo.tolist(), 0, amp)
            assert all(np.array_equal(x, y) for x, y in zip(s.export(sort=False), (lo, hi, amp)))
    finally:
        s.close()


@pytest.mark.parametrize("n", [40, 128])
@pytest.mark.parametrize("m", [2, 64, 5000, 100003])
def test_import_refuses_duplicates_and_keeps_the_state(sim, n, m):
    lo, hi, amp = W.random_state(m, m, n)
    s = sim.Simulator(n, m + 3, 1e-12, load_factor=0.9)
    try:
        s.import_state(lo, hi, amp)
        want = s.export()
        for i, j in ((0, m - 1), (m // 2, m // 2 - 1)):
            l2, h2 = lo.copy(), hi.copy()
            l2[i], h2[i] = l2[j], h2[j]
            with pytest.raises(sim.SimError, match="duplicate"):
                s.import_state(l2, h2, amp)
            l2[i] = lo[i]
            if n < 64:
                l2[j] |= np.uint64(1) << np.uint64(n)
                with pytest.raises(sim.SimError, match="above"):
                    s.import_state(l2, hi, amp)
            assert all(np.array_equal(x, y) for x, y in zip(s.export(), want))
        # The index is empty again: a gate finds its partners, and the state imports once more.
        c = W.Circuit()
        c.gate(W.K_RX, 1, param=0.3)
        c.gate(W.K_RX, 1, param=-0.3)
        s.import_state(lo[: m // 2], hi[: m // 2], amp[: m // 2])
        s.apply_ops(c.array())
        s.import_state(lo, hi, amp)
        assert all(np.array_equal(x, y) for x, y in zip(s.export(), want))
    finally:
        s.close()
