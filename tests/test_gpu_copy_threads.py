"""Imports and exports from many short-lived host threads: the pinned staging
memory they go through is shared and bounded, and several at once do not
disturb each other."""
import threading

import numpy as np
import pytest

from paper_2105_01533_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    from paper_2105_01533_amd import sim as S
    return S


def _mapped_mib():
    with open("/proc/self/statm") as f:
        return int(f.read().split()[0]) * 4096 / 2**20


def _in_thread(fn):
    err = []

    def run():
        try:
            fn()
        except Exception as e:
            err.append(e)

    t = threading.Thread(target=run)
    t.start()
    return t, err


def test_threads_share_the_staging_memory(sim):
    state = W.random_state(5, 1000, 90)
    s = sim.Simulator(90, 4096, 0.0, tuned=False)

    def round_trip():
        s.import_state(*state)
        for x, y in zip(s.export(sort=False), state):
            assert x.tobytes() == np.ascontiguousarray(y, x.dtype).tobytes()

    def threads(count):
        for _ in range(count):
            t, err = _in_thread(round_trip)
            t.join()
            assert not err, err

    try:
        threads(6)
        before = _mapped_mib()
        threads(24)
        assert _mapped_mib() - before < 64     # (24 buffers of 16 MiB would be 384)
    finally:
        s.close()


@pytest.mark.parametrize("entries", [1, 100_003, 1_200_000])
def test_concurrent_copies(sim, entries):
    """More copies at once than stages are kept; the largest takes several
    chunks of a stage."""
    import torch
    count = 20
    sims = []
    try:
        for k in range(count):
            with torch.cuda.stream(torch.cuda.Stream()):
                sims.append(sim.Simulator(90, entries, 0.0, tuned=False))
        lo, hi, amp = W.random_state(6, entries, 90)

        def work(k):
            a = amp * (k + 1)
            for _ in range(3):
                sims[k].import_state(lo, hi, a)
                got = sims[k].export(sort=False)
                assert got[0].tobytes() == lo.tobytes() and got[1].tobytes() == hi.tobytes()
                assert got[2].tobytes() == a.tobytes()

        ts = [_in_thread(lambda k=k: work(k)) for k in range(count)]
        for t, _ in ts:
            t.join()
        assert not [e for _, err in ts for e in err]
    finally:
        for s in sims:
            s.close()
