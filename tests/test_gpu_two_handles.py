"""Branching gates of several handles at once: their kernels wait, tile on tile,
for the outputs of the tiles before them, and must come to an end whatever
shares the device with them."""
import threading

import pytest

from paper_2105_01533_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    from paper_2105_01533_amd import sim as S
    return S


def _pairs(n, seed, count):
    """Branching gates that widen the state, each followed by its inverse,
    which brings it back (the other outputs are below eps)."""
    rng = W.SplitMix64(seed)
    c = W.Circuit()
    for g in range(count):
        q = rng.randint(n)
        ctrl = ((q + 3) % n,) if g % 2 else ()
        c.gate(W.K_RY, q, controls=ctrl, param=0.4 + 0.05 * g)
        c.gate(W.K_RY, q, controls=ctrl, param=-0.4 - 0.05 * g)
    return c.array()


@pytest.mark.parametrize("sizes", [
    (2100, 4096, 3000),             # the LDS index over several blocks
    (9000, 1 << 15, 20_000),        # the single pass: tiles of 256 entries
    (40_000, 1 << 16, 1 << 17),     # 256, 512 and 1024
    (3000, 60_000, 150_000),        # all of them
])
@pytest.mark.parametrize("n", [40, 90])
def test_branching_on_three_streams(sim, n, sizes):
    import torch
    ops = [_pairs(n, 17 + k, 20) for k in range(len(sizes))]
    states = [W.random_state(500 + k + e, e, n) for k, e in enumerate(sizes)]

    def run(k, stream):
        with torch.cuda.stream(stream):
            s = sim.Simulator(n, 4 * sizes[k], 1e-20, tuned=False)
            try:
                s.import_state(*states[k])
                _, _, st = s.apply_ops(ops[k])
                return st, s.export(sort=False)
            finally:
                s.close()

    streams = [torch.cuda.Stream() for _ in sizes]
    alone = [run(k, streams[k]) for k in range(len(sizes))]
    for k, e in enumerate(sizes):
        assert alone[k][0]["u2_applied"] == len(ops[k]) and len(alone[k][1][0]) == e
    for rep in range(3):
        got, errors = [None] * len(sizes), []

        def work(k):
            try:
                got[k] = run(k, streams[k])
            except Exception as e:   # (shown below)
                errors.append((k, e))

        threads = [threading.Thread(target=work, args=(k,)) for k in range(len(sizes))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not errors, errors
        for k in range(len(sizes)):
            for x, y in zip(got[k][1], alone[k][1]):
                assert x.tobytes() == y.tobytes(), (rep, k)
