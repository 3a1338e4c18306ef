"""Fused runs of the server's ticks on register planes, one launch a tick
(kb_mono_rp), at the ends of their range, against the LDS-plane tile
(SRV_FLAG_NO_RP): bit for bit the same."""
import pytest

from helpers import assert_same_state
from oracle import run_workload as oracle_run
from paper_2105_01533_amd import workloads as W
from test_gpu_serving import run_server

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2105_01533_amd import sim
    import torch
    assert torch.cuda.is_available()
    return sim


def _pruned_to_nothing(n, gates, seed):
    """A branching gate with both outputs below eps, then `gates`
    phase/permutation gates and another branching gate on no entries."""
    rng = W.SplitMix64(seed)
    c = W.Circuit()
    c.h(0)                                       # |a|^2 = 0.5 each: dropped
    for _ in range(gates):
        W._random_mono(rng, c, n, 0.7, 0.3, 0)
    c.h(1)
    return W.Workload(f"empty_{gates}", n, 0.6, c.array(), capacity=64)


@pytest.mark.parametrize("gates", [3, 16, 400])
@pytest.mark.parametrize("beside", [0, 2])
def test_runs_on_an_empty_state(S, gates, beside):
    """A request whose state has been pruned to nothing takes its runs as any
    other, alone in a tick and beside requests with entries."""
    ws = [_pruned_to_nothing(20, gates, 5), _pruned_to_nothing(70, gates, 6)]
    ws += [W.config0(71 + k, n=20, h_qubits=6, gates=600, cap=1 << 9) for k in range(beside)]
    a, sa = run_server(S, ws)
    b, _ = run_server(S, ws, flags=S.SRV_FLAG_NO_RP)
    assert sa["completed"] == len(ws) and sa["failed"] == 0
    for w, x, y in zip(ws, a, b):
        for p, q in zip(x[:4], y[:4]):
            assert p.tobytes() == q.tobytes(), w.name
        o, oout, _ = oracle_run(w)
        assert list(x[3]) == list(oout), w.name
        assert_same_state(x[:3], o.export(), what=w.name)
    assert len(a[0][0]) == 0 and len(a[1][0]) == 0


def _segments(k, n, w, count):
    """2^w entries; `count` runs of adders, controlled-phase ladders and random
    mixes in an order of request k's own, a branching gate and a measurement
    after each."""
    rng = W.SplitMix64(700 + k)
    c = W.Circuit()
    for q in range(w):
        c.h(q)
    a, b = list(range(5)), list(range(5, 10))
    for s in range(count):
        kind = (s + k) % 3
        if kind == 0:
            for _ in range(1 + k % 3):
                W.cdkm_add(c, a, b, 10, n - 2)
        elif kind == 1:
            for q in range(w):
                for j in range(1, 4 + k % 3):
                    c.gate(W.K_RZ, q, ((q + j) % w,), param=3.0 / (j + k))
        else:
            for _ in range(40 + k):
                W._random_mono(rng, c, n - 1, 0.6, 0.4, 0)
        c.h(n - 1)
        c.measure(n - 1, rng.uniform())
    return W.Workload(f"segments_{k}_{n}q", n, 1e-20, c.array(), capacity=2 << w)


def test_many_programs_side_by_side(S):
    """Ticks of more register-plane tiles (80 requests of 2^15 entries: 1,280)
    than the device has SIMDs (1,024), every request with programs of its own,
    labels of both widths."""
    ws = [_segments(k, (24, 40, 70, 100, 128)[k % 5], 15, 12) for k in range(80)]
    a, sa = run_server(S, ws, budget=2 << 30, slots=len(ws))
    b, sb = run_server(S, ws, budget=2 << 30, slots=len(ws), flags=S.SRV_FLAG_NO_RP)
    assert sa["rp_runs"] >= 12 * len(ws) and sb["rp_runs"] == 0
    # (the 12 runs of nearly all requests share their ticks)
    assert sa["ticks"] < 15 + 3 * 12 + 20
    for w, x, y in zip(ws, a, b):
        assert len(x[0]) > 1 << 13
        for p, q in zip(x[:4], y[:4]):
            assert p.tobytes() == q.tobytes(), w.name
