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
