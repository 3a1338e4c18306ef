"""A call whose branching gate turns out not to fit after later ops have been
launched: what the caller sees of those."""
import ctypes

import numpy as np
import pytest

from paper_2105_01533_amd import workloads as W

pytestmark = pytest.mark.gpu
ENTRIES, CAP = 9000, 12_000


@pytest.fixture(scope="module")
def sim():
    from paper_2105_01533_amd import sim as S
    return S


def _state(n):
    """The qubits of random labels below 2^(n - 2): two are 0 everywhere."""
    return W.random_state(61, ENTRIES, n - 2)


@pytest.mark.parametrize("n", [30, 90])
@pytest.mark.parametrize("before, after", [(0, 1), (2, 3), (1, 9)])
@pytest.mark.parametrize("static", [False, True])
def test_outcomes_end_at_the_gate(sim, n, before, after, static):
    """One outcome per measurement before the gate; the caller's array is left
    as it was past them."""
    c = W.Circuit()
    for k in range(before):
        c.measure(n - 2 + k % 2, 0.5)              # 0 everywhere: takes nothing away
    c.h(n - 1)                                     # 18,000 entries: do not fit
    for k in range(after):
        c.measure(k % 5, 0.5)
    gates = sim.sim_gates_from_ops(c.array())
    outs = np.full(before + after, 7, np.int32)
    call = sim._lib.sim_apply_gates_static if static else sim._lib.sim_apply_gates
    s = sim.Simulator(n, CAP, 0.0, tuned=False)
    try:
        s.import_state(*_state(n))
        st = sim.sim_stats()
        rc = call(s.h, sim._ptr(gates), len(gates), sim._ptr(outs), ctypes.byref(st))
        assert rc == sim.SIM_E_CAPACITY and st.gates_applied == before and st.measures == before
        assert list(outs) == [0] * before + [7] * after
        lo, hi, amp = s.export()
        assert len(lo) == ENTRIES
    finally:
        s.close()
