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


@pytest.mark.parametrize("n", [30, 90])
@pytest.mark.parametrize("after", [254, 255, 256, 3000])
def test_launches_end_soon_after_the_gate(sim, n, after):
    """At most 256 branching gates are launched whose fit is not known."""
    c = W.Circuit()
    c.h(n - 1)                                     # does not fit
    for k in range(after):
        c.gate(W.K_RX, k % (n - 2), param=0.3)
        if k % 50 == 49:
            c.x(1, (2,))
    s = sim.Simulator(n, CAP, 0.0, tuned=False)
    try:
        s.import_state(*_state(n))
        rc, _, st = s.apply_ops(c.array(), raise_on_error=False)
        assert rc == sim.SIM_E_CAPACITY and st["gates_applied"] == 0
        assert sim.sim_kernel_stats(s.h)["u2_write"]["launches"] <= 256
        lo, hi, amp = s.export(sort=False)
        for x, y in zip((lo, hi, amp), _state(n)):
            assert x.tobytes() == np.ascontiguousarray(y, x.dtype).tobytes()
    finally:
        s.close()


@pytest.mark.parametrize("n", [40, 90])
@pytest.mark.parametrize("pairs", [127, 128, 300])
def test_reads_between_gates_that_fit(sim, n, pairs):
    """Gates at the capacity that do fit run on over the reads of the count
    between them, as the two-pass form, which reads it at each."""
    state = W.random_state(62, ENTRIES, n - 2)
    c = W.Circuit()
    for k in range(pairs):
        c.h(k % 11)
        if k % 7 == 3:
            c.x(3, (5,))
            c.x(3, (5,))
        c.h(k % 11)
        if k % 16 == 15:
            c.measure(n - 1, 0.5)                  # 0 everywhere
    out = []
    for f in (0, sim.SIM_FLAG_U2_TWO_PASS):
        s = sim.Simulator(n, 2 * ENTRIES + 100, 1e-20, flags=f, tuned=False)
        try:
            s.import_state(*state)
            rc, outs, st = s.apply_ops(c.array(), raise_on_error=False)
            out.append((rc, list(outs), [st[k] for k in ("gates_applied", "updates", "u2_applied", "pruned", "peak_nnz")],
                        [x.tobytes() for x in s.export(sort=False)]))
        finally:
            s.close()
    assert out[0][0] == 0 and out[0][2][2] == 2 * pairs
    assert out[0] == out[1]


@pytest.mark.parametrize("n", [30, 90])
@pytest.mark.parametrize("flags", ["", "SIM_FLAG_U2_GLOBAL_INDEX", "SIM_FLAG_U2_TWO_PASS"])
def test_measurement_of_an_emptied_state_ends_the_call(sim, n, flags):
    """Gates that may not fit but drop everything: the measurement after them
    ends the call at its place, as in the two-pass form, which reads the count
    at each of them."""
    c = W.Circuit()
    c.h(3)                                         # every |a|^2 is below eps
    c.x(1, (2,))
    c.h(4)
    c.measure(5, 0.5)
    for k in range(3):
        c.h(6 + k)
        c.measure(k, 0.5)
    gates = sim.sim_gates_from_ops(c.array())
    outs = np.full(4, 7, np.int32)
    s = sim.Simulator(n, CAP, 1e-2, tuned=False, flags=getattr(sim, flags) if flags else 0)
    try:
        s.import_state(*_state(n))
        st = sim.sim_stats()
        rc = sim._lib.sim_apply_gates(s.h, sim._ptr(gates), len(gates), sim._ptr(outs), ctypes.byref(st))
        assert rc == sim.SIM_E_STATE
        assert (st.gates_applied, st.u2_applied, st.measures) == (3, 2, 0)
        assert list(outs) == [7] * 4
        assert sim.sim_nnz(s.h) == 0
    finally:
        s.close()
