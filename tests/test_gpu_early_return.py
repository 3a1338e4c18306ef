"""A call that returns early with an error of the HIP runtime leaves a handle
that can go on.  The error is one that the calling thread already has pending
(an invalid device asked for), which the call meets behind its first launch."""
import ctypes

import numpy as np
import pytest

from helpers import assert_same_state
from oracle import Oracle
from paper_2105_01533_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    from paper_2105_01533_amd import sim as S
    return S


def _leave_error():
    with open("/proc/self/maps") as f:
        path = next(ln.split()[-1] for ln in f if "libamdhip64" in ln)
    hip = ctypes.CDLL(path)
    assert hip.hipSetDevice(1 << 20) != 0


@pytest.mark.parametrize("n", [30, 90])
@pytest.mark.parametrize("capacity, fits", [(12_000, False), (40_000, True)])
@pytest.mark.parametrize("entries", [1500, 5000, 9000])
def test_handle_goes_on(sim, n, capacity, fits, entries):
    if entries < 9000:
        capacity = 3 * entries if fits else entries + 100
    state = W.random_state(63, entries, n - 3)
    c = W.Circuit()
    c.h(n - 1)                 # doubles the entries
    c.x(2, (1,))
    c.h(n - 2)                 # prepared by the one before
    more = W.Circuit()
    for _ in range(2):
        more.gate(W.K_RY, 4, controls=(5,), param=0.7)
        more.gate(W.K_RY, 4, controls=(5,), param=-0.7)
    more.x(7, (6,))
    s = sim.Simulator(n, capacity, 1e-20, tuned=False)
    try:
        s.import_state(*state)
        for _ in range(2):
            _leave_error()
            rc, _, _ = s.apply_ops(c.array(), raise_on_error=False)
            assert rc == sim.SIM_E_HIP
            lo, hi, amp = s.export(sort=False)
            if len(lo) == entries:      # (the gate behind the error is in or out, whole)
                for x, y in zip((lo, hi, amp), state):
                    assert x.tobytes() == np.ascontiguousarray(y, x.dtype).tobytes()
            else:
                assert fits and len(lo) == 2 * entries
            s.import_state(*state)
        if not fits:
            return
        rc, _, st = s.apply_ops(more.array(), raise_on_error=False)
        assert rc == 0 and st["u2_applied"] == 4
        o = Oracle(n, 1e-20)
        o.import_state(*state)
        o.run(more.array())
        assert_same_state(s.export(), o.export(), what="after an early return")
    finally:
        s.close()
