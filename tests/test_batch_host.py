"""Compiling batch jobs on the host (no GPU): what qk_batch_add accepts."""
import ctypes as C
import math

import pytest

from paper_1908_07187_amd import qk


@pytest.mark.parametrize("n", [3, 20])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("value", [math.nan, math.inf, -math.inf, 1e308, 0.0])
def test_any_parameter_is_accepted(dtype, n, value):
    """Parameters are not checked, here as in the per-gate path: one that is
    not finite makes amplitudes that are not, and no error."""
    lib, h, job = qk.load(), C.c_void_p(), C.c_int32()
    assert lib.qk_batch_create(qk.DTYPES[dtype], None, None, C.byref(h)) == 0
    for name, targets in (("RX", 1), ("RY", 1), ("RZ", 1), ("PHASE", 1), ("CPHASE", 2), ("RZZ", 2)):
        for controls in (0, 1):
            o = qk.QkOp()
            o.kind, o.gate, o.n_targets, o.n_controls, o.param = qk.QK_OP_GATE, qk.BUILTINS[name], targets, controls, value
            o.targets[1], o.controls[0] = 1, 2
            assert lib.qk_batch_add(h, n, 0, C.byref(o), 1, C.byref(job)) == 0, (name, lib.qk_batch_last_error(h))
    assert lib.qk_batch_destroy(h) == 0
