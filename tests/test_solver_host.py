"""Host decisions of the solver, on the CPU: whether the next product is queued ahead of the host."""
import ctypes as C

import numpy as np
import pytest


def _goes_on(run, iters, cap, est, prev, tol):
    from paper_1807_03097_amd import binding as B
    f = B._lib._ZN3ige14krylov_goes_onEiPKcPKiS3_PKdS5_S5_
    f.restype = C.c_bool
    f.argtypes = [C.c_int] + [C.c_void_p] * 6
    a = [np.array(run, np.int8), np.array(iters, np.int32), np.array(cap, np.int32)]
    a += [np.array(v, np.float64) for v in (est, prev, tol)]
    return bool(f(len(run), *(v.ctypes.data for v in a)))


@pytest.mark.parametrize("run,iters,cap,est,prev,expect", [
    ([1], [0], [5], [1.0], [0.0], True),             # first step
    ([1], [0], [1], [1.0], [0.0], False),            # its only one
    ([1], [4], [5], [1.0], [1.0], False),            # the last of five
    ([1], [3], [5], [1e-3], [1e-2], True),           # 1e-4 expected, 1e-5 wanted
    ([1], [3], [9], [5e-5], [4e-4], False),          # 6e-6 expected
    ([1], [3], [9], [5e-5], [5e-5], True),           # no progress
    ([1], [3], [9], [2e-5], [1e-5], True),           # an estimate that rose is not extrapolated
    ([1], [3], [9], [float("nan")], [1.0], True),    # left to the iteration count
    ([0], [3], [9], [1.0], [1.0], False),            # nothing runs
    ([1, 1], [4, 3], [5, 5], [1.0, 1.0], [1.0, 1.0], True),
    ([1, 0], [4, 0], [5, 9], [1.0, 1.0], [1.0, 0.0], False),
    ([1, 1], [2, 2], [9, 9], [5e-5, 1e-3], [4e-4, 1.1e-3], True),
])
def test_product_ahead_only_where_a_step_follows(run, iters, cap, est, prev, expect):
    assert _goes_on(run, iters, cap, est, prev, [1e-5] * len(run)) is expect
