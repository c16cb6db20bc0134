"""How a solve waits for the GPU: the core is given up where the process asked
for it with hipSetDeviceFlags, as hipStreamSynchronize does."""
import ctypes
import time

import numpy as np
import pytest

from paper_1411_0330_amd import inputs as I

from .gpu_util import context

pytestmark = pytest.mark.gpu

BLOCKING, YIELD = 4, 2   # hipDeviceScheduleBlockingSync, hipDeviceScheduleYield


@pytest.mark.parametrize("flag", [BLOCKING, YIELD])
def test_solve_honours_the_scheduling_flags(lsh, flag):
    shape = (128, 128, 128)
    moduli = np.stack([I.elastic_from_young(1.0, 0.3), I.elastic_from_young(10.0, 0.2)])
    ctx = context(lsh, I.random_phases(shape, 2, seed=3), moduli, I.elastic_from_young(0.5, 0.3), "elastic", "filtered",
                  "fp64", 6)
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(ln.split()[-1] for ln in f if "libamdhip64" in ln))
    before = ctypes.c_uint()
    assert hip.hipGetDeviceFlags(ctypes.byref(before)) == 0
    ref = ctx.solve(np.eye(6), "minres", tol=1e-12, maxit=30)
    A = ctx.effective()
    try:
        assert hip.hipSetDeviceFlags(flag) == 0
        wall, cpu = time.perf_counter(), time.thread_time()
        rep = ctx.solve(np.eye(6), "minres", tol=1e-12, maxit=30)
        wall, cpu = time.perf_counter() - wall, time.thread_time() - cpu
    finally:
        hip.hipSetDeviceFlags(before.value)
    assert rep["iterations"] == ref["iterations"] and np.array_equal(ctx.effective(), A)
    if flag == BLOCKING:   # iterations of 2.7 ms: the host sleeps through most of each
        assert cpu < 0.5 * wall
