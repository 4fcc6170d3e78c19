"""A waiting call follows the device's scheduling flag: where the program asked for
waits that do not spin, the calling thread does not occupy a CPU for the whole
of a long solve."""
import contextlib
import ctypes
import time

import pytest
import torch

from gpu_util import gpu_operator, problem, to_dev
from paper_1811_02605_amd import _abi as abi
from paper_1811_02605_amd import solver as S

pytestmark = pytest.mark.gpu

SCHEDULE = {"yield": 2, "blocking": 4}  # hipDeviceScheduleYield, hipDeviceScheduleBlockingSync


@contextlib.contextmanager
def schedule(flag):
    lib, old = abi.load(), ctypes.c_uint()  # the HIP runtime that the library is bound to
    assert lib.hipGetDeviceFlags(ctypes.byref(old)) == 0
    assert lib.hipSetDeviceFlags(ctypes.c_uint(flag)) == 0
    try:
        yield
    finally:
        assert lib.hipSetDeviceFlags(old) == 0


@pytest.mark.parametrize("flag", SCHEDULE)
@pytest.mark.parametrize("precond", ["pc1", "pc2"])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
def test_waiting_thread_sleeps(precision, precond, flag):
    p = problem((192, 192, 384))
    _, op = gpu_operator(p, precision)
    rhs, o = to_dev(p.rhs), S.make_opts(precision=precision, precond=precond)
    ref, _ = op.solve(rhs, o, allow_notconv=False)
    torch.cuda.synchronize()
    with schedule(SCHEDULE[flag]):
        cpu, wall = time.thread_time(), time.perf_counter()
        for _ in range(3):
            x, _ = op.solve(rhs, o, allow_notconv=False)
        cpu, wall = time.thread_time() - cpu, time.perf_counter() - wall
    print(f"{precision} {precond} {flag}: cpu {cpu / wall:.2f} of {wall / 3 * 1e3:.1f} ms")
    assert torch.equal(x, ref)
    assert cpu <= 0.5 * wall, (cpu, wall)
