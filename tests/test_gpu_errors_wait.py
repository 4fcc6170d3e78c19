"""A call that fails after it has launched kernels returns once they have ended:
the caller may free or reuse its buffers."""
import ctypes

import pytest
import torch

from gpu_util import gpu_operator, problem, to_dev
from paper_1811_02605_amd import _abi as abi
from paper_1811_02605_amd import solver as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [0, 2])  # 0: mas_pcg_solve
@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
def test_no_kernel_is_under_way_after_a_refused_right_hand_side(precision, nrhs):
    p = problem((64, 128, 256))
    _, op = gpu_operator(p, precision)
    lib, opts = abi.load(), S.make_opts(precision=precision)
    m = max(nrhs, 1)
    rhs = to_dev(p.rhs).repeat(m, 1, 1, 1).contiguous()
    rhs[-1, 0, 0, 0] = float("nan")
    x = torch.empty_like(rhs)
    need = lib.mas_pcg_multi_workspace_bytes(op.handle, m)
    work = torch.empty(need + 256, dtype=torch.uint8, device=rhs.device)
    at = (work.data_ptr() + 255) & ~255
    info = (abi.mas_pcg_info * m)()
    stream = torch.cuda.current_stream()
    for _ in range(50):
        torch.cuda.synchronize()
        if nrhs:
            st = lib.mas_pcg_solve_multi(op.handle, nrhs, rhs.data_ptr(), x.data_ptr(), ctypes.byref(opts), at, need,
                                         stream.cuda_stream, info)
        else:
            st = lib.mas_pcg_solve(op.handle, rhs.data_ptr(), x.data_ptr(), ctypes.byref(opts), at, need,
                                   stream.cuda_stream, info)
        idle = stream.query()
        assert st == abi.MAS_EINVAL and "not finite" in abi.last_error()
        assert idle
