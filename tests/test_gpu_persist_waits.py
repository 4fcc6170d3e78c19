"""Persistent runs whose blocks give up waiting.  The waits are bounded, so every
block leaves normally; a test forces them short from the host, for its own
thread."""
import contextlib
import ctypes
import time
import warnings

import pytest
import torch

from gpu_util import gpu_operator, problem, to_dev
from paper_1811_02605_amd import _abi as abi
from paper_1811_02605_amd import solver as S

pytestmark = pytest.mark.gpu


@contextlib.contextmanager
def waits(start=-1.0, wait=-1.0, refuse=False):
    """Longest waits, in seconds, for all blocks to start and at an exchange
    (negative: the library's own); or every cooperative launch refused."""
    fn = abi.load().mas_test_persist_waits
    fn.argtypes, fn.restype = [ctypes.c_double, ctypes.c_double, ctypes.c_int], None
    fn(start, wait, int(refuse))
    try:
        yield
    finally:
        fn(-1.0, -1.0, 0)


def close(a, b, rtol):
    return float((a - b).norm() / b.norm()) <= rtol


COLUMNS = ((40, 57, 130), 0)  # shape, chunk_planes: 0.3M cells, a column per thread
CELLS = ((32, 32, 64), 0)  # a cell per thread
TILES = ((32, 32, 64), 2)  # tiles of two r planes
KINDS = [COLUMNS, CELLS, TILES]
NOT_STARTED = [dict(start=0.0), dict(refuse=True)]


@pytest.mark.parametrize("forced", NOT_STARTED)
@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("shape,chunk", KINDS)
def test_runs_that_do_not_start_are_launched_per_iteration(shape, chunk, precision, forced):
    p = problem(shape)
    _, op = gpu_operator(p, precision)
    rhs = to_dev(p.rhs)
    o = dict(rtol=1e-10, precision=precision, chunk_planes=chunk)
    auto, per, asked = S.make_opts(**o), S.make_opts(launch="per_iteration", **o), S.make_opts(launch="persistent", **o)
    ref, ri = op.solve(rhs, per)
    x0 = (0.9 * ref).contiguous()
    warm, wi = op.solve(rhs, per, x0=x0.clone())
    lam, gnu, grhs, _ = op.adjoint(ref, rhs, per)
    with waits(**forced):
        x, info = op.solve(rhs, auto)
        assert info["launch"] == abi.MAS_LAUNCH_PER_ITERATION and info["iters"] == ri["iters"]
        assert torch.equal(x, ref)
        x, info = op.solve(rhs, auto, x0=x0.clone())
        assert info["iters"] == wi["iters"] and torch.equal(x, warm)
        out = op.adjoint(ref, rhs, auto)
        assert torch.equal(out[0], lam) and torch.equal(out[1], gnu) and torch.equal(out[2], grhs)
        with pytest.raises(abi.MasError) as e:
            op.solve(rhs, asked)
        assert e.value.status == abi.MAS_EHIP
    x, info = op.solve(rhs, auto)
    assert info["launch"] == abi.MAS_LAUNCH_PERSISTENT and close(x, ref, 1e-8)


@pytest.mark.parametrize("forced", NOT_STARTED)
@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("shape,chunk", [CELLS, TILES])
def test_several_rhs_that_do_not_start(shape, chunk, precision, forced):
    p = problem(shape)
    _, op = gpu_operator(p, precision)
    rhs = to_dev(p.rhs)
    b = torch.stack([rhs, torch.zeros_like(rhs), rhs.flip(2)])
    o = dict(rtol=1e-10, precision=precision, chunk_planes=chunk)
    ref, ri = op.solve_multi(b, S.make_opts(launch="per_iteration", **o))
    with waits(**forced):
        x, info = op.solve_multi(b, S.make_opts(**o))
    assert torch.equal(x, ref)
    for h in range(3):
        assert info[h]["launch"] == abi.MAS_LAUNCH_PER_ITERATION and info[h]["iters"] == ri[h]["iters"]


def test_allocation_free_solve_that_does_not_start():
    p = problem("c0")
    _, op = gpu_operator(p)
    rhs = to_dev(p.rhs)
    ref, _ = op.solve(rhs, S.make_opts(launch="per_iteration"))
    for forced in NOT_STARTED:
        with waits(**forced):
            x, info = op.solve_noalloc(rhs, S.make_opts())
        assert info["launch"] == abi.MAS_LAUNCH_PER_ITERATION and torch.equal(x, ref)


@pytest.mark.parametrize("shape,chunk", KINDS)
def test_blocks_give_up_starting_all_together(shape, chunk):
    """Start waits that follow the time that the blocks take to start, so that
    about half are too short for the last ones.  All blocks then leave at once,
    none waits 2 s for one that has left."""
    p = problem(shape)
    _, op = gpu_operator(p)
    rhs = to_dev(p.rhs)
    ref, _ = op.solve(rhs, S.make_opts(launch="per_iteration"))
    o = S.make_opts(chunk_planes=chunk)
    op.solve(rhs, o)
    us, launches = 20.0, {abi.MAS_LAUNCH_PER_ITERATION: 0, abi.MAS_LAUNCH_PERSISTENT: 0}
    for _ in range(600):
        with waits(start=us * 1e-6):
            t0 = time.perf_counter()
            x, info = op.solve(rhs, o)
            dt = time.perf_counter() - t0
        launches[info["launch"]] += 1
        assert dt < 1.0, (us, dt)
        assert close(x, ref, 1e-8), us
        us *= 0.98 if info["launch"] == abi.MAS_LAUNCH_PERSISTENT else 1.02
    assert min(launches.values()) > 50, launches


@pytest.mark.parametrize("iters", [1, 2])
@pytest.mark.parametrize("shape", [(9, 16, 32), (32, 32, 64), (40, 57, 130)])
def test_a_block_that_gives_up_last_is_not_missed(shape, iters):
    """Exchange waits that follow the time an exchange takes, so that in about half
    of the calls some blocks give up, also at the run's last exchange where others
    end it.  A call then fails; one that does not has every cell of x."""
    p = problem(shape)
    _, op = gpu_operator(p)
    rhs = to_dev(p.rhs)
    o = S.make_opts(rtol=0.0, max_iters=iters, max_restarts=0, launch="persistent")
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")  # not converged
        ref, _ = op.solve(rhs, o)
        us, failed, n = 10.0, 0, 1500
        for _ in range(n):
            try:
                with waits(wait=us * 1e-6):
                    x, _ = op.solve(rhs, o)
                assert torch.equal(x, ref), us
                us *= 0.99
            except abi.MasError as e:
                assert e.status == abi.MAS_EHIP
                failed += 1
                us *= 1.01
    assert 100 < failed < n - 100
