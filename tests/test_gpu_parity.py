"""GPU parity against the FP64 CPU oracle on seeded inputs (small and ragged
grids spanning several tiles: 64-wide phi segments, 8-row theta tiles and
32-plane r chunks, with ragged tails in every direction)."""
import math

import numpy as np
import pytest
import torch

from gpu_util import (DEV, gpu_operator, oracle_operator, oracle_plus_face_arrays, problem, rel,
                      residual_rounding_floor, to_dev, to_host)
from oracle import dense
from paper_1811_02605_amd import _abi as abi
from paper_1811_02605_amd import solver as S

pytestmark = pytest.mark.gpu

# (nr, nt, np): single tile, ragged phi (70, 129), ragged theta (7, 17), two r
# chunks (33, 65), eight 18-plane chunks with a ragged last one (137: the
# chunk length grows with nr beyond 128 planes), degenerate 1-cell
# directions, the small benchmark grid.
SHAPES = [(4, 4, 8), (5, 7, 13), (3, 9, 70), (33, 17, 129), (65, 8, 64), (137, 5, 16), (1, 3, 2),
          (6, 3, 1), (2, 1, 5), (9, 16, 32)]
BCS = [(0, 0), (1, 0), (1, 1)]

# Elementwise bound for the exported entries: both sides form each conductance
# with ~10 roundings in a different order, and the scaled storage adds a few
# more (c^ = c (1/w_a)(1/w_b), then w_a c^ w_b).  Measured at most 6 ulp for
# the couplings and 5 for the diagonal on every grid and wall set here, 8 and
# 6 on the 52.4M cells of the benchmark grid; the bound is that plus 2 ulp.
EXPORT_RTOL = 10 * 2.0 ** -52


@pytest.mark.parametrize("shape", SHAPES + ["c0"])
@pytest.mark.parametrize("bc", BCS)
def test_exported_operator_matches_oracle(shape, bc):
    p = problem(shape, bc)
    _, op = gpu_operator(p)
    got = [to_host(t) for t in op.export()]
    want = oracle_plus_face_arrays(oracle_operator(p))
    ulps = {}
    for name, g, w in zip(("cr", "ct", "cp", "diag"), got, want):
        nz = w != 0
        ulps[name] = float(np.max(np.abs(g - w)[nz] / np.spacing(np.abs(w[nz])))) if nz.any() else 0.0
        np.testing.assert_allclose(g, w, rtol=EXPORT_RTOL, atol=0, err_msg=name)
    print(f"{shape} bc={bc}: max ulp " + " ".join(f"{k} {v:.1f}" for k, v in ulps.items()))
    # exact zeros: last r plane, pole rows
    assert np.all(got[0][-1] == 0.0) and np.all(got[1][:, -1] == 0.0)


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("shape", SHAPES + ["c0"])
def test_apply_matches_oracle(shape, precision):
    p = problem(shape, (0, 1))
    _, op = gpu_operator(p, precision)
    ora = oracle_operator(p)
    x = np.random.default_rng(11).standard_normal(p.shape)
    y = to_host(op.apply(to_dev(x)))
    assert rel(y, ora.apply(x)) <= 1e-13


@pytest.mark.parametrize("shape", [(1031, 5, 3), (37, 130, 129), (40, 190, 300), (35, 257, 449)])
def test_elementwise_tiles_of_few_planes(shape):
    """The elementwise kernels with 2, 3, 8 and 12 r planes a block, the last
    block with fewer: A x, and a solve (its norms, x scaled in and out)."""
    p = problem(shape, (0, 1), q=1.001)
    _, op = gpu_operator(p)
    ora = oracle_operator(p)
    x = np.random.default_rng(12).standard_normal(p.shape)
    assert rel(to_host(op.apply(to_dev(x))), ora.apply(x)) <= 1e-13
    y, info = op.solve(to_dev(p.rhs), S.make_opts(rtol=1e-10), allow_notconv=False)
    b = ora.rhs_to_b(p.rhs)
    assert abs(info["bnorm"] - np.linalg.norm(b)) <= 1e-12 * np.linalg.norm(b)
    assert ora.rel_residual(b, to_host(y)) <= 1e-10


# r planes per chunk of the iteration kernel: 0 is the automatic choice
# (short chunks on these small grids, which cannot fill the GPU otherwise),
# 16 and 18 the chunk lengths of grids large enough to fill it
CHUNKS = [0, 16]


@pytest.mark.parametrize("chunk", CHUNKS)
@pytest.mark.parametrize("shape", SHAPES + ["c0"])
@pytest.mark.parametrize("bc", [(0, 0), (1, 1)])
def test_fp64_solve_matches_oracle(shape, bc, chunk):
    p = problem(shape, bc)
    _, op = gpu_operator(p)
    ora = oracle_operator(p)
    x, info = op.solve(to_dev(p.rhs), S.make_opts(rtol=1e-10, chunk_planes=chunk),
                       allow_notconv=False)
    x = to_host(x)
    b = ora.rhs_to_b(p.rhs)
    res = ora.rel_residual(b, x)
    assert res <= 1e-10, res
    assert info["rel_resid_true"] <= 1e-10
    # the reported residual is the oracle's up to the rounding of b - A x
    floor = residual_rounding_floor(ora, b, x)
    assert abs(info["rel_resid_true"] - res) <= floor, (info["rel_resid_true"], res, floor)
    xo, it_o, _, _ = ora.pcg(b, tol=1e-13)
    err = rel(x, xo)
    print(f"{shape} bc={bc}: iters gpu {info['iters']} oracle(1e-13) {it_o}; "
          f"residual {res:.2e}; error vs oracle {err:.2e}")
    assert err <= 1e-6


@pytest.mark.parametrize("check_every", [1, 8, 64])
@pytest.mark.parametrize("shape", ["c0", (33, 17, 129), (65, 8, 64), (9, 16, 32)])
def test_iteration_count_tracks_oracle(shape, check_every):
    """The run stops at the first iteration whose ||b - A x_k|| meets the
    tolerance, as the oracle's does: the residual norm is formed on the
    periodic check iterations and on every iteration once its value,
    predicted from (r, r), is near the threshold."""
    p = problem(shape)
    _, op = gpu_operator(p)
    ora = oracle_operator(p)
    x, info = op.solve(to_dev(p.rhs), S.make_opts(rtol=1e-10, check_every=check_every),
                       allow_notconv=False)
    _, it_o, _, _ = ora.pcg(ora.rhs_to_b(p.rhs), tol=1e-10)
    print(f"{shape} check_every={check_every}: gpu {info['iters']} oracle {it_o}")
    # the two sum their dot products in different orders (R17): the crossing
    # can move by an iteration
    assert abs(info["iters"] - it_o) <= 1, (info["iters"], it_o)


@pytest.mark.parametrize("chunk", CHUNKS + [1, 5])
@pytest.mark.parametrize("k", [0, 1, 2, 5, 20])
@pytest.mark.parametrize("shape", [(5, 7, 13), (33, 17, 129), "c0"])
def test_iterates_match_oracle(shape, k, chunk):
    # the GPU's scaled single-reduction recurrence and the oracle's classical
    # PCG produce the same iterates in exact arithmetic
    p = problem(shape)
    _, op = gpu_operator(p)
    ora = oracle_operator(p)
    x, info = op.solve(to_dev(p.rhs), S.make_opts(rtol=0.0, max_iters=k, check_every=1,
                                                  chunk_planes=chunk))
    assert info["status"] == abi.MAS_ENOTCONV and info["iters"] == k
    xo = ora.pcg(ora.rhs_to_b(p.rhs), tol=0.0, max_iters=k)[0]
    e = rel(to_host(x), xo)
    assert e <= 1e-11 * max(1, k), e


@pytest.mark.parametrize("chunk", CHUNKS)
@pytest.mark.parametrize("refine", ["reliable", "restart"])
@pytest.mark.parametrize("shape", [(5, 7, 13), (33, 17, 129), (1, 3, 2), (9, 16, 32), "c0"])
def test_mixed_precision_reaches_fp64_residual(shape, refine, chunk):
    p = problem(shape)
    _, op = gpu_operator(p, "fp32_refined")
    ora = oracle_operator(p)
    x, info = op.solve(to_dev(p.rhs), S.make_opts(rtol=1e-10, precision="fp32_refined",
                                                  refine=refine, chunk_planes=chunk),
                       allow_notconv=False)
    x = to_host(x)
    b = ora.rhs_to_b(p.rhs)
    res = ora.rel_residual(b, x)
    xo, it_o, _, _ = ora.pcg(b, tol=1e-13)
    print(f"{shape} refined/{refine}: outer {info['outer_iters']} inner {info['iters']} "
          f"(oracle FP64 at 1e-13: {it_o}) residual {res:.2e} error vs FP64 oracle {rel(x, xo):.2e}")
    assert res <= 1e-10 and info["rel_resid_true"] <= 1e-10
    floor = residual_rounding_floor(ora, b, x)
    assert abs(info["rel_resid_true"] - res) <= floor, (info["rel_resid_true"], res, floor)
    assert info["outer_iters"] >= 1
    assert rel(x, xo) <= 1e-6


def test_fp64_solve_is_bitwise_deterministic():
    p = problem((33, 17, 129))
    _, op = gpu_operator(p)
    rhs = to_dev(p.rhs)
    x1, i1 = op.solve(rhs)
    x2, i2 = op.solve(rhs)
    assert torch.equal(x1, x2) and i1["iters"] == i2["iters"]
    _, opm = gpu_operator(p, "fp32_refined")
    o = S.make_opts(precision="fp32_refined")
    y1, _ = opm.solve(rhs, o)
    y2, _ = opm.solve(rhs, o)
    assert torch.equal(y1, y2)


def test_warm_start_from_solution():
    p = problem((9, 16, 32))
    _, op = gpu_operator(p)
    ora = oracle_operator(p)
    xs = dense.dense_solve(ora, ora.rhs_to_b(p.rhs)) if p.cfg.n <= 600 else \
        ora.pcg(ora.rhs_to_b(p.rhs), tol=1e-14)[0]
    x, info = op.solve(to_dev(p.rhs), x0=to_dev(xs))
    assert info["iters"] == 0 and info["status"] == 0
    assert rel(to_host(x), xs) <= 1e-13
    # a rough warm start converges in fewer iterations than a cold one
    x0 = xs + 1e-4 * np.random.default_rng(0).standard_normal(p.shape)
    _, iw = op.solve(to_dev(p.rhs), x0=to_dev(x0))
    _, ic = op.solve(to_dev(p.rhs))
    assert iw["status"] == 0 and iw["iters"] < ic["iters"]


def test_reused_opts_keep_no_warm_start():
    """An options object used for a warm-started solve is not changed by it: a
    following adjoint and a cold solve with the same object start from zero
    and take the iterations of fresh calls."""
    p = problem((9, 16, 32))
    _, op = gpu_operator(p)
    rhs = to_dev(p.rhs)
    o = S.make_opts(rtol=1e-10)
    x, ic = op.solve(rhs, o, allow_notconv=False)
    _, iw = op.solve(rhs, o, x0=x, allow_notconv=False)  # starts at the solution
    assert o.use_x0 == 0 and iw["iters"] == 0 < ic["iters"]
    _, ic2 = op.solve(rhs, o, allow_notconv=False)
    assert ic2["iters"] == ic["iters"]
    gx = to_dev(np.random.default_rng(5).standard_normal(p.shape))
    _, _, _, ia = op.adjoint(x, gx, o, allow_notconv=False)
    _, _, _, ia_fresh = op.adjoint(x, gx, S.make_opts(rtol=1e-10), allow_notconv=False)
    assert ia["iters"] == ia_fresh["iters"]
    # use_x0 set by the caller without an x0 tensor is ignored: the output
    # buffer is fresh memory, never a starting guess
    _, iu = op.solve(rhs, S.make_opts(rtol=1e-10, use_x0=1), allow_notconv=False)
    assert iu["iters"] == ic["iters"]


def test_zero_time_step_and_zero_rhs():
    p = problem((5, 7, 13))
    _, op = gpu_operator(p, dt=0.0)
    x, info = op.solve(to_dev(p.rhs))
    assert info["iters"] <= 1 and rel(to_host(x), p.rhs) <= 1e-14
    _, op = gpu_operator(p)
    x, info = op.solve(torch.zeros(p.shape, dtype=torch.float64, device=DEV))
    assert info["iters"] == 0 and torch.count_nonzero(x) == 0


def test_status_codes_on_device():
    p = problem((5, 7, 13))
    grid = S.Grid.from_problem(p)
    nu = p.nu.copy()
    nu[2, 3, 4] = -1.0
    with pytest.raises(abi.MasError) as e:
        S.Operator(grid, to_dev(nu), p.dt)
    assert e.value.status == abi.MAS_EINVAL
    nu[2, 3, 4] = np.nan
    with pytest.raises(abi.MasError):
        S.Operator(grid, to_dev(nu), p.dt)
    _, op = gpu_operator(p)
    with pytest.raises(abi.MasError) as e:  # no single-precision coefficients in an FP64 build
        op.solve(to_dev(p.rhs), S.make_opts(precision="fp32_refined"))
    assert e.value.status == abi.MAS_EINVAL
    x, info = op.solve(to_dev(p.rhs), S.make_opts(max_iters=3))
    assert info["status"] == abi.MAS_ENOTCONV and info["iters"] == 3
    with pytest.raises(abi.MasError) as e:
        op.solve(to_dev(p.rhs), allow_notconv=False, opts=S.make_opts(max_iters=3))
    assert e.value.status == abi.MAS_ENOTCONV
    # workspace too small
    import ctypes
    o = S.make_opts()
    work, nbytes = op.workspace(o)
    info = abi.mas_pcg_info()
    rhs = to_dev(p.rhs)
    xx = torch.empty_like(rhs)
    st = abi.load().mas_pcg_solve(op.handle, rhs.data_ptr(), xx.data_ptr(), ctypes.byref(o),
                                  work.data_ptr(), nbytes - 256, 0, ctypes.byref(info))
    assert st == abi.MAS_ENOMEM


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
def test_adjoint_matches_oracle_gradient(precision):
    p = problem((16, 16, 32))
    _, op = gpu_operator(p, precision)
    ora = oracle_operator(p)
    o = S.make_opts(precision=precision)
    x, _ = op.solve(to_dev(p.rhs), o, allow_notconv=False)
    xt = ora.solve_rhs(p.rhs) * 0.9
    gx = to_host(x) - xt
    lam, gnu, grhs, info = op.adjoint(x, to_dev(gx), o, allow_notconv=False)
    xo = ora.solve_rhs(p.rhs, tol=1e-13)
    lo = ora.pcg(gx, tol=1e-13)[0]
    gnu_o, grhs_o = ora.gradient(xo, lo)
    e_nu, e_rhs = rel(to_host(gnu), gnu_o), rel(to_host(grhs), grhs_o)
    print(f"adjoint {precision}: dL/dnu rel {e_nu:.2e}, dL/drhs rel {e_rhs:.2e}")
    assert e_nu <= 1e-6 and e_rhs <= 1e-6
    # the adjoint solve meets the same tolerance
    assert ora.rel_residual(gx, to_host(lam)) <= 1e-10


# The gradient kernel's tiles: 64-cell phi segments (32 lanes x 2; 32 x 1 for
# odd np), 8 theta rows per block, 32-plane r chunks marched up or down.
GRAD_SHAPES = [(33, 17, 129), (3, 9, 70), (70, 9, 66), (65, 4, 34), (5, 9, 128), (4, 7, 64), (261, 3, 8),
               (3, 5, 2), (6, 3, 1), (2, 1, 5), (1, 2, 4), (97, 11, 130)]


@pytest.mark.parametrize("shape", GRAD_SHAPES)
@pytest.mark.parametrize("bc", [(0, 1), (1, 0), (0, 0)])
def test_gradient_kernel_matches_oracle_formula(shape, bc):
    """dL/dnu and dL/drhs at the GPU's own lambda and an arbitrary x, against the
    oracle's formula at the same fields: the kernel alone, element by element."""
    p = problem(shape, bc)
    _, op = gpu_operator(p)
    ora = oracle_operator(p)
    rng = np.random.default_rng(17)
    x = rng.standard_normal(p.shape)
    gx = rng.standard_normal(p.shape)
    lam, gnu, grhs, info = op.adjoint(to_dev(x), to_dev(gx), S.make_opts(rtol=1e-10),
                                      allow_notconv=False)
    assert info["grad_kernel_us"] == 0.0  # not sampled
    gnu_o, grhs_o = (np.asarray(t).reshape(p.shape) for t in ora.gradient(x, to_host(lam)))
    g, h = to_host(gnu), to_host(grhs)
    # each entry is a sum of at most seven products formed in the same way on
    # both sides; the bound is relative to the largest entry
    assert np.max(np.abs(g - gnu_o)) <= 1e-13 * np.max(np.abs(gnu_o))
    assert np.max(np.abs(h - grhs_o)) <= 1e-14 * np.max(np.abs(grhs_o))


def test_gradient_kernel_timing_sample():
    p = problem((9, 16, 32))
    _, op = gpu_operator(p)
    x = to_dev(np.random.default_rng(3).standard_normal(p.shape))
    _, _, _, info = op.adjoint(x, x, S.make_opts(rtol=1e-10, sample_timing=1), allow_notconv=False)
    assert info["grad_kernel_us"] > 0.0


def test_autograd_function():
    p = problem((6, 8, 16))
    grid = S.Grid.from_problem(p)
    nu = to_dev(p.nu).requires_grad_(True)
    rhs = to_dev(p.rhs).requires_grad_(True)
    x = S.solve(nu, rhs, grid, p.dt, rtol=1e-12)
    xt = torch.zeros_like(x)
    loss = 0.5 * ((x - xt) ** 2).sum()
    loss.backward()
    ora = oracle_operator(p)
    xo = ora.solve_rhs(p.rhs, tol=1e-13)
    lo = ora.pcg(xo, tol=1e-13)[0]
    gnu_o, grhs_o = ora.gradient(xo, lo)
    assert rel(to_host(nu.grad), gnu_o) <= 1e-8
    assert rel(to_host(rhs.grad), grhs_o) <= 1e-8


@pytest.mark.parametrize("nin,nout", [(8, 4), (6, 3), (7, 4), (6, 1), (2, 2), (4, 1), (1, 1)])
def test_probe_stream_writes_each_output_once(nin, nout):
    """The streaming probe over n cells (odd, several blocks and a ragged
    tail) on a buffer filled with 0.25: output array t holds 0.25 nin + t in
    every cell, the inputs and the padding keep 0.25."""
    lib = abi.load()
    n = 3 * 16384 + 1001
    nbytes = int(lib.mas_probe_stream_bytes(n, nin, nout))
    assert nbytes >= (nin + nout) * 8 * n
    buf = torch.full((nbytes // 8,), 0.25, dtype=torch.float64, device=DEV)
    with torch.cuda.device(buf.device):
        abi.check(lib.mas_probe_stream(buf.data_ptr(), nbytes, n, nin, nout,
                                       torch.cuda.current_stream().cuda_stream), "mas_probe_stream")
    torch.cuda.synchronize()
    vals, counts = torch.unique(buf, return_counts=True)
    got = dict(zip(vals.tolist(), counts.tolist()))
    want = {}
    for t in range(nout):
        v = 0.25 * nin + t
        want[v] = want.get(v, 0) + n
    for v, c in want.items():
        if v != 0.25:
            assert got.get(v, 0) == c, (v, got)
    assert set(got) <= set(want) | {0.25}
    assert lib.mas_probe_stream(buf.data_ptr(), nbytes, n, 5, 5, None) == abi.MAS_EINVAL


def test_probe_copy():
    src = torch.arange(1 << 20, dtype=torch.float64, device=DEV)
    dst = torch.empty_like(src)
    S.probe_copy(src, dst)
    torch.cuda.synchronize()
    assert torch.equal(src, dst)


# rows that are no multiple of the lanes' vector width (2 doubles, 4 floats): two
# lanes, one lane short of and one past a 32-lane segment, segments shared
# evenly, and the widths whose last segment would hold a single lane
@pytest.mark.parametrize("np_", [3, 5, 6, 7, 63, 65, 127, 129, 130, 131, 1985, 3971])
@pytest.mark.parametrize("chunk", [0, 2])
def test_ragged_rows_launched_per_iteration(np_, chunk):
    p = problem((3, 9, np_), (1, 0))
    _, op = gpu_operator(p, "fp32_refined")
    ora = oracle_operator(p)
    rhs, b = to_dev(p.rhs), ora.rhs_to_b(p.rhs)
    two = torch.stack([rhs, rhs.flip(2).contiguous()])
    for k in (1, 2, 5):
        o = S.make_opts(rtol=0.0, max_iters=k, max_restarts=0, launch="per_iteration", chunk_planes=chunk)
        x, info = op.solve(rhs, o)
        X, _ = op.solve_multi(two, o)
        xo = ora.pcg(b, tol=0.0, max_iters=k)[0]
        assert rel(to_host(x), xo) <= 1e-11 * k
        assert torch.equal(X[0], x)
    for precond in ("pc1", "pc2"):
        o = S.make_opts(rtol=1e-10, precision="fp32_refined", precond=precond, launch="per_iteration" if precond == "pc1"
                        else "auto", chunk_planes=chunk)
        x, _ = op.solve(rhs, o, allow_notconv=False)
        assert ora.rel_residual(b, to_host(x)) <= 1e-10
