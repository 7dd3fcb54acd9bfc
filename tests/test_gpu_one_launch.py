"""Solves of one source in one launch (small lattices) against the step
kernels and the oracle's true residual, at the edges of the launch: a partly
filled wavefront and block, the largest grid whose blocks read each other's
sums directly and the smallest that goes through groups, the largest lattice,
one and two parities, two and three link rows; and the step kernels taking
over when a block gives up waiting."""

import numpy as np
import pytest

import oracle
from paper_1311_2719_amd import binding, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MASS, TOL = 0.3, 1e-10
# A = m^2 - D^2 with ||D|| <= 4 (four directions, two hops of 1/2 each); both
# solutions have a residual of at most TOL ||b||, so they differ by at most
# 2 TOL ||A|| ||A^-1|| relative to ||x||
BOUND = 2 * TOL * (16 + MASS ** 2) / MASS ** 2


def solve(ctx, dims, links, src, monkeypatch, mode, **kw):
    monkeypatch.setenv("STAG_PERSIST", mode)
    f = ctx.set_gauge(dims, links)
    try:
        b, x, y = ctx.pack(f, src), ctx.new_fermion(f), ctx.new_fermion(f)
        info = ctx.cg_solve(f, b, x, y=y, mass=MASS, tol=TOL, **kw)
        torch.cuda.synchronize()
        again = ctx.new_fermion(f)
        ctx.cg_solve(f, b, again, mass=MASS, tol=TOL, **kw)
        torch.cuda.synchronize()
        assert torch.equal(x, again)  # every block adds the same sums in the same order
        return ctx.unpack(f, x).cpu().numpy(), ctx.unpack(f, y).cpu().numpy(), info
    finally:
        ctx.free_gauge(f)


@pytest.mark.parametrize("dims,fat,lanes", [
    ((2, 2, 2, 2), False, "4"),
    ((2, 4, 6, 8), True, "4"),
    ((6, 10, 14, 8), False, "2"),
    ((8, 8, 8, 16), False, "4"),    # 64 blocks
    ((8, 8, 10, 14), False, "4"),   # 70 blocks: sums through groups
    ((8, 16, 16, 16), True, "4"),   # 256 blocks, three rows
    ((16, 16, 16, 16), False, "2"),  # 256 blocks of two lanes per site
])
@pytest.mark.parametrize("precision,parity", [
    (binding.FP64, binding.ALL), (binding.FP64, binding.ODD),
    (binding.FP32_RU, binding.ALL), (binding.FP32_RU, binding.EVEN),
])
def test_one_launch_matches_the_step_kernels(gpu_ctx, monkeypatch, dims, fat, lanes, precision, parity):
    U = inputs.smooth_su3(dims, 0.5, 411)
    if fat:
        U = U * np.random.default_rng(412).uniform(0.95, 1.05, U.shape[:2])[..., None, None]
    src = inputs.gaussian_source(dims, 413)
    x1, y1, i1 = solve(gpu_ctx, dims, U, src, monkeypatch, lanes, precision=precision, parity=parity)
    x0, y0, i0 = solve(gpu_ctx, dims, U, src, monkeypatch, "0", precision=precision, parity=parity)
    assert i1["status"] == 0 and abs(i1["iters"] - i0["iters"]) <= 1, (i1, i0)
    assert np.linalg.norm(x1 - x0) <= BOUND * np.linalg.norm(x0)
    assert np.linalg.norm(y1 - y0) <= 4 * BOUND * np.linalg.norm(x0)
    if parity == binding.ALL:
        assert oracle.true_residual(dims, U, MASS, src, x1) <= TOL
    assert i1["true_rel_resid"] <= TOL


@pytest.mark.parametrize("precision", [binding.FP64, binding.FP32_RU])
def test_iteration_limit_and_zero_source(gpu_ctx, monkeypatch, precision):
    dims = (4, 4, 6, 8)
    U = inputs.smooth_su3(dims, 0.5, 421)
    src = inputs.gaussian_source(dims, 422)
    monkeypatch.setenv("STAG_PERSIST", "4")
    f = gpu_ctx.set_gauge(dims, U)
    try:
        b, x = gpu_ctx.pack(f, src), gpu_ctx.new_fermion(f)
        info = gpu_ctx.cg_solve(f, b, x, mass=MASS, tol=1e-14, maxiter=7, precision=precision, check=False)
        assert info["rc"] == binding.ENOCONV and info["iters"] == 7
        assert torch.isfinite(torch.view_as_real(x)).all() and float(x.abs().max()) > 0
        b.zero_()
        info = gpu_ctx.cg_solve(f, b, x, mass=MASS, tol=TOL, precision=precision)
        assert info["iters"] == 0 and float(x.abs().max()) == 0
    finally:
        gpu_ctx.free_gauge(f)


def test_step_kernels_take_over(gpu_ctx, monkeypatch):
    # no wait is allowed to last: if some block gives up, the solve is repeated
    # by the step kernels; the result stands either way
    dims = (8, 8, 10, 14)
    U = inputs.smooth_su3(dims, 0.5, 431)
    src = inputs.gaussian_source(dims, 432)
    monkeypatch.setenv("STAG_PERSIST_TICKS", "0")
    monkeypatch.setenv("STAG_PERSIST", "4")
    f = gpu_ctx.set_gauge(dims, U)
    try:
        b, x = gpu_ctx.pack(f, src), gpu_ctx.new_fermion(f)
        info = gpu_ctx.cg_solve(f, b, x, mass=MASS, tol=TOL)
        assert info["status"] == 0
        assert oracle.true_residual(dims, U, MASS, src, gpu_ctx.unpack(f, x).cpu().numpy()) <= TOL
    finally:
        gpu_ctx.free_gauge(f)
