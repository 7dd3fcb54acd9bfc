"""The orders in which a grid's blocks take sites and right-hand sides (0 to 3),
and the kernel that forms a step's scalars once per system, against the oracle.
Order 3 needs whole blocks per t-slice, eight or a multiple of eight: one
lattice has exactly eight, one has sixteen, and on the third the order is
refused and 1 takes its place."""

import numpy as np
import pytest

import oracle
from paper_1311_2719_amd import binding, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

DSLASH_TOL = 1e-13  # per site: sums of 24 products in FP64, as for the other shapes
MASS, TOL = 0.3, 1e-10
# A = m^2 - D^2 with ||D|| <= 4: x with a residual of TOL ||b|| is within
# TOL ||A|| ||A^-1|| of the solution, relative to ||x||
BOUND = TOL * (16 + MASS ** 2) / MASS ** 2

SIZES = [(16, 8, 8, 4), (16, 16, 8, 2), (6, 4, 4, 10)]  # 512, 1024 and 48 sites of a parity per slice


@pytest.mark.parametrize("dims", SIZES)
@pytest.mark.parametrize("order", [0, 1, 2, 3])
@pytest.mark.parametrize("parity", [binding.ALL, binding.EVEN, binding.ODD])
def test_dslash_block_orders(gpu_ctx, monkeypatch, dims, order, parity):
    monkeypatch.setenv("STAG_KERNEL_CFG", "1,64,1,0,%d" % order)
    U = inputs.haar_su3(dims, 511)
    chi = inputs.gaussian_source(dims, 512)
    ref = oracle.dslash(dims, U, chi)
    f = gpu_ctx.set_gauge(dims, U)
    try:
        b, out = gpu_ctx.pack(f, chi), gpu_ctx.new_fermion(f)
        gpu_ctx.dslash(f, b, out, out_parity=parity)
        got = gpu_ctx.unpack(f, out).cpu().numpy()
        n = np.linalg.norm(ref, axis=1)
        x = np.indices(tuple(reversed(dims))).sum(0).ravel() & 1  # lexicographic, x fastest
        on = np.ones(len(n), bool) if parity == binding.ALL else x == (0 if parity == binding.EVEN else 1)
        floor = 1e-3 * np.sqrt(np.mean(n ** 2))
        assert np.max(np.linalg.norm(got - ref, axis=1)[on] / np.maximum(n, floor)[on]) <= DSLASH_TOL
        assert not got[~on].any()
    finally:
        gpu_ctx.free_gauge(f)


@pytest.mark.parametrize("dims", SIZES)
@pytest.mark.parametrize("order", [1, 2, 3])
@pytest.mark.parametrize("precision", [binding.FP64, binding.FP32_RU, binding.FP16_RU])
@pytest.mark.parametrize("parity", [binding.ALL, binding.ODD])
def test_cg_block_orders_and_scalars_kernel(gpu_ctx, monkeypatch, dims, order, precision, parity):
    # a forced shape runs the step kernels; the scalars kernel on and off
    monkeypatch.setenv("STAG_KERNEL_CFG", "1,64,1,0,%d" % order)
    U = inputs.smooth_su3(dims, 0.5, 521)
    src = inputs.gaussian_source(dims, 522)
    got = {}
    for reduce in "01":
        monkeypatch.setenv("STAG_CG_REDUCE", reduce)
        f = gpu_ctx.set_gauge(dims, U)
        try:
            b, x = gpu_ctx.pack(f, src), gpu_ctx.new_fermion(f)
            info = gpu_ctx.cg_solve(f, b, x, mass=MASS, tol=TOL, precision=precision, parity=parity)
            assert info["status"] == 0 and info["true_rel_resid"] <= TOL
            got[reduce] = gpu_ctx.unpack(f, x).cpu().numpy()
            if parity == binding.ALL:
                assert oracle.true_residual(dims, U, MASS, src, got[reduce]) <= TOL
        finally:
            gpu_ctx.free_gauge(f)
    assert np.linalg.norm(got["1"] - got["0"]) <= 2 * BOUND * np.linalg.norm(got["0"])


@pytest.mark.parametrize("dims", [(4, 4, 4, 6), (8, 8, 8, 8)])
@pytest.mark.parametrize("rows", ["2", "3"])
@pytest.mark.parametrize("parity", [binding.EVEN, binding.ODD])
def test_one_parity_with_nontemporal_links_gives_the_same_bits(gpu_ctx, monkeypatch, dims, rows, parity):
    monkeypatch.setenv("STAG_LINK_ROWS", rows)
    monkeypatch.setenv("STAG_WILSON_LPS", "4")  # a timed choice of lanes would change the order of a sum
    U = inputs.haar_su3(dims, 531)
    chi, psi = inputs.gaussian_source(dims, 532), inputs.gaussian_spinor(dims, 533)
    got = {}
    for nt in "01":
        monkeypatch.setenv("STAG_NT_LINKS", nt)
        f, w = gpu_ctx.set_gauge(dims, U), gpu_ctx.set_gauge_wilson(dims, U)
        try:
            b, out = gpu_ctx.pack(f, chi), gpu_ctx.new_fermion(f)
            gpu_ctx.dslash(f, b, out, out_parity=parity)
            s, hop = gpu_ctx.pack_spinor(w, psi), gpu_ctx.new_spinor(w)
            gpu_ctx.wilson_dslash(w, s, hop, out_parity=parity)
            got[nt] = gpu_ctx.unpack(f, out).cpu(), gpu_ctx.unpack_spinor(w, hop).cpu()
        finally:
            gpu_ctx.free_gauge(f)
            gpu_ctx.free_gauge(w)
    assert float(got["0"][0].abs().max()) > 0 and float(got["0"][1].abs().max()) > 0
    assert torch.equal(got["0"][0], got["1"][0]) and torch.equal(got["0"][1], got["1"][1])
