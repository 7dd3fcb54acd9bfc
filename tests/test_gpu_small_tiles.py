"""Smaller shared-link tiles at the block count of a register tile with several
lanes per site: more blocks than chunks of 64 sites, so some blocks have no
site.  The tile takes over while two of four systems still run."""

import numpy as np
import pytest

import oracle
from paper_1311_2719_amd import binding, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-10
MASSES = [0.05, 0.06, 0.8, 0.9]


@pytest.mark.parametrize("dims,lanes", [((8, 8, 8, 8), 2), ((6, 6, 6, 6), 2), ((2, 4, 6, 10), 8)])
@pytest.mark.parametrize("rows", ["2", "3"])
@pytest.mark.parametrize("precision", [binding.FP32_RU, binding.FP16_RU])
@pytest.mark.parametrize("reduce", ["0", "1"])
def test_shared_tile_with_blocks_beyond_the_sites(gpu_ctx, monkeypatch, dims, lanes, rows, precision, reduce):
    sites = int(np.prod(dims)) // 2
    assert -(-sites * lanes // 64) > -(-sites // 64)  # blocks of the register tile, chunks of the shared one
    monkeypatch.setenv("STAG_KERNEL_CFG", "%d,64,4,0,1;1,128,2,0,1,1" % lanes)
    monkeypatch.setenv("STAG_CG_REDUCE", reduce)
    monkeypatch.setenv("STAG_EPOCH", "2")
    monkeypatch.setenv("STAG_LINK_ROWS", rows)
    U = inputs.smooth_su3(dims, 0.5, 181)
    srcs = [inputs.gaussian_source(dims, 1810 + i) for i in range(4)]
    f = gpu_ctx.set_gauge(dims, U)
    try:
        bs = [gpu_ctx.pack(f, s) for s in srcs]
        xs = [gpu_ctx.new_fermion(f) for _ in srcs]
        infos = gpu_ctx.cg_solve_batch(f, bs, xs, [binding.params(m, tol=TOL, precision=precision) for m in MASSES])
        torch.cuda.synchronize()
        assert min(i["iters"] for i in infos[:2]) >= max(i["iters"] for i in infos[2:]) + 8, infos
        for m, s, x, info in zip(MASSES, srcs, xs, infos):
            assert info["status"] == 0 and info["true_rel_resid"] <= TOL
            assert oracle.true_residual(dims, U, m, s, gpu_ctx.unpack(f, x).cpu().numpy()) <= TOL
    finally:
        gpu_ctx.free_gauge(f)
