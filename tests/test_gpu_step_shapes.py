"""The step kernels of one source at every number of lanes per site, with and
without neighbour tables and the scalars kernel, against the oracle."""

import pytest

import oracle
from paper_1311_2719_amd import binding, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

DIMS, MASS, TOL = (6, 4, 4, 10), 0.3, 1e-10  # 480 sites per parity: a partial wavefront


@pytest.mark.parametrize("lanes,block", [(1, 256), (2, 64), (4, 128), (8, 64), (8, 256)])
@pytest.mark.parametrize("tables", [0, 1])
@pytest.mark.parametrize("reduce", ["0", "1"])
@pytest.mark.parametrize("precision", [binding.FP64, binding.FP32_RU, binding.FP16_RU])
def test_step_shapes_of_one_source(gpu_ctx, monkeypatch, lanes, block, tables, reduce, precision):
    monkeypatch.setenv("STAG_KERNEL_CFG", "%d,%d,1,%d,1" % (lanes, block, tables))
    monkeypatch.setenv("STAG_CG_REDUCE", reduce)
    U, src = inputs.smooth_su3(DIMS, 0.5, 601), inputs.gaussian_source(DIMS, 602)
    f = gpu_ctx.set_gauge(DIMS, U)
    try:
        b, x = gpu_ctx.pack(f, src), gpu_ctx.new_fermion(f)
        info = gpu_ctx.cg_solve(f, b, x, mass=MASS, tol=TOL, precision=precision)
        shape = gpu_ctx.cg_tune_info(f, precision=precision, nrhs=1)
        assert (shape["lanes_per_site"], shape["block"], shape["reduction_kernel"]) == (lanes, block, int(reduce))
        assert info["status"] == 0
        assert oracle.true_residual(DIMS, U, MASS, src, gpu_ctx.unpack(f, x).cpu().numpy()) <= TOL
    finally:
        gpu_ctx.free_gauge(f)
