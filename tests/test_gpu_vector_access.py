"""Plain and non-temporal accesses to x and p in the FP32 and FP16 step kernels
give the same bits, in register and shared-link tiles."""

import pytest

from paper_1311_2719_amd import binding, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

DIMS, MASS, TOL = (6, 4, 4, 10), 0.3, 1e-10  # 480 sites per parity: a partial wavefront and chunk


@pytest.mark.parametrize("shape,n", [("1,64,1,0,1", 1), ("4,128,1,0,2", 1), ("1,128,2,0,2", 2), ("2,64,4,1,1", 4),
                                     ("1,128,2,0,2,1", 2), ("1,128,4,0,2,1", 4), ("1,192,3,0,2,1", 3)])
@pytest.mark.parametrize("precision", [binding.FP32_RU, binding.FP16_RU])
@pytest.mark.parametrize("parity", [binding.ALL, binding.ODD])
def test_plain_and_nontemporal_vectors_give_the_same_bits(gpu_ctx, monkeypatch, shape, n, precision, parity):
    monkeypatch.setenv("STAG_KERNEL_CFG", shape)
    U = inputs.smooth_su3(DIMS, 0.5, 571)
    srcs = [inputs.gaussian_source(DIMS, 572 + i) for i in range(n)]
    got = {}
    for nt in "01":
        monkeypatch.setenv("STAG_NT_VECTORS", nt)
        f = gpu_ctx.set_gauge(DIMS, U)
        try:
            bs, xs = [gpu_ctx.pack(f, s) for s in srcs], [gpu_ctx.new_fermion(f) for _ in srcs]
            infos = gpu_ctx.cg_solve_batch(f, bs, xs, [binding.params(MASS, tol=TOL, precision=precision, parity=parity)] * n)
            torch.cuda.synchronize()
            assert all(i["status"] == 0 and i["true_rel_resid"] <= TOL for i in infos)
            got[nt] = torch.stack(xs)
        finally:
            gpu_ctx.free_gauge(f)
    assert float(got["0"].abs().max()) > 0 and torch.equal(got["0"], got["1"])
