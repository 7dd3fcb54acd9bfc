"""What the tuners time: the kernels that are then run, and the leading shapes
of the CG step more than once."""

import re

import numpy as np
import pytest

import oracle
from paper_1311_2719_amd import binding, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nt", ["0", "1"])
def test_wilson_shapes_are_timed_on_the_kernels_that_run(monkeypatch, capfd, nt):
    dims = (4, 4, 6, 8)
    monkeypatch.setenv("STAG_TUNE_VERBOSE", "1")
    monkeypatch.setenv("STAG_NT_LINKS", nt)
    U, psi = inputs.haar_su3(dims, 541), inputs.gaussian_spinor(dims, 542)
    ref = oracle.wilson_hop(dims, U, psi)
    scale = np.sqrt(np.mean(np.sum(np.abs(ref) ** 2, axis=(1, 2))))
    timed = lambda: set(re.findall(r"(both parities|one parity) once=(\d)", capfd.readouterr().err))  # noqa: E731
    with binding.Context(device=0, arena_bytes=64 << 20) as ctx:
        f = ctx.set_gauge_wilson(dims, U)
        b, out = ctx.pack_spinor(f, psi), ctx.new_spinor(f)
        capfd.readouterr()
        ctx.wilson_dslash(f, b, out)
        assert {k for k, _ in timed()} == {"both parities"}
        # sums of 8 hops of 3 products on 4 spins in FP64
        assert np.max(np.abs(ctx.unpack_spinor(f, out).cpu().numpy() - ref)) <= 1e-13 * scale
        one = ctx.new_spinor(f)
        ctx.wilson_dslash(f, b, one, out_parity=binding.ODD)
        assert timed() == {("one parity", nt)}
        assert float((one[1] - out[1]).abs().max()) <= 1e-13 * scale and float(one[0].abs().max()) == 0
        ctx.wilson_dslash(f, b, out)
        ctx.wilson_solve(f, b, out, 0.11)  # the loads of the hop of one parity: nothing new to time
        assert timed() == set()


@pytest.mark.parametrize("slots,precision", [(1, binding.FP16_RU), (4, binding.FP32_RU)])
def test_leading_cg_shapes_are_timed_again_in_every_block_order(monkeypatch, capfd, slots, precision):
    dims = (16, 8, 8, 4)  # eight blocks of 64 sites per t-slice: every block order with 1 x 64
    monkeypatch.setenv("STAG_TUNE_VERBOSE", "1")
    U = inputs.smooth_su3(dims, 0.5, 551)
    with binding.Context(device=0, arena_bytes=256 << 20) as ctx:
        f = ctx.set_gauge(dims, U)
        bs = [ctx.pack(f, inputs.gaussian_source(dims, 560 + i)) for i in range(slots)]
        xs = [ctx.new_fermion(f) for _ in bs]
        capfd.readouterr()
        ctx.cg_solve_batch(f, bs, xs, [binding.params(0.3, precision=precision)] * slots)
        shape = ctx.cg_tune_info(f, precision=precision, nrhs=slots)
    lines = [tuple(map(int, m)) for m in re.findall(
        r"tune cg\] V=\d+ prec=\d slots=\d+ lps=(\d) block=(\d+) rtile=(\d+) shared=(\d) reduce=(\d) tables=0 remap=(\d)",
        capfd.readouterr().err)]
    taken = (shape["lanes_per_site"], shape["block"], shape["rhs_tile"], shape["shared_links"], shape["reduction_kernel"])
    times = [lines.count(taken + (order,)) for order in (0, 1, 2)]
    assert min(times) >= 1 and max(times) >= 3, (taken, times)


@pytest.mark.parametrize("precision", [0, 1, 2])
def test_dslash_of_one_parity_is_timed_by_itself(monkeypatch, capfd, precision):
    dims = (16, 8, 8, 4)
    monkeypatch.setenv("STAG_TUNE_VERBOSE", "1")
    U, chi = inputs.haar_su3(dims, 581), inputs.gaussian_source(dims, 582)
    timed = lambda: set(re.findall(r"stag tune\].* (both parities|one parity) ", capfd.readouterr().err))  # noqa: E731
    with binding.Context(device=0, arena_bytes=256 << 20) as ctx:
        f = ctx.set_gauge(dims, U)
        b = ctx.pack(f, chi)
        if precision:
            b = ctx.convert(f, b, ctx.new_fermion(f, precision), binding.F64, precision)
        out, one = ctx.new_fermion(f, precision), ctx.new_fermion(f, precision)
        capfd.readouterr()
        ctx.dslash(f, b, out, precision=precision)
        assert timed() == {"both parities"}
        ctx.dslash(f, b, one, out_parity=binding.ODD, precision=precision)
        assert timed() == {"one parity"}
        ctx.dslash(f, b, one, out_parity=binding.EVEN, precision=precision)
        assert timed() == set()
        torch.cuda.synchronize()
        assert torch.equal(one, out)  # block size and order do not change a site's sum
