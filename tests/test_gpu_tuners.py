"""What the tuners time: the leading shapes of the CG step more than once."""

import re

import pytest

from paper_1311_2719_amd import binding, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


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
