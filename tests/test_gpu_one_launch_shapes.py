"""What solves of one source in one launch leave behind for the other users of
their field: the untimed shape of the step kernels that would take over."""

import pytest

import oracle
from paper_1311_2719_amd import binding, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

DIMS, MASS, TOL = (4, 4, 6, 8), 0.3, 1e-10


@pytest.mark.parametrize("precision", [binding.FP64, binding.FP32_RU])
def test_server_of_one_slot_times_its_shape_after_a_one_launch_solve(monkeypatch, capfd, precision):
    monkeypatch.setenv("STAG_TUNE_VERBOSE", "1")
    U, src = inputs.smooth_su3(DIMS, 0.5, 441), inputs.gaussian_source(DIMS, 442)
    with binding.Context(device=0, arena_bytes=256 << 20) as ctx:
        ctx.serve_config(slots_per_field=1)
        f = ctx.set_gauge(DIMS, U)
        b, x, xs = ctx.pack(f, src), ctx.new_fermion(f), ctx.new_fermion(f)
        ctx.cg_solve(f, b, x, mass=MASS, tol=TOL, precision=precision)
        shape = ctx.cg_tune_info(f, precision=precision, nrhs=1)  # reported, by rule
        assert shape["lanes_per_site"] == 1 and shape["block"] == 256 and shape["rhs_tile"] == 1
        assert "[stag tune cg]" not in capfd.readouterr().err
        t = ctx.submit(f, b, xs, mass=MASS, tol=TOL, precision=precision)
        assert ctx.wait(t)["rc"] == 0
        ctx.release(t)
        assert "[stag tune cg]" in capfd.readouterr().err
        assert oracle.true_residual(DIMS, U, MASS, src, ctx.unpack(f, xs).cpu().numpy()) <= TOL
        # the blocking solve still runs in one launch, with the same bits
        again = ctx.new_fermion(f)
        ctx.cg_solve(f, b, again, mass=MASS, tol=TOL, precision=precision)
        torch.cuda.synchronize()
        assert torch.equal(x, again)


def test_solves_at_once_on_two_streams_give_the_bits_of_solves_alone(gpu_ctx):
    import threading

    cases = [((4, 4, 4, 4), 451, binding.FP64), ((8, 8, 10, 14), 452, binding.FP32_RU), ((16, 16, 16, 16), 453, binding.FP64)]
    links = [inputs.smooth_su3(d, 0.4, n) for d, n, _ in cases]
    srcs = [inputs.gaussian_source(d, n + 10) for d, n, _ in cases]
    out, errors = {}, []

    def work(k, passes, key):
        try:
            d, _, prec = cases[k]
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream), binding.Context(device=0, arena_bytes=256 << 20, stream=stream) as ctx:
                f = ctx.set_gauge(d, links[k])
                b = ctx.pack(f, srcs[k])
                for _ in range(passes):
                    x = ctx.new_fermion(f)
                    ctx.cg_solve(f, b, x, mass=MASS, tol=TOL, precision=prec)
                    got = ctx.unpack(f, x)
                    stream.synchronize()
                    out.setdefault((key, k), []).append(got.cpu())
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    for k in range(len(cases)):
        work(k, 1, "alone")
    threads = [threading.Thread(target=work, args=(k, 6, "at once")) for k in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(len(cases)):
        assert len(out["at once", k]) == 6
        assert all(torch.equal(g, out["alone", k][0]) for g in out["at once", k]), cases[k]
