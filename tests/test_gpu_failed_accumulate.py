"""What a Hessian accumulation is worth after a call of it that failed (host-side test hook: the n-th status check of the call reports a
failure): as it was before the call, so that the call can be made again, or closed; never a sum with a part of the call in it."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _calls(fobq, ctx, form):
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    if form.startswith("x"):
        X = torch.relu(torch.randn((400, 1500), generator=g, device="cuda"))
        return 400, [lambda lo=lo, hi=hi: fobq.fobq_hessian_accumulate(ctx, X[:, lo:hi]) for lo, hi in ((0, 600), (600, 1500))]
    c, stride = (128, 1) if form == "offsets" else (48, 2)
    maps = torch.relu(torch.randn((20, 12, 12, c), generator=g, device="cuda"))
    return 9 * c, [lambda lo=lo, hi=hi: fobq.fobq_hessian_accumulate_conv(ctx, maps[lo:hi], 3, stride, 1) for lo, hi in ((0, 15), (15, 20))]


@pytest.mark.parametrize("before", [0, 1])       # good calls before the one that fails
@pytest.mark.parametrize("form", ["offsets", "maps_i8", "x_i8"])
def test_a_call_that_failed_before_its_products_can_be_made_again(form, before):
    import paper_2509_05576_amd as fobq
    with fobq.Ctx(0) as ctx:
        ctx.set_hessian_mode(fobq.HESSIAN_INT8_SLICES)
        d, calls = _calls(fobq, ctx.handle, form)
        H, want = (torch.empty((d, d), dtype=torch.float64, device="cuda") for _ in range(2))

        def begin():
            fobq.fobq_hessian_begin(ctx.handle, d)
            for call in calls[:before]:
                call()

        begin()
        calls[before]()
        fobq.fobq_hessian_finalize(ctx.handle, want)
        assert (ctx.hessian_form() == fobq.FORM_INT8_TAP_OFFSETS) == (form == "offsets")
        for nth in range(1, 100):
            begin()
            fobq.fobq_debug_fail_after(ctx.handle, nth)
            with pytest.raises(fobq.FobqError) as e:
                calls[before]()
            assert e.value.code == fobq.EHIP and "injected" in str(e.value)
            if "xxt" in str(e.value):            # the check behind the products: they have been enqueued
                break
            fobq.fobq_debug_fail_after(ctx.handle, 0)
            calls[before]()
            H.fill_(float("nan"))
            fobq.fobq_hessian_finalize(ctx.handle, H)
            assert torch.equal(H, want), str(e.value)
        assert nth >= 3


@pytest.mark.parametrize("before", [0, 1])       # good calls before the one that fails
@pytest.mark.parametrize("form", ["offsets", "maps_i8", "maps_f64", "x_i8", "x_f64"])
def test_nothing_of_a_failed_call_is_in_the_sum(form, before):
    import paper_2509_05576_amd as fobq
    mode = fobq.HESSIAN_FP64 if form.endswith("f64") else fobq.HESSIAN_INT8_SLICES
    with fobq.Ctx(0) as ctx:
        ctx.set_hessian_mode(mode)
        d, calls = _calls(fobq, ctx.handle, form)
        H, want = (torch.empty((d, d), dtype=torch.float64, device="cuda") for _ in range(2))

        def begin():
            fobq.fobq_hessian_begin(ctx.handle, d)
            for call in calls[:before]:
                call()

        begin()
        calls[before]()
        fobq.fobq_hessian_finalize(ctx.handle, want)
        assert (ctx.hessian_form() == fobq.FORM_INT8_TAP_OFFSETS) == (form == "offsets")
        kept = closed = 0
        for nth in range(1, 100):
            begin()
            fobq.fobq_debug_fail_after(ctx.handle, nth)
            try:
                calls[before]()
                failed = False
            except fobq.FobqError as e:
                assert e.code == fobq.EHIP and "injected" in str(e)
                failed = True
            fobq.fobq_debug_fail_after(ctx.handle, 0)
            if failed:
                try:
                    calls[before]()
                    kept += 1
                except fobq.FobqError as e:
                    assert e.code == fobq.ESTATE
                    closed += 1
                    with pytest.raises(fobq.FobqError) as e:
                        fobq.fobq_hessian_finalize(ctx.handle, H)
                    assert e.value.code == fobq.ESTATE
                    continue
            H.fill_(float("nan"))
            fobq.fobq_hessian_finalize(ctx.handle, H)
            assert torch.equal(H, want), nth
            if not failed:
                break
        assert closed > 0 and nth < 99
        assert kept > 0 or form == "x_f64"          # (its first call is its products alone)
