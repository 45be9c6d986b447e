"""A call judges its own status words, whatever check of the layer before it failed (host-side test hook; every launched kernel still
runs to its end)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_calls_after_a_failed_check_read_their_own_words():
    import paper_2509_05576_amd as fobq
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    W = torch.randn((8, 96), generator=g, device="cuda")
    good = torch.eye(96, dtype=torch.float64, device="cuda") * 2.0
    bad = -good
    twice = torch.zeros((96,), dtype=torch.int32, device="cuda")      # no permutation
    with fobq.Ctx(0) as ctx:
        ctx.quantize_layer(W, good)          # the scratch is there: every later check follows a launch or a wait
        for nth in range(1, 100):
            fobq.fobq_debug_fail_after(ctx.handle, nth)
            try:
                ctx.quantize_layer(W, good)
                break
            except fobq.FobqError as e:
                assert e.code == fobq.EHIP and "injected" in str(e)
            for call, code in ((lambda: fobq.fobq_spd_inverse(ctx.handle, bad), fobq.ENOTPD),
                               (lambda: fobq.fobq_sensitivity(ctx.handle, W, good, order=fobq.ORDER_CUSTOM, perm_in=twice), fobq.EINVAL),
                               (lambda: fobq.fobq_sensitivity_static(ctx.handle, W, good, order=fobq.ORDER_CUSTOM, perm_in=twice), fobq.EINVAL),
                               (lambda: ctx.obq_rows(W, bad), fobq.ENOTPD)):
                fobq.fobq_debug_fail_after(ctx.handle, nth)
                with pytest.raises(fobq.FobqError):
                    ctx.quantize_layer(W, good)
                fobq.fobq_debug_fail_after(ctx.handle, 0)
                with pytest.raises(fobq.FobqError) as e:
                    call()
                assert e.value.code == code, nth
        assert 10 < nth < 99


@pytest.mark.parametrize("wait", [True, False])
def test_a_failed_call_has_waited_for_its_work(wait):
    import paper_2509_05576_amd as fobq
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    W = torch.randn((64, 1024), generator=g, device="cuda")
    H = torch.eye(1024, dtype=torch.float64, device="cuda")
    s = torch.cuda.Stream()
    with fobq.Ctx(0, stream=s.cuda_stream) as ctx:
        out = ctx.quantize_layer(W, H)
        torch.cuda.synchronize()
        for nth in range(1, 100):
            fobq.fobq_debug_fail_after(ctx.handle, nth)
            try:
                ctx.quantize_layer(W, H, out=out, wait=wait)
                if not wait:
                    ctx.finish()
                break
            except fobq.FobqError as e:
                assert e.code == fobq.EHIP
                assert s.query(), str(e)
        assert 10 < nth < 99
