"""The assembly of a Hessian writes the context's copy and the caller's, each entry and its mirror image (csrc/fobq_internal.h,
store_symmetric): widths at the edges of its 16 x 16 tiles and on both sides of the width from which tiles change places in LDS."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(fobq, ctx, H, buf, X):
    d, n = X.shape
    torch.cuda.synchronize()
    want = (X @ X.T.contiguous()) * (2.0 / n)
    scale = want.diagonal().sqrt()
    # fp64 sums of n products: n rounding errors at most; 1e-12: the bound of the digit products
    assert float(((H - want).abs() / (scale[:, None] * scale[None, :])).max()) <= max(1e-12, n * 2.0 ** -52)
    assert torch.equal(H, H.T)
    assert bool(torch.isnan(buf[d * d:]).all())                          # nothing behind the last row
    # the context's own copy: a layer quantized against it and against the caller's
    W = torch.randn((5, d), generator=torch.Generator(device="cuda").manual_seed(d), device="cuda")
    a, b = ctx.quantize_layer(W, damp=0.1), ctx.quantize_layer(W, H, damp=0.1)
    assert torch.equal(a.Q, b.Q) and torch.equal(a.perm, b.perm) and torch.equal(a.loss, b.loss)


@pytest.mark.parametrize("mode,d", [(m, d) for m in ("f64", "i8") for d in (1, 15, 16, 17, 255, 256, 257, 272, 273, 400, 511, 640, 1041)])
def test_both_copies_from_x(mode, d):
    import paper_2509_05576_amd as fobq
    X = torch.randn((d, 700), generator=torch.Generator(device="cuda").manual_seed(d), device="cuda")
    with fobq.Ctx(0) as ctx:
        ctx.set_hessian_mode(fobq.HESSIAN_INT8_SLICES if mode == "i8" else fobq.HESSIAN_FP64)
        buf = torch.full((d * d + 512,), float("nan"), dtype=torch.float64, device="cuda")
        H = buf[:d * d].view(d, d)
        ctx.hessian(X, H_out=H)
        _check(fobq, ctx, H, buf, X.double())


@pytest.mark.parametrize("mode", ["f64", "i8"])
@pytest.mark.parametrize("c,k,stride", [(3, 7, 2), (29, 3, 1), (255, 1, 1), (257, 1, 2), (512, 1, 1), (45, 3, 2), (64, 3, 1), (128, 2, 1)])
def test_both_copies_from_maps(mode, c, k, stride):
    import paper_2509_05576_amd as fobq
    maps = torch.randn((5, 14, 13, c), generator=torch.Generator(device="cuda").manual_seed(c), device="cuda")
    pad, d = k // 2, c * k * k
    X = torch.nn.functional.unfold(maps.permute(0, 3, 1, 2).double(), k, padding=pad, stride=stride).permute(1, 0, 2).reshape(d, -1)
    with fobq.Ctx(0) as ctx:
        ctx.set_hessian_mode(fobq.HESSIAN_INT8_SLICES if mode == "i8" else fobq.HESSIAN_FP64)
        buf = torch.full((d * d + 512,), float("nan"), dtype=torch.float64, device="cuda")
        H = buf[:d * d].view(d, d)
        ctx.hessian_conv(maps, k, stride, pad, H_out=H)
        _check(fobq, ctx, H, buf, X.contiguous())
