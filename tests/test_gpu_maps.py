"""Hessians from feature maps at the channel counts where the padding launch changes its form: channels in fours or not, maps
that are not 16-byte aligned, the channel maxima taken along with the copy or by a launch of their own."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _unfolded_hessian(maps, k, stride, pad):
    M = torch.nn.functional.pad(maps.double(), (0, 0, pad, pad, pad, pad))
    out_h, out_w = (M.shape[1] - k) // stride + 1, (M.shape[2] - k) // stride + 1
    taps = [M[:, y:y + stride * (out_h - 1) + 1:stride, x:x + stride * (out_w - 1) + 1:stride, :].reshape(-1, maps.shape[3])
            for y in range(k) for x in range(k)]
    X = torch.stack(taps, 2).reshape(taps[0].shape[0], -1)              # column c * k^2 + tap
    return (X.T.contiguous() @ X) * (2.0 / X.shape[0])


@pytest.mark.parametrize("n,h,w,c,k,stride,pad,offset", [
    (4, 13, 11, 48, 3, 2, 1, 0), (4, 13, 11, 48, 3, 2, 1, 1), (6, 12, 13, 255, 2, 1, 0, 0), (6, 12, 13, 257, 2, 2, 1, 0),
    (5, 11, 12, 1020, 1, 1, 0, 0), (5, 11, 12, 1028, 1, 1, 0, 0), (4, 13, 13, 64, 3, 1, 1, 1), (9, 9, 9, 43, 3, 1, 2, 3)])
@pytest.mark.parametrize("int8", [False, True])
def test_hessian_from_maps_at_channel_edges(n, h, w, c, k, stride, pad, offset, int8):
    import paper_2509_05576_amd as f
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (no CPU fallback exists)")
    f.load_library()
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k)
    flat = torch.randn((n * h * w * c + offset,), generator=g, device="cuda")
    maps = flat[offset:].view(n, h, w, c)
    H = torch.empty((c * k * k, c * k * k), dtype=torch.float64, device="cuda")
    with f.Ctx(0) as ctx:
        ctx.set_hessian_mode(f.HESSIAN_INT8_SLICES if int8 else f.HESSIAN_FP64)
        ctx.hessian_conv(maps, k, stride, pad, H_out=H)
    want = _unfolded_hessian(maps, k, stride, pad)
    scale = torch.sqrt(want.diagonal()[:, None] * want.diagonal()[None, :])
    # fp64 sums of n products: eps * n at most; the int8 mode's bar is 1e-12
    assert float(((H - want).abs() / scale).max()) <= (1e-12 if int8 else 1e-13)
    assert torch.equal(H, H.T)
