"""Hessians from feature maps of few, long rows, which the padding launch cuts into runs of pixels."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,c,k,pad,offset", [(1, 1, 20011, 40, 1, 0, 0), (1, 1, 20011, 43, 1, 0, 0), (2, 1, 9001, 48, 3, 1, 1), (1, 3, 7001, 44, 3, 2, 0),
                                                  (1, 1, 1503, 1028, 1, 0, 0), (3, 1, 2999, 256, 1, 3, 0)])
@pytest.mark.parametrize("int8", [False, True])
def test_hessian_of_long_rows(n, h, w, c, k, pad, offset, int8):
    import paper_2509_05576_amd as f
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (no CPU fallback exists)")
    f.load_library()
    g = torch.Generator(device="cuda")
    g.manual_seed(c + k)
    flat = torch.randn((n * h * w * c + offset,), generator=g, device="cuda")
    maps = flat[offset:].view(n, h, w, c)
    maps[-1, -1, -1] = 6.0                     # channel maxima in the last pixel of the last run
    d = c * k * k
    H = torch.empty((d, d), dtype=torch.float64, device="cuda")
    with f.Ctx(0) as ctx:
        ctx.set_hessian_mode(f.HESSIAN_INT8_SLICES if int8 else f.HESSIAN_FP64)
        ctx.hessian_conv(maps, k, 1, pad, H_out=H)
    M = torch.nn.functional.pad(maps.double(), (0, 0, pad, pad, pad, pad))
    oh, ow = M.shape[1] - k + 1, M.shape[2] - k + 1
    X = torch.stack([M[:, y:y + oh, x:x + ow, :].reshape(-1, c) for y in range(k) for x in range(k)], 2).reshape(n * oh * ow, d)
    want = (X.T.contiguous() @ X) * (2.0 / X.shape[0])
    scale = torch.sqrt(want.diagonal()[:, None] * want.diagonal()[None, :]) + 1e-300      # taps above a single row: zeros
    # fp64 sums of n products: eps * n at most; the int8 mode's bar is 1e-12
    assert float(((H - want).abs() / scale).max()) <= (1e-12 if int8 else 1e-13)
    assert torch.equal(H, H.T)
