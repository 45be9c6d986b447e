"""The fp64 Hessian at the widths whose tile depends on the length of the call: each side of that length, and accumulations whose calls
take different tiles, in either order, in scratch that held another accumulation's sums; against 64-bit products."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fobq():
    import paper_2509_05576_amd as f
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (no CPU fallback exists)")
    f.load_library()
    return f


def _close(H, X):
    want = (X @ X.T.contiguous()) * (2.0 / X.shape[1])
    scale = torch.sqrt(want.diagonal()[:, None] * want.diagonal()[None, :])
    # fp64 sums of n products in another order: a small multiple of eps * sqrt(n)
    assert float(((H - want).abs() / scale).max()) <= 1e-13
    assert torch.equal(H, H.T)


def _rand(shape, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda")


@pytest.mark.parametrize("d", [129, 147, 160, 257, 270, 288])
@pytest.mark.parametrize("cuts", [[4095], [4096], [24575], [24576], [30003], [40, 30040], [30000, 30033], [4100, 4140, 34140, 34141]])
def test_calls_of_different_length(fobq, d, cuts):
    X = _rand((d, cuts[-1]), d + len(cuts))
    H = torch.empty((d, d), dtype=torch.float64, device="cuda")
    with fobq.Ctx(0) as ctx:
        ctx.set_hessian_mode(fobq.HESSIAN_FP64)
        ctx.hessian(1e6 * X, H_out=H)
        fobq.fobq_hessian_begin(ctx.handle, d)
        lo = 0
        for hi in cuts:
            fobq.fobq_hessian_accumulate(ctx.handle, X[:, lo:hi])
            lo = hi
        fobq.fobq_hessian_finalize(ctx.handle, H)
    _close(H, X.double())


@pytest.mark.parametrize("c,k,stride", [(16, 3, 1), (3, 7, 2), (32, 3, 1)])
@pytest.mark.parametrize("images", [[1, 40], [40, 1], [3, 4]])
def test_calls_with_different_numbers_of_images(fobq, c, k, stride, images):
    side, pad = 37, k // 2
    maps = _rand((sum(images), side, side, c), c)
    H = torch.empty((c * k * k, c * k * k), dtype=torch.float64, device="cuda")
    with fobq.Ctx(0) as ctx:
        ctx.set_hessian_mode(fobq.HESSIAN_FP64)
        fobq.fobq_hessian_begin(ctx.handle, c * k * k)
        lo = 0
        for n in images:
            fobq.fobq_hessian_accumulate_conv(ctx.handle, maps[lo:lo + n], k, stride, pad)
            lo += n
        fobq.fobq_hessian_finalize(ctx.handle, H)
    M = torch.nn.functional.pad(maps.double(), (0, 0, pad, pad, pad, pad))
    o = (M.shape[1] - k) // stride + 1
    X = torch.stack([M[:, y:y + stride * (o - 1) + 1:stride, x:x + stride * (o - 1) + 1:stride, :].reshape(-1, c)
                     for y in range(k) for x in range(k)], 2).reshape(-1, c * k * k)
    _close(H, X.T.contiguous())
