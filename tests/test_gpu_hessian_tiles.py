"""The fp64 Hessian at the sizes where its tile changes (64, 96, 128 wide, or one tile of 160 for all columns), from X and from
feature maps, aligned and not, with one workgroup to a chunk and with tiles cut into pieces, against 64-bit products."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2509_05576_amd as f
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (no CPU fallback exists)")
    f.load_library()
    with f.Ctx(0) as c:
        c.set_hessian_mode(f.HESSIAN_FP64)
        yield c


def _close(H, X):
    want = (X @ X.T.contiguous()) * (2.0 / X.shape[1])
    scale = torch.sqrt(want.diagonal()[:, None] * want.diagonal()[None, :]) + 1e-300
    # fp64 sums of n products in another order: a small multiple of eps * sqrt(n)
    assert float(((H - want).abs() / scale).max()) <= 1e-13
    assert torch.equal(H, H.T)


@pytest.mark.parametrize("n", [1, 33, 700, 20003, 20004])
@pytest.mark.parametrize("d", [64, 96, 128, 129, 144, 147, 160, 161, 191, 192, 193, 257, 288, 289, 513, 576])
def test_hessian_from_x_at_tile_edges(ctx, d, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(d * 7 + n)
    X = torch.randn((d, n), generator=g, device="cuda")
    H = torch.empty((d, d), dtype=torch.float64, device="cuda")
    ctx.hessian(X, H_out=H)
    _close(H, X.double())
    for _ in range(2):          # the sums do not depend on which workgroup ends first
        again = torch.empty_like(H)
        ctx.hessian(X, H_out=again)
        assert torch.equal(H, again)


@pytest.mark.parametrize("n,side,c,k,stride,pad", [(1, 7, 15, 3, 1, 1), (3, 31, 16, 3, 2, 1), (9, 65, 3, 7, 2, 3), (2, 30, 18, 3, 1, 1),
                                                   (3, 30, 32, 3, 1, 1), (2, 25, 57, 3, 1, 0), (5, 20, 160, 1, 1, 0), (5, 20, 161, 1, 1, 0)])
def test_hessian_from_maps_at_tile_edges(ctx, n, side, c, k, stride, pad):
    g = torch.Generator(device="cuda")
    g.manual_seed(c)
    maps = torch.randn((n, side, side, c), generator=g, device="cuda")
    H = torch.empty((c * k * k, c * k * k), dtype=torch.float64, device="cuda")
    ctx.hessian_conv(maps, k, stride, pad, H_out=H)
    M = torch.nn.functional.pad(maps.double(), (0, 0, pad, pad, pad, pad))
    o = (M.shape[1] - k) // stride + 1
    X = torch.stack([M[:, y:y + stride * (o - 1) + 1:stride, x:x + stride * (o - 1) + 1:stride, :].reshape(-1, c)
                     for y in range(k) for x in range(k)], 2).reshape(n * o * o, -1)
    _close(H, X.T.contiguous())


# the first call of an accumulation stores its sums, later ones add: a later call with more slabs than the first, with fewer,
# and (int8 mode takes short calls in fp64) one in the integer form after an fp64 one; scratch that held another accumulation's sums before
@pytest.mark.parametrize("d", [100, 147, 192, 288, 512, 640])
@pytest.mark.parametrize("cuts", [[40, 20040], [20000, 20033], [1, 2, 5002, 20002]])
def test_calls_of_one_accumulation(ctx, d, cuts):
    import paper_2509_05576_amd as f
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    X = torch.randn((d, cuts[-1]), generator=g, device="cuda")
    H = torch.empty((d, d), dtype=torch.float64, device="cuda")
    ctx.hessian(1e6 * X, H_out=H)
    for int8 in (False, True):
        ctx.set_hessian_mode(f.HESSIAN_INT8_SLICES if int8 else f.HESSIAN_FP64)
        f.fobq_hessian_begin(ctx.handle, d)
        lo = 0
        for hi in cuts:
            f.fobq_hessian_accumulate(ctx.handle, X[:, lo:hi])
            lo = hi
        f.fobq_hessian_finalize(ctx.handle, H)
        ctx.set_hessian_mode(f.HESSIAN_FP64)
        want = (X.double() @ X.double().T.contiguous()) * (2.0 / X.shape[1])
        scale = torch.sqrt(want.diagonal()[:, None] * want.diagonal()[None, :])
        assert float(((H - want).abs() / scale).max()) <= (1e-12 if int8 else 1e-13)      # the integer form's bar; eps * sqrt(n)
