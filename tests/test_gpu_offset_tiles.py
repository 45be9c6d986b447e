"""Tap offsets form only the tiles that the assembly reads (csrc/hessian_i8.hip, i8_rect_needs): channel counts whose taps fill whole
128-row tiles, end inside one, or lie across them, with enough pixels that a tile is cut into several pieces; one call, and a short
call followed by a long one, which needs more slabs than the first stored into."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# (320 channels, 2 x 2: the base taps' tile rows overlap, so the whole triangle is formed; from 448 channels on the long calls deal ranges
# that lie across tiles, the short ones and those of fewer channels a piece of a tile to a workgroup; 1024, 2 x 2: more tiles than workgroups)
@pytest.mark.parametrize("images", [[6], [3, 37]])
@pytest.mark.parametrize("c,k", [(64, 3), (128, 2), (128, 3), (192, 3), (256, 2), (320, 2), (320, 3), (384, 3), (448, 3), (1024, 2)])
def test_hessian_by_offsets_matches_the_unfolded_sum(c, k, images):
    import paper_2509_05576_amd as fobq
    g = torch.Generator(device="cuda")
    g.manual_seed(100 * c + k)
    maps = torch.relu(torch.randn((sum(images), 12, 15, c), generator=g, device="cuda"))
    pad = k // 2
    M = torch.nn.functional.pad(maps, (0, 0, pad, pad, pad, pad)).double()
    ho, wo = M.shape[1] - k + 1, M.shape[2] - k + 1
    taps = [M[:, y:y + ho, x:x + wo, :].reshape(-1, c) for y in range(k) for x in range(k)]
    X = torch.stack(taps, 2).reshape(taps[0].shape[0], -1)
    want = (X.T.contiguous() @ X) * (2.0 / X.shape[0])
    with fobq.Ctx(0) as ctx:
        ctx.set_hessian_mode(fobq.HESSIAN_INT8_SLICES)
        H = torch.full((c * k * k, c * k * k), float("nan"), dtype=torch.float64, device="cuda")
        ctx.hessian_conv(1e6 * maps, k, 1, pad)              # sums of another accumulation in the slabs
        fobq.fobq_hessian_begin(ctx.handle, c * k * k)
        lo = 0
        for n in images:
            fobq.fobq_hessian_accumulate_conv(ctx.handle, maps[lo:lo + n], k, 1, pad)
            lo += n
        fobq.fobq_hessian_finalize(ctx.handle, H)
        torch.cuda.synchronize()
        assert ctx.hessian_form() == (fobq.FORM_INT8_SLICES if (c, k) == (320, 2) else fobq.FORM_INT8_TAP_OFFSETS)
    diag = want.diagonal().sqrt()
    # the digit products' own bound (19 of 25 products of 40-bit numbers), as for the other forms of this mode
    assert float(((H - want).abs() / (diag[:, None] * diag[None, :])).max()) <= 1e-12
    assert torch.equal(H, H.T)
