"""Layers with so many rows that the elimination's launch takes them in runs: runs of equal and of unequal length, ragged last group of
rows and last block, against the general form (other blocks, other kernels)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r,d,group", [(33001, 500, 0), (65535, 330, 0), (42050, 640, 64), (16385, 1100, 0), (9000, 3000, 0)])
def test_tall_layers_match_the_general_form(r, d, group):
    import paper_2509_05576_amd as f
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (no CPU fallback exists)")
    f.load_library()
    g = torch.Generator(device="cuda")
    g.manual_seed(r + d)
    W = torch.randn((r, d), generator=g, device="cuda") * 0.1
    X = torch.randn((d, 2 * d), generator=g, device="cuda").double()
    H = (X @ X.T.contiguous()) / d
    H = (0.5 * (H + H.T)).contiguous()
    with f.Ctx(0) as ctx:
        want = ctx.quantize_layer(W, H, bits=4, group=group, block=32)
        for _ in range(2):
            got = ctx.quantize_layer(W, H, bits=4, group=group)
            assert torch.equal(got.perm, want.perm)
            # both are fp64, sums in another order: a weight at a code's edge may fall on either side (1e-15 of them per ulp)
            assert int((got.codes != want.codes).sum()) <= 1
            assert torch.allclose(got.loss, want.loss, rtol=1e-9)
