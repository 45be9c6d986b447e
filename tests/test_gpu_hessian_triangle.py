"""A layer's Hessian is taken from its lower triangle: what stands above the diagonal changes nothing."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["inverse", "default", "block16", "unblocked", "batched"])
@pytest.mark.parametrize("d", [40, 65, 250])
def test_only_the_lower_triangle_is_read(form, d):
    import paper_2509_05576_amd as f
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (no CPU fallback exists)")
    f.load_library()
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    W = torch.randn((30, d), generator=g, device="cuda") * 0.1
    X = torch.randn((d, 2 * d), generator=g, device="cuda").double()
    H = (X @ X.T.contiguous()) / d
    H = (0.5 * (H + H.T)).contiguous()
    upper = torch.triu(torch.ones_like(H), 1).bool()
    with f.Ctx(0) as ctx:
        def run(h):
            if form == "inverse":
                return [f.fobq_spd_inverse(ctx.handle, h)]
            if form == "batched":
                o = ctx.quantize_layers_batched([W], [h], bits=4)[0]
            else:
                o = ctx.quantize_layer(W, h, bits=4, block={"default": 0, "block16": 16, "unblocked": 1}[form])
            return [o.codes, o.Q, o.perm, o.loss]
        want = run(H)
        for other in (float("nan"), 1e6):
            for a, b in zip(run(torch.where(upper, torch.full_like(H, other), H).contiguous()), want):
                assert torch.equal(a, b)
