"""Weights that are not finite: what they reach is undefined, but columns that were quantized before them, and other rows, keep
their codes."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["default", "block32", "batched"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
def test_columns_quantized_before_a_bad_weight_keep_their_codes(form, bad):
    import paper_2509_05576_amd as f
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (no CPU fallback exists)")
    f.load_library()
    r, d, group = 70, 160, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    W = torch.randn((r, d), generator=g, device="cuda") * 0.1
    X = torch.randn((d, 2 * d), generator=g, device="cuda").double()
    H = (X @ X.T.contiguous()) / d
    H = (0.5 * (H + H.T)).contiguous()
    bad_at = {3: 40, 68: 100, 20: 159}            # row: column (first, second and ragged last block)
    Wbad = W.clone()
    for row, col in bad_at.items():
        Wbad[row, col] = bad
    with f.Ctx(0) as ctx:
        def codes(w):
            if form == "batched":
                return ctx.quantize_layers_batched([w], [H], bits=4, group=group, order=f.ORDER_NATURAL)[0].codes
            return ctx.quantize_layer(w, H, bits=4, group=group, order=f.ORDER_NATURAL, block=32 if form == "block32" else 0).codes
        want, got = codes(W), codes(Wbad)
        again = codes(W)
    assert torch.equal(again, want)
    for row in range(r):
        upto = bad_at[row] // group * group if row in bad_at else d      # the bad weight's own group has another grid
        assert torch.equal(got[row, :upto], want[row, :upto]), (row, upto)
