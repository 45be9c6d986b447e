"""The waits inside the factorization launches: a launch that does not move is given up (forced from the host by a limit of a few
looks), drains, fails the call and leaves the context usable; one that moves is not, however long a single wait is."""
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


def _layer(r, d):
    g = torch.Generator(device="cuda")
    g.manual_seed(r + d)
    W = torch.randn((r, d), generator=g, device="cuda") * 0.1
    X = torch.randn((d, 2 * d), generator=g, device="cuda").double()
    H = (X @ X.T.contiguous()) / d
    return W, (0.5 * (H + H.T)).contiguous()


@pytest.mark.parametrize("form", ["inverse", "layer", "block32", "batched", "enqueued"])
def test_a_launch_that_is_given_up_fails_the_call_only(fobq, form):
    layers = [_layer(200, 250), _layer(70, 130), _layer(64, 256)]
    if form != "batched":
        layers = [_layer(300, 1500)]
    with fobq.Ctx(0) as ctx:
        def run():
            if form == "inverse":
                return [fobq.fobq_spd_inverse(ctx.handle, layers[0][1])]
            if form == "batched":
                outs = ctx.quantize_layers_batched([w for w, _ in layers], [h for _, h in layers], bits=4)
            else:
                outs = [ctx.quantize_layer(*layers[0], bits=4, block=32 if form == "block32" else 0, wait=form != "enqueued")]
                if form == "enqueued":
                    ctx.finish()
            return [t for o in outs for t in (o.codes, o.Q, o.perm, o.loss)]
        want = run()
        for looks in (0, 3):
            fobq.fobq_debug_wait_looks(ctx.handle, looks)
            with pytest.raises(fobq.FobqError) as e:
                run()
            assert e.value.code == fobq.EHIP and "drew no tile" in str(e.value)
            fobq.fobq_debug_wait_looks(ctx.handle, -1)
            for a, b in zip(run(), want):
                assert torch.equal(a, b)


# most of these launches' wavefronts wait for many of the chain's blocks, 15 us each, at a time: more than 768 looks of 0.16 us or
# more; the launch as a whole draws tiles all the while
@pytest.mark.parametrize("r,d", [(64, 3000), (300, 4608)])
def test_long_waits_of_a_launch_that_moves_are_waited_for(fobq, r, d):
    W, H = _layer(r, d)
    with fobq.Ctx(0) as ctx:
        want = ctx.quantize_layer(W, H, bits=4)
        fobq.fobq_debug_wait_looks(ctx.handle, 768)
        got = ctx.quantize_layer(W, H, bits=4)
    for a, b in zip((got.codes, got.Q, got.perm, got.loss), (want.codes, want.Q, want.perm, want.loss)):
        assert torch.equal(a, b)
