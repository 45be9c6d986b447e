"""The factorization launches that exchange tiles between workgroups while they run (csrc/flow.hip): the result may not
depend on which workgroup takes which tile, nor on what else runs on the GPU."""
import numpy as np
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


def _spd(d, seed):
    """(2 / n) X X^T + 1 % of its mean diagonal, n < d: the damping alone keeps it positive definite."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n = max(8, d // 2)
    X = torch.relu(torch.randn((d, n), generator=g, device="cuda")).double()
    H = (X @ X.T.contiguous()) * (2.0 / n)
    H = 0.5 * (H + H.T)
    H.diagonal().add_(0.01 * H.diagonal().mean())
    return H.contiguous()


# one to five blocks, block edges, more tiles than workgroups, several queue rows in flight
@pytest.mark.parametrize("d", [1, 63, 64, 65, 128, 129, 192, 193, 257, 500, 1216, 2048])
def test_inverse_is_the_same_every_time(fobq, d):
    H = _spd(d, d)
    with fobq.Ctx(0) as ctx:
        first = fobq.fobq_spd_inverse(ctx.handle, H)
        # residual of the first against 64-bit products: eps * kappa * d with kappa <= 1e4 here
        R = first @ H - torch.eye(d, dtype=torch.float64, device="cuda")
        assert float(R.abs().max()) <= 1e-9
        for _ in range(12):
            assert torch.equal(fobq.fobq_spd_inverse(ctx.handle, H), first)


def test_inverses_on_several_contexts_at_once(fobq):
    dims = [700, 1300, 200, 1000]
    Hs = [_spd(d, 7 + d) for d in dims]
    Ws = [torch.randn((40, d), device="cuda") for d in dims]
    streams = [torch.cuda.Stream() for _ in dims]
    ctxs = [fobq.Ctx(0, stream=s.cuda_stream) for s in streams]
    torch.cuda.synchronize()
    want = []
    for c, W, H in zip(ctxs, Ws, Hs):
        o = c.quantize_layer(W, H, bits=4)
        want.append([t.clone() for t in (o.codes, o.Q, o.perm, o.loss)])
    for _ in range(6):
        outs = [c.quantize_layer(W, H, bits=4, wait=False) for c, W, H in zip(ctxs, Ws, Hs)]
        for c in ctxs:
            c.finish()
        for o, w in zip(outs, want):
            for a, b in zip((o.codes, o.Q, o.perm, o.loss), w):
                assert torch.equal(a, b)
    for c in ctxs:
        c.close()


# single rows, ragged groups of rows, one and several rows per wavefront, ragged last block, grids per group: the launch that
# eliminates and quantizes against the general form (other blocks, other kernels); both are fp64, sums in another order
@pytest.mark.parametrize("r,d,group", [(1, 1, 0), (7, 64, 0), (9, 65, 0), (65, 129, 43), (300, 577, 0), (1030, 320, 64),
                                       (2100, 512, 128), (8200, 256, 0), (260, 2304, 0)])
def test_elimination_and_columns_match_the_general_form(fobq, r, d, group):
    H = _spd(d, 3 * d)
    g = torch.Generator(device="cuda")
    g.manual_seed(r + d)
    W = torch.randn((r, d), generator=g, device="cuda") * (2.0 / d) ** 0.5
    with fobq.Ctx(0) as ctx:
        want = ctx.quantize_layer(W, H, bits=4, group=group, block=32, debug=True)
        got = ctx.quantize_layer(W, H, bits=4, group=group, debug=True)
        assert torch.equal(got.perm, want.perm) and torch.equal(got.codes, want.codes) and torch.equal(got.Q, want.Q)
        assert torch.allclose(got.W_work, want.W_work, rtol=1e-9, atol=1e-12)
        assert torch.allclose(got.loss, want.loss, rtol=1e-11)
        assert not got.Hinv_work.any()
        for _ in range(3):
            again = ctx.quantize_layer(W, H, bits=4, group=group)
            assert torch.equal(again.codes, got.codes) and torch.equal(again.loss, got.loss)


# one layer, one to four blocks, ragged sizes, more workgroups than the GPU holds, many rows (several rows per wavefront):
# layers that share the launches against the same layers one by one; sums in the same order, so the bits are the same
@pytest.mark.parametrize("shapes", [[(1, 1)], [(40, 63), (64, 64), (3, 65), (130, 129), (9, 256)], [(17 + i % 50, 1 + i) for i in range(256)],
                                    [(3000, 250), (1, 2), (5000, 100)]])
def test_batched_layers_match_single_layers(fobq, shapes):
    g = torch.Generator(device="cuda")
    g.manual_seed(len(shapes))
    Hs = [_spd(d, 11 + d) for _, d in shapes]
    Ws = [torch.randn((r, d), generator=g, device="cuda") * (2.0 / d) ** 0.5 for r, d in shapes]
    with fobq.Ctx(0) as ctx:
        want = [ctx.quantize_layer(W, H, bits=3) for W, H in zip(Ws, Hs)]
        for _ in range(3):
            for o, w in zip(ctx.quantize_layers_batched(Ws, Hs, bits=3), want):
                assert torch.equal(o.perm, w.perm) and torch.equal(o.codes, w.codes) and torch.equal(o.Q, w.Q)
                assert torch.allclose(o.loss, w.loss, rtol=1e-11)
