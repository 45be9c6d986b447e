"""A context's first call of the forms that can do without the side stream makes none (it takes longer than the call gains), and calls
without and with it give the same bits."""
import threading

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _maps(seed, c=128):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.relu(torch.randn((8, 12, 12, c), generator=g, device="cuda"))


def _layers(seed, shapes):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    Ws, Hs = [], []
    for r, d in shapes:
        X = torch.randn((d, 600), generator=g, device="cuda").double()
        Ws.append(torch.randn((r, d), generator=g, device="cuda"))
        Hs.append((X @ X.T.contiguous() / 300).contiguous())
    return Ws, Hs


def _hessian(fobq, ctx, seed):
    ctx.set_hessian_mode(fobq.HESSIAN_INT8_SLICES)
    H = torch.full((1152, 1152), float("nan"), dtype=torch.float64, device="cuda")
    ctx.hessian_conv(_maps(seed), 3, 1, 1, H_out=H)
    assert ctx.hessian_form() == fobq.FORM_INT8_TAP_OFFSETS
    return [H]


def _batch(fobq, ctx, seed, shapes=((64, 147), (300, 64), (16, 256))):
    Ws, Hs = _layers(seed, shapes)
    return [t for o in ctx.quantize_layers_batched(Ws, Hs) for t in (o.codes, o.Q, o.perm, o.scales, o.zeros, o.loss)]


def _tall(fobq, ctx, seed):                  # one block of columns, and enough rows for the side stream
    return _batch(fobq, ctx, seed, ((15000, 40), (1000, 64)))


@pytest.mark.parametrize("call", [_hessian, _batch, _tall])
def test_a_first_call_makes_no_stream(call):
    import paper_2509_05576_amd as fobq
    said = []
    for nth in range(1, 100):
        with fobq.Ctx(0) as ctx:
            fobq.fobq_debug_fail_after(ctx.handle, nth)
            try:
                call(fobq, ctx, 1)
                break
            except fobq.FobqError as e:
                assert "injected" in str(e)
                said.append(str(e))
    assert 5 < nth < 99 and not any("side stream" in m or "event" in m for m in said), said


@pytest.mark.parametrize("call", [_hessian, _batch, _tall])
def test_calls_without_and_with_the_side_stream_agree(call):
    import paper_2509_05576_amd as fobq
    wrong = []

    def contexts(seed):                      # made and destroyed in turn; two calls without it, three with it
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for rep in range(3):
                    with fobq.Ctx(0) as ctx:
                        want = call(fobq, ctx, seed)
                        for _ in range(4):
                            got = call(fobq, ctx, seed)
                            torch.cuda.synchronize()
                            if not all(torch.equal(a, b) for a, b in zip(want, got)):
                                wrong.append((seed, rep))
        except Exception as e:               # noqa: BLE001
            wrong.append(repr(e))

    threads = [threading.Thread(target=contexts, args=(s,)) for s in (1, 2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
