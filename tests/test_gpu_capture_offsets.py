"""A convolution's Hessian by tap offsets on a stream under capture: everything stays on that stream, and every replay gives the same H."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_hessian_by_offsets_in_a_graph():
    import paper_2509_05576_amd as fobq
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    c, k = 128, 3
    maps = [torch.relu(torch.randn((8, 10, 10, c), generator=g, device="cuda")) for _ in range(2)]
    buf = maps[0].clone()
    H = torch.zeros((c * k * k, c * k * k), dtype=torch.float64, device="cuda")
    s = torch.cuda.Stream()
    with fobq.Ctx(0, stream=s.cuda_stream) as ctx:
        ctx.set_hessian_mode(fobq.HESSIAN_INT8_SLICES)
        want = []
        with torch.cuda.stream(s):
            for m in maps:                       # eager: the scratch is there afterwards
                buf.copy_(m)
                ctx.hessian_conv(buf, k, 1, 1, H_out=H)
                s.synchronize()
                want.append(H.clone())
        assert ctx.hessian_form() == fobq.FORM_INT8_TAP_OFFSETS
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            ctx.hessian_conv(buf, k, 1, 1, H_out=H)
        for i in (0, 1, 1, 0):
            buf.copy_(maps[i])
            H.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(H, want[i])
