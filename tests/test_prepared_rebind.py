"""A prepared call after rebind(): every way to launch it goes to the new stream, a `launch` that was fetched before
included, and a subclass's own launch() is the one that runs."""
import pytest

from paper_2101_05615_amd import workloads as wl


def test_a_fetched_launch_follows_and_subclasses_count(monkeypatch):
    """Host side: addresses of CPU tensors, nothing is launched."""
    import torch
    from paper_2101_05615_amd import qgemm as q

    class Weights:
        handle = None

    class Counted(q.PreparedGemm):
        def __init__(self):
            t = torch.zeros(16, dtype=torch.uint8)
            p = q.RequantParams(0, None, None, 1, 0, 0)
            self._prepare(0, (t,), t, Weights, t, None, p, (1, 16, 16, 0))
            self.calls = 0

        def launch(self):
            self.calls += 1
            return super().launch

    streams = iter([64, 128, 192])
    monkeypatch.setattr(q, "_stream", lambda: next(streams))
    c = Counted()
    before = c.launch()
    assert c.rebind() is c and c.rebind().launch().__self__ is before.__self__
    assert c.calls == 2


def test_a_call_without_arguments_is_refused():
    from paper_2101_05615_amd import qgemm as q
    with pytest.raises(q.QGemmError):   # no weights: refused before anything is enqueued
        q._binding.Call().launch()
    for args in ((), (0,), (9,) + (0,) * 14, (0,) + (0,) * 15, (0, "a") + (0,) * 13):
        with pytest.raises(TypeError):
            q._binding.Call()._set(*args)


@pytest.mark.gpu
def test_a_fetched_launch_inside_a_capture():
    import torch
    from paper_2101_05615_amd import qgemm as q
    c = wl.random_gemm(3, 70, 96, 200)
    A, B = torch.from_numpy(c.A).cuda(), q.pack_b(torch.from_numpy(c.B).cuda(), c.b_zp)
    bias, scales = torch.from_numpy(c.bias).cuda(), torch.from_numpy(c.scales).cuda()
    want = q.gemm_u8s8_requant(A, c.a_zp, B, bias, scales, c.c_zp, c.relu)
    out = torch.zeros_like(want)
    pg = q.PreparedGemm(A, c.a_zp, B, bias, scales, c.c_zp, c.relu, out)
    run = pg.launch
    run()
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    graph = torch.cuda.CUDAGraph()
    out.zero_()
    with torch.cuda.graph(graph):
        pg.rebind()
        run()
    pg.rebind()
    torch.cuda.synchronize()
    assert not bool(out.any())   # recorded, not run
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        A.add_(1)
        run()                    # on the stream of now again
        want = q.gemm_u8s8_requant(A, c.a_zp, B, bias, scales, c.c_zp, c.relu)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    s = torch.cuda.Stream()
    out.zero_()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        pg.rebind()
    run()
    s.synchronize()
    assert torch.equal(out, want)
