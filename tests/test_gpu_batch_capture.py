"""Batch runs recorded into a captured graph. A recorded run has not happened,
so the next run on the same buffers works for itself; a replay works on the
buffers that were recorded, whatever the plan ran on in between, and on no
others. Several replays, with other eager runs between, each against the
reference kernel bit for bit."""
import pytest

from tests.gpu_util import say, torch_cuda

pytestmark = pytest.mark.gpu

C = pytest.importorskip("paper_2407_11488_amd")

SMALL = [(130, 131, 5, 5), (200, 77, 3, 3), (64, 129, 17, 17), (33, 300, 9, 9)]
LARGE = [(2500, 2501, 17, 17), (1100, 900, 9, 9)]


class _Buffers:
    def __init__(self, torch, shapes, seed):
        st = torch.cuda.current_stream().cuda_stream
        self.ins, self.fs, self.refs = [], [], []
        for k, (H, W, fh, fw) in enumerate(shapes):
            x = torch.empty((H + fh - 1, W + fw - 1), device="cuda")
            f = torch.empty((fh, fw), device="cuda")
            C.conv2d_fill_uniform(x.data_ptr(), x.numel(), seed + 2 * k, 0, st)
            C.conv2d_fill_uniform(f.data_ptr(), f.numel(), seed + 2 * k + 1, 0, st)
            self.ins.append(x)
            self.fs.append(f)
            self.refs.append(C.reference(x, f))
        self.outs = [torch.empty_like(r) for r in self.refs]
        self.forget()

    def forget(self):
        for o in self.outs:
            o.fill_(float("nan"))

    def done(self, torch):
        torch.cuda.synchronize()
        return all(torch.equal(o.view(torch.int32), r.view(torch.int32)) for o, r in zip(self.outs, self.refs))

    def untouched(self, torch):
        torch.cuda.synchronize()
        return all(bool(torch.isnan(o).all()) for o in self.outs)


@pytest.mark.parametrize("shapes", [SMALL, LARGE], ids=["small", "large"])
@pytest.mark.parametrize("flags", [0, C.CONV2D_BATCH_NO_GRAPH, C.CONV2D_BATCH_BY_SIZE])
def test_recorded_runs_keep_their_buffers(shapes, flags):
    torch = torch_cuda()
    a, b = _Buffers(torch, shapes, 900), _Buffers(torch, shapes, 950)
    batch = C.Batch(shapes, flags)
    torch.cuda.synchronize()

    def run(x):
        return batch(x.ins, x.fs, x.outs)

    say(f"batch capture flags {flags}: the plan's first run is recorded")
    on_a = torch.cuda.CUDAGraph()
    with torch.cuda.graph(on_a):
        run(a)
    assert a.untouched(torch)
    run(a)                       # on the buffers just recorded, before any replay
    assert a.done(torch)
    run(b)
    assert b.done(torch)
    for rep in range(3):
        say(f"replay {rep}")
        a.forget()
        b.forget()
        torch.cuda.synchronize()
        on_a.replay()
        assert a.done(torch) and b.untouched(torch)
        run(b)                   # the plan's own table still belongs to b
        assert b.done(torch)
    say("a second recording, on the buffers of the last run")
    on_b = torch.cuda.CUDAGraph()
    with torch.cuda.graph(on_b):
        run(b)
        run(b)
    run(a)
    for rep in range(2):
        a.forget()
        b.forget()
        torch.cuda.synchronize()
        on_b.replay()
        assert b.done(torch) and a.untouched(torch)
        on_a.replay()
        assert a.done(torch)
    del on_a, on_b
    batch.close()
