"""The batched path's two ways of running: a small batch's kernels launched one
after another, a large batch's graph. Both equal the reference kernel bit for
bit, also on other buffers in a later run, and beside the same batch planned
without a graph."""
import pytest

import paper_2407_11488_amd as C

from .gpu_util import say, torch_cuda

pytestmark = pytest.mark.gpu


def _problem(torch, shape, seed):
    H, W, fh, fw = shape
    st = torch.cuda.current_stream().cuda_stream
    x = torch.empty((H + fh - 1, W + fw - 1), dtype=torch.float32, device="cuda")
    f = torch.empty((fh, fw), dtype=torch.float32, device="cuda")
    C.conv2d_fill_uniform(x.data_ptr(), x.numel(), seed, 0, st)
    C.conv2d_fill_uniform(f.data_ptr(), f.numel(), seed + 1, 0, st)
    return x, f


# one image; a few images of four filters; images large enough for the graph
@pytest.mark.parametrize("shapes", [[(130, 131, 5, 5)],
                                    [(130, 131, 5, 5), (200, 77, 3, 3), (64, 129, 17, 17), (33, 300, 9, 9)],
                                    [(2500, 2501, 17, 17), (1100, 900, 9, 9)]], ids=["one", "small", "large"])
@pytest.mark.parametrize("flags", [0, C.CONV2D_BATCH_BY_SIZE])
def test_batch_equals_reference_however_it_is_launched(shapes, flags):
    torch = torch_cuda()
    say(f"batch launch {shapes} flags {flags}")
    plans = [C.Batch(shapes, flags), C.Batch(shapes, flags | C.CONV2D_BATCH_NO_GRAPH)]
    for seed in (500, 600):
        ins, fs = zip(*[_problem(torch, s, seed + 10 * p) for p, s in enumerate(shapes)])
        refs = [C.reference(x, f) for x, f in zip(ins, fs)]
        for b in plans:
            outs = [torch.full((H, W), float("nan"), device="cuda") for H, W, _, _ in shapes]
            b(list(ins), list(fs), outs)
            torch.cuda.synchronize()
            for o, r, s in zip(outs, refs, shapes):
                assert torch.equal(o.view(torch.int32), r.view(torch.int32)), s
    for b in plans:
        b.close()
