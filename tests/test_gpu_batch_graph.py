"""Which batches run as one graph launch, and that graph's runs: many branches,
several runs with other work between them, and new buffers (the descriptors
uploaded again ahead of the graph). The reference kernel and the same batch
planned without a graph decide bit for bit."""
import pytest

from tests.gpu_util import say, torch_cuda
from tests.test_gpu_batch_launch import _problem

pytestmark = pytest.mark.gpu

C = pytest.importorskip("paper_2407_11488_amd")

ELEVEN = [(1, 1), (3, 3), (5, 5), (7, 7), (9, 9), (11, 11), (2, 6), (6, 2), (17, 17), (31, 31), (4, 4)]
MANY = [(40 + 13 * k, 70 - 5 * k, fh, fw) for k, (fh, fw) in enumerate(ELEVEN)]


# The line: 25 us of kernel time per group, taken as operations at 65 TFLOP/s.
@pytest.mark.parametrize("shapes,graph", [
    ([(130, 131, 5, 5)], False),
    ([(130, 131, 5, 5), (200, 77, 3, 3), (64, 129, 17, 17), (33, 300, 9, 9)], False),
    ([(2500, 2501, 17, 17), (1100, 900, 9, 9)], True),
    ([(1676, 1677, 17, 17)], False),          # 24.99 us, one group
    ([(1677, 1677, 17, 17)], True),           # 25.01 us
    ([(1677, 1677, 17, 17), (8, 8, 3, 3)], False),
    ([(1677, 1677, 17, 17), (1677, 1677, 17, 17), (8, 8, 3, 3)], True)])
def test_which_batches_run_as_a_graph(shapes, graph):
    torch_cuda()
    for flags, want in ((0, graph), (C.CONV2D_BATCH_NO_GRAPH, False)):
        b = C.Batch(shapes, flags)
        say(f"graph choice {shapes} flags {flags}: {b.info['graph']}")
        assert b.info["graph"] == want
        b.close()


@pytest.mark.parametrize("shapes,groups", [
    (MANY + [(3100, 3100, 31, 31)], 11),
    ([(700, 701, 3, 3), (300, 901, 5, 5), (513, 257, 9, 9), (3500, 3501, 17, 17), (64, 2000, 17, 17)], 4)])
def test_graph_runs_repeat_and_take_new_buffers(shapes, groups):
    torch = torch_cuda()
    ins, fs = zip(*[_problem(torch, s, 300 + 10 * p) for p, s in enumerate(shapes)])
    refs = [C.reference(x, f).view(torch.int32) for x, f in zip(ins, fs)]
    new = lambda: [torch.full((H, W), float("nan"), device="cuda") for H, W, _, _ in shapes]  # noqa: E731
    batch, plain = C.Batch(shapes), C.Batch(shapes, C.CONV2D_BATCH_NO_GRAPH)
    assert batch.info["graph"] and batch.info["n_groups"] == groups and not plain.info["graph"]
    outs, other = new(), new()
    for rep in range(5):
        say(f"graph run {rep} of {groups} branches")
        if rep == 2:
            outs = new()                                   # other buffers from here on
        for o in outs + other:
            o.fill_(float("nan"))                          # eager work between runs
        torch.cuda.synchronize()
        batch(ins, fs, outs)
        plain(ins, fs, other)
        torch.cuda.synchronize()
        for o, p, r, s in zip(outs, other, refs, shapes):
            assert torch.equal(o.view(torch.int32), r), (rep, s)
            assert torch.equal(p.view(torch.int32), r), (rep, s)
    batch.close()
    plain.close()
