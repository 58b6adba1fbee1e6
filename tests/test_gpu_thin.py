"""Thin images: the configurations they take in place of the winners cache's
entry for any shape, and of entries whose tiles would lie mostly outside them,
on both sides of each line, as a plan of their own, in a batch by size, and in
a plain batch, whose one kernel per filter goes by all of its images; against
the oracle."""
import json

import numpy as np
import pytest

import datagen
import oracle
import paper_2407_11488_amd as C

from .gpu_util import say, to_dev, torch_cuda

pytestmark = pytest.mark.gpu

ANY = (32, 8, 4, 2, 1, 0, 4)
NARROW, TWO, FOUR = (16, 16, 2, 2, 1, 0, 4), (128, 2, 4, 1, 0, 0, 4), (128, 2, 4, 2, 1, 0, 4)
TWO_LARGE = (64, 4, 4, 2, 1, 0, 4)      # two rows under 11 x 11 and more


def _run(torch, runs):
    """Integer data: every output equals the oracle."""
    for (H, W, fh, fw), call in runs:
        inp, f = datagen.conv_problem(H, W, fh, fw, kind="int", seed_in=H + 11, seed_f=W)
        ref, _ = oracle.conv2d_f64(inp, f)
        out = call(to_dev(inp), to_dev(f))
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().astype(np.float64), ref), (H, W, fh, fw)


@pytest.mark.parametrize("H,W,want", [
    (5000, 1, NARROW), (64, 3, NARROW), (80, 64, NARROW), (80, 65, ANY), (160, 160, NARROW), (160, 161, ANY),
    (1, 5000, TWO), (2, 513, TWO), (3, 1025, FOUR), (4, 700, FOUR), (5, 700, ANY)])
@pytest.mark.parametrize("fh,fw", [(11, 11), (1, 9), (6, 3), (10, 15)])
def test_thin_plans(H, W, want, fh, fw):
    torch = torch_cuda()
    if want == TWO and H == 2 and fh == 11:
        want = TWO_LARGE
    plan = C.Plan(H, W, fh, fw)
    say(f"thin {H}x{W} f{fh}x{fw}: {plan.config}")
    assert tuple(plan.config) == want and plan.source == "tuned-other-shape"
    _run(torch, [((H, W, fh, fw), plan)])
    plan.close()


def test_large_thin_images_of_a_tuned_filter(tmp_path, monkeypatch):
    """Above 2^22 outputs the filter's winner (here of 64 x 64 tiles, waves of 64
    x 16) serves an image unless it covers too much outside it."""
    torch = torch_cuda()
    winner = (16, 16, 4, 4, 1, 0, 0)
    wp = tmp_path / "w.jsonl"
    wp.write_text("".join(json.dumps({"arch": "gfx950", "src": C.conv2d_kernel_hash(), "shape": s, "config": list(c),
                                      "ms": 1.0}) + "\n"
                          for s, c in (([4096, 4096, 9, 9], winner), ([-1, -1, 0, 0], ANY))))
    monkeypatch.setenv("CONV2D_WINNERS", str(wp))
    for (H, W), want in (((70000, 62), winner), ((140000, 31), NARROW), ((2, 2200000), TWO), ((20, 220000), ANY),
                         ((34, 130000), winner), ((2100, 2050), winner)):
        plan = C.Plan(H, W, 9, 9)
        say(f"large thin {H}x{W}: {plan.config}")
        assert H * W > 1 << 22 and tuple(plan.config) == want
        _run(torch, [((H, W, 9, 9), plan)])
        plan.close()


# (images, configurations by size, configuration of a plain batch): an image gets
# a kernel of its own by size where its shape saves more than a launch, 5 us
@pytest.mark.parametrize("shapes,by_size,plain", [
    ([(9000, 20), (200, 300), (2, 9000), (4000, 9), (12000, 33)], {NARROW, ANY}, NARROW),
    ([(300, 20), (200, 300), (2, 900), (400, 9)], {ANY}, NARROW),
    ([(1, 900000), (2, 900000)], {TWO, TWO_LARGE}, TWO)])
def test_thin_images_in_batches(shapes, by_size, plain):
    torch = torch_cuda()
    shapes = [s + (11, 11) for s in shapes]
    probs = [datagen.conv_problem(*s, kind="int", seed_in=k + 1, seed_f=k + 9) for k, s in enumerate(shapes)]
    refs = [oracle.conv2d_f64(i, f)[0] for i, f in probs]
    for flags, want in ((C.CONV2D_BATCH_BY_SIZE, by_size), (0, {plain})):
        b = C.Batch(shapes, flags)
        say(f"thin batch flags {flags}: {b.info['groups']}")
        assert {tuple(g["config"]) for g in b.info["groups"]} == want
        outs = b([to_dev(i) for i, _ in probs], [to_dev(f) for _, f in probs])
        torch.cuda.synchronize()
        for o, r, s in zip(outs, refs, shapes):
            assert np.array_equal(o.cpu().numpy().astype(np.float64), r), s
        b.close()
