"""The winners cache's entry for any shape, (-1, -1, 0, 0): which plans take it
(filters without an entry, and small images whose filter was tuned at another
size), which do not, and their results against the oracle."""
import json

import numpy as np
import pytest

import datagen
import oracle
import paper_2407_11488_amd as C

from .gpu_util import TOL, say, to_dev, torch_cuda

pytestmark = pytest.mark.gpu

ANY, NINE, EXACT = (32, 8, 4, 2, 1, 0, 4), (64, 2, 4, 4, 1, 0, 1), (16, 16, 4, 2, 1, 0, 2)
HUGE = (128, 8, 8, 8, 1, 0, 1)          # 72 x 1032 floats of LDS and more: illegal for every filter
DEFAULT = (16, 16, 1, 1, 1, 1, 1)


def _winners(path, any_cfg):
    rows = [([4096, 4096, 9, 9], NINE), ([70, 90, 9, 9], EXACT)] + ([([-1, -1, 0, 0], any_cfg)] if any_cfg else [])
    path.write_text("".join(json.dumps({"arch": "gfx950", "src": C.conv2d_kernel_hash(), "shape": s, "config": list(c),
                                        "ms": 1.0}) + "\n" for s, c in rows))


# (shape, the configuration it takes with the entry, with an illegal entry, without one)
@pytest.mark.parametrize("shape,with_any,illegal,without", [
    ((70, 90, 9, 9), EXACT, EXACT, EXACT),             # its own entry
    ((71, 90, 9, 9), ANY, NINE, NINE),                 # small image, tuned filter
    ((2047, 2049, 9, 9), ANY, NINE, NINE),             # 2^22 - 1 outputs
    ((2048, 2048, 9, 9), NINE, NINE, NINE),            # 2^22 outputs
    ((33, 65, 5, 8), ANY, DEFAULT, DEFAULT),           # filter without an entry
    ((2050, 2050, 1, 2), ANY, DEFAULT, DEFAULT)])
def test_entry_for_any_shape(tmp_path, monkeypatch, shape, with_any, illegal, without):
    torch = torch_cuda()
    H, W, fh, fw = shape
    inp, f = datagen.conv_problem(H, W, fh, fw, seed_in=91, seed_f=92)
    ref, s = oracle.conv2d_f64(inp, f)
    d_in, d_f = to_dev(inp), to_dev(f)
    for any_cfg, want in ((ANY, with_any), (HUGE, illegal), (None, without)):
        wp = tmp_path / "w.jsonl"
        _winners(wp, any_cfg)
        monkeypatch.setenv("CONV2D_WINNERS", str(wp))
        plan = C.Plan(H, W, fh, fw)
        say(f"any-shape entry {any_cfg}: {shape} takes {plan.config} ({plan.source})")
        assert tuple(plan.config) == want
        assert plan.source == ("tuned" if want == EXACT else "default" if want == DEFAULT else "tuned-other-shape")
        out = plan(d_in, d_f)
        torch.cuda.synchronize()
        assert oracle.normalized_error(out.cpu().numpy(), ref, s) <= TOL
        plan.close()
    assert np.isfinite(ref).all()
