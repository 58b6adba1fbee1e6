"""A hotspot plan tells a winner that was tuned with the current kernel from one
of an older revision (which it still takes)."""
import json

import pytest

import paper_2407_11488_amd as C

from .gpu_util import torch_cuda


@pytest.mark.gpu
@pytest.mark.parametrize("src,want", [(None, "tuned"), ("0000000000000000", "tuned-older-kernel")])
def test_source_of_a_grids_own_entry(tmp_path, monkeypatch, src, want):
    torch_cuda()
    cfg = (64, 4, 2, 4, 4, 1, 1)
    wp = tmp_path / "hs.jsonl"
    wp.write_text(json.dumps({"arch": "gfx950", "src": src or C.hotspot_kernel_hash(), "shape": [300, 200],
                              "config": list(cfg), "ms": 1.0}) + "\n")
    monkeypatch.setenv("HOTSPOT_WINNERS", str(wp))
    plan = C.Hotspot(300, 200)
    assert (plan.source, tuple(plan.config)) == (want, cfg)
    plan.close()
    other = C.Hotspot(301, 200)
    assert (other.source, tuple(other.config)) == ("tuned-other-grid", cfg)
    other.close()
