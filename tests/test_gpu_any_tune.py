"""The tuner's choice of the winners cache's entry for any shape: the candidate
of the lowest geometric mean is stored and taken by a plan afterwards; the
current entry stays when it is as good."""
import json

import pytest

import paper_2407_11488_amd as C
from paper_2407_11488_amd import workloads

from .gpu_util import say, torch_cuda

pytestmark = pytest.mark.gpu

CANDIDATES = ((32, 8, 4, 2, 1, 0, 4), (16, 16, 1, 1, 1, 0, 1), (64, 4, 4, 4, 1, 0, 2))


def test_entry_for_any_shape_is_chosen_stored_and_taken(tmp_path, monkeypatch):
    torch_cuda()
    wp = tmp_path / "w.jsonl"
    r = workloads.any_shape_tune(((11, 11), (1, 6)), ((300, 260), (512, 700)), CANDIDATES, winners=str(wp), log=say)
    say(json.dumps(r))
    assert [c["config"] for c in r["candidates"]][0] == r["chosen"]
    assert 1.0 <= r["to_best"]["gmean"] <= r["to_best"]["worst"] and len(r["chosen_ms"]) == 4
    got, ms = C.conv2d_cache_lookup(str(wp), "gfx950", C.shape(-1, -1, 0, 0))
    assert list(got.tuple()) == r["chosen"] and ms == pytest.approx(r["gmean_ms"], rel=1e-3)
    monkeypatch.setenv("CONV2D_WINNERS", str(wp))
    plan = C.Plan(300, 300, 7, 7)
    assert list(plan.config) == r["chosen"] and plan.source == "tuned-other-shape"
    plan.close()
    kept = next(c for c in CANDIDATES if list(c) != r["chosen"])
    C.conv2d_cache_store(str(wp), "gfx950", C.shape(-1, -1, 0, 0), kept, 1.0)
    again = workloads.any_shape_tune(((11, 11),), ((300, 260),), CANDIDATES, tie_rel=1e9, winners=str(wp), store=False,
                                     log=say)
    assert again["chosen"] == list(kept)
