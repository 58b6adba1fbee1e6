"""Entries of a filter that were tuned on small sizes keep their place: a
small shape beside one takes it, before the entry for any shape, and a batch by
size does too; a winner tuned at 2^22 outputs or more still comes after."""
import json

import pytest

import paper_2407_11488_amd as C

from .gpu_util import say, torch_cuda

pytestmark = pytest.mark.gpu

ANY, NEAR = (32, 8, 4, 2, 1, 0, 4), (16, 16, 4, 2, 1, 0, 2)


# (the entry's shape, whether a 300 x 260 problem of its filter takes it)
@pytest.mark.parametrize("entry,taken", [
    ((1000, 1000, 11, 11), True), ((2047, 2049, 11, 11), True), ((2048, 2048, 11, 11), False),
    ((4096, 4096, 11, 11), False), ((0, 0, 11, 11), True), ((0, 3, 11, 11), True), ((0, 4, 11, 11), False)])
def test_a_small_entry_of_the_filter_comes_first(tmp_path, monkeypatch, entry, taken):
    torch_cuda()
    wp = tmp_path / "w.jsonl"
    wp.write_text("".join(json.dumps({"arch": "gfx950", "src": C.conv2d_kernel_hash(), "shape": list(s),
                                      "config": list(c), "ms": 1.0}) + "\n"
                          for s, c in ((entry, NEAR), ((-1, -1, 0, 0), ANY))))
    monkeypatch.setenv("CONV2D_WINNERS", str(wp))
    want = NEAR if taken else ANY
    plan = C.Plan(300, 260, 11, 11)
    say(f"entry {entry}: plan {plan.config} {plan.source}")
    assert tuple(plan.config) == want and plan.source == "tuned-other-shape"
    plan.close()
    batch = C.Batch([(300, 260, 11, 11)], C.CONV2D_BATCH_BY_SIZE)
    assert tuple(batch.info["groups"][0]["config"]) == want
    batch.close()
    other = C.Plan(300, 260, 5, 5)                  # a filter without an entry
    assert tuple(other.config) == ANY
    other.close()
