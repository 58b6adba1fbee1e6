"""The tuner's unroll refinement after a sweep at unroll 1, where no point runs
on the matrix cores: the fastest points that can (even tiles, whole waves,
filters from 3 x 3) are timed with other unrolls although plain points are
faster. The command-line tuner sweeps at an unroll where they do. No GPU."""
import numpy as np
import pytest

import paper_2407_11488_amd as C
from paper_2407_11488_amd import tune


def _matrix(c):
    return c[2] % 2 == 0 and c[3] % 2 == 0 and c[0] * c[1] % 64 == 0


@pytest.mark.parametrize("shape,reaches", [((4096, 4096, 17, 17), True), ((1000, 1000, 3, 3), True),
                                           ((1000, 1000, 2, 9), False), ((1000, 1000, 9, 1), False)])
def test_refinement_reaches_the_matrix_path(shape, reaches):
    s = C.shape(*shape)
    rng = np.random.default_rng(3)
    table = {c: float(rng.uniform(1.0, 1.1)) * (1.5 if _matrix(c) else 1.0) for c in C.conv2d_space(s, 1, 0)}
    timed = set()

    def cost(c):
        timed.add(c)
        return table[c[:6] + (1,)] * (0.5 if _matrix(c) and c[6] != 1 else 1.0)

    o = C.conv2d_tune_defaults()
    o.refine_unroll = 1
    r = C.conv2d_tune_synthetic(s, cost, o)
    best_matrix = min((c for c in table if _matrix(c)), key=table.get)
    others = {c[:6] for c in timed if c[6] != 1}
    fastest = {c[:6] for c in sorted(table, key=table.get)[:10]}
    assert fastest <= others and len(others) == (20 if reaches else 10)
    if reaches:
        assert r.best.tuple()[:6] == best_matrix[:6] and r.best.tuple()[6] != 1
    else:
        assert r.best.tuple()[:6] == min(table, key=table.get)[:6]    # equal times: the smallest unroll


def test_command_line_sweep_uses_the_matrix_path(monkeypatch):
    seen = []
    monkeypatch.setattr(tune, "tune_one", lambda shape, a, results: seen.append(a.unroll) or {})
    monkeypatch.setattr(tune, "emit", lambda rep, path: None)
    assert tune.main(["--shape", "64", "64", "5", "5"]) == 0
    assert tune.main(["--shape", "64", "64", "5", "5", "--unroll", "1"]) == 0
    assert seen == [2, 1]
