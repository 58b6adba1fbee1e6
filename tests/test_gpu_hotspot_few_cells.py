"""The hotspot kernel on both sides of the smallest tile that takes a step's
last FMA in place (4 cells per thread): bit for bit the one-step reference."""
import numpy as np
import pytest

import datagen
from tests.gpu_util import torch_cuda

STRESS = (0.2, 0.5, 0.75, 0.05, 0.25)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", [(32, 16, 2, 1, 4, 1, 1), (16, 16, 1, 2, 6, 0, 0), (64, 8, 1, 2, 6, 1, 1),
                                 (16, 16, 2, 2, 4, 1, 1), (64, 4, 1, 4, 3, 0, 1), (64, 8, 4, 1, 3, 1, 0)])
@pytest.mark.parametrize("rows,cols,steps", [(300, 500, 17), (49, 113, 8)])
def test_few_cells_match_the_reference(cfg, rows, cols, steps):
    C = pytest.importorskip("paper_2407_11488_amd")
    torch = torch_cuda()
    if C.hotspot_config_check(C.hotspot_shape(rows, cols), cfg) != 0:
        pytest.fail(f"not a legal configuration: {cfg}")
    temp = torch.from_numpy(datagen.uniform_pm1(71, rows * cols).reshape(rows, cols)).cuda()
    power = torch.from_numpy(datagen.uniform_pm1(72, rows * cols).reshape(rows, cols)).cuda()
    ref = C.reference_hotspot(temp, power, steps, STRESS)
    out = torch.full((rows, cols), float("nan"), device="cuda")
    plan = C.Hotspot(rows, cols, cfg)
    plan(temp, power, steps, STRESS, out=out)
    torch.cuda.synchronize()
    plan.close()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.cpu().numpy().view(np.uint32))
