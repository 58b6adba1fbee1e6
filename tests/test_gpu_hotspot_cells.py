"""The hotspot kernel on both sides of the tile size up to which a step's last
FMA writes the cells in place (8 cells per thread): bit for bit the one-step
reference, for odd and even step counts and more than one launch."""
import numpy as np
import pytest

import datagen
from tests.gpu_util import torch_cuda

STRESS = (0.2, 0.5, 0.75, 0.05, 0.25)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", [(32, 8, 1, 1, 1, 1, 1), (32, 16, 2, 4, 8, 1, 1), (32, 16, 2, 4, 8, 0, 1),
                                 (64, 8, 4, 2, 6, 1, 0), (128, 4, 2, 4, 4, 0, 0), (16, 16, 4, 4, 8, 1, 1)])
@pytest.mark.parametrize("rows,cols,steps", [(1, 1, 3), (300, 500, 17), (49, 113, 8)])
def test_cells_match_the_reference(cfg, rows, cols, steps):
    C = pytest.importorskip("paper_2407_11488_amd")
    torch = torch_cuda()
    temp = torch.from_numpy(datagen.uniform_pm1(71, rows * cols).reshape(rows, cols)).cuda()
    power = torch.from_numpy(datagen.uniform_pm1(72, rows * cols).reshape(rows, cols)).cuda()
    ref = C.reference_hotspot(temp, power, steps, STRESS)
    out = torch.full((rows, cols), float("nan"), device="cuda")
    plan = C.Hotspot(rows, cols, cfg)
    plan(temp, power, steps, STRESS, out=out)
    torch.cuda.synchronize()
    plan.close()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.cpu().numpy().view(np.uint32))
