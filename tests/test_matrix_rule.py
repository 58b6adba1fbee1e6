"""Which builds of the convolution kernel use the matrix cores: all that can
with the tile in LDS, but for 2 x 2 outputs under tall filters; without LDS
those whose arithmetic outweighs the loads of the taps. Both sides of each
line, in the compiled code. No GPU needed."""
import subprocess

import pytest

import paper_2407_11488_amd as C

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


# (fh, fw), (tile_x, tile_y, use_lds, unroll), on the matrix cores
@pytest.mark.parametrize("f,t,matrix", [
    ((3, 3), (2, 2, 1, 2), True), ((3, 3), (2, 2, 1, 1), False), ((2, 9), (4, 4, 1, 2), False),
    ((12, 3), (2, 2, 1, 4), True), ((13, 3), (2, 2, 1, 4), False), ((13, 3), (2, 2, 1, 0), False),
    ((13, 3), (4, 2, 1, 4), True),
    ((9, 9), (2, 2, 0, 2), False), ((15, 15), (2, 2, 0, 2), False), ((15, 15), (2, 2, 0, 0), True),
    ((14, 15), (2, 2, 0, 0), False),
    ((10, 11), (4, 2, 0, 2), False), ((11, 11), (4, 2, 0, 2), True), ((11, 12), (2, 4, 0, 4), True),
    ((8, 9), (8, 2, 0, 2), False), ((9, 9), (8, 2, 0, 2), True), ((9, 9), (2, 8, 0, 0), True),
    ((5, 5), (2, 8, 0, 2), False), ((5, 5), (4, 4, 0, 2), True), ((5, 5), (4, 4, 0, 0), False),
    ((12, 3), (4, 4, 0, 2), True), ((13, 3), (4, 4, 0, 2), False)])
def test_builds_on_the_matrix_cores(f, t, matrix):
    cfg = (16, 16, t[0], t[1], t[2], 0, t[3])
    for path in (C.conv2d_compile(C.shape(4096, 4096, *f), cfg, 4, 4),
                 C.conv2d_compile_batch(C.shape(4096, 4096, *f), cfg)):
        isa = subprocess.run([OBJDUMP, "-d", path], capture_output=True, text=True).stdout
        assert ("v_mfma_f32_4x4x1" in isa) == matrix
