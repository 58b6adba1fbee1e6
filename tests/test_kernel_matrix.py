"""The convolution kernel's matrix path on the CPU (tests/emu): the tunable
kernel source with the matrix instruction emulated (each lane's four fused
multiply-adds, the taps taken from the broadcast block), under
AddressSanitizer. Filters at the edges of a tap register (16 interior columns:
filter widths 16, 17, 18, 33, 34), the smallest filters the path takes, block
rows that never all lie inside the filter at once, and images that end inside a
2 x 2 block or leave whole waves outside. No GPU needed."""
import concurrent.futures as cf
import hashlib
import os
import subprocess

import numpy as np
import pytest

import datagen
import oracle

from .test_kernel_emu import BIN_DIR, CXX, EMU, KERNEL, run

# (H, W, fh, fw) and the configurations (block_x, block_y, tile_x, tile_y,
# use_lds, filter_in_const, unroll) run on it.
CASES = [
    ((9, 131, 3, 3), [(64, 1, 2, 2, 0, 0, 0), (32, 2, 4, 2, 1, 1, 2)]),
    ((7, 61, 4, 16), [(16, 4, 4, 4, 1, 0, 4), (64, 1, 2, 2, 0, 1, 2)]),
    ((5, 70, 3, 17), [(16, 4, 8, 2, 0, 0, 2), (32, 4, 2, 4, 1, 0, 0)]),
    ((11, 35, 17, 18), [(16, 4, 4, 4, 0, 0, 2)]),
    ((3, 33, 5, 33), [(64, 1, 4, 2, 1, 0, 2)]),
    ((2, 18, 3, 34), [(32, 2, 2, 8, 0, 0, 0)]),
    ((19, 37, 9, 5), [(16, 4, 2, 8, 1, 0, 2), (16, 8, 8, 8, 0, 0, 4)]),
    ((1, 1, 3, 3), [(64, 1, 8, 2, 0, 0, 4)]),
]


def _build(cfg, fh, fw):
    bx, by, tx, ty, lds, fc, un = cfg
    defs = dict(BX=bx, BY=by, TX=tx, TY=ty, USE_LDS=lds, FCONST=fc, UNROLL=un, FH=fh, FW=fw, VIN=4, VOUT=4)
    srcs = [KERNEL] + [os.path.join(EMU, n) for n in ("emu_direct.cpp", "emu_direct_matrix.cpp", "emu_matrix.h",
                                                      "hip_emu.h")]
    key = hashlib.sha1(("".join(open(p).read() for p in srcs) + repr(sorted(defs.items()))).encode()).hexdigest()[:16]
    os.makedirs(BIN_DIR, exist_ok=True)
    exe = os.path.join(BIN_DIR, f"emum_{key}")
    if not os.path.exists(exe):
        cmd = [CXX, "-std=c++20", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
               "-fno-omit-frame-pointer", *[f"-DCONV_{k}={v}" for k, v in defs.items()],
               os.path.join(EMU, "emu_direct_matrix.cpp"), "-o", exe + f".{os.getpid()}.tmp", "-lpthread"]
        subprocess.run(cmd, check=True, capture_output=True)
        os.replace(exe + f".{os.getpid()}.tmp", exe)
    return exe


@pytest.fixture(scope="module")
def binaries():
    jobs = [(cfg, shape[2], shape[3]) for shape, cfgs in CASES for cfg in cfgs]
    with cf.ThreadPoolExecutor(os.cpu_count() or 4) as ex:
        return dict(zip(jobs, ex.map(lambda j: _build(*j), jobs)))


@pytest.mark.parametrize("shape,cfgs", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_matrix_path_exact_on_integers(binaries, shape, cfgs, tmp_path):
    H, W, fh, fw = shape
    inp, f = datagen.conv_problem(H, W, fh, fw, kind="int", seed_in=H + 7, seed_f=W)
    ref, _ = oracle.conv2d_f64(inp, f)
    for cfg in cfgs:
        got = run(binaries[(cfg, fh, fw)], inp, f, H, W, str(tmp_path))
        assert np.array_equal(got.astype(np.float64), ref), cfg


def test_infinity_reaches_only_its_outputs(binaries, tmp_path):
    """An infinite input pixel makes exactly the outputs whose window holds it
    non-finite (no product with a padding zero is added to others)."""
    (H, W, fh, fw), cfgs = CASES[6]
    inp, f = datagen.conv_problem(H, W, fh, fw, kind="int", seed_in=3, seed_f=4)
    f[f == 0] = 1.0
    inp[11, 20] = np.inf
    want = np.ones((H, W), bool)
    want[11 - fh + 1:12, 20 - fw + 1:21] = False
    for cfg in cfgs:
        got = run(binaries[(cfg, fh, fw)], inp, f, H, W, str(tmp_path))
        assert np.array_equal(np.isfinite(got), want), cfg
