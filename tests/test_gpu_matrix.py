"""The convolution kernel's matrix path (unroll other than 1, even tiles, whole
waves, filters from 3 x 3) on the GPU: its whole configuration space, filters
of one to four tap registers and of unequal sides, and the values on which a
matrix instruction could round or flush differently from a fused multiply-add
(subnormal products and sums, infinities, NaN). The oracle or the reference
kernel, which is plain fused multiply-adds, decides bit for bit."""
import numpy as np
import pytest

import datagen
import oracle
from tests.gpu_util import VEC, nan_like, precompile, run_config, say, to_dev, torch_cuda

pytestmark = pytest.mark.gpu

C = pytest.importorskip("paper_2407_11488_amd")

# (block_x, block_y, tile_x, tile_y, use_lds, filter_in_const, unroll)
CONFIGS = [(16, 16, 4, 4, 1, 0, 0), (32, 8, 4, 2, 1, 0, 4), (64, 1, 2, 2, 0, 1, 2), (16, 4, 8, 4, 1, 1, 4),
           (128, 2, 2, 8, 0, 0, 2), (64, 4, 8, 2, 0, 0, 0)]
SMALLEST_UNIT = 2.0 ** -149    # spacing of subnormal FP32 values


def _bits(t):
    return t.cpu().numpy().view(np.uint32)


def test_whole_matrix_space_integer_data_bitwise():
    """Every configuration that can take the path at unroll 2, on a ragged shape
    that spans several tiles: integer data makes every partial sum exact. The
    filter is large enough that most do take it also without LDS."""
    H, W, fh, fw = 70, 45, 11, 12
    s = C.shape(H, W, fh, fw)
    every = [c for c in C.conv2d_space(s, 2, -1) if c[2] % 2 == 0 and c[3] % 2 == 0 and c[0] * c[1] % 64 == 0]
    assert len(every) == 576
    # without the four that spill: scratch that a queue keeps upsets tests that fill the memory
    cfgs = [c for c in every if C.conv2d_lds_bytes(fh, fw, c) <= 163840 and
            not (c[0] * c[1] == 1024 and c[2] * c[3] == 64 and c[4] == 0)]
    precompile(C, s, cfgs, VEC, VEC)
    inp, f = datagen.conv_problem(H, W, fh, fw, kind="int", seed_in=8, seed_f=9)
    ref, _ = oracle.conv2d_f64(inp, f)
    di, df = to_dev(inp), to_dev(f)
    bad = []
    for k, c in enumerate(cfgs):
        if k % 100 == 0:
            say(f"matrix space: config {k}/{len(cfgs)} {c}")
        got = run_config(C, di, df, c).cpu().numpy().astype(np.float64)
        if not np.array_equal(got, ref):
            bad.append(c)
    assert not bad, f"{len(bad)} configurations differ, first {bad[:5]}"


@pytest.mark.parametrize("fh,fw", [(3, 3), (4, 7), (17, 17), (3, 33), (18, 34), (31, 31), (5, 63), (63, 4), (49, 50)])
def test_filters_equal_the_reference(fh, fw):
    """Filters with 2 to 62 interior columns, uniform data, ragged images."""
    H, W = 71, 205
    s = C.shape(H, W, fh, fw)
    cfgs = [c[:6] + (u,) for c in CONFIGS for u in (c[6], 2) if (u != 0 or (fh <= 31 and fh * fw <= 400)) and
            C.conv2d_config_check(s, c) == 0]
    precompile(C, s, cfgs, VEC, VEC)
    inp, f = datagen.conv_problem(H, W, fh, fw, seed_in=30 + fh, seed_f=40 + fw)
    di, df = to_dev(inp), to_dev(f)
    ref = _bits(C.reference(di, df, out=nan_like(H, W)))
    for c in cfgs:
        say(f"matrix {H}x{W} f{fh}x{fw} cfg {c}")
        assert np.array_equal(_bits(run_config(C, di, df, c)), ref), c


def _special(kind, H, W, fh, fw):
    inp, f = datagen.conv_problem(H, W, fh, fw, seed_in=55, seed_f=56)
    if kind == "products":           # normal factors, subnormal products and sums
        inp, f = inp * np.float32(2.0 ** -70), f * np.float32(2.0 ** -72)
    elif kind == "inputs":           # subnormal pixels, taps near 1
        inp = inp * np.float32(2.0 ** -130)
    elif kind == "taps":             # subnormal taps, pixels near 1
        f = f * np.float32(2.0 ** -130)
    elif kind == "edge":             # sums on both sides of the smallest normal value
        inp, f = inp * np.float32(2.0 ** -64), f * np.float32(2.0 ** -63)
    elif kind == "zeros":            # negative zeros among both
        inp[::2], f[::2] = np.float32(-0.0), np.float32(-0.0)
    else:                            # sums that overflow, infinities and NaN
        inp = inp * np.float32(2.0 ** 126)
        f = f * np.float32(2.0)
        inp[H // 2, W // 3], inp[3, W - 2], inp[H - 3, 4] = np.inf, -np.inf, np.nan
    return np.ascontiguousarray(inp, np.float32), np.ascontiguousarray(f, np.float32)


@pytest.mark.parametrize("fh,fw", [(3, 3), (17, 17), (5, 33)])
@pytest.mark.parametrize("kind", ["products", "inputs", "taps", "edge", "zeros", "nonfinite"])
def test_special_values_equal_the_reference(kind, fh, fw):
    """Configurations of the path and one of the batched kernel give the
    reference kernel's bits (any NaN for a NaN). The subnormal kinds are also
    held to the 64-bit sums: each of the fh * fw fused multiply-adds rounds by
    at most half a unit of 2^-149 there, and twice that covers sums up to twice
    the smallest normal value."""
    torch = torch_cuda()
    H, W = 66, 131
    inp, f = _special(kind, H, W, fh, fw)
    di, df = to_dev(inp), to_dev(f)
    assert np.array_equal(_bits(di).reshape(-1), inp.view(np.uint32).reshape(-1))
    ref_dev = C.reference(di, df, out=nan_like(H, W))
    torch.cuda.synchronize()
    ref = ref_dev.cpu().numpy()
    if kind in ("products", "inputs", "taps", "edge"):
        tiny = (ref != 0) & (np.abs(ref) < 2.0 ** -126)
        assert tiny.mean() > 0.01
        exact, _ = oracle.conv2d_f64(inp, f)
        assert np.abs(ref.astype(np.float64) - exact).max() <= fh * fw * SMALLEST_UNIT * max(
            1.0, np.abs(exact).max() / 2.0 ** -125)
    if kind == "nonfinite":
        assert np.isnan(ref).any() and np.isinf(ref).any()
    batch = C.Batch([(H, W, fh, fw)])
    got = {"batch": batch([di], [df])[0]}
    for c in CONFIGS:
        if C.conv2d_config_check(C.shape(H, W, fh, fw), c) == 0:
            got[c] = run_config(C, di, df, c)
    torch.cuda.synchronize()
    for c, o in got.items():
        say(f"{kind} f{fh}x{fw} {c}")
        o = o.cpu().numpy()
        assert np.array_equal(np.isnan(o), np.isnan(ref)), c
        fin = ~np.isnan(ref)
        assert np.array_equal(o.view(np.uint32)[fin], ref.view(np.uint32)[fin]), c
    batch.close()
