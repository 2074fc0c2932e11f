"""The split-operand conv launch (conv mfma 2 and 3 at unroll depth 1, 3x3
filters, whole groups of eight channels) on the GPU.

* Small-integer inputs: bit-exact against the oracle (every plane product and
  partial sum is an integer below 2**24), outputs all written, nothing past
  the end; shapes with ragged K, odd image sizes, padding 0 and 2, bands
  across images and reduction splits.
* Precision: its error against the fp64 oracle is no larger than that of the
  fp32-MFMA program of the same tile (a deeper unroll), on inputs of several
  scales.  Both errors are sums of rounding errors of the same kind, so the
  ratio of their 2-norms over thousands of outputs is stable; 1.1 leaves room
  for its spread.
* Values the bf16 planes cannot hold (infinities, NaN, floats that round past
  the largest bf16, tiles of tiny values): the same outputs as the fp32
  program, non-finite where and as it has them; rectangles, bands over several
  images with a reduction split and ragged channels, stride 2.
"""
import numpy as np
import pytest

import synthdata
from oracle import kernels as ok

pytestmark = pytest.mark.gpu

CANARY = 12345.0
TAIL = 64

# shape, tile knobs (tk, th, tw, tc, ks, mfma)
POINTS = [
    ((2, 32, 28, 28, 64, 3, 3, 1, 1), (64, 16, 16, 4, 1, 2)),
    ((2, 16, 30, 33, 70, 3, 3, 1, 1), (64, 8, 16, 8, 1, 2)),
    ((1, 8, 20, 18, 33, 3, 3, 1, 0), (32, 16, 16, 4, 1, 2)),
    ((1, 24, 19, 17, 40, 3, 3, 1, 2), (32, 8, 16, 8, 1, 2)),
    ((3, 64, 14, 14, 96, 3, 3, 1, 1), (64, 16, 8, 4, 8, 3)),
    ((5, 16, 9, 9, 64, 3, 3, 1, 1), (64, 16, 16, 4, 2, 3)),
    ((2, 40, 13, 11, 48, 3, 3, 1, 1), (32, 16, 8, 4, 1, 3)),
    ((1, 48, 12, 40, 32, 3, 3, 1, 1), (32, 4, 64, 4, 2, 3)),
    ((1, 16, 18, 18, 32, 3, 3, 2, 1), (32, 16, 8, 4, 1, 3)),
    ((2, 32, 10, 20, 40, 3, 3, 2, 1), (32, 8, 16, 4, 2, 3)),
]


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2406_20037_amd import _lib
    return torch, _lib


def points(L, sh, knobs):
    """(space, the split-operand schedule, an fp32-MFMA schedule of its tile)."""
    tk, th, tw, tc, ks, mfma = knobs
    space = L.Space(L.DS_OP_CONV2D_NCHW, sh)
    kn = dict(tk=tk, th=th, tw=tw, tc=tc, unroll=0, lds=1, ks=ks, mfma=mfma, vec=1)
    split = space.sched_of(**kn)
    if not space.valid(split.index()):
        split = space.sched_of(**dict(kn, vec=4))
    info = space.kernel_info(split.index())
    assert info["params"][5:] == [1], (sh, kn, info)
    # a deeper unroll of the same tile and split runs on fp32 MFMAs
    for ch in (8, 16, 32):
        for unroll in (16, 64, 512):
            for vec in (4, 1):
                f32 = space.sched([vals.index(v) if v in vals else -1 for vals, v in zip(
                    space.values, dict(kn, tc=ch, unroll=unroll, vec=vec).values())])
                if -1 not in f32.index() and space.valid(f32.index()) and (
                        space.kernel_info(f32.index())["params"][5:] != [1]):
                    return space, split, f32
    raise AssertionError(sh)


def run(torch, L, s, x, w, n):
    y = torch.full((n + TAIL,), float("nan"), device="cuda:0")
    y[n:] = CANARY
    L.kernel_run(L.DS_OP_CONV2D_NCHW, s, x, w, y)
    torch.cuda.synchronize()
    assert bool((y[n:] == CANARY).all()), "write past the end of y"
    return y[:n].cpu().numpy().astype(np.float64)


def dev(torch, a, shift=0):
    buf = torch.zeros(a.size + shift, dtype=torch.float32, device="cuda:0")
    buf[shift:] = torch.from_numpy(np.ascontiguousarray(a).ravel()).to("cuda:0")
    return buf[shift:]


IDS = ["x".join(map(str, p[0])) for p in POINTS]


@pytest.mark.parametrize("sh,knobs", POINTS, ids=IDS)
def test_split_bit_exact_on_integers(env, sh, knobs):
    torch, L = env
    _, split, _ = points(L, sh, knobs)
    x, w = synthdata.conv_inputs(sh, "int")
    ref = ok.conv2d_f64(x, w, sh).ravel()
    for shift in (0, 1):
        print("conv split int", sh, knobs, shift, flush=True)
        got = run(torch, L, split, dev(torch, x, shift), dev(torch, w, shift), ref.size)
        assert np.array_equal(got, ref)


@pytest.mark.parametrize("scale", [1.0, 1e-12, 1e15])
@pytest.mark.parametrize("sh,knobs", POINTS, ids=IDS)
def test_split_no_less_precise_than_fp32_mfma(env, sh, knobs, scale):
    torch, L = env
    _, split, f32 = points(L, sh, knobs)
    x, w = synthdata.conv_inputs(sh, "he")
    x = (x * np.float32(scale)).astype(np.float32)
    ref = ok.conv2d_f64(x, w, sh).ravel()
    xd, wd = dev(torch, x), dev(torch, w)
    print("conv split precision", sh, knobs, scale, flush=True)
    e = [np.linalg.norm(run(torch, L, s, xd, wd, ref.size) - ref) for s in (split, f32)]
    print(f"  error {e[0] / np.linalg.norm(ref):.3g}, fp32 MFMA {e[1] / np.linalg.norm(ref):.3g}")
    assert e[0] <= 1.1 * e[1]


# a rectangle, a band over three images in eight splits with ragged channels, and
# one of stride 2
SPECIAL_POINTS = [POINTS[0], POINTS[4], POINTS[9]]


@pytest.mark.parametrize("kind", ["inf", "nan", "max", "tiny", "winf"])
@pytest.mark.parametrize("sh,knobs", SPECIAL_POINTS,
                         ids=["x".join(map(str, p[0])) for p in SPECIAL_POINTS])
def test_split_special_values(env, sh, knobs, kind):
    torch, L = env
    _, split, f32 = points(L, sh, knobs)
    x, w = synthdata.conv_inputs(sh, "he")
    at = (1, 5, min(13, sh[2] - 1), 9)
    if kind == "inf":
        x[at] = np.inf
        x[0, 0, 0, 0] = -np.inf
    elif kind == "nan":
        x[at] = np.nan
    elif kind == "max":       # rounds past the largest bf16, the products stay finite
        x[at] = 3.4e38
        w *= np.float32(0.25)
    elif kind == "tiny":      # the planes past the first are denormal
        x *= np.float32(1e-36)
    else:
        w[3, 2, 1, 1] = np.inf
    P, Q = synthdata.conv_out_hw(sh[2], sh[3], sh[5], sh[6], sh[7], sh[8])
    n = sh[0] * sh[4] * P * Q
    xd, wd = dev(torch, x), dev(torch, w)
    print("conv split special", sh, knobs, kind, flush=True)
    got, want = (run(torch, L, s, xd, wd, n) for s in (split, f32))
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf])
    fin = np.isfinite(want)
    # both within fp32 rounding of the same sums: 9 terms a channel, each below
    # the tile's largest output
    scale = np.abs(want[fin]).max()
    assert np.abs(got[fin] - want[fin]).max() <= 9 * sh[1] * 2.0 ** -24 * scale


# a rectangle, ragged K, a band over three images in eight splits, stride 2
GUARD_POINTS = [POINTS[0], POINTS[1], POINTS[4],
                ((1, 16, 18, 18, 40, 3, 3, 2, 1), (32, 16, 8, 4, 2, 3))]


def scaled(kind, x, w):
    x, w = x.astype(np.float64), w.astype(np.float64)
    if kind == "column":          # tiny pixels beside normal ones
        x[:, :, :, 5] *= 1e-38
        x[-1, :, 3, :] = 0        # and empty ones
    elif kind == "channel":       # a tiny output channel beside normal ones
        w[7] *= 1e-39
        x *= 1e20
    elif kind == "one":           # a single tiny operand that alone makes its outputs
        x[:, :, 4:7, 4:7] = 0
        x[0, 3, 5, 5] = 1.2345e-38
        w *= 1e20
    else:
        sx, sw = map(float, kind.split("*"))
        x *= sx
        w *= sw
    return x.astype(np.float32), w.astype(np.float32)


@pytest.mark.parametrize("kind", ["1e-36*1e20", "1e-38*1e20", "1e-39*1e30", "1e-39*1", "1e20*1e-38",
                                  "1e-16*1e-17", "1e-20*1e-22", "1e-30*1e30", "column", "channel",
                                  "one"])
@pytest.mark.parametrize("sh,knobs", GUARD_POINTS,
                         ids=["x".join(map(str, p[0])) for p in GUARD_POINTS])
def test_split_small_operands(env, sh, knobs, kind):
    """Operands whose bf16 planes lose bits, or whose products leave the normal
    range: every output within what n fp32 sums may lose (each rounds to 2^-24 of
    at most sum |x w|, a few more for the product and the splits, and to 2^-149),
    and the errors relative to sum |x w| no larger than the fp32 program's (2-norm;
    1.1 as above)."""
    torch, L = env
    _, split, f32 = points(L, sh, knobs)
    x, w = scaled(kind, *synthdata.conv_inputs(sh, "he"))
    ref = ok.conv2d_f64(x, w, sh).ravel()
    mag = ok.conv2d_f64(np.abs(x), np.abs(w), sh).ravel()
    n = sh[1] * 9 + 8
    xd, wd = dev(torch, x), dev(torch, w)
    print("conv split small", sh, knobs, kind, flush=True)
    e = [np.abs(run(torch, L, s, xd, wd, ref.size) - ref) for s in (split, f32)]
    some = mag > 0
    rel = [np.linalg.norm(v[some] / mag[some]) / np.sqrt(some.sum()) * 2.0 ** 24 for v in e]
    print(f"  error in 2^-24 sum|xw|: {rel[0]:.3g}, fp32 MFMA {rel[1]:.3g}")
    assert (e[0] <= n * (2.0 ** -24 * mag + 2.0 ** -149)).all()
    assert (e[0][~some] == 0).all()
    assert rel[0] <= 1.1 * rel[1]
