"""The split-operand conv kernel's index arithmetic, replayed on the CPU.

`tests/replay/conv_split_replay.cpp` walks every workgroup, thread and lane of
conv_split with the library's own launch set-up: global reads inside their
tensors, LDS units inside the workgroup's LDS and written before they are read,
every output written once per split, and the fp64 result of the replayed
multiply-adds equal to a direct convolution.  Shapes: strides, padding, ragged
K, odd image sizes, reduction splits, bands across images.

Also which points take the kernel at all: rectangles of 32 pixels a wave in splits
of a single stage, whose weights the fp32 program copies 16 bytes at a time, stay on
that program.
"""
import os
import random
import shutil
import subprocess

import pytest

from oracle import space as sp

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

SHAPES = [
    (2, 16, 14, 14, 40, 3, 3, 1, 1),
    (3, 24, 17, 16, 33, 3, 3, 1, 1),
    (2, 16, 13, 13, 70, 3, 3, 1, 1),
    (4, 40, 12, 10, 32, 3, 3, 1, 0),
    (1, 8, 5, 40, 32, 3, 3, 1, 1),
    (5, 64, 9, 9, 64, 3, 3, 1, 1),
    (1, 32, 40, 33, 64, 3, 3, 1, 2),
    (1, 16, 18, 18, 32, 3, 3, 2, 1),
    (2, 24, 10, 20, 40, 3, 3, 2, 1),
]
PER_SHAPE = 10


@pytest.fixture(scope="module")
def replay_bin(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx or not os.path.exists(os.path.join(ROCM, "include", "hip")):
        pytest.skip("needs g++ and the ROCm headers")
    out = str(tmp_path_factory.mktemp("replay") / "conv_split_replay")
    subprocess.run([gxx, "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2406_20037_amd", "csrc"),
                    os.path.join(HERE, "replay", "conv_split_replay.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("sh", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_conv_split_index_replay(replay_bin, sh):
    s = sp.Space(sp.OP_CONV, sh)
    pts = []
    for p in s.valid_points():
        v, g = s.knobs(p), s.geometry(p)
        if v["mfma"] >= 2 and v["unroll"] == 0 and g["t0"] >= 2 and g["t1"] >= 2:
            pts.append((v, g))
    assert pts
    rng = random.Random(hash(sh) & 0xFFFF)
    lines = []
    for v, g in rng.sample(pts, min(PER_SHAPE, len(pts))):
        lines.append(" ".join(map(str, list(sh) + [
            v["tk"], v["th"], v["tw"], v["tc"], g["unroll_eff"], v["ks"], v["vec"],
            int(v["mfma"] == 3)])))
    r = subprocess.run([replay_bin], input="\n".join(lines) + "\n", capture_output=True, text=True,
                       timeout=600)
    out = r.stdout.strip().splitlines()
    assert r.returncode == 0 and len(out) == len(lines), (
        f"{lines[len(out) - 1] if out else lines[0]}: {out[-1:]} {r.stderr[-2000:]}")
    assert any(o.startswith("ok") for o in out), out


# tile knobs (tk, th, tw, tc, ks, mfma, vec); takes the split-operand kernel?
ROUTES = [
    ((16, 64, 112, 112, 128, 3, 3, 1, 1), (64, 32, 4, 4, 8, 2, 4), False),
    ((16, 64, 112, 112, 128, 3, 3, 1, 1), (32, 32, 4, 4, 8, 2, 4), False),
    ((16, 64, 112, 112, 128, 3, 3, 1, 1), (64, 32, 4, 4, 4, 2, 4), True),    # two stages
    ((16, 64, 112, 112, 128, 3, 3, 1, 1), (64, 32, 8, 4, 8, 2, 4), True),    # 64 pixels a wave
    ((3, 40, 61, 53, 90, 3, 3, 1, 1), (64, 8, 16, 4, 8, 2, 4), False),
    ((3, 40, 61, 53, 90, 3, 3, 1, 1), (64, 8, 16, 4, 8, 2, 1), True),        # 4-byte copies
    ((16, 8, 56, 56, 128, 3, 3, 1, 1), (64, 32, 4, 8, 1, 2, 4), True),       # no split
    ((16, 256, 14, 14, 512, 3, 3, 1, 1), (64, 16, 8, 4, 32, 3, 4), True),    # a band
]


@pytest.mark.parametrize("sh,knobs,taken", ROUTES)
def test_single_stage_rectangles_keep_the_fp32_program(sh, knobs, taken):
    from paper_2406_20037_amd import _lib as L
    space = L.Space(L.DS_OP_CONV2D_NCHW, sh)
    kn = dict(zip(("tk", "th", "tw", "tc", "ks", "mfma", "vec"), knobs), unroll=0, lds=1)
    s = space.sched_of(**kn)
    assert space.valid(s.index())
    assert (space.kernel_info(s.index())["params"][5:] == [1]) == taken
