"""Timed cases of the library's kernel path.

A user of this library tunes a conv2d or matmul once and then launches the
schedule it found, again and again, through ``kernel_run``; the tuner itself
spends its time in trials (``ds_measure``).  The listed cases are those calls
at the shapes of the repository's workloads (synthdata/workloads.py) with the
schedules the tuner picks for them, and at odd sizes that no tile divides.
Drawn cases take other sizes of the same ranges, with a schedule chosen by
rules of thumb in place of a tuning run.

conv shape = N,C,H,W,K,R,S,stride,pad; matmul shape = M,N,K; all tensors fp32.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_2406_20037_amd import _lib as L

CONV, MATMUL = L.DS_OP_CONV2D_NCHW, L.DS_OP_MATMUL_RM
LARGEST = 16 * 64 * 64 * 224 * 224 * 9       # multiply-adds of the largest listed case


def _case(name, op, shape, sched, kind, call="run"):
    return dict(name=name, op=op, shape=shape, sched=sched, kind=kind, call=call)


def listed():
    return [
        # The smallest calls: one image, one layer, ten microseconds each, where
        # launches and per-workgroup latency count.
        _case("conv3x3_c64_56", "conv", "1,64,56,56,64,3,3,1,1",
              "tk=16,th=2,tw=32,tc=64,unroll=512,lds=1,ks=4,mfma=2,vec=4", "uniform"),
        # ResNet-50 stem at batch 1 (three channels, 7x7 filter, stride 2).
        _case("conv7x7_s2_c3_224", "conv", "1,3,224,224,64,7,7,2,3",
              "tk=16,th=8,tw=16,tc=1,unroll=16,lds=1,ks=1,mfma=1,vec=4", "uniform"),
        # ResNet-50's last 3x3 stride-2 layer at batch 1: 49 output pixels, a
        # 4608-long reduction split over workgroups, and its reduce launch.
        _case("resnet50_s4_3x3_s2", "conv", "1,512,14,14,512,3,3,2,1",
              "tk=32,th=8,tw=8,tc=8,unroll=0,lds=1,ks=32,mfma=3,vec=4", "he"),
        # One trial of the tuner at its default settings (parity launch, warm-up,
        # timed repeats of at least 0.5 ms each) on ResNet-50's most repeated
        # layer at batch 1: what tuning does some 300 times a kernel.
        _case("trial_resnet50_s3_1x1", "conv", "1,256,14,14,1024,1,1,1,0",
              "tk=32,th=2,tw=8,tc=64,unroll=512,lds=1,ks=4,mfma=2,vec=4", "he", "trial"),
        # The classifier at batch 1: a matrix-vector product.
        _case("resnet50_fc", "matmul", "1,1000,2048",
              "bm=16,bn=16,bk=64,unroll=64,dbuf=1,mfma=0,ks=8,vec=4", "he"),
        _case("matmul_1024", "matmul", "1024,1024,1024",
              "bm=64,bn=64,bk=16,unroll=64,dbuf=1,mfma=1,ks=1,vec=4", "uniform"),
        # No tile divides these: bounds-checked staging, 4-byte copies.
        _case("matmul_ragged", "matmul", "1003,1501,777",
              "bm=64,bn=64,bk=16,unroll=64,dbuf=1,mfma=1,ks=1,vec=1", "uniform"),
        _case("conv5x5_ragged", "conv", "3,37,61,53,90,5,5,1,2",
              "tk=16,th=8,tw=16,tc=4,unroll=0,lds=1,ks=1,mfma=2,vec=1", "uniform"),
        # VGG-16 at batch 16: the first layer (memory-bound), the largest
        # layer, a deep layer (reduction split over workgroups) and the last
        # ones (14x14 images).
        _case("vgg16_L1", "conv", "16,3,224,224,64,3,3,1,1",
              "tk=64,th=8,tw=32,tc=1,unroll=0,lds=1,ks=1,mfma=2,vec=1", "he"),
        _case("vgg16_L2", "conv", "16,64,224,224,64,3,3,1,1",
              "tk=64,th=16,tw=16,tc=4,unroll=0,lds=1,ks=1,mfma=2,vec=4", "he"),
        _case("vgg16_L10", "conv", "16,512,28,28,512,3,3,1,1",
              "tk=64,th=8,tw=32,tc=4,unroll=0,lds=1,ks=8,mfma=3,vec=4", "he"),
        _case("vgg16_L12", "conv", "16,512,14,14,512,3,3,1,1",
              "tk=64,th=16,tw=8,tc=4,unroll=0,lds=1,ks=16,mfma=3,vec=4", "he"),
    ]


def _shape(case):
    return tuple(int(v) for v in case["shape"].split(","))


def _op(case):
    return CONV if case["op"] == "conv" else MATMUL


def _out_shape(case):
    sh = _shape(case)
    if case["op"] == "matmul":
        return sh[0], sh[1]
    N, C, H, W, K, R, S, st, pd = sh
    return N, K, (H + 2 * pd - R) // st + 1, (W + 2 * pd - S) // st + 1


def _macs(case):
    sh = _shape(case)
    if case["op"] == "matmul":
        return sh[0] * sh[1] * sh[2]
    return math.prod(_out_shape(case)) * sh[1] * sh[5] * sh[6]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    """A conv (three in four) or matmul of the listed ranges: batch 1 to 16,
    3 to 512 channels, images of 7 to 224 rows and columns, filters of 1 to 5
    (7 for three channels), strides 1 and 2; matrices of 1 to 2048 rows and
    columns."""
    while True:
        if rng.random() < 0.25:
            m = 1 if rng.random() < 0.2 else _log_int(rng, 16, 2048)
            case = dict(op="matmul", kind="uniform",
                        shape=f"{m},{_log_int(rng, 64, 2048)},{_log_int(rng, 64, 2048)}")
        else:
            st = rng.choice([1, 1, 1, 2])
            # half the image sizes and channel counts are multiples of 4 and 16, as
            # in the networks, the others any
            h = _log_int(rng, 7, 224)
            w = h if rng.random() < 0.5 else _log_int(rng, 7, 224)
            c = 3 if rng.random() < 0.1 else _log_int(rng, 3, 512)
            r = rng.choice([3, 7] if c == 3 else [1, 3, 3, 3, 5])
            k = _log_int(rng, 16, 512)
            if rng.random() < 0.5:
                h, w = max(8, h // 4 * 4), max(8, w // 4 * 4)
                c, k = (c if c < 16 else c // 16 * 16), max(16, k // 16 * 16)
            case = dict(op="conv", kind=rng.choice(["uniform", "he"]),
                        shape=f"{_log_int(rng, 1, 16)},{c},{h},{w},{k},{r},{r},{st},{r // 2}")
        case["unroll"] = rng.choice([0, 0, 16, 64])
        case["call"] = "run"
        if 2e5 <= _macs(case) <= LARGEST:
            return case


def _pick(space, case):
    """A schedule by rules of thumb: of a few dozen valid points, the one whose
    tiles waste the least work and fill the chip."""
    best = None

    def consider(knobs, waste, per_wave):
        nonlocal best
        idx = []
        for n, vals in zip(space.names, space.values):
            if knobs[n] not in vals:
                return
            idx.append(vals.index(knobs[n]))
        if not space.valid(idx):
            return
        g = space.geometry(idx)
        waves = g["grid"] * g["threads"] / 64
        cost = waste(g) * max(1.0, 2048 / waves) * (1 + 8 / per_wave) * (1 + 0.02 * knobs["ks"])
        cost *= 1.0 if knobs["vec"] == 4 else 1.1
        if best is None or cost < best[0]:
            best = (cost, idx)

    out = _out_shape(case)
    if case["op"] == "matmul":
        M, N, K = _shape(case)
        for bm in (16, 32, 64, 128):
            for bn in (16, 32, 64, 128):
                for bk in (16, 32, 64):
                    for ks in (1, 2, 4, 8):
                        for vec in (4, 1):
                            consider(dict(bm=bm, bn=bn, bk=bk, unroll=case["unroll"], dbuf=1,
                                          mfma=int(bm >= 32 and bn >= 32), ks=ks, vec=vec),
                                     lambda g: (-(-M // bm) * bm * -(-N // bn) * bn) / (M * N),
                                     bm * bn / 256)
    else:
        C = _shape(case)[1]
        F_ = out[0] * out[2] * out[3]
        for tk in (64, 32, 16):
            for th, tw in ((16, 16), (8, 32), (4, 64), (16, 8), (8, 16), (4, 32), (8, 8), (4, 16),
                           (2, 32), (4, 8), (2, 16), (4, 4)):
                for mfma in (1, 2, 3):
                    if mfma < 3:
                        px = out[0] * -(-out[2] // th) * th * -(-out[3] // tw) * tw
                    else:
                        px = -(-F_ // (th * tw)) * th * tw
                    waste = px * (-(-out[1] // tk) * tk) / (F_ * out[1])
                    # the tabled family (mfma 1) is the pick for the 7x7 stem only
                    waste *= 8 if mfma == 1 and (C > 3 or _shape(case)[5] < 7) else 1
                    for tc in ((1,) if C < 4 else (4, 8, 16)):
                        for ks in (1, 2, 4, 8, 16, 32):
                            for vec in (4, 1):
                                consider(dict(tk=tk, th=th, tw=tw, tc=tc, unroll=case["unroll"],
                                              lds=1, ks=ks, mfma=mfma, vec=vec),
                                         lambda g: waste * (1 + 2 / tc), tk * th * tw / 256)
    if best is None and case["unroll"]:      # deep unrolling fits no tile of so few channels
        return _pick(space, dict(case, unroll=0))
    return best[1]


def _schedule(case):
    space = L.Space(_op(case), _shape(case))
    if "sched" in case:
        return space.sched_of(**{k: int(v) for k, v in
                                 (kv.split("=") for kv in case["sched"].split(","))})
    return space.sched(_pick(space, case))


def _inputs(case, seed):
    """x, w as the networks hold them: normal activations with He-normal weights,
    or U[-1, 1) for the single kernels."""
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    sh = _shape(case)
    if case["op"] == "matmul":
        xs, ws, fan_in = (sh[0], sh[2]), (sh[2], sh[1]), sh[2]
    else:
        xs, ws, fan_in = sh[:4], (sh[4], sh[1], sh[5], sh[6]), sh[1] * sh[5] * sh[6]
    if case["kind"] == "uniform":
        return [torch.rand(s, generator=g, device="cuda:0") * 2 - 1 for s in (xs, ws)]
    x = torch.randn(xs, generator=g, device="cuda:0")
    return [x, torch.randn(ws, generator=g, device="cuda:0") * math.sqrt(2.0 / fan_in)]


def prepare(case, seed):
    x, w = _inputs(case, seed)
    y = torch.empty(_out_shape(case), device="cuda:0")
    state = dict(op=_op(case), sched=_schedule(case), x=x, w=w, y=y,
                 stream=torch.cuda.current_stream())
    if case["call"] == "trial":
        ref = torch.empty_like(y)
        L.kernel_run_reference(_op(case), _shape(case), x, w, ref, state["stream"])
        state["io"] = L.make_io(x, w, y, ref, state["stream"])
        state["ref"] = ref
    return state


def run(state):
    if "io" in state:
        L.ds_measure(state["sched"], state["io"])
        return state["y"]
    L.kernel_run(state["op"], state["sched"], state["x"], state["w"], state["y"], state["stream"])
    return state["y"]


def work(case):
    sh = _shape(case)
    out = math.prod(_out_shape(case))
    if case["op"] == "matmul":
        elems = sh[0] * sh[2] + sh[2] * sh[1] + out
    else:
        elems = math.prod(sh[:4]) + sh[4] * sh[1] * sh[5] * sh[6] + out
    # a trial launches its kernel at least 16 times: parity, 3 warm-up, 12 repeats
    launches = 16 if case["call"] == "trial" else 1
    return {"bytes": 4 * elems * launches, "flops": 2 * _macs(case) * launches}


def tolerance(case):
    return {"rel": 2e-6, "max": 2e-5}


def exact(case, seed):
    x, w = (t.double() for t in _inputs(case, seed))
    if case["op"] == "matmul":
        return x @ w
    N, C, H, W, K, R, S, st, pd = _shape(case)
    y = torch.empty(_out_shape(case), dtype=torch.float64, device="cuda:0")
    for n in range(N):
        cols = F.unfold(x[n:n + 1], (R, S), padding=pd, stride=st)[0]
        y[n] = (w.view(K, -1) @ cols).view(y[n].shape)
    return y
