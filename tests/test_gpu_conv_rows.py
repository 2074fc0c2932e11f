"""The builds of the channel-quad conv for 3x3 and 5x5 filters, which walk rows of
taps, on the GPU, beside the step-by-step loop's (1x1, 1x3, 7x7): every such build
the shapes reach, up to the largest tiles that have one (eight blocks a wave for
3x3, four for 5x5), odd and even numbers of quad blocks per chunk, ragged
channels.  Small-integer inputs, so every output must equal the oracle's."""
import numpy as np
import pytest

import synthdata
from oracle import kernels as ok
from oracle import space as osp

pytestmark = pytest.mark.gpu

# blocks a wave: what the shape's builds must reach (output-channel blocks x
# pixel blocks), {} where the filter has none of its own
SHAPES = [
    ((1, 37, 15, 13, 40, 5, 5, 1, 2), {1, 2}),
    ((2, 36, 24, 20, 70, 5, 5, 1, 2), {1, 2, 4}),
    ((2, 29, 14, 14, 33, 3, 3, 1, 1), {1, 2}),
    ((2, 28, 24, 20, 66, 3, 3, 1, 1), {1, 2, 4, 8}),
    ((1, 64, 9, 9, 48, 3, 3, 2, 1), {1, 2}),
    ((1, 70, 12, 12, 32, 1, 1, 1, 0), set()),
    ((1, 16, 11, 20, 17, 1, 3, 1, 0), set()),
    ((1, 3, 30, 30, 16, 7, 7, 2, 3), set()),
]
IDS = ["x".join(map(str, s)) for s, _ in SHAPES]


def row_points(L, sh):
    """[(point, knobs, params)]: one per build, chunk depth, split and tile kind."""
    space, o = L.Space(1, sh), osp.Space(1, sh)
    size = sh[5] if sh[5] == sh[6] and sh[5] in (3, 5) else 0
    seen = {}
    for p in o.valid_points():
        g, k = o.geometry(p), o.knobs(p)
        blocks = g["t0"] * g["t1"]
        if k["mfma"] < 2 or blocks > (8 if size == 3 else 4 if size else 2):
            continue
        key = (g["t0"], g["t1"], g["unroll_eff"], k["tc"], min(k["ks"], 8), k["mfma"], k["vec"])
        if key in seen:
            continue
        params = space.kernel_info(p)["params"]
        if params[5:] in ([1], [2]):              # split-operand or few-channel kernel
            continue
        # the quads a loop step multiplies (1, 2, 4)
        if size and blocks <= 4 and params[2] < 4:
            assert params[5:] == [size], (sh, k, params)
        elif not size:
            assert params[5:] == [], (sh, k, params)
        seen[key] = (p, k, params)
    return space, list(seen.values())


@pytest.mark.parametrize("sh,blocks", SHAPES, ids=IDS)
def test_row_builds_bit_exact(sh, blocks):
    import torch
    from paper_2406_20037_amd import _lib as L
    x, w = synthdata.conv_inputs(sh, "int")
    ref = ok.conv2d_f64(x, w, sh).ravel()
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    y = torch.empty(ref.size, device="cuda:0")
    space, pts = row_points(L, sh)
    for p, k, params in pts:
        print("rows", sh, k, params, flush=True)
        y.fill_(float("nan"))
        L.kernel_run(1, space.sched(p), xd, wd, y)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy().astype(np.float64), ref), k
    assert len(pts) >= 3
    assert blocks <= {q[0] * q[1] for _, _, q in pts if q[5:]}
