"""The row-wise loops of the channel-quad conv's small tiles on the GPU: 3x3 and
5x5 filters beside the step-by-step loop's (1x1, 1x3, 7x7), odd and even numbers
of quad blocks per chunk, ragged channels.  Small-integer inputs, so
every output must equal the oracle's."""
import numpy as np
import pytest

import synthdata
from oracle import kernels as ok
from oracle import space as osp

pytestmark = pytest.mark.gpu

SHAPES = [
    (1, 37, 15, 13, 40, 5, 5, 1, 2),
    (2, 29, 14, 14, 33, 3, 3, 1, 1),
    (1, 64, 9, 9, 48, 3, 3, 2, 1),
    (1, 70, 12, 12, 32, 1, 1, 1, 0),
    (1, 16, 11, 20, 17, 1, 3, 1, 0),
    (1, 3, 30, 30, 16, 7, 7, 2, 3),
]


@pytest.mark.parametrize("sh", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_small_tiles_bit_exact(sh):
    import torch
    from paper_2406_20037_amd import _lib as L
    x, w = synthdata.conv_inputs(sh, "int")
    ref = ok.conv2d_f64(x, w, sh).ravel()
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    y = torch.empty(ref.size, device="cuda:0")
    space, o = L.Space(1, sh), osp.Space(1, sh)
    seen = set()
    for p in o.valid_points():
        g, k = o.geometry(p), o.knobs(p)
        if k["mfma"] < 2 or g["t0"] * g["t1"] > 2:
            continue
        # one point per block shape, quads per step, chunk depth and split
        key = (g["t0"], g["t1"], g["unroll_eff"], k["tc"], k["ks"] if k["ks"] < 8 else 8, k["mfma"])
        if key in seen:
            continue
        seen.add(key)
        print("rows", sh, k, flush=True)
        y.fill_(float("nan"))
        L.kernel_run(1, space.sched(p), xd, wd, y)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy().astype(np.float64), ref), k
    assert len(seen) >= 3
