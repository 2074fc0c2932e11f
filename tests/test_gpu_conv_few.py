"""3x3 convolutions over up to three channels (conv_few) on the GPU: one point of
every block shape and tile kind, ragged images and channel tiles, strides, no
padding, several images in a band.  Small-integer inputs, so every output must
equal the oracle's; and infinities and NaN reach exactly the outputs whose
windows hold them (the padding taps of a k-step and taps off the image do not
spread them)."""
import numpy as np
import pytest

import synthdata
from oracle import kernels as ok
from oracle import space as osp

pytestmark = pytest.mark.gpu

SHAPES = [
    (2, 3, 17, 23, 40, 3, 3, 1, 1),
    (1, 3, 32, 64, 64, 3, 3, 1, 1),
    (3, 2, 21, 20, 33, 3, 3, 2, 1),
    (2, 1, 9, 31, 70, 3, 3, 1, 0),
    (5, 3, 7, 8, 128, 3, 3, 1, 2),
]


@pytest.mark.parametrize("sh", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_few_channels(sh):
    import torch
    from paper_2406_20037_amd import _lib as L
    x, w = synthdata.conv_inputs(sh, "int")
    ref = ok.conv2d_f64(x, w, sh).ravel()
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    odd = x.copy()
    odd[0, 0, 0, 0], odd[-1, -1, -1, -1], odd[-1, 0, 3, 4] = np.inf, np.nan, -np.inf
    assert not (w == 0).all()
    odd_ref = torch.nn.functional.conv2d(torch.from_numpy(odd).double(), torch.from_numpy(w).double(),
                                         stride=sh[7], padding=sh[8]).numpy().ravel()
    od = torch.from_numpy(odd).cuda()
    y = torch.empty(ref.size + 64, device="cuda:0")
    space, o = L.Space(1, sh), osp.Space(1, sh)
    seen = set()
    for p in o.valid_points():
        info, k = space.kernel_info(p), o.knobs(p)
        if info["family"] != 5 or info["params"][5:] != [2]:
            continue
        key = (info["params"][0], info["params"][1], k["mfma"], k["tw"] if k["mfma"] == 2 else 0,
               k["th"] * k["tw"])
        if key in seen:
            continue
        seen.add(key)
        print("few channels", sh, k, flush=True)
        for inp, want in ((xd, ref), (od, odd_ref)):
            y[: ref.size].fill_(float("nan"))
            y[ref.size:] = 12345.0
            L.kernel_run(1, space.sched(p), inp, wd, y)
            torch.cuda.synchronize()
            assert bool((y[ref.size:] == 12345.0).all()), k
            got = y[: ref.size].cpu().numpy().astype(np.float64)
            assert np.array_equal(got, want, equal_nan=True), k
    assert len(seen) >= 6
