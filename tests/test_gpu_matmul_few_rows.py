"""Matmuls of up to four rows whose split runs inside one workgroup (mm_rows), on
the GPU: every point that takes it, small-integer inputs bit-exact against the
oracle, and B off a 16-byte boundary (which keeps the tiled kernel) the same."""
import numpy as np
import pytest

import synthdata
from oracle import kernels as ok
from oracle import space as osp

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1000, 2048), (2, 20, 515), (3, 132, 64), (4, 64, 1023), (1, 16, 33)]


@pytest.mark.parametrize("sh", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_few_rows_exact(sh):
    import torch
    from paper_2406_20037_amd import _lib as L
    a, b = synthdata.matmul_inputs(sh, "int")
    ref = ok.matmul_f64(a, b).ravel()
    ad = torch.from_numpy(a).cuda()
    bufs = []
    for shift in (0, 1):
        t = torch.zeros(b.size + shift, device="cuda:0")
        t[shift:] = torch.from_numpy(b.ravel()).cuda()
        bufs.append(t[shift:])
    y = torch.empty(ref.size + 64, device="cuda:0")
    o, space, taken = osp.Space(2, sh), L.Space(2, sh), 0
    for p in o.valid_points():
        info = space.kernel_info(p)
        if info["family"] != 3 or len(info["params"]) != 6:
            continue
        taken += 1
        assert info["splits"] == 1 and info["params"][5] in (1, 2, 4)
        print("few rows", sh, o.knobs(p), flush=True)
        for bd in bufs:
            y[: ref.size].fill_(float("nan"))
            y[ref.size:] = 12345.0
            L.kernel_run(2, space.sched(p), ad, bd, y)
            torch.cuda.synchronize()
            assert bool((y[ref.size:] == 12345.0).all())
            assert np.array_equal(y[: ref.size].cpu().numpy().astype(np.float64), ref), o.knobs(p)
    assert taken > 0
