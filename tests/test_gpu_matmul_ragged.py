"""Matmul sizes that no tile divides, on the GPU: the pipelined MFMA loop's clamped
rows and columns, its zero-filled last K-tile and both copy widths.  Small-integer
inputs, so every output must equal the oracle's; a non-finite value next to the
end of a row must not leak into the row before it."""
import numpy as np
import pytest

import synthdata
from oracle import kernels as ok
from oracle import space as osp

pytestmark = pytest.mark.gpu

# odd everything; 16-byte rows with ragged tiles; K below and just past a K-tile; rows
# of B or of A alone in 16-byte groups, few K-tiles (staged through registers) and many
SHAPES = [(257, 195, 203), (260, 196, 204), (130, 129, 15), (65, 71, 65), (129, 260, 68),
          (65, 72, 66), (66, 71, 264), (70, 132, 151)]


def run(torch, L, s, a, b, n):
    y = torch.full((n + 64,), float("nan"), device="cuda:0")
    y[n:] = 12345.0
    L.kernel_run(L.DS_OP_MATMUL_RM, s, a, b, y)
    torch.cuda.synchronize()
    assert bool((y[n:] == 12345.0).all()), "write past the end of C"
    return y[:n].cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("sh", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_every_mfma_class_exact(sh):
    import torch
    from paper_2406_20037_amd import _lib as L
    a, b = synthdata.matmul_inputs(sh, "int")
    ref = ok.matmul_f64(a, b).ravel()
    ad, bd = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    o, space = osp.Space(2, sh), L.Space(2, sh)
    seen = set()
    for p in o.valid_points():
        k = o.knobs(p)
        cls = (k["bm"], k["bn"], k["bk"], k["dbuf"], min(k["ks"], 4), k["unroll"] >= 16, k["vec"])
        if k["mfma"] != 1 or cls in seen:
            continue
        seen.add(cls)
        print("matmul", sh, k, flush=True)
        assert np.array_equal(run(torch, L, space.sched(p), ad, bd, ref.size), ref), k
    assert len(seen) > 40


@pytest.mark.parametrize("sh", SHAPES[:2], ids=["x".join(map(str, s)) for s in SHAPES[:2]])
def test_values_past_a_row_do_not_leak(sh):
    import torch
    from paper_2406_20037_amd import _lib as L
    M, N, K = sh
    a, b = synthdata.matmul_inputs(sh, "int")
    a[5, :4] = np.inf          # the floats after row 4
    b[3, :4] = np.nan          # the floats after row 2
    b[3, N - 1] = np.nan
    ref = a.astype(np.float64) @ np.nan_to_num(b).astype(np.float64)
    space = L.Space(L.DS_OP_MATMUL_RM, sh)
    s = space.sched_of(bm=64, bn=64, bk=16, unroll=64, dbuf=1, mfma=1, ks=1, vec=1)
    y = run(torch, L, s, torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), M * N).reshape(M, N)
    rows = np.arange(M) != 5
    cols = np.ones(N, bool)
    cols[[0, 1, 2, 3, N - 1]] = False
    assert np.array_equal(y[np.ix_(rows, cols)], ref[np.ix_(rows, cols)])
    assert not np.isfinite(y[5]).any() and np.isnan(y[:, :4]).all() and np.isnan(y[:, N - 1]).all()
