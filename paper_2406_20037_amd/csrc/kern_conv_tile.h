// Tiles, outputs and stores of a channel-quad conv point (conv_mfma2's rules), for
// the kernels that take such points in its place.
#pragma once

#include "kern_common.h"

namespace ds {

namespace {

__device__ __forceinline__ int fdv(int n, FastDiv f) {
    return int((__umulhi(unsigned(n), f.m) + unsigned(n)) >> f.s);
}

// Tile of a workgroup (tile order: k, q, p, split, image): channel tile kt,
// pixel tile (pt, qt) of image n, split z over chunks [ci0, ci1).  A band tile
// starts at pixel qt * npx of the flattened output: image n0, padded row g0 of
// that image; its halo is the `rows` padded rows from there (image boundaries
// included), each one whole output row wide.
struct Tile {
    int kt, qt, pt, n, z, ci0, ci1, n0, g0, rows;
    __device__ __forceinline__ explicit Tile(const Conv2Args &a) {
        const int t0 = xcd_tile(blockIdx.x, gridDim.x);
        const int t1 = fdv(t0, a.f_tk);
        kt = t0 - t1 * a.tiles_k;
        const int t2 = fdv(t1, a.f_tq);
        qt = t1 - t2 * a.tiles_q;
        const int t3 = fdv(t2, a.f_tp);
        pt = t2 - t3 * a.tiles_p;
        n = fdv(t3, a.f_ksw);
        z = t3 - n * a.ksw;
        ci0 = z * a.cps;
        ci1 = min(ci0 + a.cps, a.chunks);
        n0 = n;
        g0 = 0;
        rows = a.hs;
        if (a.band) {
            const int f0 = qt * a.npx, fl = min(f0 + a.npx, a.F) - 1;
            const int r0 = fdv(f0, a.f_q), rl = fdv(fl, a.f_q);
            n0 = fdv(r0, a.f_p);
            const int nl = fdv(rl, a.f_p);
            g0 = (r0 - n0 * a.P) * a.st;
            rows = (nl - n0) * a.hp + (rl - nl * a.P) * a.st + a.R - g0;
        }
    }
};

// Output of the tile's image (the split's partial output when ksw > 1).
__device__ __forceinline__ float *out_base(const Conv2Args &a, const Tile &T) {
    const int PQ = a.P * a.Q;
    return (a.ksw > 1 ? a.part + (size_t)T.z * a.N * a.K * PQ : a.y) + (size_t)T.n * a.K * PQ;
}

// Stores 4 consecutive tile pixels, from pix on, of output channel k.
__device__ __forceinline__ void put(const Conv2Args &a, const Tile &T, float *yn, int k, int pix,
                                    floatx4 val) {
    const int PQ = a.P * a.Q;
    if (k >= a.K) return;
    if (a.band) {
        const int f = T.qt * a.npx + pix;
        if (a.st4 && f + 3 < a.F) {
            const int img = fdv(f, a.f_pq);
            *reinterpret_cast<floatx4 *>(yn + (size_t)img * a.K * PQ + (size_t)k * PQ +
                                         (f - img * PQ)) = val;
            return;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int fe = f + e;
            if (fe >= a.F) break;
            const int img = fdv(fe, a.f_pq);
            yn[(size_t)img * a.K * PQ + (size_t)k * PQ + (fe - img * PQ)] = val[e];
        }
    } else {
        const int py = pix >> a.ltw, px = pix & (a.tw - 1);
        const int p = T.pt * a.th + py, q = T.qt * a.tw + px;
        if (a.st4 && p < a.P && q + 3 < a.Q) {
            *reinterpret_cast<floatx4 *>(yn + (size_t)k * PQ + p * a.Q + q) = val;
            return;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int pe = T.pt * a.th + ((pix + e) >> a.ltw), qe = T.qt * a.tw + ((pix + e) & (a.tw - 1));
            if (pe < a.P && qe < a.Q) yn[(size_t)k * PQ + pe * a.Q + qe] = val[e];
        }
    }
}

}  // namespace

}  // namespace ds
