// CPU replay of the split-operand conv kernel's index arithmetic
// (kern_conv_split.hip: conv_split), for tests only.
//
// For one schedule it walks every workgroup, thread and lane with the launch
// set-up of conv2_setup and conv2_split_setup and checks what the GPU cannot
// report: global reads inside their tensors, LDS units and the unit table
// inside the workgroup's LDS size, no unit read before it was written, every
// output written once per split, and the fp64 result equal to a direct
// convolution.  It mirrors the kernel by hand: a change to one needs the same
// change here.
//
// stdin, one schedule per line:
//   N C H W K R S stride pad  tk th tw tc depth ks vec band
// stdout: "ok ...", "fp32 ..." (the point does not take this kernel) or
// "FAIL ..." per line; exit status 1 on the first failure.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "ds_internal.h"

namespace ds {
void set_error(const char *, ...) {}
}
using namespace ds;

namespace {

int fdv(int n, FastDiv f) {
    const unsigned hi = unsigned((uint64_t(unsigned(n)) * uint64_t(f.m)) >> 32);
    return int((hi + unsigned(n)) >> f.s);
}

int xcd_tile(int b, int nwg) {   // kern_common.h
    const int q = nwg >> 3, r = nwg & 7;
    const int x = b & 7, j = b >> 3;
    return x * q + (x < r ? x : r) + j;
}

long g_errors = 0;
#define CHECK(c, ...)                                         \
    do {                                                      \
        if (!(c) && g_errors++ < 8) {                         \
            fprintf(stderr, __VA_ARGS__);                     \
            fprintf(stderr, "\n");                            \
        }                                                     \
    } while (0)

struct Unit {
    double v[8];
    int stage = -1;   // stage that wrote it (1 << 30: the zero padding)
};

const char *replay(const int64_t *sh, int tk, int th, int tw, int tc, int depth, int ks, int vec,
                   bool band, char *summary, size_t nsum) {
    Conv2Args a;
    const Conv2Shape c = conv2_setup(sh, tk, th, tw, tc, depth, ks, vec, band, a);
    summary[0] = 0;
    if (!c.valid) return "FAIL invalid point";
    int64_t lds = 0;
    if (!conv2_split_setup(a, c, &lds)) return "fp32";
    const int TB = c.tkb / 2, NB = c.npb / 2, nthr = c.threads, RS = a.R * a.S, HW = a.H * a.W;
    const int PQ = a.P * a.Q;
    const size_t nx = size_t(a.N) * a.C * HW, nwt = size_t(a.K) * a.C * RS, ny = size_t(a.N) * a.K * PQ;
    CHECK(lds <= kLdsLimit && lds >= c.lds, "lds %ld", (long)lds);
    
    CHECK(a.sxo % 16 == 0 && a.sxo >= a.tk * kConvSplitRow && a.sxo + 48 * a.scs <= lds, "layout");
    const int HU = kConvSplitHalo, WU = (32 * TB * 9 + 255) / 256;
    std::mt19937 rng(20240620);
    std::uniform_real_distribution<double> ud(-1, 1);
    std::vector<double> x(nx), w(nwt);
    for (auto &v : x) v = ud(rng);
    for (auto &v : w) v = ud(rng);
    std::vector<double> part(size_t(a.ksw) * ny, 0);
    std::vector<int> written(size_t(a.ksw) * ny, 0);
    for (int64_t g = 0; g < c.grid; ++g) {
        const int t0 = xcd_tile(int(g), int(c.grid));
        const int t1 = fdv(t0, a.f_tk), kt = t0 - t1 * a.tiles_k;
        const int t2 = fdv(t1, a.f_tq), qt = t1 - t2 * a.tiles_q;
        const int t3 = fdv(t2, a.f_tp), pt = t2 - t3 * a.tiles_p;
        const int n = fdv(t3, a.f_ksw), z = t3 - n * a.ksw;
        const int ci0 = z * a.cps, ci1 = std::min(ci0 + a.cps, a.chunks);
        if (ci0 >= ci1) continue;
        int n0 = n, g0 = 0, rows = a.hs;
        if (a.band) {
            const int f0 = qt * a.npx, fl = std::min(f0 + a.npx, a.F) - 1;
            const int r0 = fdv(f0, a.f_q), rl = fdv(fl, a.f_q);
            n0 = fdv(r0, a.f_p);
            const int nl = fdv(rl, a.f_p);
            g0 = (r0 - n0 * a.P) * a.st;
            rows = (nl - n0) * a.hp + (rl - nl * a.P) * a.st + a.R - g0;
        }
        const int hy0 = pt * a.th * a.st - a.pd, hx0 = (a.band ? 0 : qt * a.tw * a.st) - a.pd;
        const int kvalid = a.K - kt * a.tk;
        const int c_beg = ci0 * a.tc, c_end = std::min(ci1 * a.tc, a.C);
        const int stages = (c_end - c_beg) >> 3;
        const int64_t xn = (int64_t(n0) * a.C + c_beg) * HW, wk = (int64_t(kt) * a.tk * a.C + c_beg) * RS;
        const int nh = a.scs, nw = a.tk * 9;
        CHECK((c_end - c_beg) % 8 == 0, "partial stage");
        CHECK(HU * nthr >= nh && WU * nthr >= nw, "units");
        // weights by (row, tap; tap 9 the zero padding), halo by position
        std::vector<Unit> LW(size_t(a.tk) * 10), LX(nh);
        for (int row = 0; row < a.tk; ++row) {
            LW[size_t(row) * 10 + 9].stage = 1 << 30;
            for (double &v : LW[size_t(row) * 10 + 9].v) v = 0;
        }
        std::vector<double> acc(size_t(tk) * a.npx, 0);
        auto gx_at = [&](int64_t i) { CHECK(i >= 0 && i < int64_t(nx), "x read %ld of %zu", (long)i, nx); return x[size_t(i)]; };
        auto gw_at = [&](int64_t i) { CHECK(i >= 0 && i < int64_t(nwt), "w read %ld of %zu", (long)i, nwt); return w[size_t(i)]; };
        for (int s = 0; s < stages; ++s) {
            const int64_t xb = xn + int64_t(s) * 8 * HW, wb = wk + int64_t(s) * 8 * RS;
            for (int u = 0; u < HU; ++u)
                for (int tid = 0; tid < nthr; ++tid) {
                    const int e = std::min(u * nthr + tid, nh - 1);
                    const int hy = fdv(e, a.f_sws), hx = e - hy * a.sws;
                    int gy, img = 0;
                    if (a.band) {
                        const int gr = g0 + hy;
                        img = fdv(gr, a.f_hp);
                        gy = gr - img * a.hp - a.pd;
                    } else {
                        gy = hy0 + hy;
                    }
                    const int gx = hx0 + hx;
                    const bool in = hy < rows && gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
                    const int sx = in ? (img * a.C * a.H + gy) * a.W + gx : -1;
                    LX[e].stage = s;
                    for (int j = 0; j < 8; ++j) {
                        const double v = gx_at(xb + int64_t(j) * HW + std::max(sx, 0));
                        LX[e].v[j] = in ? v : 0;
                    }
                }
            for (int u = 0; u < WU; ++u)
                for (int tid = 0; tid < nthr; ++tid) {
                    const int e = std::min(u * nthr + tid, nw - 1);
                    const int row = e / 9, t = e - row * 9;
                    Unit &U = LW[size_t(row) * 10 + t];
                    U.stage = s;
                    for (int j = 0; j < 8; ++j)
                        U.v[j] = gw_at(wb + int64_t(j) * RS + std::min(row, kvalid - 1) * a.C * 9 + t);
                }
            for (int wp = 0; wp < a.wpx; ++wp)
                for (int b = 0; b < NB; ++b)
                    for (int li = 0; li < 32; ++li) {
                        const int pix = (wp * NB + b) * 32 + li;
                        CHECK(pix < a.npx, "pixel %d", pix);
                        int pos;
                        if (a.band) {
                            const int f = std::min(qt * a.npx + pix, a.F - 1);
                            const int r = fdv(f, a.f_q), q = f - r * a.Q;
                            const int img = fdv(r, a.f_p), p = r - img * a.P;
                            pos = ((img - n0) * a.hp + p * a.st - g0) * a.sws + q * a.st;
                        } else {
                            const int py = pix >> a.ltw, px = pix & (a.tw - 1);
                            pos = py * a.st * a.sws + px * a.st;
                        }
                        for (int t = 0; t < 10; ++t) {
                            const int tap = std::min(t, 8), bu = pos + tap / 3 * a.sws + tap % 3;
                            CHECK(bu >= 0 && bu < nh && LX[bu].stage == s, "operand unit %d of %d", bu, nh);
                            if (bu < 0 || bu >= nh) continue;
                            for (int row = 0; row < 32 * TB; ++row) {
                                const Unit &A = LW[size_t(row) * 10 + t];
                                CHECK(A.stage == s || A.stage == 1 << 30, "weight row %d unit %d", row, t);
                                for (int j = 0; j < 8; ++j) acc[size_t(row) * a.npx + pix] += A.v[j] * LX[bu].v[j];
                            }
                        }
                    }
        }
        for (int row = 0; row < tk; ++row)
            for (int pix = 0; pix < a.npx; ++pix) {
                const int k = kt * tk + row;
                if (k >= a.K) continue;
                int64_t at;
                if (a.band) {
                    const int f = qt * a.npx + pix;
                    if (f >= a.F) continue;
                    const int img = fdv(f, a.f_pq);
                    at = (int64_t(img) * a.K + k) * PQ + f - img * PQ;
                } else {
                    const int p = pt * th + (pix >> a.ltw), q = qt * tw + (pix & (tw - 1));
                    if (p >= a.P || q >= a.Q) continue;
                    at = (int64_t(n) * a.K + k) * PQ + p * a.Q + q;
                }
                part[size_t(z) * ny + at] = acc[size_t(row) * a.npx + pix];
                written[size_t(z) * ny + at]++;
            }
    }
    const int nsplit = (a.chunks + a.cps - 1) / a.cps;
    double maxerr = 0, maxref = 0;
    for (size_t e = 0; e < ny; ++e) {
        double s = 0;
        for (int zz = 0; zz < nsplit; ++zz) {
            CHECK(written[zz * ny + e] == 1, "output %zu of split %d written %d times", e, zz, written[zz * ny + e]);
            s += part[zz * ny + e];
        }
        const int q = int(e % a.Q), p = int(e / a.Q % a.P), k = int(e / PQ % a.K), nn = int(e / (size_t(PQ) * a.K));
        double ref = 0;
        for (int ch = 0; ch < a.C; ++ch)
            for (int r = 0; r < a.R; ++r)
                for (int s2 = 0; s2 < a.S; ++s2) {
                    const int iy = p * a.st - a.pd + r, ix = q * a.st - a.pd + s2;
                    if (iy < 0 || iy >= a.H || ix < 0 || ix >= a.W) continue;
                    ref += x[((size_t(nn) * a.C + ch) * a.H + iy) * a.W + ix] * w[((size_t(k) * a.C + ch) * a.R + r) * a.S + s2];
                }
        maxerr = std::max(maxerr, std::fabs(s - ref));
        maxref = std::max(maxref, std::fabs(ref));
    }
    CHECK(maxerr <= 1e-9 * std::max(1.0, maxref), "max error %g (max |ref| %g)", maxerr, maxref);
    snprintf(summary, nsum, "band=%d tb=%d nb=%d halo=%d lds=%ld ksw=%d grid=%ld err=%.2g",
             a.band, TB, NB, a.scs, (long)lds, a.ksw, (long)c.grid, maxerr);
    return g_errors == 0 ? "ok" : "FAIL";
}

}  // namespace

int main() {
    int64_t sh[9];
    int tk, th, tw, tc, depth, ks, vec, band;
    while (scanf("%ld %ld %ld %ld %ld %ld %ld %ld %ld %d %d %d %d %d %d %d %d", &sh[0], &sh[1], &sh[2],
                 &sh[3], &sh[4], &sh[5], &sh[6], &sh[7], &sh[8], &tk, &th, &tw, &tc, &depth, &ks, &vec,
                 &band) == 17) {
        char summary[256];
        const char *r = replay(sh, tk, th, tw, tc, depth, ks, vec, band != 0, summary, sizeof summary);
        printf("%s %s\n", r, summary);
        fflush(stdout);
        if (r[0] == 'F') return 1;
    }
    return 0;
}
