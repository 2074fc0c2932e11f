// 3x3 conv over up to three channels for gfx950 (conv mfma = 2 and 3): the first
// layer of a network, at most 27 products an output and as many bytes stored as
// the rest of the layer needs time for.
//
// The channel-quad loop pads three channels to four (nine MFMA steps, here seven
// of four taps each), computes its copy sources as it goes and takes every output
// through LDS; fp32 MFMAs hold the vector unit meanwhile, so the 69 us of
// 16x3x224x224 (64 channels) were the sum of the three.  Here a lane reads its
// taps straight from global memory (16 consecutive pixels a tap: 64 bytes in a
// row), the weights stay in registers, and the outputs go from the accumulators
// to memory without LDS.  What that takes, measured on that layer:
//   - weights through LDS: read from their rows in global memory each lane is a
//     request of its own (91 us; 75 through LDS);
//   - blocks of 16 pixels next to each other stored one after the other, so that
//     128-byte lines fill at once (75 -> 59 us), two of them at a time: four need
//     149 registers, three waves per SIMD (57 us with two);
//   - non-temporal stores where a wave's pixels are whole lines (57 -> 47 us; 64-byte pieces would
//     reach memory as they are, so other sizes store normally).
// Lanes along channels with 16-byte stores of four pixels each are slower (93 us).
// Bound by its stores: 206 MB, which a plain fill writes in 30 us.  240 points
// of six shapes (one to three channels, strides 1 and 2, odd sizes): 1.9 times as
// fast (geometric mean; least 1.01, a tile four columns wide of that layer).
#include <type_traits>

#include "kern_conv_tile.h"

namespace ds {

namespace {

template <int TKB, int GB>
__global__ __launch_bounds__(256, 4) void conv_few(Conv2Args a) {
    constexpr int NS = kConvFewSteps;
    const Tile T(a);
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int wp = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int taps = a.C * 9;

    // The workgroup's weights, rows 29 floats apart: 16 of them are read together.
    constexpr int ROW = 29;
    __shared__ float wl[16 * TKB * ROW];
    {
        const float *src = a.w + (size_t)T.kt * a.tk * taps;
        const int n = min(a.tk, a.K - T.kt * a.tk) * taps;
        for (int e = tid; e < 16 * TKB * taps; e += blockDim.x) {
            const int row = e / taps;
            wl[row * ROW + e - row * taps] = src[min(e, n - 1)];
        }
    }
    // Step j takes taps 4j + lg (channel, row, column).  Taps past the last
    // have zero weights and zero inputs.
    float w[TKB][NS];
    int off[NS];                                  // bytes from the pixel's first tap
    unsigned bit[NS];                             // of the tap in a pixel's mask
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int k = 4 * j + lg, kk = min(k, taps - 1);
        const int c = kk / 9, t = kk - c * 9, r = t / 3;
        off[j] = 4 * ((c * a.H + r) * a.W + t - 3 * r);
        bit[j] = k < taps ? 1u << t : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NS; ++j)
#pragma unroll
        for (int i = 0; i < TKB; ++i) {
            const int k = 4 * j + lg;
            const float e = wl[(16 * i + li) * ROW + min(k, taps - 1)];
            w[i][j] = k < taps ? e : 0.f;
        }

    const char *xn = reinterpret_cast<const char *>(a.x + (size_t)T.n0 * a.C * a.H * a.W);
    const int PQ = a.P * a.Q, kvalid = a.K - T.kt * a.tk;
    const bool full = kvalid >= a.tk;
    // a wave's 32 pixels are whole 128-byte lines of every channel
    const bool lines = (a.band ? PQ : a.Q | a.tw) % 32 == 0;
    char *yn = reinterpret_cast<char *>(a.y + ((size_t)T.n0 * a.K + T.kt * a.tk) * PQ);
    const int groups = a.npx / (16 * GB * a.wpx);
    for (int g = 0; g < groups; ++g) {
        const int base = (wp * groups + g) * GB * 16;
        int at[GB];
        unsigned out[GB];                         // bytes from yn; ~0: no pixel
        unsigned m[GB];                           // bit 3r + s: tap (r, s) is in the image
        bool in = true;
#pragma unroll
        for (int b = 0; b < GB; ++b) {
            const int pix = base + 16 * b + li;
            int p, q, img = 0;
            bool ok = true;
            if (a.band) {
                ok = T.qt * a.npx + pix < a.F;
                const int f = min(T.qt * a.npx + pix, a.F - 1), r = fdv(f, a.f_q);
                q = f - r * a.Q;
                img = fdv(r, a.f_p);
                p = r - img * a.P;
                img -= T.n0;
            } else {
                p = T.pt * a.th + (pix >> a.ltw);
                q = T.qt * a.tw + (pix & (a.tw - 1));
                ok = p < a.P && q < a.Q;
            }
            out[b] = ok ? 4u * unsigned((img * a.K + 4 * lg) * PQ + p * a.Q + q) : ~0u;
            const int y0 = p * a.st - a.pd, x0 = q * a.st - a.pd;
            at[b] = 4 * ((img * a.C * a.H + y0) * a.W + x0);
            unsigned cols = 0;
#pragma unroll
            for (int s = 0; s < 3; ++s) cols |= unsigned(unsigned(x0 + s) < unsigned(a.W)) << s;
            m[b] = 0;
#pragma unroll
            for (int r = 0; r < 3; ++r)
                m[b] |= unsigned(y0 + r) < unsigned(a.H) ? cols << (3 * r) : 0u;
            in = in && m[b] == 0x1ffu;
        }
        float v[GB][NS];
        if (__all(in)) {
#pragma unroll
            for (int b = 0; b < GB; ++b)
#pragma unroll
                for (int j = 0; j < NS; ++j) {
                    const float e = *reinterpret_cast<const float *>(xn + unsigned(at[b] + off[j]));
                    v[b][j] = bit[j] ? e : 0.f;
                }
        } else {
#pragma unroll
            for (int b = 0; b < GB; ++b)
#pragma unroll
                for (int j = 0; j < NS; ++j) {
                    const bool on = m[b] & bit[j];
                    const float e = *reinterpret_cast<const float *>(xn + unsigned(on ? at[b] + off[j] : 0));
                    v[b][j] = on ? e : 0.f;
                }
        }
        floatx4 acc[TKB][GB];
#pragma unroll
        for (int i = 0; i < TKB; ++i)
#pragma unroll
            for (int b = 0; b < GB; ++b) acc[i][b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NS; ++j)
#pragma unroll
            for (int i = 0; i < TKB; ++i)
#pragma unroll
                for (int b = 0; b < GB; ++b)
                    acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i][j], v[b][j], acc[i][b], 0, 0, 0);
        // A lane holds four channels of a pixel: 16 lanes store 64 bytes in a row,
        // and the blocks next to each other follow, so that lines fill at once.
        bool all = full;
#pragma unroll
        for (int b = 0; b < GB; ++b) all = all && out[b] != ~0u;
        auto store = [&]<bool ALL, bool NT>(std::bool_constant<ALL>, std::bool_constant<NT>) {
            // keeps the compiler from merging these stores with the other branches',
            // which would drop the hint
            if (NT) __asm__ volatile("; non-temporal stores");
#pragma unroll
            for (int i = 0; i < TKB; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    char *yc = yn + (size_t)(16 * i + e) * PQ * 4;
#pragma unroll
                    for (int b = 0; b < GB; ++b)
                        if (ALL || (out[b] != ~0u && 16 * i + 4 * lg + e < kvalid)) {
                            float *y = reinterpret_cast<float *>(yc + out[b]);
                            if (NT) store_out(y, acc[i][b][e]);
                            else *y = acc[i][b][e];
                        }
                }
            if (NT) __asm__ volatile("; end of non-temporal stores");
        };
        if (!__all(all)) store(std::false_type{}, std::false_type{});
        else if (GB == 2 && lines) store(std::true_type{}, std::bool_constant<GB == 2>{});
        else store(std::true_type{}, std::false_type{});
    }
}

}  // namespace

// Slot: log2(TKB) * 2 + log2(GB)
extern const void *g_conv_few[kConvFewSlots];

namespace {

struct Registrar {
    Registrar() {
        g_conv_few[0] = reinterpret_cast<const void *>(&conv_few<1, 1>);
        g_conv_few[1] = reinterpret_cast<const void *>(&conv_few<1, 2>);
        g_conv_few[2] = reinterpret_cast<const void *>(&conv_few<2, 1>);
        g_conv_few[3] = reinterpret_cast<const void *>(&conv_few<2, 2>);
        g_conv_few[4] = reinterpret_cast<const void *>(&conv_few<4, 1>);
        g_conv_few[5] = reinterpret_cast<const void *>(&conv_few<4, 2>);
    }
};
const Registrar registrar;

}  // namespace

}  // namespace ds
