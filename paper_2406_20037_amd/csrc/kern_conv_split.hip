// Split-operand 3x3 conv for gfx950 (conv mfma = 2 and 3 at unroll depth 1): fp32
// products on the bf16 matrix cores.
//
// Every operand is written as the sum of three bf16 values, x = x0 + x1 + x2
// (x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1): 24 bits, so the sum
// is exact), and a product of two operands becomes the six products x_i * w_j
// with i + j <= 2, each a v_mfma_f32_32x32x16_bf16 accumulating in fp32, the
// smallest first.  What is left out is below 2^-24 of the product.  Six bf16
// MFMAs take 6/16 of the cycles of the fp32 MFMAs they replace, and round less
// often: against fp64 the error is 0.8 of the fp32 MFMA program's (3x3 over 64
// channels: 3.6e-7 against 4.3e-7 of the result's 2-norm).
//
// That holds output by output, for every finite input: a workgroup whose
// operands or outputs lie where it would not runs its tile again on fp32 MFMAs
// (kExact and what follows it, below).  Sums of bf16 values in place of fp32 operands:
// Henry, Tang, Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype
// For Higher-Precision Computations", ARITH 2019.
//
// A workgroup computes the tile of the fp32 program (conv_mfma2): tk channels x
// th * tw pixels, four waves of 32 TB channels x 32 NB pixels.  Its reduction
// runs in stages of eight channels; a stage's operands sit in LDS as bf16
// planes, eight channels (16 bytes a plane, one MFMA operand) at a halo position
// or weight tap, so the loop reads them with one ds_read_b128 each and the
// splitting is done once per element instead of once per tap and wave.  An MFMA
// step takes two taps (one per half-wave); the tenth tap is zero weights.
//
// What bounds it: two waves a SIMD with two barriers a stage and operands read
// from LDS.  The matrix cores are busy for 58% of the cycles on 16x64x224x224, 60%
// on 16x512x28x28 (8 splits) and 42% on 16x256x56x56 in bands of 128 pixels (a wave
// of 64 x 32 reads 9 operands for 12 MFMAs, one of 64 x 64 12 for 24); bank
// conflicts are 19 to 31% of the LDS-active cycles.  With the padded tap the first
// runs 1.16 PFLOP/s of bf16 products; the library's product of 8192^2 matrices
// 1.40 on the same card.  fp32 MFMAs hold the vector unit, bf16 ones do not: 64
// vector instructions between 32 of them cost nothing, but only between MFMAs of
// the same wave, so the next stage is split between the MFMAs of this one and kept
// in registers until the planes in LDS are free (splitting it after the loop, when
// this was tried: 28x28x512 392 us against 361).  VGG-16 at batch 16, against the
// fp32 program of the same schedule: 64x224x224 532 -> 338 us, 512x28x28 (8
// reduction splits, their reduce included) 571 -> 348, 512x14x14 (16 splits)
// 177 -> 130.  The LDS it reserves is what the point's geometry states, the double
// buffer of the fp32 program, which with large chunks is more than it uses.
#include <type_traits>

#include "kern_conv_tile.h"

namespace ds {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
    const bf16x2 r = {(__bf16)a, (__bf16)b};
    unsigned p = __builtin_bit_cast(unsigned, r);
    // keeps the conversion of the pair from being repeated for one half
    __asm__("" : "+v"(p));
    return p;
}

// The three bf16 planes of two floats (each plane packed in one word).
__device__ __forceinline__ void split_pair(float x, float y, unsigned (&p)[3]) {
    p[0] = pack_bf16(x, y);
    x -= __uint_as_float(p[0] << 16);
    y -= __uint_as_float(p[0] & 0xffff0000u);
    p[1] = pack_bf16(x, y);
    x -= __uint_as_float(p[1] << 16);
    y -= __uint_as_float(p[1] & 0xffff0000u);
    p[2] = pack_bf16(x, y);
}

// Where the split products are as good as fp32 ones.  The bf16 MFMA keeps
// denormals, in its operands and its sums, so a plane holds multiples of 2^-133
// and a sum multiples of 2^-149, as an fp32 one does.
//   - From kExact = 2^-110 on, an operand's last bit (2^-23 of it) is at least
//     2^-133: its planes add up to it.  Smaller ones may lose up to 2^-134.
//   - The products of operands whose product is kWhole = 2^-100 or more have,
//     plane by plane, no bit below 2^-149.  Those of smaller ones may lose 2^-149
//     each.
//   - What a term loses either way is below 2^-92 where no operand is above
//     kLarge = 2^40.  An output of kSmall = 2^-40 or more then loses less than 2^-52
//     of itself a term, nothing beside the rounding of its fp32 sums.
// So a loop that meets a large operand, or leaves a small output (zero among
// them), looks at its operands again for the first two.  The loop itself only keeps
// their largest magnitude, one instruction a pair (14x14x512: 131.8 -> 133.0 us);
// their smallest but zero takes three (132.0 -> 136.4 us).  Where every tile looks
// again 64x224x224 takes 426 us, where every tile runs again 970 to 1020.
constexpr float kLarge = 0x1p40f, kSmall = 0x1p-40f;
// The largest and smallest of three magnitudes, NaN if any is (v_maximum3_f32).
__device__ __forceinline__ float max3(float m, float a, float b) {
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(a), fabsf(b)), m);
}
__device__ __forceinline__ float min3(float m, float a, float b) {
    return __builtin_elementwise_minimum(__builtin_elementwise_minimum(fabsf(a), fabsf(b)), m);
}
// Magnitudes as twice their bits less one: zero, which is exact, is the largest.
__device__ __forceinline__ unsigned mag(float v) { return 2u * __float_as_uint(v) - 1u; }
constexpr unsigned kExact = 2u * (unsigned(127 - 110) << 23) - 1u;
constexpr unsigned kWhole = 2 * 127 - 100;   // sum of the biased exponents

// The three bf16 planes of the eight channels of a unit, 16 bytes each; largest
// is kept at the largest magnitude split so far.
struct Planes {
    uintx4 q[3];
};
__device__ __forceinline__ void split_unit(const float (&v)[8], Planes &o, float &largest) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        largest = max3(largest, v[2 * j], v[2 * j + 1]);
        unsigned p[3];
        split_pair(v[2 * j], v[2 * j + 1], p);
#pragma unroll
        for (int i = 0; i < 3; ++i) o.q[i][j] = p[i];
    }
}
__device__ __forceinline__ void store_unit(char *dst, const Planes &o) {
#pragma unroll
    for (int i = 0; i < 3; ++i) *reinterpret_cast<uintx4 *>(dst + 16 * i) = o.q[i];
}

// Workgroup barrier for LDS only: loads from global memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int TB, int NB>
__global__ __launch_bounds__(256, 2) void conv_split(Conv2Args a) {
    constexpr int HU = kConvSplitHalo, WU = (32 * TB * 9 + 255) / 256, U = HU + WU;
    constexpr int STEPS = 5;                      // 9 taps, two a step
    constexpr int ROWB = kConvSplitRow;
    extern __shared__ float smem[];
    char *lds = reinterpret_cast<char *>(smem);
    const Tile T(a);
    if (T.ci0 >= T.ci1) return;

    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63;
    const int wp = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lg = lane >> 5;
    const int HW = a.H * a.W;
    const int hy0 = T.pt * a.th * a.st - a.pd;
    const int hx0 = (a.band ? 0 : T.qt * a.tw * a.st) - a.pd;
    const int kvalid = a.K - T.kt * a.tk;
    const int c_beg = T.ci0 * a.tc, c_end = min(T.ci1 * a.tc, a.C);
    const int stages = (c_end - c_beg) >> 3;
    const char *xb = reinterpret_cast<const char *>(a.x + ((size_t)T.n0 * a.C + c_beg) * HW);
    const char *wb = reinterpret_cast<const char *>(a.w + ((size_t)T.kt * a.tk * a.C + c_beg) * 9);
    const int nh = a.scs, nw = a.tk * 9;

    // Source (byte offset from the stage's first channel; -1: outside the
    // image) and LDS position of this thread's units; a unit is eight channels
    // at one halo position or one weight tap.  Threads past the last unit
    // repeat it.
    int src[U], dw[WU];
#pragma unroll
    for (int u = 0; u < HU; ++u) {
        const int e = min(u * nthr + tid, nh - 1);
        const int hy = fdv(e, a.f_sws), hx = e - hy * a.sws;
        int gy, img = 0;
        if (a.band) {
            const int gr = T.g0 + hy;
            img = fdv(gr, a.f_hp);
            gy = gr - img * a.hp - a.pd;
        } else {
            gy = hy0 + hy;
        }
        const int gx = hx0 + hx;
        const bool in = hy < T.rows && gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
        src[u] = in ? 4 * ((img * a.C * a.H + gy) * a.W + gx) : -1;
    }
#pragma unroll
    for (int u = 0; u < WU; ++u) {
        const int e = min(u * nthr + tid, nw - 1);
        const int row = e / 9, t = e - row * 9;
        src[HU + u] = 4 * (min(row, kvalid - 1) * a.C * 9 + t);
        dw[u] = row * ROWB + 48 * t;
    }
    auto dst = [&](int u) {
        return lds + (u < HU ? a.sxo + 48 * min(u * nthr + tid, nh - 1) : dw[max(u - HU, 0)]);
    };
    float raw[U][8];
    // unit u of stage s; past the last stage every lane reads one address
    auto load = [&](int u, int s) {
        const int on = s < stages ? -1 : 0;
        const char *b = u < HU ? xb + (size_t)(s & on) * 8 * HW * 4 : wb + (size_t)(s & on) * 8 * 9 * 4;
        const unsigned o = unsigned(max(src[u], 0) & on);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            raw[u][j] = *reinterpret_cast<const float *>(b + (u < HU ? (size_t)j * HW * 4 : j * 9 * 4) + o);
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load(u, 0);

    // zeros: halo positions outside the image, the weights of the padding tap
#pragma unroll
    for (int u = 0; u < HU; ++u)
        if (src[u] < 0) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                *reinterpret_cast<uintx4 *>(dst(u) + 16 * i) = uintx4{0u, 0u, 0u, 0u};
        }
    for (int e = tid; e < 3 * a.tk; e += nthr) {
        const int row = e / 3, k = e - row * 3;
        *reinterpret_cast<uintx4 *>(lds + row * ROWB + 48 * 9 + 16 * k) = uintx4{0u, 0u, 0u, 0u};
    }

    // lane bases (bytes), and the offset of step t's tap 2t + lg from a
    // pixel's halo position (the padding tap: the last one's)
    int bb[NB], off[STEPS / 2 + 1];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int pix = (wp * NB + b) * 32 + li;
        int pos;
        if (a.band) {
            const int f = min(T.qt * a.npx + pix, a.F - 1);
            const int r = fdv(f, a.f_q), q = f - r * a.Q;
            const int img = fdv(r, a.f_p), p = r - img * a.P;
            pos = ((img - T.n0) * a.hp + p * a.st - T.g0) * a.sws + q * a.st;
        } else {
            const int py = pix >> a.ltw, px = pix & (a.tw - 1);
            pos = py * a.st * a.sws + px * a.st;
        }
        bb[b] = a.sxo + 48 * pos;
    }
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
        const int u0 = 2 * t, u1 = cmin(2 * t + 1, 8);
        const int o = 48 * (lg ? u1 / 3 * a.sws + u1 % 3 : u0 / 3 * a.sws + u0 % 3);
        if (t & 1) off[t / 2] |= o << 16;      // both below 2^15: halos of at most 512 positions
        else off[t / 2] = o;
    }
    const int ab = li * ROWB + 48 * lg;

    floatx16 acc[TB][NB];
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[i][b] = floatx16{};

    struct Ops {
        bf16x8 A[TB][3], B[NB][3];
    };
    auto read = [&](int t, Ops &o) {
#pragma unroll
        for (int i = 0; i < TB; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                o.A[i][k] = *reinterpret_cast<const bf16x8 *>(lds + ab + i * 32 * ROWB + 96 * t + 16 * k);
        const int ot = t & 1 ? off[t / 2] >> 16 : off[t / 2] & 0xffff;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                o.B[b][k] = *reinterpret_cast<const bf16x8 *>(lds + bb[b] + ot + 16 * k);
    };
    auto mma = [&](const Ops &o) {
        constexpr int pa[6] = {0, 2, 1, 0, 1, 0}, pb[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
        for (int e = 0; e < 6; ++e)
#pragma unroll
            for (int i = 0; i < TB; ++i)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[i][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.A[i][pa[e]], o.B[b][pb[e]],
                                                                        acc[i][b], 0, 0, 0);
    };
    // The last stage has no next one to split: a build of its own saves that work.
    // One stage of eight channels, 8x8x100x100: 16.6 -> 14.7 us, where the fp32
    // program takes 14.5; 14x14x512 in 16 splits of four stages: 1%.  For waves of
    // 64 x 64 it spills, and their stages slow down by 1 to 4%.
    constexpr bool TAIL = TB * NB < 4;
    Planes pl[U];
    float largest = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        split_unit(raw[u], pl[u], largest);
        if (!TAIL || stages > 1) load(u, 1);
    }
    // each step's MFMAs, with the split of one unit of the next stage and the
    // loads of the one after it between them
    auto run_stage = [&]<bool LAST>(std::bool_constant<LAST>, int s) {
        if (s > 0) lds_barrier();       // every wave is past its reads of the last stage
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u >= HU || src[u] >= 0) store_unit(dst(u), pl[u]);
        lds_barrier();
        Ops o[2];
        read(0, o[0]);
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
            if (t + 1 < STEPS) read(t + 1, o[(t + 1) & 1]);
            if (!LAST && t < U) {
                split_unit(raw[t], pl[t], largest);
                load(t, s + 2);
            }
            mma(o[t & 1]);
            constexpr int NM = 6 * TB * NB;
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (m < 3 * (TB + NB)) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                if (LAST) continue;
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
                if (m >= NM - 8) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int s = 0; s < stages - TAIL; ++s) run_stage(std::false_type{}, s);
    if (TAIL) run_stage(std::true_type{}, stages - 1);

    // Infinities, NaN and values that round up past bf16's largest leave NaN or
    // infinities in the accumulators.  With any of them, or operands too small for their
    // outputs, the workgroup's tile runs again on fp32 MFMAs: its operands are
    // shared between the waves, so one vote decides for all.
    float large = 0.f, small = kSmall;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        // A rectangle's pixels past the image are zeros that nobody reads, and no
        // reason to look again (8x16x100x90 in rectangles of 8x16: 45.2 us with them,
        // 38.4 without).
        const int pix = (wp * NB + b) * 32 + li;
        const bool kept = a.band || (T.pt * a.th + (pix >> a.ltw) < a.P &&
                                     T.qt * a.tw + (pix & (a.tw - 1)) < a.Q);
        float least = kSmall;
#pragma unroll
        for (int i = 0; i < TB; ++i)
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                large = max3(large, acc[i][b][v], acc[i][b][v + 1]);
                least = min3(least, acc[i][b][v], acc[i][b][v + 1]);
            }
        small = kept ? __builtin_elementwise_minimum(small, least) : small;
    }
    const int vote = (__any(!(large < INFINITY)) ? 1 : 0) |
                     (__any(!(largest < kLarge) || small < kSmall) ? 2 : 0);
    unsigned *votes = reinterpret_cast<unsigned *>(lds);
    lds_barrier();
    if (lane == 0) votes[wp] = vote;
    lds_barrier();
    int again = 0;
    for (int w = 0; w < a.wpx; ++w) again |= votes[w];
    again = __builtin_amdgcn_readfirstlane(again);
    if (again == 2) {
        unsigned least[2] = {~0u, ~0u};           // of the image, of the weights
        for (int s = 0; s < stages; ++s)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                load(u, s);
#pragma unroll
                for (int j = 0; j < 8; ++j) least[u >= HU] = min(least[u >= HU], mag(raw[u][j]));
            }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
            for (int d = 1; d < 64; d *= 2) least[k] = min(least[k], unsigned(__shfl_xor(int(least[k]), d)));
            if (lane == 0) votes[4 + 4 * k + wp] = least[k];
        }
        lds_barrier();
#pragma unroll
        for (int k = 0; k < 2; ++k)
            for (int w = 0; w < a.wpx; ++w) least[k] = min(least[k], votes[4 + 4 * k + w]);
        const bool lost = min(least[0], least[1]) < kExact || (least[0] >> 24) + (least[1] >> 24) < kWhole;
        again = __builtin_amdgcn_readfirstlane(int(lost));
    }
    lds_barrier();
    if (again & 1) {
        // the lane's coordinates anew, so that nothing of this path is kept in
        // registers through the loop above
        int ln = lane;
        __asm__ volatile("" : "+v"(ln));
        const int lj = ln & 31, lh = ln >> 5;
#pragma unroll
        for (int i = 0; i < TB; ++i)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[i][b] = floatx16{};
        const float *pw[TB], *px[NB];
        int at[NB];
        unsigned ok[NB];                          // bit t: tap t is inside the image
#pragma unroll
        for (int i = 0; i < TB; ++i)
            pw[i] = a.w + ((size_t)(T.kt * a.tk + min(i * 32 + lj, kvalid - 1)) * a.C + c_beg + lh) * 9;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int pix = (wp * NB + b) * 32 + lj;
            int img = T.n, p, q;
            if (a.band) {
                const int f = min(T.qt * a.npx + pix, a.F - 1), r = fdv(f, a.f_q);
                q = f - r * a.Q;
                img = fdv(r, a.f_p);
                p = r - img * a.P;
            } else {
                p = T.pt * a.th + (pix >> a.ltw);
                q = T.qt * a.tw + (pix & (a.tw - 1));
            }
            const int y0 = p * a.st - a.pd, x0 = q * a.st - a.pd;
            px[b] = a.x + ((size_t)img * a.C + c_beg + lh) * HW;
            at[b] = y0 * a.W + x0;
            ok[b] = 0;
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int y = y0 + t / 3, x = x0 + t % 3;
                ok[b] |= unsigned(y >= 0 && y < a.H && x >= 0 && x < a.W) << t;
            }
        }
        for (int c = 0; c < 8 * stages; c += 2) {
            float A[TB][9], B[NB][9];
#pragma unroll
            for (int i = 0; i < TB; ++i)
#pragma unroll
                for (int t = 0; t < 9; ++t) A[i][t] = pw[i][c * 9 + t];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const bool in = ok[b] >> t & 1;
                    const float v = px[b][(size_t)c * HW + (in ? at[b] + t / 3 * a.W + t % 3 : 0)];
                    B[b][t] = in ? v : 0.f;
                }
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int i = 0; i < TB; ++i)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[i][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(A[i][t], B[b][t], acc[i][b],
                                                                        0, 0, 0);
        }
    }

    // Output through LDS, 16 channels x up to 64 pixels of a wave at a time, as
    // in conv2_body.  A 32x32 block leaves lane (lg, li) rows 8*(v/4) + 4*lg +
    // v%4 of column li.
    constexpr int BG = NB < 2 ? NB : 2;
    constexpr int ROW = 32 * BG + 4;
    constexpr int LPR = 8 * BG;
    float *stage = smem + wp * (16 * 68);
    float *yn = out_base(a, T);
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int b0 = 0; b0 < NB; b0 += BG)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int b = 0; b < BG; ++b)
#pragma unroll
                    for (int v = 0; v < 8; ++v)
                        stage[(8 * (v / 4) + 4 * lg + v % 4) * ROW + b * 32 + li] =
                            acc[i][b0 + b][8 * h + v];
#pragma unroll
                for (int r0 = 0; r0 < 16; r0 += 64 / LPR) {
                    const int row = r0 + lane / LPR, c4 = lane % LPR;
                    const floatx4 val = *reinterpret_cast<const floatx4 *>(stage + row * ROW + 4 * c4);
                    put(a, T, yn, T.kt * a.tk + i * 32 + h * 16 + row,
                            (wp * NB + b0) * 32 + 4 * c4, val);
                }
            }
}

}  // namespace

// Slot: log2(TB) * 2 + log2(NB)
extern const void *g_conv_split[kConvSplitSlots];

namespace {

// Two waves per SIMD (256 registers): the operands of a step are read while the
// step before multiplies.  Three waves without that ran slower when it was tried
// (28x28x512 379 us against 363, 14x14x512 147 against 137).
struct Registrar {
    Registrar() {
        g_conv_split[0] = reinterpret_cast<const void *>(&conv_split<1, 1>);
        g_conv_split[1] = reinterpret_cast<const void *>(&conv_split<1, 2>);
        g_conv_split[2] = reinterpret_cast<const void *>(&conv_split<2, 1>);
        g_conv_split[3] = reinterpret_cast<const void *>(&conv_split<2, 2>);
    }
};
const Registrar registrar;

}  // namespace

}  // namespace ds
