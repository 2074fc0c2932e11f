// Row-major fp32 matmul kernel family for gfx950: C[M,N] = A[M,K] * B[K,N].
//
// A workgroup of 256 threads computes a BM x BN tile of C over the K-tiles of
// its split.  Each K-tile (BK deep) is staged through LDS:
//   As[BM][BK]  k contiguous in 16-byte slots; slot j of row r is stored at
//               j ^ swz(r), so the 16-byte reads of eight consecutive rows at
//               one k land on distinct banks without padding,
//   Bs[BK][BN]  n contiguous.
// MFMA tiles with two or more stages run pipelined (mm_mfma_pipe): K-tiles travel
// straight from global memory into LDS (global_load_lds, no register staging),
// 16 bytes per lane when rows of A and B are whole aligned 16-byte groups, else
// 4, and the next ST-1 K-tiles are in flight while the current one is consumed
// (ST = 3 stages when they fit in LDS, else 2).  The other kernels do the same
// without the pipelined reads when every tile is also full (a.direct), and
// otherwise stage tiles through registers with bounds checks (zero outside A
// and B), written with dbuf to the other LDS stage after the current one is
// consumed.
//
//   mm_valu: VALU FMA; thread (ty, tx) of a 16x16 grid owns RM rows x RN
//            columns (contiguous).
//   mm_mfma: KG groups of 2x2 waves; each wave a WM x WN tile of fp32 MFMA
//            blocks (v_mfma_f32_32x32x2f32 when WM, WN >= 32, else
//            v_mfma_f32_16x16x4f32).  Group g consumes the g-th of KG equal
//            k ranges of every K-tile; the groups' accumulators are summed
//            through LDS at the end (two waves per SIMD hide each other's
//            waits).  Lane group g feeds k = kk + VEC*g + v (v < VEC) to both
//            operands, so one VEC-wide LDS read of A serves VEC MFMA steps.
// A split (ks > 1) stores its partial C tile; a reduce kernel sums the splits
// into C in split order.
#include <utility>

#include "kern_common.h"

namespace ds {

namespace {

#define DS_GLOBAL(p) ((const __attribute__((address_space(1))) void *)(p))
#define DS_LOCAL(p) ((__attribute__((address_space(3))) void *)(p))

// Tiles in groups of a.gm tile rows (chosen on the host: the XCD's range of
// tiles square in elements), column-major inside a group, so the contiguous
// tile range of one XCD touches few rows of A and columns of B.
__device__ __forceinline__ void mm_tile_coords(const MatmulArgs &a, int &mt, int &nt, int &z) {
    const int tiles = a.tiles_m * a.tiles_n;
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    z = t / tiles;
    const int r = t - z * tiles;
    const int gm = a.gm;
    const int gsz = gm * a.tiles_n;
    const int g = r / gsz, first = g * gm;
    const int rows = min(a.tiles_m - first, gm);
    const int rg = r - g * gsz;
    mt = first + rg % rows;
    nt = rg / rows;
}

// Lane exchange inside quads of lanes (DPP quad_perm).
template <int CTRL>
__device__ __forceinline__ float quad_perm(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}

// 4x4 transpose across the four lanes of a quad: lane b's x[j] becomes lane
// j's x[b].  Two rounds of 2x2 swaps: lanes b, b^1 on register pairs (0,1),
// (2,3), then lanes b, b^2 on pairs (0,2), (1,3).
__device__ __forceinline__ void quad_transpose(float (&x)[4], int b) {
    const bool o1 = b & 1, o2 = b & 2;
#pragma unroll
    for (int p = 0; p < 4; p += 2) {
        const float r = quad_perm<0xB1>(o1 ? x[p] : x[p + 1]);   // lanes [1,0,3,2]
        x[p] = o1 ? r : x[p];
        x[p + 1] = o1 ? x[p + 1] : r;
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const float r = quad_perm<0x4E>(o2 ? x[p] : x[p + 2]);   // lanes [2,3,0,1]
        x[p] = o2 ? r : x[p];
        x[p + 2] = o2 ? x[p + 2] : r;
    }
}

// Slot permutation of A row r (BK/4 slots per row).
template <int BK>
__device__ __forceinline__ int a_swz(int r) {
    constexpr int SPR = BK / 4;
    if constexpr (SPR >= 8) return r & 7;
    else return ((r * SPR) >> 3) & (SPR - 1);
}

// Float offset of A element (row, k) inside a stage.
template <int BK>
__device__ __forceinline__ int a_off(int row, int k) {
    return row * BK + (((k >> 2) ^ a_swz<BK>(row)) << 2) + (k & 3);
}

// Waits for every vector-memory operation of the wave, then for LDS, then
// barriers the workgroup without a memory fence (the waits above make the LDS
// writes of every wave complete before any wave passes).
// s_waitcnt immediate for vmcnt(n) (expcnt, lgkmcnt not waited on).
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x70 | 0xF00; }

template <int VM = 0>
__device__ __forceinline__ void stage_barrier() {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(VM));
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// Global -> LDS copy of one full, aligned K-tile (16 bytes per lane per
// instruction; the LDS destination of a wave's instruction is contiguous).
template <int BM, int BN, int BK, int NT>
__device__ __forceinline__ void direct_load(const MatmulArgs &a, int m0, int n0, int kt, float *As,
                                            float *Bs) {
    constexpr int SPR = BK / 4, A4 = BM * SPR, B4 = BK * BN / 4;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < (A4 + NT - 1) / NT; ++j) {
        const int base = j * NT + wid * 64;
        const int c = base + lane;
        if (A4 % NT == 0 || c < A4) {
            const int row = c / SPR, slot = c % SPR;
            const float *src = a.A + (size_t)(m0 + row) * a.K + kt * BK + 4 * (slot ^ a_swz<BK>(row));
            __builtin_amdgcn_global_load_lds(DS_GLOBAL(src), DS_LOCAL(As + base * 4), 16, 0, 0);
        }
    }
#pragma unroll
    for (int j = 0; j < (B4 + NT - 1) / NT; ++j) {
        const int base = j * NT + wid * 64;
        const int c = base + lane;
        if (B4 % NT == 0 || c < B4) {
            const int k = c / (BN / 4), n4 = c % (BN / 4);
            const float *src = a.B + (size_t)(kt * BK + k) * a.N + n0 + 4 * n4;
            __builtin_amdgcn_global_load_lds(DS_GLOBAL(src), DS_LOCAL(Bs + base * 4), 16, 0, 0);
        }
    }
}

// Global -> register staging of one K-tile (float4 slots; zero outside A, B).
template <int BM, int BN, int BK, int NT>
struct Stager {
    static constexpr int A4 = BM * BK / 4, B4 = BK * BN / 4;
    static constexpr int AL = (A4 + NT - 1) / NT, BL = (B4 + NT - 1) / NT;
    floatx4 ra[AL], rb[BL];

    __device__ __forceinline__ void load(const MatmulArgs &a, int m0, int n0, int kt) {
        const int tid = threadIdx.x;
#pragma unroll
        for (int u = 0; u < AL; ++u) {
            const int e = tid + NT * u;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (A4 % NT == 0 || e < A4) {
                const int m = e / (BK / 4), k4 = e - m * (BK / 4);
                const int gm = m0 + m, gk = kt * BK + 4 * k4;
                if (gm < a.M) {
                    const float *src = a.A + (size_t)gm * a.K + gk;
                    if (a.vecA && gk + 3 < a.K) {
                        v = *reinterpret_cast<const floatx4 *>(src);
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (gk + i < a.K) v[i] = src[i];
                    }
                }
            }
            ra[u] = v;
        }
#pragma unroll
        for (int u = 0; u < BL; ++u) {
            const int e = tid + NT * u;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (B4 % NT == 0 || e < B4) {
                const int k = e / (BN / 4), n4 = e - k * (BN / 4);
                const int gk = kt * BK + k, gn = n0 + 4 * n4;
                if (gk < a.K) {
                    const float *src = a.B + (size_t)gk * a.N + gn;
                    if (a.vecB && gn + 3 < a.N) {
                        v = *reinterpret_cast<const floatx4 *>(src);
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (gn + i < a.N) v[i] = src[i];
                    }
                }
            }
            rb[u] = v;
        }
    }

    __device__ __forceinline__ void store(float *As, float *Bs) const {
        const int tid = threadIdx.x;
#pragma unroll
        for (int u = 0; u < AL; ++u) {
            const int e = tid + NT * u;
            if (A4 % NT == 0 || e < A4) {
                const int m = e / (BK / 4), k4 = e - m * (BK / 4);
                *reinterpret_cast<floatx4 *>(As + a_off<BK>(m, 4 * k4)) = ra[u];
            }
        }
#pragma unroll
        for (int u = 0; u < BL; ++u) {
            const int e = tid + NT * u;
            if (B4 % NT == 0 || e < B4) {
                const int k = e / (BN / 4), n4 = e - k * (BN / 4);
                *reinterpret_cast<floatx4 *>(Bs + k * BN + 4 * n4) = rb[u];
            }
        }
    }
};

// The K-loop shared by both families: stages K-tiles [kt0, kt1) through LDS
// and calls compute(As, Bs) on each.  NT threads; ST LDS stages (1: stage,
// barrier, compute; >= 2: the next tiles are in flight during compute).
template <int BM, int BN, int BK, int ST, int NT, class F>
__device__ __forceinline__ void k_loop(const MatmulArgs &a, int m0, int n0, int kt0, int kt1,
                                       float *smem, F &&compute) {
    constexpr int STAGE = BM * BK + BK * BN;
    if (a.direct) {
        if constexpr (ST >= 2) {
            // Each thread issues the same L copies per tile when the tile
            // divides into whole rounds of NT threads; then waiting until at
            // most L*(ST-2) copies are outstanding means tile kt has landed.
            constexpr int A4 = BM * BK / 4, B4 = BK * BN / 4;
            constexpr bool EXACT = A4 % NT == 0 && B4 % NT == 0;
            constexpr int L = A4 / NT + B4 / NT;
#pragma unroll
            for (int p = 0; p < ST - 1; ++p)
                if (kt0 + p < kt1)
                    direct_load<BM, BN, BK, NT>(a, m0, n0, kt0 + p, smem + p * STAGE,
                                                smem + p * STAGE + BM * BK);
            int s = 0;
            for (int kt = kt0; kt < kt1; ++kt) {
                if (EXACT && ST > 2 && kt + ST - 2 < kt1) stage_barrier<EXACT ? L * (ST - 2) : 0>();
                else stage_barrier<0>();
                if (kt + ST - 1 < kt1) {
                    int sn = s + ST - 1;
                    if (sn >= ST) sn -= ST;
                    float *nx = smem + sn * STAGE;
                    direct_load<BM, BN, BK, NT>(a, m0, n0, kt + ST - 1, nx, nx + BM * BK);
                }
                compute(smem + s * STAGE, smem + s * STAGE + BM * BK);
                if (++s == ST) s = 0;
            }
        } else {
            for (int kt = kt0; kt < kt1; ++kt) {
                stage_barrier();
                direct_load<BM, BN, BK, NT>(a, m0, n0, kt, smem, smem + BM * BK);
                stage_barrier();
                compute(smem, smem + BM * BK);
            }
        }
        return;
    }
    Stager<BM, BN, BK, NT> st;
    if constexpr (ST >= 2) {
        st.load(a, m0, n0, kt0);
        st.store(smem, smem + BM * BK);
        __syncthreads();
        for (int kt = kt0; kt < kt1; ++kt) {
            const int s = (kt - kt0) & 1;
            const bool more = kt + 1 < kt1;
            if (more) st.load(a, m0, n0, kt + 1);
            compute(smem + s * STAGE, smem + s * STAGE + BM * BK);
            if (more) st.store(smem + (s ^ 1) * STAGE, smem + (s ^ 1) * STAGE + BM * BK);
            __syncthreads();
        }
    } else {
        for (int kt = kt0; kt < kt1; ++kt) {
            st.load(a, m0, n0, kt);
            __syncthreads();
            st.store(smem, smem + BM * BK);
            __syncthreads();
            compute(smem, smem + BM * BK);
        }
    }
}

template <int RM, int RN, int BK, int UF, int DB>
__global__ __launch_bounds__(256) void mm_valu(MatmulArgs a) {
    constexpr int BM = 16 * RM, BN = 16 * RN;
    constexpr int ST = mm_stages(BM, BN, BK, DB);
    constexpr int U4 = UF >= 4 ? UF / 4 : 1;
    extern __shared__ float smem[];
    int mt, nt, z;
    mm_tile_coords(a, mt, nt, z);
    const int kt0 = z * a.kps, kt1 = min(kt0 + a.kps, a.nkt);
    if (kt0 >= kt1) return;
    const int m0 = mt * BM, n0 = nt * BN;
    const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;

    float acc[RM][RN];
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j) acc[i][j] = 0.f;

    auto compute = [&](const float *As, const float *Bs) {
#pragma unroll U4
        for (int kk = 0; kk < BK; kk += 4) {
            floatx4 av[RM];
#pragma unroll
            for (int i = 0; i < RM; ++i)
                av[i] = *reinterpret_cast<const floatx4 *>(As + a_off<BK>(ty * RM + i, kk));
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float bv[RN];
                const float *brow = Bs + (kk + v) * BN + tx * RN;
                if constexpr (RN >= 4) {
#pragma unroll
                    for (int j = 0; j < RN; j += 4) {
                        const floatx4 b4 = *reinterpret_cast<const floatx4 *>(brow + j);
                        bv[j] = b4[0];
                        bv[j + 1] = b4[1];
                        bv[j + 2] = b4[2];
                        bv[j + 3] = b4[3];
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < RN; ++j) bv[j] = brow[j];
                }
#pragma unroll
                for (int i = 0; i < RM; ++i)
#pragma unroll
                    for (int j = 0; j < RN; ++j) acc[i][j] = fmaf(av[i][v], bv[j], acc[i][j]);
            }
        }
    };
    k_loop<BM, BN, BK, ST, 256>(a, m0, n0, kt0, kt1, smem, compute);

    float *cbase = a.ks > 1 ? a.part + (size_t)z * a.M * a.N : a.C;
#pragma unroll
    for (int i = 0; i < RM; ++i) {
        const int gm = m0 + ty * RM + i;
        if (gm >= a.M) continue;
        float *crow = cbase + (size_t)gm * a.N;
#pragma unroll
        for (int j = 0; j < RN; ++j) {
            const int gn = n0 + tx * RN + j;
            if (gn < a.N) crow[gn] = acc[i][j];
        }
    }
}

// Geometry of one wave group's MFMA work on a K-tile.
template <int WM, int WN, int BK, int KG>
struct MfmaShape {
    static constexpr bool BIG = WM >= 32 && WN >= 32;
    static constexpr int IM = BIG ? 32 : 16;          // MFMA output tile edge
    static constexpr int NG = 64 / IM;                // lane groups along k
    static constexpr int KR = BK / KG;                // k of every K-tile per wave group
    static constexpr int VEC = cmin(4, KR / NG);      // k values per lane per LDS read
    static constexpr int KGS = NG * VEC;              // k consumed per chunk
    static constexpr int NCH = KR / KGS;              // chunks per K-tile
    static constexpr int MB = WM / IM, NB = WN / IM;
    static constexpr int NV = BIG ? 16 : 4;           // accumulator values per lane
};

// Whether K-tiles run software-pipelined (mm_mfma_pipe) with copies of W floats
// per lane: at least two stages, every thread issuing the same number of copies
// per K-tile, at most 32, and at least two chunks per K-tile.  The loop waits for
// all copies but those of one K-tile, a count that must fit the six bits of the
// wait (63).  With two tiles of 32 copies in flight the counter is full before the
// last one, which then waits to be issued (W = 1: 64x64x64, 128x128x32, 256x256x16).
template <int WM, int WN, int BK, int DB, int KG, int W>
constexpr bool mm_pipelined() {
    using S = MfmaShape<WM, WN, BK, KG>;
    constexpr int BM = 2 * WM, BN = 2 * WN, NT = 256 * KG;
    return mm_stages(BM, BN, BK, DB) >= 2 && (BM * BK / W) % NT == 0 && (BK * BN / W) % NT == 0 &&
           (BM + BN) * BK / W / NT <= 32 && S::NCH >= 2;
}

// K-loop of global -> LDS copies, W floats per lane, with the LDS operand reads
// software-pipelined across MFMA chunks.  Rows of A past M and columns of B past
// N re-read the last one (their outputs are not stored); in the last K-tile,
// when K does not fill it, positions past K are written as zeros instead of
// copied.  W = 1 takes any alignment.  Bound by the MFMAs, which hold the vector
// unit: every vector instruction in the loop costs as much MFMA time, so it has
// none (addresses are scalar bases plus lane offsets, LDS stages immediates).
// 64x64x16 tiles: 1024^3 22.1 -> 20.3 us (106 TFLOP/s); 1003x1501x777 58.8 ->
// 28.4 us (staged through registers with checked loads before).  A chunk is one k step of every MFMA block of the wave
// (KGS k values).  The operands of chunk c + D are read while the MFMAs of
// chunk c run, from a ring of D + 1 operand sets (D = 3 with unroll >= 16 when
// the chunks of a K-tile divide into whole rings, else 1).  The stage barrier
// sits before the last D chunks of every K-tile: past it every wave has
// finished reading the current tile and the next tile has landed, so the next
// tile's first reads overlap the current tile's last MFMAs, and the stage of
// the tile just consumed is refilled in the next iteration.  Each K-tile's
// copies are spread over the chunks before the barrier.  Past the end of the
// split the last K-tile is loaded again into a stage nobody reads, so every
// iteration has the same copies in flight and the wait counts are constants.
template <int WM, int WN, int BK, int UF, int DB, int KG, int W, class Acc, int MB, int NB>
__device__ __forceinline__ void mm_mfma_pipe(const MatmulArgs &a, int m0, int n0, int kt0, int kt1,
                                             float *smem, Acc (&acc)[MB][NB]) {
    using S = MfmaShape<WM, WN, BK, KG>;
    constexpr int BM = 2 * WM, BN = 2 * WN, NT = 256 * KG;
    constexpr int ST = mm_stages(BM, BN, BK, DB);
    constexpr int STAGE = BM * BK + BK * BN;
    constexpr int AL = BM * BK / W / NT, BL = BK * BN / W / NT, L = AL + BL;
    constexpr int IM = S::IM, VEC = S::VEC, KGS = S::KGS, NCH = S::NCH;
    constexpr int D = UF >= 16 && NCH % 4 == 0 ? 3 : 1;
    constexpr int RG = D + 1;
    constexpr bool RING = NCH % RG == 0;   // chunk c always uses ring slot c % RG
    constexpr int PRE = NCH - D;           // chunks before the stage barrier
    constexpr int PER = (L + PRE - 1) / PRE;
    static_assert(PRE >= 1, "the copies of a tile are issued before its barrier");

    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wsc = __builtin_amdgcn_readfirstlane(wid);
    const int kg = wid >> 2, wq = wid & 3;
    const int wr = wq >> 1, wc = wq & 1;
    const int li = lane % IM, lg = lane / IM;

    // Copy j's position in the stage is (j * NT + thread) * W, its source row r of
    // A at k (slot permuted) or row k of B at column c; both from a base that
    // moves with the K-tile.
    auto a_src = [&](int j, int &row, int &k) {
        const int p = (j * NT + tid) * W;
        row = p / BK;
        k = ((((p % BK) >> 2) ^ a_swz<BK>(row)) << 2) + p % 4;
    };
    unsigned oa[AL], ob[BL];
#pragma unroll
    for (int j = 0; j < AL; ++j) {
        int row, k;
        a_src(j, row, k);
        row = min(m0 + row, a.M - 1);
        oa[j] = 4u * (unsigned(row - m0) * unsigned(a.K) + k);
    }
#pragma unroll
    for (int j = 0; j < BL; ++j) {
        const int p = (j * NT + tid) * W, k = p / BN, c = min(n0 + p % BN, a.N - W);
        ob[j] = 4u * (unsigned(k) * unsigned(a.N) + c);
    }
    const float *abase = a.A + (size_t)m0 * a.K;
    // copy j of K-tile kt into the stage at st (the LDS slot is wave-uniform);
    // TAIL: the tile may reach past K
    auto copy = [&]<bool TAIL>(std::bool_constant<TAIL>, int kt, float *st, int j) {
        const bool isa = j < AL;
        const int jb = j - AL;
        float *dst = st + (isa ? 0 : BM * BK) + ((isa ? j : jb) * NT + wsc * 64) * W;
        if constexpr (TAIL) {
            int row, k;
            if (isa) a_src(j, row, k);
            else k = (jb * NT + tid) * W / BN;
            if (kt * BK + k >= a.K) {
#pragma unroll
                for (int v = 0; v < W; ++v) dst[lane * W + v] = 0.f;
                return;
            }
        }
        const char *base = reinterpret_cast<const char *>(isa ? abase + (size_t)kt * BK
                                                              : a.B + (size_t)kt * BK * a.N);
        // scalar base plus 32-bit lane offset is an address form of the copy; with
        // either out of sight (summed or widened before the loop) each copy takes a
        // 64-bit vector addition
        __asm__("" : "+s"(base));
        unsigned &o = isa ? oa[isa ? j : 0] : ob[isa ? 0 : jb];
        __asm__ volatile("" : "+v"(o));
        if constexpr (W == 4)
            __builtin_amdgcn_global_load_lds(DS_GLOBAL(base + o), DS_LOCAL(dst), 16, 0, 0);
        else
            __builtin_amdgcn_global_load_lds(DS_GLOBAL(base + o), DS_LOCAL(dst), 4, 0, 0);
    };

    struct Ops {
        float a[MB][VEC];
        float b[VEC][NB];
    };
    const int arow = wr * WM + li;
    const int brow = BM * BK + wc * WN + li + (kg * S::KR + VEC * lg) * BN;
    auto read = [&](const float *st, int c, Ops &o) {
        const int k = kg * S::KR + c * KGS + VEC * lg;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const float *src = st + a_off<BK>(arow + i * IM, k);
            if constexpr (VEC == 4) {
                const floatx4 t = *reinterpret_cast<const floatx4 *>(src);
                o.a[i][0] = t[0];
                o.a[i][1] = t[1];
                o.a[i][2] = t[2];
                o.a[i][3] = t[3];
            } else if constexpr (VEC == 2) {
                const float2 t = *reinterpret_cast<const float2 *>(src);
                o.a[i][0] = t.x;
                o.a[i][1] = t.y;
            } else {
                o.a[i][0] = src[0];
            }
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v)
#pragma unroll
            for (int j = 0; j < NB; ++j) o.b[v][j] = st[brow + (c * KGS + v) * BN + j * IM];
    };
    auto mma = [&](const Ops &o) {
#pragma unroll
        for (int v = 0; v < VEC; ++v)
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    if constexpr (S::BIG)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.a[i][v], o.b[v][j],
                                                                        acc[i][j], 0, 0, 0);
                    else
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.a[i][v], o.b[v][j],
                                                                        acc[i][j], 0, 0, 0);
                }
    };
    // one LDS read between consecutive MFMAs of a chunk
    auto interleave = [&]() {
        constexpr int NM = VEC * MB * NB, NDS = MB + (VEC * NB + 1) / 2;
#pragma unroll
        for (int t = 0; t < NM; ++t) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (t < NDS && t + 1 < NM) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };

    // A K-tile that reaches past K is the last of the last split: the iterations
    // whose copies may touch it (and a prologue that does) take the checked copies,
    // some lanes of which issue nothing, so they wait for every copy in flight.  As
    // they count on no number of copies they load nothing again past the end, which
    // was most of a short loop (640x1284x85 in 64x32x64 tiles 10.4 -> 8.2 us,
    // 128x4000x36 in 32x32x32 4.86 -> 4.13, 1003x1501x777 28.4 -> 27.7).
    const bool tail = kt1 == a.nkt && a.K % BK != 0;
    const int kmain = tail ? max(kt0, kt1 - ST) : kt1;
    // prologue: K-tiles kt0 .. kt0+ST-2, then wait for the first
#pragma unroll
    for (int p = 0; p < ST - 1; ++p) {
        const int kt = min(kt0 + p, kt1 - 1);
        if (tail && kt0 + p >= kt1) break;
#pragma unroll
        for (int j = 0; j < L; ++j) {
            if (tail && kt == kt1 - 1) copy(std::true_type{}, kt, smem + p * STAGE, j);
            else copy(std::false_type{}, kt, smem + p * STAGE, j);
        }
    }
    if (tail) stage_barrier<0>();
    else stage_barrier<L * (ST - 2)>();
    Ops o[RG];
#pragma unroll
    for (int c = 0; c < D; ++c) read(smem, c, o[c]);

    // K-tile kt in stage s
    auto tile = [&]<bool TAIL>(std::bool_constant<TAIL> t, int kt, int s) {
        const int sp = s == 0 ? ST - 1 : s - 1, sn = s == ST - 1 ? 0 : s + 1;
        const float *cur = smem + s * STAGE, *nxt = smem + sn * STAGE;
        float *fill = smem + sp * STAGE;
        const int ktf = min(kt + ST - 1, kt1 - 1);
        const bool more = !TAIL || kt + ST - 1 < kt1;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (c == PRE) stage_barrier<TAIL ? 0 : L * (ST - 2)>();
            Ops &rd = RING ? o[(c + D) % RG] : o[D];
            if (c + D < NCH) read(cur, c + D, rd);
            else read(nxt, c + D - NCH, rd);
            mma(RING ? o[c % RG] : o[0]);
            if (c < PRE && more) {
#pragma unroll
                for (int q = 0; q < PER; ++q)
                    if (c * PER + q < L) copy(t, ktf, fill, c * PER + q);
            }
            interleave();
            if constexpr (!RING) {
#pragma unroll
                for (int r = 0; r < D; ++r) o[r] = o[r + 1];
            }
        }
    };
    int kt = kt0, s = 0;
    // Small tiles run the stages of the ring unrolled: their LDS addresses are
    // immediates then (an fp32 MFMA holds the vector unit an addition needs).
    if constexpr (NCH * VEC * MB * NB <= 32)
        for (; kt + ST <= kmain; kt += ST)
#pragma unroll
            for (int q = 0; q < ST; ++q) tile(std::false_type{}, kt + q, q);
    for (; kt < kmain; ++kt) {
        tile(std::false_type{}, kt, s);
        if (++s == ST) s = 0;
    }
    for (; kt < kt1; ++kt) {
        tile(std::true_type{}, kt, s);
        if (++s == ST) s = 0;
    }
    // the reloads past the end are still in flight
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
}

template <int WM, int WN, int BK, int UF, int DB, int KG>
__global__ __launch_bounds__(256 * KG) void mm_mfma(MatmulArgs a) {
    constexpr int BM = 2 * WM, BN = 2 * WN;
    constexpr int ST = mm_stages(BM, BN, BK, DB);
    constexpr int KR = BK / KG;                // k of every K-tile per wave group
    constexpr bool BIG = WM >= 32 && WN >= 32;
    constexpr int IM = BIG ? 32 : 16;          // MFMA output tile edge
    constexpr int NG = 64 / IM;                // lane groups along k
    static_assert(KR >= NG, "every wave group needs one k step per lane group");
    constexpr int VEC = cmin(4, KR / NG);      // k values per lane per LDS read
    constexpr int KGS = NG * VEC;              // k consumed per group step
    constexpr int MB = WM / IM, NB = WN / IM;
    constexpr int KSTEP = BIG ? 2 : 4;
    constexpr int UG = cmax(1, UF * KSTEP / KGS);
    using Acc = typename std::conditional<BIG, floatx16, floatx4>::type;

    extern __shared__ float smem[];
    int mt, nt, z;
    mm_tile_coords(a, mt, nt, z);
    const int kt0 = z * a.kps, kt1 = min(kt0 + a.kps, a.nkt);
    if (kt0 >= kt1) return;
    const int m0 = mt * BM, n0 = nt * BN;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int kg = wid >> 2, wq = wid & 3;
    const int wr = wq >> 1, wc = wq & 1;
    const int li = lane % IM, lg = lane / IM;

    Acc acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = Acc{};

    auto compute = [&](const float *As, const float *Bs) {
#pragma unroll UG
        for (int kk = kg * KR; kk < (kg + 1) * KR; kk += KGS) {
            float av[MB][VEC];
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const float *src = As + a_off<BK>(wr * WM + i * IM + li, kk + VEC * lg);
                if constexpr (VEC == 4) {
                    const floatx4 t = *reinterpret_cast<const floatx4 *>(src);
                    av[i][0] = t[0];
                    av[i][1] = t[1];
                    av[i][2] = t[2];
                    av[i][3] = t[3];
                } else if constexpr (VEC == 2) {
                    const float2 t = *reinterpret_cast<const float2 *>(src);
                    av[i][0] = t.x;
                    av[i][1] = t.y;
                } else {
                    av[i][0] = src[0];
                }
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                float bv[NB];
                const float *brow = Bs + (kk + VEC * lg + v) * BN + wc * WN + li;
#pragma unroll
                for (int j = 0; j < NB; ++j) bv[j] = brow[j * IM];
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j) {
                        if constexpr (BIG)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i][v], bv[j],
                                                                            acc[i][j], 0, 0, 0);
                        else
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][v], bv[j],
                                                                            acc[i][j], 0, 0, 0);
                    }
            }
        }
    };
    constexpr bool P4 = mm_pipelined<WM, WN, BK, DB, KG, 4>(),
                   P1 = mm_pipelined<WM, WN, BK, DB, KG, 1>();
    if constexpr (P4) {
        if (a.pipe == 4) mm_mfma_pipe<WM, WN, BK, UF, DB, KG, 4>(a, m0, n0, kt0, kt1, smem, acc);
    }
    if constexpr (P1) {
        if (a.pipe == 1) mm_mfma_pipe<WM, WN, BK, UF, DB, KG, 1>(a, m0, n0, kt0, kt1, smem, acc);
    }
    if (!(P4 && a.pipe == 4) && !(P1 && a.pipe == 1))
        k_loop<BM, BN, BK, ST, 256 * KG>(a, m0, n0, kt0, kt1, smem, compute);

    constexpr int NV = BIG ? 16 : 4;
    if constexpr (KG > 1) {
        // group 1 hands its partial tile to group 0 through LDS (16 bytes
        // per lane per access: value quad q of block b at ((b*NV/4 + q)*64 + lane)*4)
        __syncthreads();
        float *rb = smem + wq * (WM * WN);
        if (kg == 1) {
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int q = 0; q < NV / 4; ++q)
                        *reinterpret_cast<floatx4 *>(rb + (((i * NB + j) * (NV / 4) + q) * 64 + lane) * 4) =
                            floatx4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2],
                                    acc[i][j][4 * q + 3]};
        }
        __syncthreads();
        if (kg == 1) return;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int q = 0; q < NV / 4; ++q) {
                    const floatx4 t = *reinterpret_cast<const floatx4 *>(
                        rb + (((i * NB + j) * (NV / 4) + q) * 64 + lane) * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += t[e];
                }
    }

    // Output layout: 32x32 block, lane holds rows 8*(v/4) + 4*lg + v%4 of
    // column li (v < 16); 16x16 block, rows 4*lg + v of column li (v < 4).
    float *cbase = a.ks > 1 ? a.part + (size_t)z * a.M * a.N : a.C;
    if constexpr (!BIG && NB % 4 == 0) {
        // Four 16x16 blocks side by side: lane 4q+b holds columns 16j + 4q + b
        // (j < 4) of a row; a 4x4 transpose inside each lane quad leaves it
        // columns 16b + 4q .. +3, so every lane stores 16 contiguous bytes and
        // a row's 64 columns go out as whole 256-byte segments (non-temporal,
        // like the 32x32 blocks).  Full aligned tiles only.
        if (a.direct && (reinterpret_cast<uintptr_t>(cbase) & 15) == 0) {
            const int b = li & 3, q4 = li >> 2;
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int gm = m0 + wr * WM + i * IM + 4 * lg + v;
#pragma unroll
                    for (int jq = 0; jq < NB / 4; ++jq) {
                        float x[4] = {acc[i][4 * jq][v], acc[i][4 * jq + 1][v],
                                      acc[i][4 * jq + 2][v], acc[i][4 * jq + 3][v]};
                        quad_transpose(x, b);
                        const int gn = n0 + wc * WN + jq * 64 + 16 * b + 4 * q4;
                        __builtin_nontemporal_store(
                            floatx4{x[0], x[1], x[2], x[3]},
                            reinterpret_cast<floatx4 *>(cbase + (size_t)gm * a.N + gn));
                    }
                }
            return;
        }
    }
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int gn = n0 + wc * WN + j * IM + li;
            if (gn >= a.N) continue;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int row = BIG ? 8 * (v / 4) + 4 * lg + (v % 4) : 4 * lg + v;
                const int gm = m0 + wr * WM + i * IM + row;
                if (gm >= a.M) continue;
                // 32x32 blocks write whole 128-byte row segments per half-wave:
                // those go out with the non-temporal hint; the 64-byte segments of
                // 16x16 blocks stay in L2 to be merged (with the hint they cost
                // up to 1.5x the HBM writes)
                if constexpr (BIG) store_out(cbase + (size_t)gm * a.N + gn, acc[i][j][v]);
                else cbase[(size_t)gm * a.N + gn] = acc[i][j][v];
            }
        }
}

// A few rows of C (M <= 4, the matrix-vector products of a classifier at small
// batch): a workgroup owns 16 columns and the whole reduction, so a split (ks >=
// 2) needs no partials and no second launch.  Its 128 * ks threads take four
// columns each (16 bytes of a row of B) of every (32 * ks)-th row, up to four rows in
// flight per thread (one with unroll 0), and meet by lane exchange and LDS.
// Bound by the latency of the loads (63 workgroups hold 256 rows of 2048x1000 in
// flight at once), large matrices by their bytes.  In a graph, against the tiles
// and reduce launch of the same point: 1x1000x2048, ks 8, 7.8 -> 3.6 us; 4x1000x2048
// 8.1 -> 4.5; 1x4096x4096 32.0 -> 13.7 (4.9 TB/s).  2640 points of 140 shapes with 1
// to 4 rows 2.4 times as fast (geometric mean; the least 1.4).
template <int MR>
__global__ __launch_bounds__(1024) void mm_rows(MatmulArgs a) {
    __shared__ float red[16][MR][16];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, nw = blockDim.x >> 6;
    const int n0 = xcd_tile(blockIdx.x, gridDim.x) * 16;
    const int n = n0 + 4 * (tid & 3);
    const int r0 = tid >> 2, step = blockDim.x >> 2;
    const float *B = a.B + min(n, a.N - 4);       // N is a multiple of 4
    floatx4 acc[MR];
#pragma unroll
    for (int m = 0; m < MR; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    // D rows, one step apart, from row k on, all loaded before the first is used
    auto rows = [&]<int D>(std::integral_constant<int, D>, int k) {
        floatx4 b[D];
        float av[D][MR];
#pragma unroll
        for (int u = 0; u < D; ++u) {
            b[u] = *reinterpret_cast<const floatx4 *>(B + (size_t)(k + u * step) * a.N);
#pragma unroll
            for (int m = 0; m < MR; ++m) av[u][m] = a.A[(size_t)min(m, a.M - 1) * a.K + k + u * step];
        }
        // (left alone, the scheduler loads a row at a time to save registers)
        if constexpr (D > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < D; ++u)
#pragma unroll
            for (int m = 0; m < MR; ++m)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[m][j] = fmaf(av[u][m], b[u][j], acc[m][j]);
    };
    // every thread has `left` rows, the first K % step of them one more
    int k = r0, left = a.K / step;
    // 256 rows of B in flight a workgroup (4096x4096 and one row, 1, 2, 4, 8 a thread: ks
    // 8 13.9 14.6 15.2 15.6 us, ks 4 14.1 13.4 14.0 13.7, ks 2 21.2 14.9 13.3 14.0; 2048x1000
    // 3.7 at 8 x 1, 3.8 at 4 x 2 and 2 x 4)
    const int flight = min(a.uf, 1024 / int(blockDim.x));
    auto blocks = [&]<int D>(std::integral_constant<int, D> d) {
        if (flight < D) return;
        for (; left >= D; left -= D, k += D * step) rows(d, k);
    };
    blocks(std::integral_constant<int, 4>{});
    blocks(std::integral_constant<int, 2>{});
    blocks(std::integral_constant<int, 1>{});
    if (k < a.K) rows(std::integral_constant<int, 1>{}, k);
    // Lanes 4 apart hold the same columns.  Each exchange halves the sums a lane
    // holds (it sends the half its partner keeps) until one is left, so a wave's 16
    // rows meet in 5 to 15 exchanges instead of the 16 to 64 of whole sums.
    float v[4 * MR];
#pragma unroll
    for (int e = 0; e < 4 * MR; ++e) v[e] = acc[e / 4][e % 4];
    int at = 0;                                   // sum the lane is left with
    bool own = true;                              // (one of its copies)
#pragma unroll
    for (int d = 4, n = 4 * MR; d < 64; d *= 2, n = n > 1 ? n / 2 : 1) {
        const bool up = lane & d;
        if (n > 1) {
#pragma unroll
            for (int e = 0; e < n / 2; ++e) {
                const float lo = v[e], hi = v[e + n / 2];
                v[e] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, d);
            }
            at += up ? n / 2 : 0;
        } else {
            v[0] += __shfl_xor(v[0], d);
            own = own && !up;
        }
    }
    if (own) red[wid][at >> 2][4 * (lane & 3) + (at & 3)] = v[0];
    __syncthreads();
    if (tid < 16 * MR) {
        const int m = tid >> 4, c = tid & 15;
        float s = red[0][m][c];
        for (int w = 1; w < nw; ++w) s += red[w][m][c];
        if (m < a.M && n0 + c < a.N) a.C[(size_t)m * a.N + n0 + c] = s;
    }
}

}  // namespace

extern const void *g_mm_rows[3];
extern const void *g_mm_valu[kMmValuSlots];
extern const void *g_mm_mfma[kMmMfmaSlots];

#ifndef DS_SLICE
#define DS_SLICE 0
#define DS_NSLICES 1
#endif

namespace {

constexpr int kMmBkList[5] = {4, 8, 16, 32, 64};
constexpr int kMmWaveList[4] = {16, 32, 64, 128};

// slot = (((log2 RM * 5 + log2 RN) * 5 + ibk) * 7 + log2 UF) * 2 + DB
template <int I>
void reg_mm_valu() {
    constexpr int DB = I % 2, iuf = (I / 2) % 7, ibk = (I / 14) % 5, irn = (I / 70) % 5,
                  irm = I / 350;
    constexpr int RM = 1 << irm, RN = 1 << irn, BK = kMmBkList[ibk], UF = 1 << iuf;
    constexpr int lds = mm_stages(16 * RM, 16 * RN, BK, DB) * (16 * RM * BK + BK * 16 * RN) * 4;
    if constexpr (RM * RN <= 128 && UF <= BK && lds <= kLdsLimit &&
                  mm_uf_reachable(BK, RM * RN, UF) && I % DS_NSLICES == DS_SLICE)
        g_mm_valu[I] = reinterpret_cast<const void *>(&mm_valu<RM, RN, BK, UF, DB>);
}

// slot = ((((iwm * 4 + iwn) * 5 + ibk) * 7 + log2 UF) * 2 + DB) * 2 + (KG - 1)
template <int I>
void reg_mm_mfma() {
    constexpr int KG = 1 + I % 2, DB = (I / 2) % 2, iuf = (I / 4) % 7, ibk = (I / 28) % 5,
                  iwn = (I / 140) % 4, iwm = I / 560;
    constexpr int WM = kMmWaveList[iwm], WN = kMmWaveList[iwn], BK = kMmBkList[ibk],
                  UF = 1 << iuf;
    constexpr bool BIG = WM >= 32 && WN >= 32;
    constexpr int KSTEP = BIG ? 2 : 4;
    constexpr int blocks = BIG ? (WM / 32) * (WN / 32) : (WM / 16) * (WN / 16);
    constexpr int lds = mm_stages(2 * WM, 2 * WN, BK, DB) * (2 * WM * BK + BK * 2 * WN) * 4;
    if constexpr (lds <= kLdsLimit && UF <= BK / KSTEP && mm_uf_reachable(BK / KSTEP, blocks, UF) &&
                  (KG == 1 || BK >= 8) && I % DS_NSLICES == DS_SLICE)
        g_mm_mfma[I] = reinterpret_cast<const void *>(&mm_mfma<WM, WN, BK, UF, DB, KG>);
}

template <size_t... I>
void reg_all_valu(std::index_sequence<I...>) {
    (reg_mm_valu<int(I)>(), ...);
}
// in halves: one fold over every slot would exceed the compiler's nesting limit
template <size_t Off, size_t... I>
void reg_all_mfma(std::index_sequence<I...>) {
    (reg_mm_mfma<int(Off + I)>(), ...);
}

struct Registrar {
    Registrar() {
        if constexpr (DS_SLICE == 0) {
            g_mm_rows[0] = reinterpret_cast<const void *>(&mm_rows<1>);
            g_mm_rows[1] = reinterpret_cast<const void *>(&mm_rows<2>);
            g_mm_rows[2] = reinterpret_cast<const void *>(&mm_rows<4>);
        }
        reg_all_valu(std::make_index_sequence<kMmValuSlots>{});
        reg_all_mfma<0>(std::make_index_sequence<kMmMfmaSlots / 2>{});
        reg_all_mfma<kMmMfmaSlots / 2>(std::make_index_sequence<kMmMfmaSlots - kMmMfmaSlots / 2>{});
    }
};
const Registrar registrar;

}  // namespace

}  // namespace ds
