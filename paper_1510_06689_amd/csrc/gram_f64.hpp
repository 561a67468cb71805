// Tiled FP64 Gram kernels (stage 1 of gram.hip): their schedules, which the
// plans need too, and the kernels, which gram_f64_double.hip and
// gram_f64_float.hip compile for one storage type each (the unrolled copies
// take a while to build).
#pragma once

#include <type_traits>

#include "tile_io.hpp"
#include "tk_common.hpp"

namespace tk {

typedef double d4_t __attribute__((ext_vector_type(4)));

// Calls f with the block count nb (at most 16) as a constant.
template <int NB = 1, class F>
static int with_blocks(int nb, F&& f) {
    if constexpr (NB <= 16) {
        if (nb == NB) return f(std::integral_constant<int, NB>{});
        return with_blocks<NB + 1>(nb, f);
    } else {
        return fail(TK_ERR_UNSUPPORTED, "Gram: %d row blocks", nb);
    }
}

// Pair index p -> (bi, bj), upper-triangle blocks in row-major order.
__device__ __forceinline__ void pair_of(int p, int nb, int& bi, int& bj) {
    int row = 0;
    int start = 0;
    while (p >= start + (nb - row)) {
        start += nb - row;
        ++row;
    }
    bi = row;
    bj = row + (p - start);
}

// Schedule of the tiled FP64 Gram for NB = ceil(J / 16) blocks and its
// NP = NB (NB + 1) / 2 block pairs.
//   NB <= 6: 4 waves, each with all pairs and every fourth k-step (KS = 4), so
//     that a k-step reads each block once;
//   NB <= 8: 4 waves, each with a quarter of the pairs (NPW) and all k-steps;
//   above:   8 waves, each with an eighth of the pairs.
// Up to NB = 8 a CU has two workgroups, one multiplying while the other stands
// at its barrier.  KT, the tile's columns: what LDS holds; small extents take
// wide tiles, which keep more loads in flight (FEW, up to NB = 4: 32 columns,
// for tensors that fill few tiles).
template <int NB, bool FEW = false>
struct GramSched {
    static constexpr int W = NB <= 8 ? 4 : 8;
    static constexpr int T = 64 * W;  // threads
    static constexpr int KS = NB <= 6 ? W : 1;
    static constexpr int KT = NB <= 2 && !FEW ? 128 : NB <= 4 && !FEW ? 64 : 32;
    static constexpr int NP = NB * (NB + 1) / 2;
    static constexpr int NPW = KS == 1 ? (NP + W - 1) / W : NP;
    static constexpr int kLds = 2 * kTileBuf<NB, KT>;  // doubles
    static constexpr int kPerCu = NB <= 8 ? 2 : 1;
};

// Column of a lane's first fragment value within 32 columns (see gram_f64_walk).
__device__ __forceinline__ int frag_col(int k4) { return 16 * (k4 & 1) + (k4 >> 1); }

// One workgroup's share, tiles [t0, t1): writes NP * 256 partial sums at
// `out`, in pair_of order.  While the products of tile t run, the stage's
// elements of tile t + 1 go to the other buffer and those of tile t + 2 are
// loaded, a few after each k-step.  Below J = 64 or so HBM bounds it; above,
// the products and what feeds them: at J = 128 on 8.6 GB it does 49 TFLOP/s of
// products (44 counted), where an FP64 GEMM of the library reaches 70 on this
// card, so this is not the card's limit.  A wave takes consecutive pairs of the
// list and reads both fragments of each from LDS, 18 reads per nine products; 26
// reads per 36 products (a set of pairs per wave at compile time) were 5% faster
// there and took sixteen minutes to build.  Before and after (one conversion per
// load, a branch per element, all pairs rounded up to 32, 64, 128, 256 rows): J =
// 128 FP64 3.46 -> 3.16 ms (8.6 GB), FP32 0.61 -> 0.30 ms (0.4 GB); J = 250, L =
// 10 1.23 -> 0.94 ms (1.25 GB); J = 25 1.04 -> 0.67 ms (3.1 GB, 4.6 TB/s); J = 97
// 57 -> 40 us (81 MB).  From NB = 13 on 12 to 17 accumulators and 16 staged
// doubles per lane exceed 256 registers: 17, 6, 11 and 31 are spilled (FP32 0,
// 28, 12, 16).
// SKIP (batches, J below the extent class): pairs with a block at or past
// ceil(J / 16) sum zeros only and skip their products (their partials stay 0).
template <typename T, int NB, bool FEW, bool SKIP, bool PACKED>
__device__ __forceinline__ void gram_f64_walk(const T* __restrict__ y, const TileMap& tm,
                                              int64_t t0, int64_t t1, double* __restrict__ out,
                                              double* lds) {
    typedef GramSched<NB, FEW> S;
    constexpr int P = S::KT + 1, NPW = S::NPW, NP = S::NP, BUF = kTileBuf<NB, S::KT>;
    constexpr int KQ = S::KT / 8 / S::KS;  // steps of eight columns, of a wave per tile
    constexpr bool ALL = S::KS > 1;        // a wave has all pairs
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, k4 = lane >> 4;
    const int nbv = SKIP ? __builtin_amdgcn_readfirstlane((tm.J + 15) >> 4) : NB;

    TileStage<T, NB, S::KT, S::T, PACKED> st;
    constexpr int PER = decltype(st)::kPer;
    if (t0 < t1) {
        // tile t0 to the first buffer, tile t0 + 1 on its way to the registers
        st.begin(y, tm, t0, t1);
#pragma unroll
        for (int q = 0; q < PER; ++q) st.load(q);
        st.advance();
        __syncthreads();  // zeroing done before the first store
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            st.store(lds, q);
            st.load(q);
        }
        st.advance();
    }
    // this wave's pairs: p0 .. p0 + NPW - 1, spare slots repeat the last one
    const int p0 = ALL ? 0 : wave * NPW;
    int bi[NPW], bj[NPW];
    {
        int i, j;
        if (ALL) i = j = 0;
        else pair_of(min(p0, NP - 1), NB, i, j);
#pragma unroll
        for (int q = 0; q < NPW; ++q) {
            bi[q] = i;
            bj[q] = j;
            if (ALL || p0 + q + 1 < NP) {
                ++j;
                if (j == NB) {
                    ++i;
                    j = i;
                }
            }
        }
    }
    d4_t acc[NPW];
#pragma unroll
    for (int q = 0; q < NPW; ++q) acc[q] = d4_t{0.0, 0.0, 0.0, 0.0};
    __syncthreads();
    // Of every 32 columns product s takes columns 16 (k4 & 1) + (k4 >> 1) + 2 s
    // for the lanes of quarter k4: at the odd pitch a half-wave's 32 values then
    // lie in 32 different bank pairs.  A step is two products.
    const double* fr = lds + r16 * P + frag_col(k4) + (ALL ? 16 / S::KS * wave : 0);
    auto frag = [&](const double* at) { return double2{at[0], at[2]}; };
    int b = 0;
    for (int64_t t = t0; t < t1; ++t) {
        const double* cur = fr + b * BUF;
        double* nxt = lds + (1 - b) * BUF;
#pragma unroll
        for (int kq = 0; kq < KQ; ++kq) {
            // KS = 1: four steps per 32 columns; KS = 4: one
            const double* at = cur + (ALL ? 32 * kq : 32 * (kq / 4) + 4 * (kq % 4));
            static_assert(S::KS == 1 || S::KS == 4, "step addresses");
            if constexpr (ALL) {
                double2 f[NB];
#pragma unroll
                for (int B = 0; B < NB; ++B) f[B] = frag(at + B * 16 * P);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0, q = 0; i < NB; ++i)
#pragma unroll
                        for (int j = i; j < NB; ++j, ++q)
                            if (!SKIP || j < nbv)  // uniform
                                acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                    h ? f[i].y : f[i].x, h ? f[j].y : f[j].x, acc[q], 0, 0, 0);
            } else {
                double2 fi[NPW], fj[NPW];
#pragma unroll
                for (int q = 0; q < NPW; ++q) {
                    fi[q] = frag(at + bi[q] * 16 * P);
                    fj[q] = frag(at + bj[q] * 16 * P);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int q = 0; q < NPW; ++q)
                        if (!SKIP || bj[q] < nbv)  // uniform; bi <= bj
                            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                h ? fi[q].y : fi[q].x, h ? fj[q].y : fj[q].x, acc[q], 0, 0, 0);
            }
#pragma unroll
            for (int e = PER * kq / KQ; e < PER * (kq + 1) / KQ; ++e) {
                st.store(nxt, e);
                st.load(e);
            }
        }
        st.advance();
        b ^= 1;
        __syncthreads();
    }

    // v_mfma_f64_16x16x4f64 leaves D[row][col] in lane col + 16 * (row % 4),
    // register row / 4, i.e. row = 4 * v + lane / 16, col = lane % 16.
    if constexpr (!ALL) {
#pragma unroll
        for (int q = 0; q < NPW; ++q)
            if (p0 + q < NP) {  // uniform
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    out[(p0 + q) * 256 + (4 * v + k4) * 16 + r16] = acc[q][v];
            }
    } else {
        // the waves' slices of each pair are added in order, QR pairs at a
        // time through the tile buffers
        constexpr int room = 2 * BUF / (S::W * 256);
        constexpr int QR = room < NPW ? room : NPW;
        static_assert(QR >= 1, "the fold needs room for one pair per wave");
#pragma unroll
        for (int q0 = 0; q0 < NPW; q0 += QR) {
            if (q0 > 0) __syncthreads();
#pragma unroll
            for (int q = 0; q < QR; ++q)
                if (q0 + q < NPW) {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        lds[(wave * QR + q) * 256 + (4 * v + k4) * 16 + r16] =
                            acc[q0 + q < NPW ? q0 + q : 0][v];
                }
            __syncthreads();
            for (int e = tid; e < QR * 256 && q0 * 256 + e < NP * 256; e += S::T) {
                double s = 0.0;
#pragma unroll
                for (int w = 0; w < S::W; ++w) s += lds[w * QR * 256 + e];
                out[q0 * 256 + e] = s;
            }
        }
    }
}

template <typename T, int NB, bool FEW, bool SKIP>
__device__ __forceinline__ void gram_f64_body(const T* __restrict__ y, const TileMap& tm,
                                              int64_t t0, int64_t t1, double* __restrict__ out,
                                              double* lds) {
    typedef GramSched<NB, FEW> S;
    for (int e = threadIdx.x; e < S::kLds; e += S::T) lds[e] = 0.0;
    if (tm.packed)
        gram_f64_walk<T, NB, FEW, SKIP, true>(y, tm, t0, t1, out, lds);
    else
        gram_f64_walk<T, NB, FEW, SKIP, false>(y, tm, t0, t1, out, lds);
}

// P tile ranges, one workgroup each; J <= 256.
template <typename T, int NB, bool FEW>
__global__ __launch_bounds__((GramSched<NB, FEW>::T), 2) void gram_partial_f64(
    const T* __restrict__ y, TileMap tm, int P, double* __restrict__ partial) {
    extern __shared__ double lds[];
    const int p = blockIdx.x;
    const int64_t t0 = tm.ntiles * (int64_t)p / P;
    const int64_t t1 = tm.ntiles * (int64_t)(p + 1) / P;
    gram_f64_body<T, NB, FEW, false>(y, tm, t0, t1, partial + (int64_t)p * GramSched<NB>::NP * 256,
                                     lds);
}

// J > 256: 153 to 528 block pairs do not fit one workgroup's accumulators, so
// G groups of at most kWidePairs of them, dealt at run time, share each tile
// range (P ranges x G groups, one workgroup each, xcd_range_group).  J = 400
// FP32, 93 MB: 404 -> 210 us, J = 512 FP64, 164 MB: 412 -> 370 us, J = 301
// FP64 unchanged (139 us), against nine groups and a stage of 512 rows.
// J > 160 takes it too where there are few columns, in many small groups.
constexpr int kWideThreads = 512, kWideWaves = kWideThreads / 64;
constexpr int kWideNpw = 14, kWidePairs = kWideWaves * kWideNpw, kWideKt = 16;
// NB: the block count rounded up to a multiple of four (it sizes the stage).
template <int NB>
constexpr int kWideBuf = kTileBuf<NB, kWideKt>;

template <typename T, int NB, bool PACKED>
__device__ __forceinline__ void gram_wide_body(const T* __restrict__ y, const TileMap& tm, int nb,
                                               int q0, int nq, int64_t t0, int64_t t1,
                                               double* __restrict__ out, double* lds) {
    constexpr int PT = kWideKt + 1, KQ = kWideKt / 8;
    const int tid = threadIdx.x, lane = tid & 63;
    const int r16 = lane & 15, k4 = lane >> 4;
    int aoff[kWideNpw], boff[kWideNpw];
    d4_t acc[kWideNpw];
#pragma unroll
    for (int q = 0; q < kWideNpw; ++q) {
        int bi, bj;
        pair_of(q < nq ? q0 + q : 0, nb, bi, bj);
        aoff[q] = (bi * 16 + r16) * PT + 2 * k4;
        boff[q] = (bj * 16 + r16) * PT + 2 * k4;
        acc[q] = d4_t{0.0, 0.0, 0.0, 0.0};
    }
    TileStage<T, NB, kWideKt, kWideThreads, PACKED> st;
    if (t0 < t1) {
        st.begin(y, tm, t0, t1);
#pragma unroll
        for (int q = 0; q < st.kPer; ++q) st.load(q);
        st.advance();
        __syncthreads();
#pragma unroll
        for (int q = 0; q < st.kPer; ++q) {
            st.store(lds, q);
            st.load(q);
        }
        st.advance();
    }
    __syncthreads();
    for (int64_t t = t0; t < t1; ++t) {
        const int b = (int)((t - t0) & 1);
        const double* cur = lds + b * kWideBuf<NB>;
        double* nxt = lds + (1 - b) * kWideBuf<NB>;
#pragma unroll
        for (int ks = 0; ks < KQ; ++ks) {
#pragma unroll
            for (int q = 0; q < kWideNpw; ++q)
                if (q < nq) {  // uniform over the wave
                    const double* fa = cur + aoff[q] + ks * 8;
                    const double* fb = cur + boff[q] + ks * 8;
                    acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[0], fb[0], acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[1], fb[1], acc[q], 0, 0, 0);
                }
#pragma unroll
            for (int e = st.kPer * ks / KQ; e < st.kPer * (ks + 1) / KQ; ++e) {
                st.store(nxt, e);
                st.load(e);
            }
        }
        st.advance();
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < kWideNpw; ++q)
        if (q < nq) {
#pragma unroll
            for (int v = 0; v < 4; ++v) out[q * 256 + (4 * v + k4) * 16 + r16] = acc[q][v];
        }
}

template <typename T, int NB>
__global__ __launch_bounds__(kWideThreads, 2) void gram_partial_wide(
    const T* __restrict__ y, TileMap tm, int nb, int npairs, int pairs_per_group, int P, int G,
    double* __restrict__ partial) {
    extern __shared__ double lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int p, g;
    xcd_range_group(blockIdx.x, G, p, g);
    const int npg = min(npairs - g * pairs_per_group, pairs_per_group);
    const int64_t t0 = tm.ntiles * (int64_t)p / P;
    const int64_t t1 = tm.ntiles * (int64_t)(p + 1) / P;
    // this wave's pairs: nq of the group's, from pair q0 on
    const int q0 = g * pairs_per_group + npg * wave / kWideWaves;
    const int nq = g * pairs_per_group + npg * (wave + 1) / kWideWaves - q0;
    for (int e = threadIdx.x; e < 2 * kWideBuf<NB>; e += kWideThreads) lds[e] = 0.0;
    double* out = partial + ((int64_t)p * npairs + q0) * 256;
    if (tm.packed)
        gram_wide_body<T, NB, true>(y, tm, nb, q0, nq, t0, t1, out, lds);
    else
        gram_wide_body<T, NB, false>(y, tm, nb, q0, nq, t0, t1, out, lds);
}

// P tile ranges (times pl.G pair groups above extent 256) into `partial`.
int launch_gram_f64(const double* y, const ModeView& v, const GramPlan& pl, double* partial,
                    hipStream_t st);
int launch_gram_f64(const float* y, const ModeView& v, const GramPlan& pl, double* partial,
                    hipStream_t st);

template <typename T>
static int launch_gram_f64_t(const T* y, const ModeView& v, const GramPlan& pl, double* partial,
                            hipStream_t st) {
    const TileMap tm = make_tiles(v, pl.KT);
    if (pl.KT != kWideKt)
        return with_blocks(pl.nb, [&](auto nbc) -> int {
            constexpr int NB = decltype(nbc)::value;
            auto launch = [&](auto few) -> int {
                constexpr bool FEW = decltype(few)::value;
                typedef GramSched<NB, FEW> S;
                const size_t lds = S::kLds * sizeof(double);
                auto fn = gram_partial_f64<T, NB, FEW>;
                TK_HIP(hipFuncSetAttribute((const void*)fn,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
                hipLaunchKernelGGL(fn, dim3(pl.P), dim3(S::T), lds, st, y, tm, pl.P, partial);
                TK_HIP(hipGetLastError());
                return TK_OK;
            };
            if constexpr (NB <= 4)
                if (pl.KT != GramSched<NB>::KT) return launch(std::true_type{});
            return launch(std::false_type{});
        });
    if (v.J > TK_MAX_MODE_DIM)
        return fail(TK_ERR_UNSUPPORTED, "mode extent %d exceeds %d", v.J, TK_MAX_MODE_DIM);
    auto launch = [&](auto nbc) -> int {
        constexpr int NB = decltype(nbc)::value;
        const size_t lds = 2 * kWideBuf<NB> * sizeof(double);
        auto fn = gram_partial_wide<T, NB>;
        TK_HIP(hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds));
        hipLaunchKernelGGL(fn, dim3(pl.P * pl.G), dim3(kWideThreads), lds, st, y, tm, pl.nb,
                           pl.npairs, pl.pairs_per_group, pl.P, pl.G, partial);
        TK_HIP(hipGetLastError());
        return TK_OK;
    };
    if (pl.nb <= 16) return launch(std::integral_constant<int, 16>{});
    if (pl.nb <= 20) return launch(std::integral_constant<int, 20>{});
    if (pl.nb <= 24) return launch(std::integral_constant<int, 24>{});
    if (pl.nb <= 28) return launch(std::integral_constant<int, 28>{});
    return launch(std::integral_constant<int, 32>{});
}

}  // namespace tk
