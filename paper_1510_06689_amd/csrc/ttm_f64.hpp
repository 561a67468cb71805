// FP64 TTM with the operator in registers (ttm.hip chooses it): many output
// rows, where the products and not the tensor's bytes take the time.
// ttm_f64_double.hip and ttm_f64_float.hip compile it for one storage type each.
#pragma once

#include <type_traits>

#include "tile_io.hpp"
#include "tk_common.hpp"

namespace tk {

typedef double d4_t __attribute__((ext_vector_type(4)));

// 8 waves.  Wave (wr, wc) owns the 16 output rows of block wr (WR = 4 or 8
// blocks per workgroup; more rows go to grid.y) and every WC-th block of 16
// tile columns, WC = 8 / WR; its part of op(M), 16 x J, stays in registers, so
// a k-step reads one value of Y per product from LDS.  Y's tiles pass through
// two LDS buffers as in the FP64 Gram: elements of the next tile are stored,
// and those of the one after it loaded, between the products.  Of every 32
// rows of Y product s takes rows 16 (k4 & 1) + (k4 >> 1) + 2 s for the lanes
// of quarter k4 (the sum's order is free): at the odd pitch a half-wave's
// values then lie in 32 different bank pairs.  JC: J rounded up to 128,
// 192 or 256 (the rows past J are zero in LDS).
constexpr int kRegThreads = 512;
template <int JC>
constexpr int kRegKt = JC <= 128 ? 64 : 32;
template <int JC>
constexpr size_t kRegLds = (size_t)2 * kTileBuf<JC / 16, kRegKt<JC>> * sizeof(double);

// ZT: form Z^T blocks, so that the lanes of a quarter-wave write consecutive
// output rows r (columns of the tile fewer than 16 apart in memory, L < 16);
// else consecutive columns.
template <typename T, int JC, int WR, bool PACKED, bool ZT>
__global__ __launch_bounds__(kRegThreads, 2) void ttm_reg_f64(
    const T* __restrict__ y, TileMap tm, const double* __restrict__ m, int64_t ldm, int K,
    int transpose, T* __restrict__ z) {
    extern __shared__ double lds[];
    constexpr int KT = kRegKt<JC>, P = KT + 1, BUF = kTileBuf<JC / 16, KT>;
    constexpr int WC = 8 / WR, CB = KT / 16;
    constexpr int NC = CB / WC;  // column blocks per wave
    static_assert(CB % WC == 0, "column blocks over waves");
    constexpr int FS = 4, NG = JC / 4 / FS;     // steps per tile
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, k4 = lane >> 4;
    const int wr = wave % WR, wc = wave / WR;
    const int J = tm.J;
    const int r0 = (int)blockIdx.y * 16 * WR + 16 * wr;  // the wave's first output row
    const int64_t t0 = tm.ntiles * (int64_t)blockIdx.x / gridDim.x;
    const int64_t t1 = tm.ntiles * (int64_t)(blockIdx.x + 1) / gridDim.x;
    if (t0 >= t1) return;  // uniform over the workgroup

    for (int e = tid; e < 2 * BUF; e += kRegThreads) lds[e] = 0.0;
    TileStage<T, JC / 16, KT, kRegThreads, PACKED> st;
    constexpr int PER = decltype(st)::kPer;
    st.begin(y, tm, t0, t1);
#pragma unroll
    for (int q = 0; q < PER; ++q)
        st.load(q);
    st.advance();
    // op(M)'s rows r0 + c16, in the order of the products
    const int i0 = 16 * (k4 & 1) + (k4 >> 1);
    double a[JC / 4];
#pragma unroll
    for (int s = 0; s < JC / 4; ++s) {
        const int i = 32 * (s / 8) + 2 * (s % 8) + i0, r = r0 + c16;
        a[s] = i < J && r < K ? (transpose ? m[i + ldm * r] : m[r + ldm * i]) : 0.0;
    }
    // this lane's output columns: offset of column kk inside a tile
    constexpr int NV = ZT ? 4 : 1;
    int col[NC * NV];
    int64_t zoff[NC * NV];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int kk = 16 * (wc + WC * c) + (ZT ? 4 * v + k4 : c16);
            col[c * NV + v] = kk;
            zoff[c * NV + v] = PACKED ? tile_col_offset(kk, tm.L, K) : kk;
        }
    __syncthreads();  // zeroing done before the first store
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        st.store(lds, q);
        st.load(q);
    }
    st.advance();
    // op(M) has arrived: without this the compiler waits for it, and so for
    // every load under way, at the first product of each tile
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // the output tile: first element and columns, walked like the stage's
    const Tile zt = tile_at(tm, t0, K);
    T* zp = z + zt.base;
    int ncols = zt.ncols;
    int64_t bleft = tm.B - t0 * tm.nbb;                   // PACKED: b-blocks from this tile on
    int64_t seg = PACKED ? 0 : t0 % tm.lsegs;             // strided: segment of this tile
    int b = 0;
    for (int64_t t = t0; t < t1; ++t) {
        const double* cur = lds + b * BUF + i0 * P + 16 * wc + c16;
        double* nxt = lds + (1 - b) * BUF;
        d4_t acc[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = d4_t{0.0, 0.0, 0.0, 0.0};
        // steps of FS products per column block: the next step's values of Y
        // are read before this step's products
        double f[2][FS * NC];
        auto read = [&](int g, double (&to)[FS * NC]) {
#pragma unroll
            for (int s = 0; s < FS; ++s)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int p = FS * g + s;
                    to[s * NC + c] = cur[(32 * (p / 8) + 2 * (p % 8)) * P + 16 * WC * c];
                }
        };
        read(0, f[0]);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) read(g + 1, f[(g + 1) & 1]);
            // else they sink to their products (with more in flight it spills)
            if constexpr (NC <= 2 && JC <= 192) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < FS; ++s)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const double yv = f[g & 1][s * NC + c], av = a[FS * g + s];
                    acc[c] = ZT ? __builtin_amdgcn_mfma_f64_16x16x4f64(yv, av, acc[c], 0, 0, 0)
                                : __builtin_amdgcn_mfma_f64_16x16x4f64(av, yv, acc[c], 0, 0, 0);
                }
#pragma unroll
            for (int q = PER * g / NG; q < PER * (g + 1) / NG; ++q) {
                st.store(nxt, q);
                st.load(q);
            }
        }
        st.advance();
        // D[row][col] sits in lane col + 16 (row % 4), register row / 4
        {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = r0 + (ZT ? c16 : 4 * v + k4);
                    const int w = c * NV + (ZT ? v : 0);
                    if (r < K && col[w] < ncols) zp[zoff[w] + (int64_t)r * tm.L] = (T)acc[c][v];
                }
        }
        if (PACKED) {
            zp += (int64_t)tm.nbb * K * tm.L;
            bleft -= tm.nbb;
            ncols = (int)((bleft < tm.nbb ? bleft : tm.nbb) * tm.L);
        } else {
            const bool wrap = seg + 1 == tm.lsegs;
            zp += wrap ? (int64_t)K * tm.L - seg * KT : KT;
            seg = wrap ? 0 : seg + 1;
            const int64_t w = tm.L - seg * KT;
            ncols = (int)(w < KT ? w : KT);
        }
        b ^= 1;
        __syncthreads();
    }
}

// Z = op(M) Y for J <= 256 and any K (meant for J > 64, K > 32).
int launch_ttm_reg(const double* y, const ModeView& v, const double* m, int64_t ldm, int K,
                   int transpose, double* z, hipStream_t st);
int launch_ttm_reg(const float* y, const ModeView& v, const double* m, int64_t ldm, int K,
                   int transpose, float* z, hipStream_t st);

template <typename T, int JC, int WR>
static int launch_ttm_reg_t(const T* y, const ModeView& v, const double* m, int64_t ldm, int K,
                            int transpose, T* z, hipStream_t st) {
    const TileMap tm = make_tiles(v, kRegKt<JC>);
    auto fn = !tm.packed ? ttm_reg_f64<T, JC, WR, false, false>
              : v.L < 16 ? ttm_reg_f64<T, JC, WR, true, true>
                         : ttm_reg_f64<T, JC, WR, true, false>;
    const int G = (K + 16 * WR - 1) / (16 * WR);
    // one resident workgroup per CU (two where LDS holds two tile pairs), each
    // with a contiguous range of tiles
    const int64_t want = (kRegLds<JC> * 2 <= 160 * 1024 ? 2 : 1) * (int64_t)device_cu_count();
    int64_t P = want / G;
    P = P < 1 ? 1 : P;
    if (tm.ntiles < P) P = tm.ntiles;
    TK_HIP(hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kRegLds<JC>));
    hipLaunchKernelGGL(fn, dim3((int)P, G), dim3(kRegThreads), kRegLds<JC>, st, y, tm, m, ldm, K,
                       transpose, z);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

template <typename T, int JC>
static int launch_ttm_reg_jc(const T* y, const ModeView& v, const double* m, int64_t ldm, int K,
                             int transpose, T* z, hipStream_t st) {
    if (K <= 64) return launch_ttm_reg_t<T, JC, 4>(y, v, m, ldm, K, transpose, z, st);
    return launch_ttm_reg_t<T, JC, 8>(y, v, m, ldm, K, transpose, z, st);
}

template <typename T>
static int launch_ttm_reg_any(const T* y, const ModeView& v, const double* m, int64_t ldm, int K,
                              int transpose, T* z, hipStream_t st) {
    if (v.J <= 128) return launch_ttm_reg_jc<T, 128>(y, v, m, ldm, K, transpose, z, st);
    if (v.J <= 192) return launch_ttm_reg_jc<T, 192>(y, v, m, ldm, K, transpose, z, st);
    return launch_ttm_reg_jc<T, 256>(y, v, m, ldm, K, transpose, z, st);
}

}  // namespace tk
