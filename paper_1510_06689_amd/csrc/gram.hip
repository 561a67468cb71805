// Gram matrix S = Y_(n) Y_(n)^T of a mode-n unfolding (Alg. 1, Gram step),
// computed in the natural layout without permuting data (Sec. V-C, local
// part), exploiting symmetry: only 16x16 blocks (bi <= bj) are formed.
//
// Stage 1 (gram_partial_f64; above extent 256 gram_partial_wide): a workgroup
// streams its contiguous range of column tiles (TileMap) through a
// double-buffered LDS tile and accumulates block pairs in registers.  Each
// wave owns a compile-time set of pairs (GramSched) and a k-slice of each
// tile.  One barrier per tile: while the MFMAs read buffer t % 2 the
// registers holding tile t + 1 are written to the other buffer.  It writes
// one partial per pair to the workspace.
// Stage 2 (gram_reduce): sums the partials over p in a fixed order (so S is
// bitwise reproducible) and mirrors the upper blocks into both triangles.
//
// FP64 path: v_mfma_f64_16x16x4f64 on FP64 data (FP32 input is widened
// exactly while staging).  Narrow modes (J <= 32 over long contiguous runs)
// replace stage 1 by gram_narrow_f64, which needs no LDS tile.
#include "gram_f64.hpp"
#include "tk_common.hpp"

namespace tk {

// acc + partial[q n + idx] over q = g, g + 4, ... < P, added in that order;
// eight loads go out per trip so that they overlap.
__device__ __forceinline__ double sum_partials(const double* __restrict__ partial, int P,
                                               int n, int idx, int g) {
    double acc = 0.0;
    int q = g;
    for (; q + 28 < P; q += 32) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = partial[(int64_t)(q + 4 * u) * n + idx];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; q < P; q += 4) acc += partial[(int64_t)q * n + idx];
    return acc;
}

// {sum over p of aux[2 p], max over p of aux[2 p + 1]} -> out[0..1], summed
// by the first wave of a workgroup in a fixed order (lane-strided partial
// sums, then lane by lane).
__device__ __forceinline__ void reduce_split_stats(const double* __restrict__ aux, int P,
                                                   double* __restrict__ out, double* part) {
    const int lane = threadIdx.x;
    if (lane < 64) {
        double d = 0.0, e = -125.0;
        for (int q = lane; q < P; q += 64) {
            d += aux[2 * q];
            e = fmax(e, aux[2 * q + 1]);
        }
        part[lane] = d;
        part[64 + lane] = e;
    }
    __syncthreads();
    if (lane == 0) {
        double d = 0.0, e = -125.0;
        for (int k = 0; k < 64; ++k) {
            d += part[k];
            e = fmax(e, part[64 + k]);
        }
        out[0] = d;
        out[1] = e;
    }
}

// S[r + J c] for the upper block pairs.  Each workgroup reduces 64 outputs;
// its 4 wave-sized groups sum the partials p = g, g + 4, ... and the four
// group sums are added in a fixed order.  With aux, one more workgroup
// reduces the split statistics into stats.
__global__ __launch_bounds__(256) void gram_reduce(const double* __restrict__ partial, int P,
                                                   int npairs, int nb, int J,
                                                   double* __restrict__ s,
                                                   const double* __restrict__ aux,
                                                   double* __restrict__ stats) {
    __shared__ double part[4][64];
    if (aux && blockIdx.x == gridDim.x - 1) {  // uniform over the workgroup
        reduce_split_stats(aux, P, stats, &part[0][0]);
        return;
    }
    const int o = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int idx = blockIdx.x * 64 + o;
    const int n = npairs * 256;
    const double acc = idx < n ? sum_partials(partial, P, n, idx, g) : 0.0;
    part[g][o] = acc;
    __syncthreads();
    if (g != 0 || idx >= n) return;
    const double tot = ((part[0][o] + part[1][o]) + part[2][o]) + part[3][o];
    int p = idx >> 8, e = idx & 255;
    int bi, bj;
    pair_of(p, nb, bi, bj);
    int r = bi * 16 + (e >> 4), c = bj * 16 + (e & 15);
    if (r >= J || c >= J) return;
    if (bi == bj && r > c) return;  // diagonal blocks: upper triangle only, then mirror
    s[r + (int64_t)J * c] = tot;
    s[c + (int64_t)J * r] = tot;
}

// trace(S) = ||Y||^2, summed in a fixed order by one wave.
__global__ void gram_trace(const double* __restrict__ s, int J, double* __restrict__ out) {
    __shared__ double part[64];
    int lane = threadIdx.x;
    double acc = 0.0;
    for (int i = lane; i < J; i += 64) acc += s[i + (int64_t)J * i];
    part[lane] = acc;
    __syncthreads();
    if (lane == 0) {
        double t = 0.0;
        for (int k = 0; k < 64; ++k) t += part[k];
        *out = t;
    }
}

// ------------------------------------------------------------ narrow modes
//
// J <= 32 where every unfolding row is made of long contiguous runs (L a
// multiple of 8): no LDS tile.  A step is 32 consecutive l of one slab b.
// Lane t of a wave owns unfolding row t % 16 (and 16 + t % 16 when J > 16)
// and the eight columns l0 + 8 (t / 16) + e of a step, read with one vector
// load per row straight from HBM.  For MFMA call e each lane's element is
// both A[t % 16][t / 16] and B[t / 16][t % 16], so the eight calls sum
// y_i y_j over the step's 32 columns.  A wave takes U consecutive steps at a
// time (one contiguous run of 32 U elements per row); its accumulators stay
// in registers until the end, where the 8 waves of a workgroup fold them
// through LDS, in a fixed order, into one partial per workgroup.
constexpr int kNarrowThreads = 512;
constexpr int kNarrowWaves = kNarrowThreads / 64;

template <typename T>
struct Run8;
template <>
struct Run8<float> {
    typedef float type __attribute__((ext_vector_type(8)));
};
template <>
struct Run8<double> {
    typedef double type __attribute__((ext_vector_type(8)));
};

// Block pairs of the narrow kernel: (0,0) for J <= 16; (0,0), (0,1), (1,1)
// (pair_of order with nb = 2) for 16 < J <= 32.
template <int JN>
constexpr int kNarrowPairs = JN == 16 ? 1 : 3;

template <typename T, int JN, int U>
__global__ __launch_bounds__(kNarrowThreads) void gram_narrow_f64(
    const T* __restrict__ y, int64_t L, int J, int64_t nsteps, int P,
    double* __restrict__ partial) {
    constexpr int NR = JN / 16;  // row blocks per lane
    constexpr int NP = kNarrowPairs<JN>;
    constexpr int NA = JN == 16 ? 2 : 3;  // J <= 16: two accumulator chains
    typedef typename Run8<T>::type run_t;
    __shared__ double red[kNarrowWaves * NP * 256];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, k4 = lane >> 4;
    const int p = blockIdx.x;
    const int64_t s0 = nsteps * p / P, s1 = nsteps * (p + 1) / P;
    const int64_t sb = (L + 31) >> 5;  // steps per slab
    const int64_t slab = (int64_t)J * L;
    int64_t roff[NR];
    bool rok[NR];
#pragma unroll
    for (int h = 0; h < NR; ++h) {
        const int r = 16 * h + r16;
        rok[h] = r < J;
        roff[h] = (int64_t)(rok[h] ? r : 0) * L + 8 * k4;
    }
    d4_t acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = d4_t{0.0, 0.0, 0.0, 0.0};

    for (int64_t q = s0 + (int64_t)wave * U; q < s1; q += (int64_t)kNarrowWaves * U) {
        int64_t b = q / sb;
        int64_t l0 = (q - b * sb) << 5;
        run_t v[U][NR];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = q + u < s1 && l0 + 8 * k4 < L;
            const T* base = y + b * slab + l0;
#pragma unroll
            for (int h = 0; h < NR; ++h) {
                if (ok && rok[h])
                    v[u][h] = *reinterpret_cast<const run_t*>(base + roff[h]);
                else
                    v[u][h] = run_t(0);
            }
            l0 += 32;
            if (l0 >= L) {
                l0 = 0;
                ++b;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const double a0 = (double)v[u][0][e];
                if constexpr (JN == 16) {
                    acc[e & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, a0, acc[e & 1], 0, 0, 0);
                } else {
                    const double a1 = (double)v[u][1][e];
                    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, a0, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, a1, acc[1], 0, 0, 0);
                    acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, a1, acc[2], 0, 0, 0);
                }
            }
    }
    if constexpr (JN == 16) acc[0] += acc[1];

    // D[row][col] of pair c sits in lane col + 16 (row % 4), register row / 4
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            red[(wave * NP + c) * 256 + (4 * r + k4) * 16 + r16] = acc[c][r];
    __syncthreads();
    for (int e = threadIdx.x; e < NP * 256; e += kNarrowThreads) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kNarrowWaves; ++w) s += red[w * NP * 256 + e];
        partial[(int64_t)p * NP * 256 + e] = s;
    }
}

// ------------------------------------------------------------------ host

// Narrow-mode plan: one partial per workgroup, at most 2 per CU, each
// workgroup holding at least one batch of steps per wave.
constexpr int kNarrowStepsF32 = 4, kNarrowStepsF64 = 2;  // U: steps per batch

static int64_t narrow_steps(const ModeView& v) { return v.B * ((v.L + 31) / 32); }

static GramPlan plan_narrow(const ModeView& v, int elem_bytes) {
    GramPlan pl{};
    pl.narrow = v.J <= 16 ? 16 : 32;
    pl.nb = pl.narrow / 16;
    pl.npairs = pl.nb * (pl.nb + 1) / 2;
    pl.G = 1;
    pl.pairs_per_group = pl.npairs;
    const int U = elem_bytes == 8 ? kNarrowStepsF64 : kNarrowStepsF32;
    const int64_t per_wg = (int64_t)kNarrowWaves * U;
    const int64_t cap = 2 * (int64_t)device_cu_count();
    int64_t P = (narrow_steps(v) + per_wg - 1) / per_wg;
    pl.P = (int)(P < 1 ? 1 : P > cap ? cap : P);
    pl.partial_bytes = (size_t)pl.P * pl.npairs * 256 * sizeof(double);
    pl.partial_bound = (size_t)cap * pl.npairs * 256 * sizeof(double);
    return pl;
}

// Few columns, whose tiles don't fill the chip, take other schedules; the line
// is about where they stop to pay.  Times against one tile per workgroup of the
// schedules for many columns, both types, L = 1 .. 300:
//   J <= 64: tiles of 32 columns instead of 64 or 128, which a small tensor
//     doesn't fill.  J = 17 .. 64: 100 columns 0.75 - 0.91, 1500 0.83 - 0.98,
//     3500 0.85 - 1.04, 4500 0.95 - 1.06, 8000 1.00 - 1.34 (more partials to
//     reduce).
//   J > 160: the block pairs over many workgroups (gram_partial_wide), so that a
//     tile's products are spread, and at most 32 ranges of tiles, since every
//     range costs the reduction a partial per pair.  J = 161 .. 512: 600 columns
//     0.65 - 0.89, 3000 0.67 - 0.99, 4000 0.73 - 1.05, 6000 0.82 - 1.20.  (16
//     ranges took 0.82 - 1.13 times the time of 32 at 600 columns and 1.00 - 1.48
//     at 3000, 64 ranges 1.04 - 1.30 and 0.92 - 1.15.)  J = 145: 0.82 - 0.89, 0.94
//     - 1.04, 0.99 - 1.10, not worth a stage of its own.
constexpr double kFewColumns = 4096;
constexpr int kFewRanges = 32;

static GramPlan plan_tiled(const ModeView& v) {
    GramPlan pl{};
    pl.nb = (v.J + 15) / 16;
    pl.npairs = pl.nb * (pl.nb + 1) / 2;
    const bool few = (double)v.L * (double)v.B <= kFewColumns;
    int64_t want = device_cu_count();
    pl.G = 1;
    if (pl.nb <= 16) {
        with_blocks(pl.nb, [&](auto nbc) {
            constexpr int NB = decltype(nbc)::value;
            pl.KT = few && NB <= 4 ? GramSched<NB, true>::KT : GramSched<NB>::KT;
            want *= GramSched<NB>::kPerCu;
            return (int)TK_OK;
        });
    } else {
        pl.KT = kWideKt;
        pl.G = (pl.npairs + kWidePairs - 1) / kWidePairs;
        want = xcd_round_want(want / pl.G, pl.G);
    }
    pl.partial_bound = (size_t)want * pl.npairs * 256 * sizeof(double);
    if (few && pl.nb > 10) {
        pl.KT = kWideKt;
        want = want < kFewRanges ? want : kFewRanges;
        const int64_t p = xcd_ranges(make_tiles(v, pl.KT).ntiles, want, 2);
        int G = device_cu_count() / (int)p;
        if (G > pl.npairs / 16) G = pl.npairs / 16;
        if (G > pl.G) pl.G = G;
    }
    pl.pairs_per_group = (pl.npairs + pl.G - 1) / pl.G;
    pl.P = xcd_ranges(make_tiles(v, pl.KT).ntiles, want, pl.G);
    pl.partial_bytes = (size_t)pl.P * pl.npairs * 256 * sizeof(double);
    return pl;
}

// The narrow kernel's plan where the view qualifies; its workspace bounds
// also cover the tiled plan, which runs instead when the data pointer is not
// aligned for the kernel's vector loads.
GramPlan plan_gram(const ModeView& v, int precision, int elem_bytes) {
    if (precision == TK_GRAM_SPLIT_BF16) return plan_gram_mixed(v);
    GramPlan tiled = plan_tiled(v);
    if (!gram_narrow_view(v)) return tiled;
    GramPlan pl = plan_narrow(v, elem_bytes);
    if (tiled.partial_bytes > pl.partial_bytes) pl.partial_bytes = tiled.partial_bytes;
    if (tiled.partial_bound > pl.partial_bound) pl.partial_bound = tiled.partial_bound;
    return pl;
}

template <typename T, int JN>
static int launch_narrow(const T* y, const ModeView& v, const GramPlan& pl, double* partial,
                         hipStream_t st) {
    constexpr int U = sizeof(T) == 8 ? kNarrowStepsF64 : kNarrowStepsF32;
    hipLaunchKernelGGL((gram_narrow_f64<T, JN, U>), dim3(pl.P), dim3(kNarrowThreads), 0, st, y,
                       v.L, v.J, narrow_steps(v), pl.P, partial);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

template <typename T>
static int dispatch_narrow(const T* y, const ModeView& v, const GramPlan& pl, double* partial,
                           hipStream_t st) {
    return pl.narrow == 16 ? launch_narrow<T, 16>(y, v, pl, partial, st)
                           : launch_narrow<T, 32>(y, v, pl, partial, st);
}

static int launch_gram_reduce(const double* partial, const GramPlan& pl, int J, double* s,
                              const double* aux, double* stats, hipStream_t st) {
    int n = pl.npairs * 256;
    const int nblk = (n + 63) / 64 + (aux ? 1 : 0);
    hipLaunchKernelGGL(gram_reduce, dim3(nblk), dim3(256), 0, st, partial, pl.P, pl.npairs,
                       pl.nb, J, s, aux, stats);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

// One launch reduces the partials of every problem of a batch (and forms the
// trace of those that need ||X||^2), in the same fixed order as gram_reduce.
__global__ __launch_bounds__(256) void gram_reduce_batched(const BatchReduceTask* __restrict__ tasks,
                                                           int ntasks, int conditional) {
    __shared__ double part[4][64];
    int lo = 0, hi = ntasks - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tasks[mid].wg_begin <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
    }
    BatchReduceTask tk = tasks[lo];
    tk.partial = uni_global(tk.partial);  // global, not flat, accesses
    tk.s = uni_global(tk.s);
    if (conditional && !(*tk.status & 4)) return;  // uniform over the workgroup
    const int w = blockIdx.x - tk.wg_begin;
    const int o = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int n = tk.npairs * 256;
    const int P = *tk.nparts;  // slots the Gram launch wrote (<= tk.P)
    // split statistics: a split Gram's, not a redo's nor an FP64-only problem's
    const bool split = tk.aux != nullptr && !conditional && !(tk.status && (*tk.status & 8));
    const bool extra = tk.nu != nullptr || split;
    if (w < tk.nwg - 1 || !extra) {
        const int idx = w * 64 + o;
        const double acc = idx < n ? sum_partials(tk.partial, P, n, idx, g) : 0.0;
        part[g][o] = acc;
        __syncthreads();
        if (g != 0 || idx >= n) return;
        const double tot = ((part[0][o] + part[1][o]) + part[2][o]) + part[3][o];
        const int p = idx >> 8, e = idx & 255;
        int bi, bj;
        pair_of(p, tk.nb, bi, bj);
        const int r = bi * 16 + (e >> 4), c = bj * 16 + (e & 15);
        if (r >= tk.J || c >= tk.J) return;
        if (bi == bj && r > c) return;
        tk.s[r + (int64_t)tk.J * c] = tot;
        tk.s[c + (int64_t)tk.J * r] = tot;
    } else {
        // the problem's last workgroup: split statistics of the unconditional
        // (split) pass, and the trace of its diagonal from the partials
        // (diagonal 16-blocks p = bi nb - bi (bi - 1) / 2), fixed order
        if (split) {
            reduce_split_stats(tk.aux, P, tk.stats, &part[0][0]);
            __syncthreads();
        }
        if (tk.nu == nullptr) return;
        // each diagonal entry summed as the other workgroups sum S's entries
        // (four slot groups, eight loads in flight each, then added in a
        // fixed order), the entries then lane by lane
        double acc = 0.0;
        for (int i0 = 0; i0 < tk.J; i0 += 64) {  // uniform
            const int i = i0 + o;
            const int bi = i >> 4, p = bi * tk.nb - bi * (bi - 1) / 2;
            const int idx = p * 256 + (i & 15) * 17;
            part[g][o] = i < tk.J ? sum_partials(tk.partial, P, n, idx, g) : 0.0;
            __syncthreads();
            if (g == 0) acc += ((part[0][o] + part[1][o]) + part[2][o]) + part[3][o];
            __syncthreads();
        }
        if (g == 0) part[0][o] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int k = 0; k < 64; ++k) t += part[0][k];
            *tk.nu = t;
        }
    }
}

// Clears status words with a kernel (no memset node in a captured graph).
__global__ void fill_i32(int* __restrict__ p, int n, int v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

int launch_fill_i32(int* p, int n, int v, hipStream_t st) {
    if (n <= 0) return TK_OK;
    hipLaunchKernelGGL(fill_i32, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

int launch_gram_reduce_batched(const BatchReduceTask* tasks_dev, int ntasks, int total_wg,
                               int conditional, hipStream_t st) {
    hipLaunchKernelGGL(gram_reduce_batched, dim3(total_wg), dim3(256), 0, st, tasks_dev, ntasks,
                       conditional);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

// One thread per task: the problem's FP64 Gram work at its actual shape
// (the truncated extents come from the device ranks) decides bit 8.
__global__ __launch_bounds__(64) void batch_mark_fp64(const BatchGramTask* __restrict__ tasks,
                                                      int ntasks, double max_flops) {
    const int t = blockIdx.x * 64 + threadIdx.x;
    if (t >= ntasks) return;
    const BatchGramTask tk = tasks[t];
    const ModeView v = batch_mode_view(tk.v);
    const double flops = 2.0 * (double)v.J * (double)v.J * (double)v.L * (double)v.B;
    if (flops <= max_flops) *const_cast<int*>(tk.status) |= 8;  // the task is the word's only writer here
}

int launch_batch_mark_fp64(const BatchGramTask* tasks_dev, int ntasks, double max_flops,
                           hipStream_t st) {
    if (ntasks <= 0) return TK_OK;
    hipLaunchKernelGGL(batch_mark_fp64, dim3((ntasks + 63) / 64), dim3(64), 0, st, tasks_dev,
                       ntasks, max_flops);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

int launch_gram(const void* y, int dtype, const ModeView& v, int precision, double* s,
                double* sumsq, void* ws, size_t ws_bytes, hipStream_t st,
                double* split_stats, const hipEvent_t* ev) {
    GramPlan pl = plan_gram(v, precision, (int)dtype_size(dtype));
    if (ws_bytes < pl.partial_bytes)
        return fail(TK_ERR_WORKSPACE, "gram workspace %zu < %zu", ws_bytes, pl.partial_bytes);
    double* partial = (double*)ws;
    // the narrow kernel's 8-element vector loads need the run's own alignment
    if (pl.narrow && (uintptr_t)y % (8 * dtype_size(dtype)) != 0) pl = plan_tiled(v);
    if (ev) TK_HIP(hipEventRecord(ev[0], st));
    if (precision == TK_GRAM_SPLIT_BF16) {
        TK_TRY(launch_gram_mixed((const float*)y, v, pl, partial, st));
    } else if (pl.narrow) {
        if (dtype == TK_F64)
            TK_TRY(dispatch_narrow((const double*)y, v, pl, partial, st));
        else
            TK_TRY(dispatch_narrow((const float*)y, v, pl, partial, st));
    } else if (dtype == TK_F64) {
        TK_TRY(launch_gram_f64((const double*)y, v, pl, partial, st));
    } else {
        TK_TRY(launch_gram_f64((const float*)y, v, pl, partial, st));
    }
    if (ev) TK_HIP(hipEventRecord(ev[1], st));
    const bool split = precision == TK_GRAM_SPLIT_BF16;
    const double* aux = split && split_stats ? partial + (size_t)pl.P * pl.npairs * 256 : nullptr;
    TK_TRY(launch_gram_reduce(partial, pl, v.J, s, aux, split_stats, st));
    if (sumsq) {
        hipLaunchKernelGGL(gram_trace, dim3(1), dim3(64), 0, st, s, v.J, sumsq);
        TK_HIP(hipGetLastError());
    }
    return TK_OK;
}

}  // namespace tk
