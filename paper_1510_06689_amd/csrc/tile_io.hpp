// Column-tile staging shared by the streaming kernels (Gram, TTM).
//
// A tile is J x KT columns of the block-column view Y[B][J][L] (TileMap).
// ColumnTile loads one tile into registers with a thread mapping that keeps
// every wave's global loads contiguous, and writes it to LDS, widened to the
// compute type (a conversion at the load would wait for the data), as
// [i][kk] with a row pitch of KT + 1 elements (an odd
// pitch in 8-byte words spreads both the row-wise and the column-wise
// accesses across banks).
//   L == 1 : column kk is J contiguous elements -> thread t reads row
//            i = t % JB of column t / JB (+ column passes);
//   L  > 1 : rows are runs along kk -> thread t reads column kk = t % KT of
//            row t / KT (+ row passes); the column's offset inside the tile
//            is fixed per thread.
// Elements outside the tile (rows >= J, columns >= the tile's width) are 0.
#pragma once

#include "tk_common.hpp"

namespace tk {

// Offset (relative to a tile's base) of tile column kk: kk = bb * L + l maps
// to bb * J * L + l.  For strided tiles (L >= KT) this is kk itself.
__device__ __forceinline__ int64_t tile_col_offset(int kk, int64_t L, int J) {
    int64_t bb = kk / L;
    return bb * J * L + (kk - bb * L);
}

template <typename T, typename C, int JB, int KT, int THREADS>
struct ColumnTile {
    static_assert(JB * KT % THREADS == 0, "tile must split evenly over threads");
    static_assert(THREADS % JB == 0 && THREADS % KT == 0, "thread mappings need JB, KT | THREADS");
    static constexpr int kPer = JB * KT / THREADS;
    static constexpr int P = KT + 1;  // LDS row pitch (elements)
    T v[kPer];
    int64_t coff;  // L > 1: offset of this thread's column
    int kk0, i0;   // this thread's first (i, kk)
    bool unit;     // L == 1

    __device__ __forceinline__ void setup(const TileMap& tm, int tid) {
        unit = tm.L == 1;
        if (unit) {
            i0 = tid % JB;
            kk0 = tid / JB;
            coff = 0;
        } else {
            kk0 = tid % KT;
            i0 = tid / KT;
            coff = tile_col_offset(kk0, tm.L, tm.J);
        }
    }

    __device__ __forceinline__ void load(const T* __restrict__ y, const TileMap& tm,
                                         const Tile& t) {
        if (unit) {
            constexpr int colstep = THREADS / JB;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                int kk = kk0 + q * colstep;
                T val = T(0);
                if (i0 < tm.J && kk < t.ncols) val = y[t.base + (int64_t)kk * tm.J + i0];
                v[q] = val;
            }
        } else {
            constexpr int rowstep = THREADS / KT;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                int i = i0 + q * rowstep;
                T val = T(0);
                if (i < tm.J && kk0 < t.ncols) val = y[t.base + coff + (int64_t)i * tm.L];
                v[q] = val;
            }
        }
    }

    __device__ __forceinline__ void store(C* lds) const {
        if (unit) {
            constexpr int colstep = THREADS / JB;
#pragma unroll
            for (int q = 0; q < kPer; ++q) lds[i0 * P + kk0 + q * colstep] = (C)v[q];
        } else {
            constexpr int rowstep = THREADS / KT;
#pragma unroll
            for (int q = 0; q < kPer; ++q) lds[(i0 + q * rowstep) * P + kk0] = (C)v[q];
        }
    }
};

// Stages the tiles of a workgroup's range one after another: registers hold
// one tile (16 NB rows by KT columns at most) in its storage type, which is
// widened and written to LDS ([i][kk], pitch KT + 1) one element at a time
// while the next tile's elements are loaded into the freed registers.  The
// element-wise calls have no branches, so that they can be spread between the
// products of the tile being multiplied; loads are clamped into the tile
// instead, and a store puts zero for what lies outside.  (With a branch per
// element, and all waves of a CU staging at once, an FP64 Gram's matrix cores
// idled for a third of the time; a conversion at the load instead of the
// store doubled the time of one on FP32 data.)
//   PACKED (TileMap::packed): the tile is one contiguous range and is read as
//   such, so lanes stay dense and lines are read once whatever L and J are.
//   strided: thread t reads column t % KT of row t / KT (+ passes).
// LDS: rows at or past J and a packed tile's padding columns are never
// written and must be zeroed first.  A buffer (kTileBuf) ends with 64 doubles
// that take the stores of lanes without an element: they belong to the buffer,
// so every offset is valid from the start of either one.
template <int NB, int KT>
constexpr int kTileBuf = 16 * NB * (KT + 1) + 64;

template <typename T, int NB, int KT, int THREADS, bool PACKED>
struct TileStage {
    static_assert(16 * NB * KT % THREADS == 0 && THREADS % KT == 0, "tile over threads");
    static constexpr int kPer = 16 * NB * KT / THREADS;
    static constexpr int P = KT + 1;
    static constexpr int RS = THREADS / KT;  // rows per pass
    static constexpr int kTrash = kTileBuf<NB, KT> - 64;
    T v[kPer];
    int at[PACKED ? kPer : 1];  // offset of each element in a buffer; strided: of the first row
    int64_t row0;               // strided: offset of this thread's first row
    int tid, kk, J;
    int64_t L;
    // the tile to load next (uniform): first element, elements (PACKED) or
    // columns it has, its place, and how many tiles follow it
    const T* p;
    int n;
    int64_t place, left, span;  // PACKED: b-blocks after it; strided: its segment
    int nreg;                   // n of the tile in the registers

    // Tiles t0 .. t1 - 1 (t0 < t1), the last one repeated when asked for more.
    __device__ __forceinline__ void begin(const T* __restrict__ y, const TileMap& tm, int64_t t0,
                                          int64_t t1) {
        tid = threadIdx.x;
        J = tm.J;
        L = tm.L;
        const Tile t = tile_at(tm, t0, tm.J);
        p = y + t.base;
        left = t1 - 1 - t0;
        if constexpr (PACKED) {
            span = (int64_t)tm.nbb * tm.J * tm.L;
            n = (int)t.nvalid;
            place = tm.B - (t0 + 1) * tm.nbb;
            // element tid + THREADS q is (bb, i, l) in mixed radix (., J, L);
            // THREADS is added digit by digit
            const int Li = (int)tm.L, total = (int)span;
            int r = tid / Li, l = tid - r * Li;
            int bb = r / J, i = r - bb * J;
            const int r1 = THREADS / Li, l1 = THREADS - r1 * Li;
            const int b1 = r1 / J, i1 = r1 - b1 * J;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int in = i * P + bb * Li + l;
                at[q] = tid + q * THREADS < total ? in : kTrash + (tid & 63);
                l += l1;
                i += i1;
                bb += b1;
                const int cl = l >= Li ? 1 : 0;
                l -= cl ? Li : 0;
                i += cl;
                const int ci = i >= J ? 1 : 0;
                i -= ci ? J : 0;
                bb += ci;
            }
        } else {
            span = tm.lsegs;
            n = t.ncols;
            place = t0 % tm.lsegs;
            kk = tid % KT;
            const int i0 = min(tid / KT, J - 1);
            row0 = (int64_t)i0 * L;
            at[0] = i0 * P + kk;
        }
    }

    __device__ __forceinline__ void advance() {
        nreg = n;
        if (left <= 0) return;
        --left;
        if constexpr (PACKED) {
            p += span;
            const int64_t nb = place * J * L;  // place >= 1: there is another tile
            n = (int)(nb < span ? nb : span);
            place -= span / ((int64_t)J * L);
        } else {
            const bool wrap = place + 1 == span;
            p += wrap ? J * L - place * KT : KT;
            place = wrap ? 0 : place + 1;
            const int64_t w = L - place * KT;
            n = (int)(w < KT ? w : KT);
        }
    }

    // First row of pass q: the last passes repeat rows (the same values go to
    // the same places twice) rather than leave the tile.
    __device__ __forceinline__ int pass_row(int q) const {
        return max(0, min(q * RS, J - RS));
    }

    __device__ __forceinline__ void load(int q) {
        if constexpr (PACKED)
            v[q] = p[min(tid + q * THREADS, n - 1)];
        else
            v[q] = (p + (int64_t)pass_row(q) * L)[row0 + min(kk, n - 1)];
    }

    __device__ __forceinline__ void store(double* buf, int q) const {
        if constexpr (PACKED)
            buf[at[q]] = tid + q * THREADS < nreg ? (double)v[q] : 0.0;
        else
            buf[at[0] + pass_row(q) * P] = kk < nreg ? (double)v[q] : 0.0;
    }
};

}  // namespace tk
