"""Staging of the tiled FP64 Gram and of the FP64 TTM with the operator in
registers (tile_io.hpp), compiled for the host: every store lies inside the
buffer it is given, in each of the two, and what a tile leaves there is the
tile, for the schedules of every block count and packed, strided, partial and
repeated tiles."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <algorithm>
#include <cstdio>
#include <cmath>
#include <utility>
#include <vector>
using std::max;
using std::min;
struct Dim { int x, y, z; };
static Dim threadIdx, blockIdx, gridDim;
static int __builtin_amdgcn_readfirstlane(int x) { return x; }
#include "tile_io.hpp"

using namespace tk;

template <class T, int NB, int KT, int THREADS, bool PACKED>
static int walk(const ModeView& v) {
    constexpr int BUF = kTileBuf<NB, KT>, P = KT + 1;
    const TileMap tm = make_tiles(v, KT);
    const int64_t n = v.L * v.J * v.B;
    std::vector<T> mem(n + 128, (T)NAN);  // nothing around the tensor may be used
    T* y = mem.data() + 64;
    for (int64_t i = 0; i < n; ++i) y[i] = (T)(1 + i % 8191);
    // two buffers of the size the kernels launch with, and a guard area behind
    std::vector<double> lds(2 * BUF + 4 * BUF, -1.0);
    std::fill(lds.begin(), lds.begin() + 2 * BUF, 0.0);
    std::vector<TileStage<T, NB, KT, THREADS, PACKED>> st(THREADS);
    const int per = st[0].kPer;
    const int64_t t0 = tm.ntiles / 3, t1 = tm.ntiles;
    for (int t = 0; t < THREADS; ++t) {
        threadIdx.x = t;
        st[t].begin(y, tm, t0, t1);
        for (int q = 0; q < per; ++q) st[t].load(q);
        st[t].advance();
    }
    for (int64_t tile = t0; tile < t1; ++tile) {
        double* buf = lds.data() + (tile - t0) % 2 * BUF;
        const std::vector<double> other(lds.data() + (1 - (tile - t0) % 2) * BUF,
                                        lds.data() + (2 - (tile - t0) % 2) * BUF);
        for (int t = 0; t < THREADS; ++t) {
            for (int q = 0; q < per; ++q) {
                st[t].store(buf, q);
                st[t].load(q);
            }
            st[t].advance();
        }
        if (!std::equal(other.begin(), other.end(), lds.data() + (1 - (tile - t0) % 2) * BUF))
            return printf("a store reached the other buffer\n"), 1;
        for (size_t i = 2 * BUF; i < lds.size(); ++i)
            if (lds[i] != -1.0) return printf("a store at %zu of %d\n", i, 2 * BUF), 1;
        const Tile g = tile_at(tm, tile, v.J);
        for (int i = 0; i < 16 * NB; ++i)
            for (int k = 0; k < KT; ++k) {
                const bool in = i < v.J && k < g.ncols;
                const double want = in ? (double)y[g.base + tile_col_offset(k, v.L, v.J) + i * v.L] : 0.0;
                if (buf[i * P + k] != want) return printf("row %d column %d of a tile\n", i, k), 1;
            }
    }
    return 0;
}

template <class T, int NB, int KT, int THREADS>
static int check(int jmax) {
    for (int J : {jmax, jmax - 1, jmax - 7, jmax - 15, 16 * (NB - 1) / 2 + 1, 3, 1}) {
        if (J < 1) continue;
        for (int64_t L : {1, 2, 3, 5, 10, 16, 31, 32, 33, 64, 100, 128, 130, 257}) {
            for (int64_t B : {1, 2, 7, 150}) {
                if (L > 30 && B > 7) continue;
                const ModeView v{L, B, J};
                const int bad = L <= KT ? walk<T, NB, KT, THREADS, true>(v) : walk<T, NB, KT, THREADS, false>(v);
                if (bad) {
                    printf("NB %d KT %d threads %d: J %d L %d B %d\n", NB, KT, THREADS, J, (int)L, (int)B);
                    return 1;
                }
            }
        }
    }
    return 0;
}

// the staged shapes of gram_f64.hpp and ttm_f64.hpp
template <int NB>
static int gram() {
    constexpr int KT = NB <= 2 ? 128 : NB <= 4 ? 64 : 32, THREADS = NB <= 8 ? 256 : 512;
    if constexpr (NB <= 4)
        if (check<double, NB, 32, THREADS>(16 * NB)) return 1;
    return check<double, NB, KT, THREADS>(16 * NB) || check<float, NB, KT, THREADS>(16 * NB);
}

int main() {
    return gram<1>() || gram<2>() || gram<3>() || gram<4>() || gram<5>() || gram<6>() || gram<7>() || gram<8>() ||
           gram<9>() || gram<12>() || gram<13>() || gram<16>() || check<float, 16, 16, 512>(256) ||
           check<double, 20, 16, 512>(320) ||
           check<float, 24, 16, 512>(384) || check<double, 28, 16, 512>(448) || check<float, 32, 16, 512>(512) ||
           check<double, 8, 64, 512>(128) || check<float, 12, 32, 512>(192) || check<double, 16, 32, 512>(256);
}
"""


def test_stores_stay_in_their_buffer(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("needs g++")
    src, exe = tmp_path / "stage.cpp", tmp_path / "stage"
    src.write_text(SOURCE)
    subprocess.run([cxx, "-O1", "-w", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1510_06689_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
