// FP64 symmetric eigensolver + rank truncation for one J x J Gram matrix
// (Alg. 1, eigenvector and rank steps; Sec. V-D uses a LAPACK subset solver,
// this is the same family of method on one workgroup):
//
//   1. Householder reduction to tridiagonal form T = Q^T S Q.  Each step
//      derives the reflector from the pivot row, forms p = tau A22 v, then
//      applies the rank-2 update A22 -= v w^T + w v^T.  For J <= 128 the
//      matrix lives in one workgroup's registers; otherwise the first
//      J - 192 columns, if any, are reduced by 64 single-wave workgroups that
//      hold it together (eig_reduce_grid), one workgroup brings the last 192
//      to 128 (eig_reduce_mid) and one finishes those (eig_reduce_tail); the
//      reflectors go to global scratch;
//   2. all eigenvalues of T by multisection: groups of threads per
//      eigenvalue evaluate Sturm counts with the three-term determinant
//      recurrence of T scaled by a power of two (exact), rescaled (exactly)
//      every eight rows; a ballot picks the sub-interval;
//   3. rank rule R = min R >= 1 with sum_{r>R} max(lambda_r,0) <= eps^2 nu / N
//      (tail sums accumulated smallest first), or a fixed rank;
//   4. the R leading eigenvectors of T by inverse iteration (tridiagonal LU
//      with partial pivoting from both ends to the middle, kept in LDS,
//      reciprocal pivots, two iterations),
//      in batches that fit in LDS, then modified Gram-Schmidt (twice) inside
//      eigenvalue clusters by one wave;
//   5. back-transformation X <- Q X, 16 lanes per eigenvector with the
//      vector in registers (no barriers), and a sign rule (largest |entry|
//      positive, lowest index on ties), written to the factor output.
// Extents above 128 and ranks of more than one batch run step 4's inverse
// iteration on a workgroup per batch, and the rest in two more launches once
// the host knows the rank (launch_eig_finish).
// Barriers never wait on global stores inside loops: global memory is only
// written between phases.  One workgroup of 1024 threads, except that from
// J = 64 on step 2 runs in a launch of its own (eig_multisect, one wave per
// eigenvalue) between two launches of the solver; no host sync.
#include <cfloat>
#include <type_traits>

#include "tk_common.hpp"

namespace tk {

constexpr int kEigThreads = 1024;
constexpr int kEigWaves = kEigThreads / 64;
constexpr int kInvIters = 2;
constexpr int kLuArrays = 6;  // u0 (reciprocal), u1, u2, multiplier, pivot flag, x
constexpr int kSweepRows = 4;  // rows per block of the inverse-iteration sweeps

// Rows of the inverse-iteration arrays: half of J (two threads carry a
// vector), padded to whole sweep blocks, and the doubles of one of the two
// records: kLuArrays per row and one more.
__host__ __device__ constexpr int eig_sweep_rows(int J) {
    return ((J + 1) / 2 + kSweepRows - 1) / kSweepRows * kSweepRows;
}
__host__ __device__ constexpr int eig_record_doubles(int J) {
    return kLuArrays * eig_sweep_rows(J) + 1;
}

// Moves a double across lanes with one DPP pattern (applied to both 32-bit
// halves); lanes the pattern does not write receive 0.
template <int CTRL, int ROW_MASK, bool BOUND_CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const long long bits = __double_as_longlong(v);
    int lo = (int)(bits & 0xffffffffll), hi = (int)(bits >> 32);
    lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROW_MASK, 0xf, BOUND_CTRL);
    hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROW_MASK, 0xf, BOUND_CTRL);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Calls f(std::integral_constant<int, I>) for I = B .. E - 1 in order.
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

__device__ __forceinline__ double read_lane(double v, int lane) {
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(bits & 0xffffffffll), lane);
    const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum over the 64 lanes of a wave, in a fixed order, returned to every lane.
// Row prefix sums by row_shr 1, 2, 4, 8 leave each 16-lane row's total in its
// lane 15; row_bcast 15 and 31 then carry the row totals into lane 63.  Must
// be called with all lanes active.
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_move<0x111, 0xf, true>(v);   // row_shr:1
    v += dpp_move<0x112, 0xf, true>(v);   // row_shr:2
    v += dpp_move<0x114, 0xf, true>(v);   // row_shr:4
    v += dpp_move<0x118, 0xf, true>(v);   // row_shr:8
    v += dpp_move<0x142, 0xa, false>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_move<0x143, 0xc, false>(v);  // row_bcast:31 into rows 2 and 3
    return read_lane(v, 63);
}

// 1/q from the hardware reciprocal refined by one Newton step.
__device__ __forceinline__ double recip(double q) {
    double r = __builtin_amdgcn_rcp(q);
    double err = fma(-q, r, 1.0);
    return fma(r, err, r);
}

// 1/sqrt(s) (s > 0 finite) from the hardware estimate refined by two Newton
// steps r <- r + r (1 - s r^2) / 2.
__device__ __forceinline__ double rsq(double s) {
    double r = __builtin_amdgcn_rsq(s);
    double err = fma(-(s * r), r, 1.0);
    r = fma(0.5 * r, err, r);
    err = fma(-(s * r), r, 1.0);
    return fma(0.5 * r, err, r);
}

// Deterministic start vector entry in [-1, 1) for inverse iteration: the
// pair (a, b) goes through SplitMix64's golden-ratio increment and its
// published 64-bit finaliser (Steele, Lea and Flood, 2014).
__device__ __forceinline__ double hash_unit(uint32_t a, uint32_t b) {
    uint64_t z = ((uint64_t)a << 32) ^ (uint64_t)b ^ 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;  // [-1, 1)
}

// J <= 128: an unused J x J area (its start is the hand-off of a split solve)
// and the reflectors H (J x J).  J > 128: the exchange slots of the reduction
// over many waves (products, J x J), H, the exchange slots of the pivot rows
// (J x J) and the hand-off.
size_t eig_scratch_doubles(int J) {
    return J > 128 ? (size_t)3 * J * J + (size_t)6 * J + 64 : (size_t)2 * J * J + 64;
}

// small per-matrix arrays, and room for the four vector buffers of the register
// reduction (4 JP <= 512 doubles of the last 1024)
static size_t eig_small_doubles(int J) { return (size_t)8 * J + 64 + 8 + (size_t)kEigThreads; }

// LDS doubles for the matrix (J <= 128) and later the inverse-iteration
// batch; region + small arrays stay within the 160 KB of LDS.
static size_t eig_region_doubles(int J) {
    const size_t lds_doubles = 160 * 1024 / sizeof(double);
    size_t cap = lds_doubles - eig_small_doubles(J) - 128;
    if (cap > 16384) cap = 16384;                 // J <= 128 also holds A here (J*J <= 16384)
    // room for every vector in one batch: two records and two scale factors
    const size_t want = ((size_t)2 * eig_record_doubles(J) + 2) * J;
    return (want < cap ? want : cap) & ~size_t(1);  // even: what follows holds 16-byte pairs
}

// Number of eigenvalues of the (scaled) tridiagonal matrix below x: sign
// changes along the leading principal minors
//   p_0 = 1,  p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}.
// The squares are at least kMinE2 (scale_t raises smaller ones: a change of T
// by 2^-70 of its norm), so an exactly zero minor is followed by one of the
// opposite sign to its predecessor: one sign change over the two steps
// whichever sign the zero takes, and nothing needs to replace it.
//
// What bounds it: a wave's own instructions, since a solve's few waves leave
// SIMDs idle.  A step is three FP64 instructions, of which one fma is in the
// chain, and one that shifts its sign into a word; signs are compared and
// counted once per block of eight rows, and the pair (p_{i-1}, p_i) is
// rescaled once per block (exact): it grows by less than 2^16 and, losing a
// rounding and a smallest square every second step, shrinks by less than
// 2^-780, so from 2^kTop it neither overflows nor vanishes.  Rows are read
// a block ahead: through the scalar unit from the hand-off area in the split
// solves (no vector instruction, no LDS; T is the same for every lane), from
// LDS in the one-launch solver.  Both may read, and do not use, up to eight
// rows behind the last one; what follows T in both places is longer.  One wave per eigenvalue, J = 128:
// testing and counting every minor in floating point 50 us, in integers every
// step with rows through LDS 42 us, this form 27 us (J = 301
// 120, 100, 46).  Four rows ahead instead of eight left the scalar loads'
// latency in sight: 34 us.
constexpr double kMinE2 = 0x1p-140;
constexpr double kSectTol = 2.0 * DBL_EPSILON;  // width of a found interval; T is scaled to norm <= 1
struct TRows {
    double d[8], e2[8];  // eight rows of T: d_i, e_{i-1}^2
};

struct LdsRows {
    const double2* t;  // (d_i, e_{i-1}^2)
    __device__ __forceinline__ void load(int i, TRows& q) const {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const double2 v = t[i + r];
            q.d[r] = v.x;
            q.e2[r] = v.y;
        }
    }
    __device__ __forceinline__ void sent() const {}
    __device__ __forceinline__ void arrive() const {}  // LDS returns in order: the compiler's waits do
};

struct ScalarRows {
    using cdouble = const __attribute__((address_space(4))) double;
    cdouble* t;  // pairs as above, written by an earlier launch
    __device__ __forceinline__ explicit ScalarRows(const double* p)
        : t(reinterpret_cast<cdouble*>(reinterpret_cast<uint64_t>(p))) {}
    __device__ __forceinline__ void load(int i, TRows& q) const {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            q.d[r] = t[2 * (i + r)];
            q.e2[r] = t[2 * (i + r) + 1];
        }
    }
    // scalar loads return in any order, so a wait is for all of them: here,
    // before the next ones go out
    __device__ __forceinline__ void arrive() const {
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void sent() const { __builtin_amdgcn_sched_barrier(0); }
};

template <class Rows>
__device__ __forceinline__ int sturm_count(const Rows& rows, double d0, int J, double x) {
    constexpr int kTop = 800;
    double p0 = 0x1p800, p1 = (d0 - x) * 0x1p800;
    unsigned sg = (unsigned)__double2hiint(p1) >> 31;  // signs, the latest in bit 0
    int c = (int)sg;
    auto step = [&](const TRows& q, int r) {
        const double p2 = fma(q.d[r] - x, p1, -q.e2[r] * p0);
        sg = __builtin_amdgcn_alignbit(sg, (unsigned)__double2hiint(p2), 31);  // sg << 1 | sign
        p0 = p1;
        p1 = p2;
    };
    auto block = [&](const TRows& q) {
#pragma unroll
        for (int r = 0; r < 8; ++r) step(q, r);
        c += __popc((sg ^ (sg >> 1)) & 0xffu);
        const unsigned ex = (unsigned)__double2hiint(fmax(fabs(p0), fabs(p1))) & 0x7ff00000u;
        const double f = __hiloint2double((int)(((2 * 1023u + kTop) << 20) - ex), 0);
        p0 *= f;
        p1 *= f;
    };
    auto tail = [&](const TRows& q, int left) {  // 0 to 7 rows
#pragma unroll
        for (int r = 0; r < 7; ++r)
            if (r < left) step(q, r);
        return c + __popc((sg ^ (sg >> 1)) & ((1u << left) - 1u));
    };
    TRows qa, qb;
    rows.load(1, qa);
    int i = 1;
    for (; i + 15 < J; i += 16) {
        rows.arrive();
        rows.load(i + 8, qb);
        rows.sent();
        block(qa);
        rows.arrive();
        rows.load(i + 16, qa);
        rows.sent();
        block(qb);
    }
    if (i + 7 < J) {
        rows.arrive();
        rows.load(i + 8, qb);
        rows.sent();
        block(qa);
        rows.arrive();
        return tail(qb, J - i - 8);
    }
    rows.arrive();
    return tail(qa, J - i);
}

// Sum over the 8 consecutive lanes of a row group (every lane gets the same
// bits: each step adds the same two values in either order).
__device__ __forceinline__ double row8_sum(double v) {
    v += dpp_move<0xb1, 0xf, false>(v);   // quad_perm [1,0,3,2]
    v += dpp_move<0x4e, 0xf, false>(v);   // quad_perm [2,3,0,1]
    v += dpp_move<0x141, 0xf, false>(v);  // row_half_mirror
    return v;
}

// Sum over the 16 lanes of a row (every lane gets the same bits).
__device__ __forceinline__ double row16_sum(double v) {
    v = row8_sum(v);
    v += dpp_move<0x140, 0xf, false>(v);  // row_mirror
    return v;
}

// Householder tridiagonalisation of a symmetric Jr x Jr block held in
// registers (Jr <= JP): element (i, j) of the block is src[i + ld j].  Its
// diagonal, off-diagonal and reflector scalars go to d, e, beta at offset
// koff, and reflector koff + k (length Jr - k - 1) to H[(koff + k) J ..].
// With koff = 0, Jr = J this is the whole reduction; with koff > 0 it
// finishes one whose first koff columns the kernels for extents above 128 have
// reduced.
template <int JP>
__device__ __forceinline__ void tridiag_regs(const double* __restrict__ src, int ld, int Jr,
                                             int koff, int J, double* reg, double* red,
                                             double* d, double* e, double* beta, double* H) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // ---- 1. Householder tridiagonalisation, A in registers ---------------
    // Thread t owns rows 2 (t / 16) and the next and of them the columns
    // j = t % 16 + 16 q.  Per column k: the 16 owners of row k form the
    // reflector and publish v; (A22 v)_i is a sum over the row's 16 lanes and
    // p = tau A22 v is published; each thread then updates its own elements.
    // Vectors alternate between two LDS buffers so that two barriers per
    // column suffice; reflectors collect in LDS and go to the global scratch
    // once at the end.
    //
    // What bounds a column: the chain of the reflector and the two exchanges,
    // and every row's reading v and p from LDS.  Two rows per thread halve
    // those reads against one row on eight lanes, and v and p fit in
    // registers between the product and the update: J = 128 154 -> 130 us,
    // J = 100 128 -> 107.  (A 32 x 32 grid of threads whose waves each form
    // the reflector, for one barrier per column, was issue-bound: 280 us.)
    constexpr int NQ = JP / 16;
    const int rp = tid >> 4, rc = tid & 15, r0 = 2 * rp;
    double av[2][NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int j = rc + 16 * q;
        av[0][q] = (r0 < Jr && j < Jr) ? src[r0 + (size_t)ld * j] : 0.0;
        av[1][q] = (r0 + 1 < Jr && j < Jr) ? src[r0 + 1 + (size_t)ld * j] : 0.0;
    }
    double* Hs = reg;
    // Every load below stays inside the reflector store (zeroed first, so
    // that entries no step writes are exact zeros: reflector k is written
    // from column k + 1 on) and four JP-long vector buffers in the area after
    // misc (zeroed too).  Finished rows and columns see v = p = 0, so the
    // register loops need no masks.
    static_assert(4 * JP <= kEigThreads, "vector buffers must fit the area after misc");
    double* vbuf = red + 64 + 8;
    for (int i = tid; i < 4 * JP; i += kEigThreads) vbuf[i] = 0.0;
    for (int i = tid; i < (Jr > 2 ? Jr - 2 : 0) * JP; i += kEigThreads) Hs[i] = 0.0;
    __syncthreads();
    // Columns run in blocks of 16, the block index KB and the parity of k
    // compile-time constants: chunks below KB are finished for every column of
    // the block (their v and p are zero), so each loop starts at chunk KB with
    // no test, and only chunks KB and KB + 1 can hold the pivot column k + 1.
    static_for<0, NQ>([&](auto kbc) {
        constexpr int KB = decltype(kbc)::value;
        auto column = [&](int k, auto parity) {
            constexpr int PR = decltype(parity)::value;  // k & 1
            double* vs = Hs + (size_t)k * JP;    // v = reflector k: v_{k+1} = 1, zero outside k < j < Jr
            double* ps = vbuf + (2 + PR) * JP;   // p = tau A22 v, zero outside k < i < Jr
            double* sg = red + 40 + PR;          // tau of column k
            // The pair index goes through an empty asm so that the compiler
            // cannot use rp == k / 2 to replace the uniform k by the per-lane
            // row inside the owner branch (that turns every column test below
            // into a per-lane mask held across the loop).
            int rp_k = rp;
            asm volatile("" : "+v"(rp_k));
            if (rp_k == (k >> 1)) {
                // The owners of row k (= column k, x = its part beyond the
                // diagonal) form the reflector alone, in the form of LAPACK's
                // dlarfg: alpha = -sign(x_0) |x|, tau = 1 + |x_0| / |x|,
                // v = x / (x_0 - alpha) (one reciprocal square root and one
                // reciprocal), and publish v.
                double sq[2] = {0.0, 0.0};
#pragma unroll
                for (int q = KB; q < NQ; ++q) {
                    const double m = (q > KB + 1 || rc + 16 * q >= k + 2) ? av[PR][q] : 0.0;
                    sq[q & 1] = fma(m, m, sq[q & 1]);
                }
                const double sigma = row16_sum(sq[0] + sq[1]);
                // a_kk and a_k,k+1 from the lanes of row k that hold them:
                // column k lies in chunk KB, column k + 1 in KB or KB + 1
                const int l0 = 16 * ((k >> 1) & 3);
                const double akk = read_lane(av[PR][KB], l0 + (k & 15));
                const double x0 =
                    read_lane(((k + 1) >> 4) == KB ? av[PR][KB] : av[PR][KB + 1 < NQ ? KB + 1 : KB],
                              l0 + ((k + 1) & 15));
                double tau = 0.0, alpha = x0, inv_v0 = 0.0;
                if (sigma != 0.0) {
                    const double ss = fma(x0, x0, sigma);
                    const double r = rsq(ss);  // 1 / |x|
                    const double mu = ss * r;
                    const double sgn = x0 < 0.0 ? -1.0 : 1.0;
                    alpha = -sgn * mu;
                    tau = fma(fabs(x0), r, 1.0);
                    inv_v0 = sgn * recip(fabs(x0) + mu);
                }
#pragma unroll
                for (int q = KB; q < NQ; ++q) {
                    const int j = rc + 16 * q;
                    const double vj = av[PR][q] * inv_v0;  // av is 0 beyond Jr
                    vs[j] = q > KB + 1 ? vj : (j == k + 1 ? 1.0 : (j > k + 1 ? vj : 0.0));
                }
                if (rc == 0) {
                    *sg = tau;
                    d[koff + k] = akk;
                    e[koff + k] = alpha;
                    beta[koff + k] = tau;
                }
            }
            __syncthreads();
            const double tau = *sg;
            // A wave whose 8 rows are all <= k has nothing to form or update (uniform).
            const bool wact = 8 * wave + 7 > k;
            double part = 0.0;
            double vq[NQ];
            if (wact) {  // formed before tau is tested, so that v's loads do not wait for it
                double s0[2] = {0.0, 0.0}, s1[2] = {0.0, 0.0};
#pragma unroll
                for (int q = KB; q < NQ; ++q) {
                    vq[q] = vs[rc + 16 * q];
                    s0[q & 1] = fma(av[0][q], vq[q], s0[q & 1]);
                    s1[q & 1] = fma(av[1][q], vq[q], s1[q & 1]);
                }
                // (A22 v)_i of the first row to lanes 0-7, of the second to 8-15
                const double a0 = s0[0] + s0[1], a1 = s1[0] + s1[1];
                const bool hi = rc >= 8;
                part = row8_sum((hi ? a1 : a0) + dpp_move<0x140, 0xf, false>(hi ? a0 : a1));
            }
            if (tau == 0.0) return;  // uniform: the reflector is the identity
            const int rw = r0 + (rc >> 3);
            if ((rc & 7) == 0 && rw < JP) ps[rw] = (wact && rw > k && rw < Jr) ? tau * part : 0.0;
            __syncthreads();
            if (!wact) return;  // uniform over the wave; it still meets every barrier
            // A22 -= v w^T + w v^T with w = p - (tau/2)(p.v) v, two fused
            // multiply-adds per element; entries outside the trailing block
            // see v = w = 0.  Every row's lanes form p.v from the same values
            // with the same bits.  The update rounds a_ij and a_ji
            // differently, so A is symmetric up to rounding; only each row's
            // own elements are ever read, so the reduction is that of a matrix
            // within rounding of the exact iterate.
            const int rr = r0 < JP ? r0 : 0;
            const double v0 = vs[rr], v1 = vs[rr + 1], p0 = ps[rr], p1 = ps[rr + 1];
            double pq[NQ], pv[2] = {0.0, 0.0};
#pragma unroll
            for (int q = KB; q < NQ; ++q) {
                pq[q] = ps[rc + 16 * q];
                pv[q & 1] = fma(pq[q], vq[q], pv[q & 1]);
            }
            const double half = 0.5 * tau * row16_sum(pv[0] + pv[1]);
            const double w0 = fma(-half, v0, p0), w1 = fma(-half, v1, p1);
#pragma unroll
            for (int q = KB; q < NQ; ++q) {
                const double wj = fma(-half, vq[q], pq[q]);
                av[0][q] = fma(-w0, vq[q], fma(-v0, wj, av[0][q]));
                av[1][q] = fma(-w1, vq[q], fma(-v1, wj, av[1][q]));
            }
        };
        const int kend = min(16 * KB + 16, Jr - 2);
        for (int k = 16 * KB; k < kend; k += 2) {
            column(k, std::integral_constant<int, 0>{});
            if (k + 1 < kend) column(k + 1, std::integral_constant<int, 1>{});
        }
    });
    // the trailing 2 x 2 block (or 1 x 1)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int ri = r0 + h;
        if (ri < Jr - 2 || ri >= Jr) continue;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int j = rc + 16 * q;
            if (j == ri) d[koff + ri] = av[h][q];
            if (ri == Jr - 2 && j == Jr - 1) e[koff + Jr - 2] = av[h][q];
        }
    }
    if (tid == 0) {
        if (Jr >= 2) beta[koff + Jr - 2] = 0.0;
        e[koff + Jr - 1] = 0.0;
        beta[koff + Jr - 1] = 0.0;
    }
    __syncthreads();
    // reflector koff + k has length J - (koff + k) - 1 = Jr - k - 1
    for (int idx = tid; idx < (Jr - 2) * Jr; idx += kEigThreads) {
        const int k = idx / Jr, i = idx - k * Jr;
        if (i < Jr - k - 1) H[(size_t)(koff + k) * J + i] = Hs[(size_t)k * JP + k + 1 + i];
    }
    __syncthreads();
}

// Hand-off area of a split solve (6 J + 4 doubles): for J <= 128 the start of
// the scratch when it fits there, else the 64 spare doubles behind the
// reflectors (J <= 6); for J > 128 the end of the scratch.
__host__ __device__ inline double* eig_handoff(double* scratch, int J) {
    if (J > 128) return scratch + (size_t)3 * J * J;
    return 6 * J + 4 <= J * J ? scratch : scratch + (size_t)2 * J * J;
}

// Bounds and scale of T (all threads of the workgroup): red[32..35] receive
// the widened Gershgorin interval of the scaled T, the scale (a power of two
// that brings |entries| to at most 1) and the norm bound; ts the scaled T as
// sturm_count reads it.  The interval is a minimum and a maximum, so the
// split over threads changes no bit.
__device__ __forceinline__ void scale_t(const double* d, const double* e, int J, double* red,
                                        double2* ts) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double gl = DBL_MAX, gu = -DBL_MAX;
    for (int i = tid; i < J; i += kEigThreads) {
        const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < J ? fabs(e[i]) : 0.0);
        gl = fmin(gl, d[i] - r);
        gu = fmax(gu, d[i] + r);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        gl = fmin(gl, __shfl_xor(gl, off, 64));
        gu = fmax(gu, __shfl_xor(gu, off, 64));
    }
    if (lane == 0) {
        red[wave] = gl;
        red[kEigWaves + wave] = gu;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kEigWaves; ++w) {
            gl = fmin(gl, red[w]);
            gu = fmax(gu, red[kEigWaves + w]);
        }
        const double tnorm = fmax(fabs(gl), fabs(gu));
        // scale T by a power of two so that |entries| <= 1 (exact)
        int ex = 0;
        frexp(tnorm > 0.0 ? tnorm : 1.0, &ex);
        const double sc = ldexp(1.0, -ex);
        // widen slightly so that count(gl) = 0 and count(gu) = J hold exactly
        red[32] = (gl - 2.0 * DBL_EPSILON * tnorm * J) * sc - 0x1p-900;
        red[33] = (gu + 2.0 * DBL_EPSILON * tnorm * J) * sc + 0x1p-900;
        red[34] = sc;
        red[35] = tnorm;
    }
    __syncthreads();
    const double sc = red[34];
    for (int i = tid; i < J; i += kEigThreads) {
        const double es = i > 0 ? e[i - 1] * sc : 0.0;
        ts[i] = double2{d[i] * sc, i > 0 ? fmax(es * es, kMinE2) : 0.0};
    }
    __syncthreads();
}

// T, beta and the bounds to the hand-off area of a split solve.
__device__ __forceinline__ void write_handoff(double* ho, int J, const double* d, const double* e,
                                              const double* beta, const double2* ts,
                                              const double* red) {
    const int tid = threadIdx.x;
    for (int i = tid; i < J; i += kEigThreads) {
        ho[i] = d[i];
        ho[J + i] = e[i];
        ho[2 * J + i] = beta[i];
        ho[3 * J + 2 * i] = ts[i].x;
        ho[3 * J + 2 * i + 1] = ts[i].y;
    }
    if (tid < 4) ho[5 * J + tid] = red[32 + tid];  // gl, gu, sc, tnorm
}

// ---------------------------------------------- reduction of extents > 128
//
// The first J - 192 columns of a matrix too large for one workgroup's
// registers.  One workgroup streaming A22 from L2 took 12 us per column at
// J = 256 (one CU's load path and three barriers); here kGridWaves single-wave
// workgroups hold all of A in registers for the whole reduction (wave w owns
// rows w + 64 q, lane t of it the columns t + 64 s), so a column costs one
// exchange between them and no barrier: about 3 us, most of it the trip of a
// value from one XCD to another.  Whole reductions, with these columns and the
// last 192 in one workgroup: J = 187 0.80 -> 0.25 ms, J = 250 1.72 -> 0.48,
// J = 301 3.69 -> 0.68.  All waves on one XCD was slower (J - 128 columns of
// J = 301: 0.85 against 0.64 ms).  In column k
//   - every wave holds the pivot row k and forms the reflector (v, tau) from
//     it redundantly, with the same bits;
//   - it publishes p_i = tau (A v)_i for its rows i > k, and the owner of row
//     k + 1 that row, both as of before this column's update;
//   - it reads all of p and the row back, forms w = p - (tau / 2)(p.v) v, the
//     next pivot row, and updates its own rows, A -= v w^T + w v^T.
// Every (column, entry) has a slot of its own in the scratch, filled with
// kNotYet beforehand, so a value carries its own arrival: no flags, no order
// between stores, and 64-bit relaxed agent-scope atomics are all it needs.
// A result equal to the fill pattern (a NaN payload) is published as the
// default NaN.  The 64 waves wait for one another, so all have to be
// resident.  They take at most half a SIMD's registers and no LDS, 2048 of
// them fit the GPU, and a queue has at most one partly dispatched kernel; but
// work of other streams or processes can keep some from starting for as long
// as it runs, and a stream's CU mask for good.  So a wave that has found
// something missing kGridPolls times in all sets flag bit 4 and waits no more,
// the others follow, and the workgroup that takes over the last 192 rows first
// does these columns itself (reduce_alone): the same operations in the same
// order, so the same bits.  A poll takes 0.17 us, the limit 11 ms; the columns
// by one workgroup take 1.4 ms at J = 250, 3.2 at J = 301, 17 at J = 512.
constexpr int kGridWaves = 64;
constexpr int kMidRows = 192;   // rows left to one workgroup,
constexpr int kGridTail = 128;  // of them those left to the register reduction
constexpr unsigned long long kNotYet = 0xFFF7A5C39B1E64D2ull;
constexpr int kGridPolls = 1 << 16;
constexpr int kGaveUp = 16;  // flag bit 4

__device__ __forceinline__ void slot_put(double* p, double v) {
    unsigned long long b = (unsigned long long)__double_as_longlong(v);
    if (b == kNotYet) b = 0x7FF8000000000000ull;
    __hip_atomic_store((unsigned long long*)p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long slot_get(const double* p) {
    return __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(256) void eig_slots_fill(unsigned long long* __restrict__ a,
                                                      unsigned long long* __restrict__ b,
                                                      int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) a[i] = b[i] = kNotYet;
}

// Entry g of a vector spread over the lanes (x[s] of lane t is entry
// t + 64 s); g is uniform.
template <int NS>
__device__ __forceinline__ double grid_entry(const double (&x)[NS], int g) {
    const int l = g & 63, s = g >> 6;
    double r = read_lane(x[0], l);
#pragma unroll
    for (int q = 1; q < NS; ++q) {
        const double t = read_lane(x[q], l);
        r = s == q ? t : r;
    }
    return r;
}

// Reflector of x = (x_0, rest) with |rest|^2 = sigma: alpha = -sign(x_0) |x|,
// v = (1, rest inv_v0), tau; the identity (tau = 0) for sigma = 0.
__device__ __forceinline__ void grid_reflector(double x0, double sigma, double& tau,
                                               double& alpha, double& inv_v0) {
    tau = 0.0;
    alpha = x0;
    inv_v0 = 0.0;
    if (sigma != 0.0) {
        const double ss = fma(x0, x0, sigma);
        const double rs = rsq(ss);
        const double mu = ss * rs;
        const double sgn = x0 < 0.0 ? -1.0 : 1.0;
        alpha = -sgn * mu;
        tau = fma(fabs(x0), rs, 1.0);
        inv_v0 = sgn * recip(fabs(x0) + mu);
    }
}

// NS = ceil(J / 64) slots per lane; rows and columns at or past J are zero.
template <int NS>
__global__ __launch_bounds__(64) void eig_reduce_grid(const double* __restrict__ S, int J,
                                                      double* __restrict__ scratch,
                                                      int* flags, int polls) {
    const int lane = threadIdx.x;
    const int w = blockIdx.x;
    double* P = scratch;                        // [J - 192][J] products
    double* H = scratch + (size_t)J * J;        // reflectors
    double* Rw = scratch + (size_t)2 * J * J;   // [J - 192][J] pivot rows
    double* ho = eig_handoff(scratch, J);
    const int kend = J - kMidRows;
    double a[NS][NS];  // a[q][s]: row w + 64 q, column lane + 64 s
    double r[NS];      // pivot row, 0 before column k
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int i = w + 64 * q, j = lane + 64 * s;
            a[q][s] = (i < J && j < J) ? S[(size_t)i * J + j] : 0.0;
        }
#pragma unroll
    for (int s = 0; s < NS; ++s) r[s] = lane + 64 * s < J ? S[lane + 64 * s] : 0.0;
    if (w == 0 && lane == 0) ho[0] = r[0];  // d_0

    for (int k = 0; k < kend; ++k) {
        // the owner of row k + 1 publishes it first: it is ready
        if (w == ((k + 1) & 63)) {
#pragma unroll
            for (int q = 0; q < NS; ++q)
                if (q == ((k + 1) >> 6)) {
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        const int j = lane + 64 * s;
                        if (j > k && j < J) slot_put(Rw + (size_t)k * J + j, a[q][s]);
                    }
                }
        }
        // reflector of the pivot row's part beyond the diagonal, in the form
        // of LAPACK's dlarfg (as in the register reduction)
        const double x0 = grid_entry<NS>(r, k + 1);
        double sq = 0.0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const double m = lane + 64 * s >= k + 2 ? r[s] : 0.0;
            sq = fma(m, m, sq);
        }
        double tau, alpha, inv_v0;
        grid_reflector(x0, wave_sum(sq), tau, alpha, inv_v0);
        double v[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int j = lane + 64 * s;
            v[s] = j >= k + 2 ? r[s] * inv_v0 : (j == k + 1 ? 1.0 : 0.0);
        }
        // p of the own rows; lane q ends with row w + 64 q's
        double mine = 0.0;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            if (w + 64 * q > k) {  // uniform
                double t = 0.0;
#pragma unroll
                for (int s = 0; s < NS; ++s) t = fma(a[q][s], v[s], t);
                t = tau * wave_sum(t);
                mine = lane == q ? t : mine;
            }
        }
        if (lane < NS) {
            const int i = w + 64 * lane;
            if (i > k && i < J) slot_put(P + (size_t)k * J + i, mine);
        }
        if (w == (k & 63)) {  // one wave, another each column, keeps what is found
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int j = lane + 64 * s;
                if (j > k && j < J) H[(size_t)k * J + (j - k - 1)] = v[s];
            }
            if (lane == 0) {
                ho[J + k] = alpha;
                ho[2 * J + k] = tau;
            }
        }
        // everyone's p, and row k + 1
        double p[NS], rn[NS];
        for (;;) {
            bool wait = false;
            unsigned long long bp[NS], br[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int j = lane + 64 * s;
                const bool need = j > k && j < J;
                bp[s] = need ? slot_get(P + (size_t)k * J + j) : 0ull;
                br[s] = need ? slot_get(Rw + (size_t)k * J + j) : 0ull;
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                wait = wait || bp[s] == kNotYet || br[s] == kNotYet;
                p[s] = __longlong_as_double((long long)bp[s]);
                rn[s] = __longlong_as_double((long long)br[s]);
            }
            if (!__any(wait)) break;
            // another wave has given up (looked at now and then), or this one does:
            // what is missing is a NaN (kNotYet), and what follows is not used
            if ((--polls & 63) == 0 &&
                (uni(__hip_atomic_load(flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) & kGaveUp))
                polls = 0;
            if (polls <= 0) {
                polls = 0;
                if (lane == 0) atomicOr(flags, kGaveUp);
                break;
            }
        }
        double pv = 0.0;
#pragma unroll
        for (int s = 0; s < NS; ++s) pv = fma(p[s], v[s], pv);
        const double half = 0.5 * tau * wave_sum(pv);
        double ww[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) ww[s] = fma(-half, v[s], p[s]);
        const double w1 = grid_entry<NS>(ww, k + 1);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            // as a row of A is updated, with v_{k+1} = 1
            const double x = fma(-w1, v[s], rn[s] - ww[s]);
            r[s] = lane + 64 * s > k ? x : 0.0;
            if (w == 0 && lane + 64 * s == k + 1) ho[k + 1] = x;  // d_{k+1}
        }
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            if (w + 64 * q > k) {  // uniform
                const double vi = read_lane(v[q], w), wi = read_lane(ww[q], w);
#pragma unroll
                for (int s = 0; s < NS; ++s) a[q][s] = fma(-wi, v[s], fma(-vi, ww[s], a[q][s]));
            }
        }
    }
    // the trailing 192 x 192 block, in the room of the reflectors still to come
    double* T = H + (size_t)kend * J;
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        const int i = w + 64 * q - kend;
        if (i >= 0 && i < kMidRows) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int j = lane + 64 * s - kend;
                if (j >= 0 && j < kMidRows) T[(size_t)i * kMidRows + j] = a[q][s];
            }
        }
    }
}

// What eig_reduce_grid does, by one workgroup, with A in the scratch (where the
// products' slots were).  Every wave sum has the lanes, and every element the
// operations, of there.  lds: 3 TK_MAX_MODE_DIM doubles.
__device__ __forceinline__ void reduce_alone(const double* __restrict__ S, int J, double* scratch,
                                             double* lds) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double* A = scratch;
    double* H = scratch + (size_t)J * J;
    double* ho = eig_handoff(scratch, J);
    double* rs = lds;                        // pivot row, 0 before column k
    double* vs = lds + TK_MAX_MODE_DIM;      // v
    double* ps = lds + 2 * TK_MAX_MODE_DIM;  // p
    const int kend = J - kMidRows;
    for (int i = tid; i < J * J; i += kEigThreads) A[i] = S[i];
    for (int j = tid; j < J; j += kEigThreads) rs[j] = S[j];
    if (tid == 0) ho[0] = S[0];
    __syncthreads();
    for (int k = 0; k < kend; ++k) {
        const int s0 = (k + 1) & ~63;  // columns before it see v = w = 0
        double sq = 0.0;
        for (int j = s0 + lane; j < J; j += 64) {
            const double m = j >= k + 2 ? rs[j] : 0.0;
            sq = fma(m, m, sq);
        }
        double tau, alpha, inv_v0;
        grid_reflector(rs[k + 1], wave_sum(sq), tau, alpha, inv_v0);
        if (wave == 0) {
            for (int j = s0 + lane; j < J; j += 64) {
                const double v = j >= k + 2 ? rs[j] * inv_v0 : (j == k + 1 ? 1.0 : 0.0);
                vs[j] = v;
                if (j > k) H[(size_t)k * J + (j - k - 1)] = v;
                if (j <= k) ps[j] = 0.0;
            }
            if (lane == 0) {
                ho[J + k] = alpha;
                ho[2 * J + k] = tau;
            }
        }
        __syncthreads();
        for (int i = wave; i < J; i += kEigWaves) {
            if (i <= k) continue;  // uniform
            double t = 0.0;
            for (int j = s0 + lane; j < J; j += 64) t = fma(A[(size_t)i * J + j], vs[j], t);
            t = tau * wave_sum(t);
            if (lane == 0) ps[i] = t;
        }
        __syncthreads();
        double pv = 0.0;
        for (int j = s0 + lane; j < J; j += 64) pv = fma(ps[j], vs[j], pv);
        const double half = 0.5 * tau * wave_sum(pv);
        const double w1 = fma(-half, vs[k + 1], ps[k + 1]);
        for (int i = wave; i < J; i += kEigWaves) {
            if (i <= k) continue;  // uniform
            const double vi = vs[i], wi = fma(-half, vi, ps[i]);
            for (int j = s0 + lane; j < J; j += 64) {
                const double a = A[(size_t)i * J + j], v = vs[j], w = fma(-half, v, ps[j]);
                if (i == k + 1) {  // the next pivot row, from the row as it was
                    const double x = fma(-w1, v, a - w);
                    rs[j] = j > k ? x : 0.0;
                    if (j == k + 1) ho[k + 1] = x;
                }
                A[(size_t)i * J + j] = fma(-wi, v, fma(-vi, w, a));
            }
        }
        __syncthreads();
    }
    double* T = H + (size_t)kend * J;
    for (int i = kend + wave; i < J; i += kEigWaves)
        for (int j = kend + lane; j < J; j += 64)
            T[(size_t)(i - kend) * kMidRows + (j - kend)] = A[(size_t)i * J + j];
}

// The columns that bring a symmetric block of n = 129 .. 192 rows to 128, in
// one workgroup's registers; element (i, j) is src[i ld + j].  Thread t owns
// the rows t / 16 + 64 h, h < 3, of the block set at the lower end of 192
// positions, and of them the columns t % 16 + 16 q: the rows that finish here
// are those of h = 0, and the 128 that remain need no test.  Columns run as in
// the register reduction of at most 128 rows (tridiag_regs), two exchanges
// through LDS each; its store for the reflectors has room for these 64
// columns, not for all of 192.  What bounds a column is the same chain and
// the rows' reads of v and p from LDS: 2.0 us each at 192 rows, where one
// exchange between workgroups on different XCDs takes 3.2.  Whole reductions,
// with these 64 columns in place of the grid's: J = 187 295 -> 245 us,
// J = 250 540 -> 475, J = 301 755 -> 680.
constexpr int kMidLds = (64 * kMidRows + 2 * kMidRows + 3 * 64 + 2) * (int)sizeof(double);

// S, flags: eig_reduce_grid's, where it ran before; NULL elsewhere.
__global__ __launch_bounds__(kEigThreads) void eig_reduce_mid(const double* src, int ld, int n,
                                                              int J, double* scratch,
                                                              const double* S, int* flags) {
    extern __shared__ double smem[];
    if (flags && (*flags & kGaveUp)) {  // uniform
        reduce_alone(S, J, scratch, smem);
        __syncthreads();
        if (threadIdx.x == 0) *flags &= ~kGaveUp;
    }
    constexpr int NQ = kMidRows / 16;
    double* Hs = smem;                      // reflector k at row k, zero up to k
    double* pb = smem + 64 * kMidRows;      // p, two buffers
    double* dv = pb + 2 * kMidRows;         // d, e, beta
    double* sgb = dv + 3 * 64;              // tau, two buffers
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = tid >> 4, rc = tid & 15;
    const int off = kMidRows - n;           // position of the block's first row
    const int koff = J - n;
    double av[3][NQ];
#pragma unroll
    for (int h = 0; h < 3; ++h)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int i = g + 64 * h - off, j = rc + 16 * q - off;
            av[h][q] = i >= 0 && j >= 0 ? src[(size_t)i * ld + j] : 0.0;
        }
    for (int i = tid; i < 64 * kMidRows; i += kEigThreads) Hs[i] = 0.0;
    __syncthreads();
    static_for<0, 4>([&](auto kbc) {
        constexpr int KB = decltype(kbc)::value;  // chunks below KB are finished
        for (int k = max(16 * KB, off); k < 16 * KB + 16; ++k) {
            double* vs = Hs + k * kMidRows;
            double* ps = pb + (k & 1) * kMidRows;
            double* sg = sgb + (k & 1);
            int g_k = g;  // as in tridiag_regs: k stays uniform inside the branch
            asm volatile("" : "+v"(g_k));
            if (g_k == k) {
                double sq[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int q = KB; q < NQ; ++q) {
                    const double m = (q > KB + 1 || rc + 16 * q >= k + 2) ? av[0][q] : 0.0;
                    sq[q & 3] = fma(m, m, sq[q & 3]);
                }
                const double sigma = row16_sum((sq[0] + sq[1]) + (sq[2] + sq[3]));
                const int l0 = 16 * (k & 3);
                const double akk = read_lane(av[0][KB], l0 + (k & 15));
                const double x0 = read_lane(((k + 1) >> 4) == KB ? av[0][KB] : av[0][KB + 1],
                                            l0 + ((k + 1) & 15));
                double tau = 0.0, alpha = x0, inv_v0 = 0.0;
                if (sigma != 0.0) {
                    const double ss = fma(x0, x0, sigma);
                    const double r = rsq(ss);  // 1 / |x|
                    const double mu = ss * r;
                    const double sgn = x0 < 0.0 ? -1.0 : 1.0;
                    alpha = -sgn * mu;
                    tau = fma(fabs(x0), r, 1.0);
                    inv_v0 = sgn * recip(fabs(x0) + mu);
                }
#pragma unroll
                for (int q = KB; q < NQ; ++q) {
                    const int j = rc + 16 * q;
                    const double vj = av[0][q] * inv_v0;
                    vs[j] = q > KB + 1 ? vj : (j == k + 1 ? 1.0 : (j > k + 1 ? vj : 0.0));
                }
                if (rc == 0) {
                    *sg = tau;
                    dv[k] = akk;
                    dv[64 + k] = alpha;
                    dv[128 + k] = tau;
                }
            }
            __syncthreads();
            const double tau = *sg;
            const bool top = 4 * wave + 3 > k;  // uniform: a row of h = 0 is left
            double vq[NQ], s0 = 0.0, s1[2] = {0.0, 0.0}, s2[2] = {0.0, 0.0};
#pragma unroll
            for (int q = KB; q < NQ; ++q) {
                vq[q] = vs[rc + 16 * q];
                s1[q & 1] = fma(av[1][q], vq[q], s1[q & 1]);
                s2[q & 1] = fma(av[2][q], vq[q], s2[q & 1]);
            }
            if (top) {
                double t[2] = {0.0, 0.0};
#pragma unroll
                for (int q = KB; q < NQ; ++q) t[q & 1] = fma(av[0][q], vq[q], t[q & 1]);
                s0 = row16_sum(t[0] + t[1]);
            }
            // the sum of row 64 + g to lanes 0-7, of row 128 + g to 8-15
            const double a1 = s1[0] + s1[1], a2 = s2[0] + s2[1];
            const bool hi = rc >= 8;
            const double part = row8_sum((hi ? a2 : a1) + dpp_move<0x140, 0xf, false>(hi ? a1 : a2));
            if (tau == 0.0) continue;  // uniform: the reflector is the identity
            if ((rc & 7) == 0) ps[g + 64 + 64 * (rc >> 3)] = tau * part;
            if (rc == 0) ps[g] = g > k ? tau * s0 : 0.0;
            __syncthreads();
            double pv = 0.0;
#pragma unroll
            for (int h = 0; h < 3; ++h) pv = fma(ps[lane + 64 * h], vs[lane + 64 * h], pv);
            const double half = 0.5 * tau * wave_sum(pv);
            double vi[3], wi[3];
#pragma unroll
            for (int h = 0; h < 3; ++h) {
                vi[h] = vs[g + 64 * h];
                wi[h] = fma(-half, vi[h], ps[g + 64 * h]);
            }
#pragma unroll
            for (int q = KB; q < NQ; ++q) {
                const double wj = fma(-half, vq[q], ps[rc + 16 * q]);
                if (top) av[0][q] = fma(-wi[0], vq[q], fma(-vi[0], wj, av[0][q]));
                av[1][q] = fma(-wi[1], vq[q], fma(-vi[1], wj, av[1][q]));
                av[2][q] = fma(-wi[2], vq[q], fma(-vi[2], wj, av[2][q]));
            }
        }
    });
    __syncthreads();
    double* H = scratch + (size_t)J * J;
    double* ho = eig_handoff(scratch, J);
    for (int k = off + wave; k < 64; k += kEigWaves)
        for (int i = lane; i < kMidRows - k - 1; i += 64)
            H[(size_t)(koff + k - off) * J + i] = Hs[k * kMidRows + k + 1 + i];
    if (tid >= off && tid < 64) {
        const int k = koff + tid - off;
        ho[k] = dv[tid];
        ho[J + k] = dv[64 + tid];
        ho[2 * J + k] = dv[128 + tid];
    }
    // the trailing 128 x 128 block, in the room of the reflectors still to come
    double* T = H + (size_t)(J - kGridTail) * J;
#pragma unroll
    for (int h = 1; h < 3; ++h)
#pragma unroll
        for (int q = 4; q < NQ; ++q)
            T[(size_t)(g + 64 * (h - 1)) * kGridTail + rc + 16 * (q - 4)] = av[h][q];
}

// Extents above 128: the register reduction of the trailing block, then the
// scaling of T; d, e and beta of the first J - 128 columns come from the
// hand-off, where T goes as for PH = 1 of the solver.
// LDS: the block's reflectors, five vectors, the reduction's small areas.
constexpr int kTailRegion = (kGridTail - 2) * kGridTail;
static size_t eig_tail_lds_bytes(int J) {
    return ((size_t)kTailRegion + 5 * J + 64 + 8 + 4 * kGridTail) * sizeof(double);
}

__global__ __launch_bounds__(kEigThreads) void eig_reduce_tail(double* __restrict__ scratch,
                                                               int J) {
    extern __shared__ double smem[];
    double* reg = smem;
    double2* ts = reinterpret_cast<double2*>(smem + kTailRegion);
    double* d = smem + kTailRegion + 2 * J;
    double* e = d + J;
    double* beta = e + J;
    double* red = beta + J;  // 64, then 8, then the vector buffers
    double* H = scratch + (size_t)J * J;
    double* ho = eig_handoff(scratch, J);
    const int kend = J - kGridTail;
    for (int i = threadIdx.x; i < kend; i += kEigThreads) {
        d[i] = ho[i];
        e[i] = ho[J + i];
        beta[i] = ho[2 * J + i];
    }
    tridiag_regs<kGridTail>(H + (size_t)kend * J, kGridTail, kGridTail, kend, J, reg, red, d, e,
                            beta, H);
    scale_t(d, e, J, red, ts);
    write_handoff(ho, J, d, e, beta, ts, red);
}

// Writes a vector held by 16 lanes (element t = 32 p + 2 l16 + h) to column j
// of X, its largest |entry| (lowest index on ties) made positive.
template <int NP>
__device__ __forceinline__ void signed_store(double* __restrict__ X, int J, int j, bool jok,
                                             int l16, const double2 (&xr)[NP]) {
                double bv = -1.0;
                int bi = J;
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const int t = 32 * p + 2 * l16;
                    if (t < J && fabs(xr[p].x) > bv) {
                        bv = fabs(xr[p].x);
                        bi = t;
                    }
                    if (t + 1 < J && fabs(xr[p].y) > bv) {
                        bv = fabs(xr[p].y);
                        bi = t + 1;
                    }
                }
#pragma unroll
                for (int off = 8; off > 0; off >>= 1) {  // within the 16-lane group
                    const double ov = __shfl_xor(bv, off, 64);
                    const int oi = __shfl_xor(bi, off, 64);
                    if (ov > bv || (ov == bv && oi < bi)) {
                        bv = ov;
                        bi = oi;
                    }
                }
                double at = 0.0;
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const int t = 32 * p + 2 * l16;
                    if (t == bi) at = xr[p].x;
                    if (t + 1 == bi) at = xr[p].y;
                }
                const double sgn = row16_sum(at) < 0.0 ? -1.0 : 1.0;
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const int t = 32 * p + 2 * l16;
                    if (jok && t < J) X[(size_t)j * J + t] = sgn * xr[p].x;
                    if (jok && t + 1 < J) X[(size_t)j * J + t + 1] = sgn * xr[p].y;
                }
}

// JP = 32, 64, 96, 128: A lives in registers during the tridiagonalisation
// (J <= JP); JP = 0: J > 128, PH = 3 only (launch_eig_reduce does the rest).
// PH = 0: the whole solver in one launch.  PH = 1: steps 1 and the scaling of
// T, then T, beta and the bounds go to the hand-off area (eig_handoff) and the
// launch ends; eig_multisect then finds the eigenvalues with one workgroup each
// and PH = 3 picks everything up for steps 3 to 5.
// MULTI (PH = 3): one workgroup per batch of vectors.  Each repeats the rank
// rule (the first one writes its results) and runs the inverse iteration of
// its own batch.  With J <= 128 and a rank of one batch the first workgroup
// goes on to the end; otherwise the vectors of T are left in u for
// eig_gs_* and eig_back.
template <int JP, int PH, bool MULTI>
__device__ __forceinline__ void eig_body(const EigArgs& a, int region) {
    extern __shared__ double smem[];
    const int J = a.J;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool lead = !MULTI || blockIdx.x == 0;  // uniform: writes the rank rule's results
    double* reg = smem;                        // A (J <= 128) then the LU batch
    double* sv = smem + region;  // region is even
    double2* ts = reinterpret_cast<double2*>(sv);  // J: the scaled T (step 2)
    double* d = sv + 2 * J;      // J
    double* e = d + J;           // J
    double* beta = e + J;        // J
    double* vals = beta + J;     // J: the rank rule's terms
    double* lam = vals + J;      // J (descending)
    double* shift = lam + J;     // J
    double* red = shift + J;     // 64
    int* misc = (int*)(red + 64);  // [0] = R
    double* H = a.scratch + (size_t)J * J;    // reflector k at H[k * J], length J - k - 1
    double* X = a.u;                          // column-major J x R
    double* ho = eig_handoff(a.scratch, J);   // hand-off between split launches
    double sc, tnorm;
    // the rank rule's global inputs, loaded now so that their latency
    // overlaps the earlier phases
    double nu_in = 0.0, stat_d2 = 0.0, stat_e = 0.0;
    if constexpr (PH != 1) {
        if (tid == 0) {
            if (a.fixed_rank <= 0) nu_in = *a.nu;
            if (a.guard > 0.0 && a.split_stats) {
                stat_d2 = a.split_stats[0];
                stat_e = a.split_stats[1];
            }
        }
    }

    if constexpr (PH != 3) {
    // ---- 1. Householder tridiagonalisation, A in registers ---------------
    tridiag_regs<JP>(a.s, J, J, 0, J, reg, red, d, e, beta, H);
    scale_t(d, e, J, red, ts);
    sc = red[34];
    tnorm = red[35];
    if constexpr (PH == 1) {
        write_handoff(ho, J, d, e, beta, ts, red);
        return;
    }

    // ---- 2. eigenvalues by multisection ---------------------------------
    {
        const double gl = red[32], gu = red[33];
        int jp = 32;
        while (jp < J) jp *= 2;
        // about 512 active lanes (two waves per SIMD): more sample points per
        // eigenvalue add work faster than they remove iterations
        const int tpe = jp >= 512 ? 1 : 512 / jp;  // threads (sample points) per eigenvalue
        const int k = tid / tpe, s = tid - (tid / tpe) * tpe;
        const int gofs = (lane / tpe) * tpe;
        const uint64_t gmask = (((1ull << tpe) - 1ull) << gofs);
        (void)wave;
        double lo = gl, hi = gu;
        if (k < J) {
            for (int it = 0; it < 160; ++it) {
                const double tol = fmax(kSectTol, kSectTol * fmax(fabs(lo), fabs(hi)));
                if (hi - lo <= tol) break;
                const double h = (hi - lo) / (double)(tpe + 1);
                const int c = sturm_count(LdsRows{ts}, ts[0].x, J, lo + h * (double)(s + 1));
                const uint64_t bal = __ballot(c > k) & gmask;
                const int sstar = bal ? (__ffsll((long long)bal) - gofs) : tpe + 1;  // 1-based point
                const double nlo = sstar == 1 ? lo : lo + h * (double)(sstar - 1);
                const double nhi = sstar == tpe + 1 ? hi : lo + h * (double)sstar;
                lo = nlo;
                hi = nhi;
            }
            if (s == 0) lam[J - 1 - k] = 0.5 * (lo + hi) / sc;
        }
    }
    __syncthreads();
    } else {
        for (int i = tid; i < J; i += kEigThreads) {
            d[i] = ho[i];
            e[i] = ho[J + i];
            beta[i] = ho[2 * J + i];
            lam[i] = ho[5 * J + 4 + i];
        }
        sc = ho[5 * J + 2];
        tnorm = ho[5 * J + 3];
        __syncthreads();
    }
    (void)sc;
    // Jordan-Wielandt input: the leading half of the spectrum is sigma(R)
    const int Jv = a.aug ? J / 2 : J;
    // Tail sums: negative rounding eigenvalues count as 0 -- except for a
    // split Gram, whose subtracted quantization energy leaves small negative
    // eigenvalues in noise-level directions; there the raw sum is the
    // estimate of the exact tail (clamping would raise it).
    const bool raw = a.guard > 0.0 && a.split_stats != nullptr && !a.aug;
    auto val = [&](int r) {
        const double l = raw ? lam[r] : fmax(lam[r], 0.0);
        return a.aug ? l * l : l;
    };
    // the values of the tail sums, formed in parallel
    for (int i = tid; i < Jv; i += kEigThreads) {
        const double v = val(i);
        vals[i] = v;
        if (lead) a.lambda[i] = a.aug ? v : lam[i];
    }
    __syncthreads();

    // ---- 3. rank rule ---------------------------------------------------
    if (tid == 0) {
        int R;
        double tail = 0.0;
        const bool eps_rule = a.fixed_rank <= 0;
        const double tau = eps_rule ? a.eps2_over_n * nu_in : 0.0;
        if (!eps_rule) {
            R = a.fixed_rank < Jv ? a.fixed_rank : Jv;
            for (int r = Jv - 1; r >= R; --r) tail += vals[r];
        } else {
            // R = Jv; while (R > 1 && tail + val(R - 1) <= tau) tail += val(--R),
            // with the values loaded eight at a time ahead of the running sum
            R = Jv;
            bool more = true;
            double vb[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) vb[u] = vals[max(R - 1 - u, 0)];  // unused past r = 1
            while (more) {
                double nb8[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) nb8[u] = vals[max(R - 9 - u, 0)];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const double t = tail + vb[u];
                    more = more && R > 1 && t <= tau;
                    tail = more ? t : tail;
                    R -= more ? 1 : 0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) vb[u] = nb8[u];
            }
        }
        double bound = 0.0;
        if (a.guard > 0.0 && a.split_stats) {
            // The cut must survive the split representation's error in the
            // tail sums (EigArgs::guard): a model standard deviation at each
            // side, sqrt(4 delta^2 t + 2 K delta^4 (J - r)) for the tail t
            // beyond rank r.  R = J discards nothing and is exact.
            const double d2 = stat_d2;
            const double dl2 = ldexp(1.0, 2 * ((int)stat_e - 16)) / 3.0;
            auto margin = [&](double t, int r) {
                return a.guard * sqrt(4.0 * dl2 * t + 2.0 * a.ncols * dl2 * dl2 * (double)(Jv - r)) +
                       kSplitModelError * d2;
            };
            const double next = tail + val(R - 1);
            bound = R == Jv ? 0.0 : margin(fmax(tail, 0.0), R);
            if (eps_rule) {
                const bool below = tau - tail >= bound;
                const bool above = R == 1 || next - tau >= margin(fmax(next, 0.0), R - 1);
                if (lead && !(below && above)) a.flags[0] |= 4;
            }
        }
        if (lead && a.tail_bound) *a.tail_bound = bound;
        int flag = 0;
        if (R > a.max_rank) {
            flag |= 2;
            R = a.max_rank;
        }
        if (lead) {  // single writer: thread 0 of one workgroup
            *a.rank_out = R;
            *a.disc_out = fmax(tail, 0.0);
            if (flag) a.flags[0] |= flag;
        }
        misc[0] = R;
        // shifts for inverse iteration: separate (near-)equal eigenvalues
        const double pert = 10.0 * DBL_EPSILON * tnorm;
        double prev = 0.0;
        for (int j0 = 0; j0 < R; j0 += 8) {
            double lb[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) lb[u] = lam[min(j0 + u, R - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int j = j0 + u;
                if (j < R) {
                    double sj = lb[u];
                    if (j > 0 && prev - sj < pert) sj = prev - pert;
                    shift[j] = sj;
                    prev = sj;
                }
            }
        }
    }
    __syncthreads();
    const int R = misc[0];


    // ---- 4. inverse iteration, batches of vectors held in LDS -----------
    // Two threads, neighbouring lanes, carry a vector: they eliminate T - sg I
    // from its two ends (the rows are taken in even number: behind an odd J
    // comes one that is coupled to nothing) and meet in the middle, where one
    // row each with the two middle unknowns is left, a 2 x 2 system with
    // pivoting; both sweeps then run towards and away from there.  What bounds
    // this is the chain from row to row of one wave, about 400 cycles in the
    // factorisation and 230 per iteration; each thread walks half the rows
    // (the launch at J = 128, 16 vectors 114 -> 92 us, J = 100 66 -> 53,
    // J = 250, 100 vectors 102 -> 64).  Two sets of four rows beside the rest of
    // the kernel exceed the 128 registers of a 1024-thread workgroup: PH = 3
    // with J <= 128 keeps 68 bytes per lane in scratch memory, PH = 0 spills 5
    // registers (24 bytes); JP = 0 and the batched kernels have no scratch.
    // Each thread works on a record of its own in
    // LDS: row i holds (x, reciprocal pivot, u1, u2, multiplier, pivot flag)
    // at rec[kLuArrays i ..], so every access is the thread's base plus an
    // immediate offset; the record's last double is x of row Jb (zero), and
    // records are an odd number of doubles apart, which keeps the lanes of a
    // wave in distinct banks.  Loads are never conditional (a guarded load
    // waits for its value inside the guard).  Operands are read a block
    // of kSweepRows rows ahead of the recurrence (a load that follows a store
    // to the same record waits for it), and rows are padded to whole blocks
    // with exact zeros, which every sweep maps to zeros.  A sweep's
    // normalisation is applied when the next sweep (or the copy-out) reads
    // its result, with the same two roundings as an in-place pass.
    const double tiny = DBL_EPSILON * tnorm + DBL_MIN;
    const int Jb = eig_sweep_rows(J);
    const int half = (J + 1) / 2;  // rows of either thread, counted from its end
    const int recd = eig_record_doubles(J);
    const int batch = (int)((size_t)region / ((size_t)2 * recd + 2));
    constexpr int oX = 0, oRP = 1, oU1 = 2, oU2 = 3, oLM = 4, oPV = 5;
    const int jfirst = MULTI ? (int)blockIdx.x * batch : 0;
    const int jlast = MULTI ? min(R, jfirst + batch) : R;
    if (MULTI && jfirst >= R) return;  // uniform over the workgroup
    for (int j0 = jfirst; j0 < jlast; j0 += batch) {
        const int nb = min(batch, R - j0);
        double* SC1 = reg + (size_t)2 * recd * nb;  // nb: pending scale factors of x
        double* SC2 = SC1 + nb;
        __syncthreads();  // the region is free (A or the previous batch)
        // deterministic start vectors, zero in the padding rows and row Jb
        for (int idx = tid; idx < (Jb + 1) * 2 * nb; idx += kEigThreads) {
            const int rr = idx / (Jb + 1), i = idx - rr * (Jb + 1);
            const int t = rr & 1 ? 2 * half - 1 - i : i;  // row of T
            reg[(size_t)rr * recd + kLuArrays * i + oX] =
                i < half && t < J ? hash_unit((uint32_t)(j0 + (rr >> 1)), (uint32_t)t) : 0.0;
        }
        __syncthreads();
        // meanwhile the last wave hands the call's scalars to the host, which
        // waits for the rank: it can enqueue what follows while this runs
        if (lead && a.host != nullptr && j0 == jfirst && wave == kEigWaves - 1) {
            if (lane < kHostScalars)
                __hip_atomic_store(a.host + lane, a.host_scal[lane], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
            __threadfence_system();
            if (lane == 0)
                __hip_atomic_store((uint64_t*)(a.host + kHostScalars), a.host_seq,
                                   __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        if (tid < 2 * nb) {
            constexpr int IB = kSweepRows;
            constexpr int W = kLuArrays;
            const int jj = tid >> 1, j = j0 + jj;
            const bool low = tid & 1;  // from the last row up
            double* rec = reg + (size_t)tid * recd;
            // row i of this thread's half and its coupling to row i + 1
            const int st = low ? -1 : 1;
            const double* dp = low ? d + (2 * half - 1) : d;
            const double* ep = low ? e + (2 * half - 2) : e;
            auto partner = [](double v) { return dpp_move<0xb1, 0xf, false>(v); };
            // Row i0 of the record.  The offset goes through an empty asm so
            // that each block forms one address and reaches its rows by
            // immediate offsets (the compiler otherwise keeps one address per
            // row and field across the sweep loops).
            auto row = [&](int i0) {
                int o = W * i0;
                asm volatile("" : "+s"(o));
                return rec + o;
            };
            const double sg = shift[j];
            const double rtiny = recip(tiny);  // recip(-tiny) = -recip(tiny) exactly
            // LU factorisation of T - sg I with partial pivoting
            double ai = low && (J & 1) ? 1.0 : dp[low && (J & 1) ? -1 : 0] - sg;
            double bi = ep[0];  // e[J - 1] is 0
            for (int i0 = 0; i0 + 1 < half; i0 += IB) {
                double cb[IB], anb[IB], bnb[IB];
#pragma unroll
                for (int u = 0; u < IB; ++u) {
                    const int i = min(i0 + u, half - 2);
                    cb[u] = ep[st * i];
                    anb[u] = dp[st * (i + 1)] - sg;
                    bnb[u] = ep[st * (i + 1)];
                }
                double* rr = row(i0);
#pragma unroll
                for (int u = 0; u < IB; ++u) {
                    if (i0 + u + 1 < half) {  // uniform
                        // Without interchange (|a_i| >= |c_i|) the pivot is a_i,
                        // raised to +-tiny if smaller; with it the pivot is c_i
                        // (|c_i| > |a_i|), the multiplier uses c_i itself and only
                        // the stored reciprocal is that of +-tiny.  Selects, not
                        // branches: lanes of a wave take either case.
                        const double ci = cb[u], an = anb[u], bn = bnb[u];
                        const bool keep = fabs(ai) >= fabs(ci);
                        const double pa = fabs(ai) < tiny ? (ai < 0.0 ? -tiny : tiny) : ai;
                        const double rl = recip(keep ? pa : ci);
                        const double l = (keep ? ci : ai) * rl;
                        const double rp = (!keep && fabs(ci) < tiny) ? (ci < 0.0 ? -rtiny : rtiny) : rl;
                        const double u1 = keep ? bi : an;
                        const double u2 = keep ? 0.0 : bn;
                        const double pf = keep ? 0.0 : 1.0;
                        const double ain = keep ? an - l * bi : bi - l * an;
                        bi = keep ? bn : -l * bn;
                        ai = ain;
                        rr[W * u + oRP] = rp;
                        rr[W * u + oU1] = u1;
                        rr[W * u + oU2] = u2;
                        rr[W * u + oLM] = l;
                        rr[W * u + oPV] = pf;
                    }
                }
            }
            // The last row's unknown comes from the middle system; it and the
            // padding rows are all zero (their pivot reciprocal included).
            for (int i = half - 1; i < Jb; ++i) {
                rec[W * i + oRP] = 0.0;
                rec[W * i + oU1] = 0.0;
                rec[W * i + oU2] = 0.0;
                rec[W * i + oLM] = 0.0;
                rec[W * i + oPV] = 0.0;
            }
            // Middle system a1 y + b1 z = r1, b2 y + a2 z = r2 (1: the thread
            // from the first row, y its last unknown): the pivot row has p, pc,
            // the other one multiplier ml and pivot q.  Both threads form the
            // same bits.
            const double ao = partner(ai), bo = partner(bi);
            const double a1 = low ? ao : ai, b1 = low ? bo : bi;
            const double a2 = low ? ai : ao, b2 = low ? bi : bo;
            const bool swp = fabs(b2) > fabs(a1);
            auto raised = [&](double v) { return fabs(v) < tiny ? (v < 0.0 ? -tiny : tiny) : v; };
            const double pc = swp ? a2 : b1;
            const double rpm = recip(raised(swp ? b2 : a1));
            const double ml = (swp ? a1 : b2) * rpm;
            const double rqm = recip(raised(fma(-ml, pc, swp ? b1 : a2)));
            double f1 = 1.0, f2 = 1.0;  // x = (stored x f1) f2
            // Both sweeps alternate two register sets: the next block's loads
            // are issued before this block's arithmetic and stores.  Rows past
            // the half (all in the last block) carry zeros: the forward sweep
            // maps a zero row to zero, the backward one forces them.
            for (int it = 0; it < kInvIters; ++it) {
                // forward: row interchanges and multipliers, running value in xc
                double xA[IB], pA[IB], lA[IB], xB[IB], pB[IB], lB[IB];
                auto fload = [&](int i0, double (&xb)[IB], double (&pb)[IB], double (&lb)[IB]) {
                    const double* rr = row(i0);
#pragma unroll
                    for (int u = 0; u < IB; ++u) {
                        xb[u] = (rr[W * (u + 1) + oX] * f1) * f2;  // row Jb: zero
                        pb[u] = rr[W * u + oPV];
                        lb[u] = rr[W * u + oLM];
                    }
                };
                double xc = (rec[oX] * f1) * f2;
                auto fstep = [&](int i0, const double (&xb)[IB], const double (&pb)[IB],
                                 const double (&lb)[IB]) {
                    double ob[IB];
#pragma unroll
                    for (int u = 0; u < IB; ++u) {
                        double xn = xb[u];
                        if (pb[u] != 0.0) {
                            const double t = xc;
                            xc = xn;
                            xn = t;
                        }
                        ob[u] = xc;
                        xc = xn - lb[u] * xc;
                    }
                    double* rw = row(i0);
#pragma unroll
                    for (int u = 0; u < IB; ++u) rw[W * u + oX] = ob[u];
                };
                fload(0, xA, pA, lA);
                for (int i0 = 0;; i0 += 2 * IB) {
                    fload(min(i0 + IB, Jb - IB), xB, pB, lB);
                    fstep(i0, xA, pA, lA);
                    if (i0 + IB >= Jb) break;
                    fload(min(i0 + 2 * IB, Jb - IB), xA, pA, lA);
                    fstep(i0 + IB, xB, pB, lB);
                    if (i0 + 2 * IB >= Jb) break;
                }
                // backward substitution
                double u1A[IB], u2A[IB], rA[IB], u1B[IB], u2B[IB], rB[IB];
                auto bload = [&](int i0, double (&xb)[IB], double (&u1b)[IB], double (&u2b)[IB],
                                 double (&rb)[IB]) {
                    const double* rr = row(i0);
#pragma unroll
                    for (int u = 0; u < IB; ++u) {
                        xb[u] = rr[W * u + oX];
                        u1b[u] = rr[W * u + oU1];
                        u2b[u] = rr[W * u + oU2];
                        rb[u] = rr[W * u + oRP];
                    }
                };
                const double rl = rec[W * (half - 1) + oX], ro = partner(rl);
                const double r1 = low ? ro : rl, r2 = low ? rl : ro;
                const double rp1 = swp ? r2 : r1, rs1 = swp ? r1 : r2;
                const double zm = fma(-ml, rp1, rs1) * rqm;
                const double ym = fma(-pc, zm, rp1) * rpm;
                double x1 = low ? zm : ym, x2 = low ? ym : zm, amax = fabs(x1);
                auto bstep = [&](auto top, int i0, const double (&xb)[IB], const double (&u1b)[IB],
                                 const double (&u2b)[IB], const double (&rb)[IB]) {
                    double ob[IB];
#pragma unroll
                    for (int u = IB - 1; u >= 0; --u) {
                        if constexpr (decltype(top)::value) {
                            if (i0 + u >= half - 1) {  // uniform
                                ob[u] = i0 + u == half - 1 ? x1 : 0.0;
                                continue;
                            }
                        }
                        double v = xb[u];
                        v = fma(-u1b[u], x1, v);
                        v = fma(-u2b[u], x2, v);
                        v *= rb[u];
                        ob[u] = v;
                        x2 = x1;
                        x1 = v;
                        amax = fmax(amax, fabs(v));
                    }
                    double* rw = row(i0);
#pragma unroll
                    for (int u = 0; u < IB; ++u) rw[W * u + oX] = ob[u];
                };
                bload(Jb - IB, xA, u1A, u2A, rA);
                for (int i0 = Jb - IB;; i0 -= 2 * IB) {
                    bload(max(i0 - IB, 0), xB, u1B, u2B, rB);
                    if (i0 == Jb - IB)
                        bstep(std::true_type{}, i0, xA, u1A, u2A, rA);
                    else
                        bstep(std::false_type{}, i0, xA, u1A, u2A, rA);
                    if (i0 == 0) break;
                    bload(max(i0 - 2 * IB, 0), xA, u1A, u2A, rA);
                    bstep(std::false_type{}, i0 - IB, xB, u1B, u2B, rB);
                    if (i0 == IB) break;
                }
                amax = fmax(amax, partner(amax));
                double nrm2 = 0.0;
                const double scl = amax > 0.0 ? 1.0 / amax : 1.0;
#pragma unroll 8
                for (int i = 0; i < half; ++i) {
                    const double v = rec[W * i + oX] * scl;
                    nrm2 += v * v;
                }
                nrm2 += partner(nrm2);
                f1 = scl;
                f2 = nrm2 > 0.0 ? 1.0 / sqrt(nrm2) : 0.0;
            }
            if (!low) {
                SC1[jj] = f1;
                SC2[jj] = f2;
            }
        }
        __syncthreads();
        for (int idx = tid; idx < J * nb; idx += kEigThreads) {
            const int jj = idx / J, i = idx - jj * J;
            const bool low = i >= half;
            const double* x = reg + (size_t)(2 * jj + low) * recd + oX;
            X[(size_t)(j0 + jj) * J + i] =
                (x[kLuArrays * (low ? 2 * half - 1 - i : i)] * SC1[jj]) * SC2[jj];
        }
    }
    if constexpr (MULTI)
        if (JP == 0 || R > batch) return;  // eig_gs_* and eig_back go on
    if constexpr (JP > 0) {
    __syncthreads();

    // Modified Gram-Schmidt, twice, inside clusters (descending order), by
    // wave 0 with the working vector in registers and the others in LDS;
    // cluster starts are found in one pass over the eigenvalues.
    const int nslot = (J + 63) / 64;
    constexpr int kGsSlots = (JP + 63) / 64;  // per-lane slots of a vector
    const double ortol = 1e-3 * tnorm;
    const bool clustered =
        __syncthreads_or(tid >= 1 && tid < R && lam[tid - 1] - lam[tid] <= ortol);
    if (clustered) {
        // vector j at XL[j J ..]: a copy in LDS when the region holds all R
        const bool in_lds = (size_t)R * J <= (size_t)region;
        double* XL = in_lds ? reg : X;
        if (in_lds)
            for (int idx = tid; idx < R * J; idx += kEigThreads) XL[idx] = X[idx];
        __syncthreads();
        if (wave == 0) {
            int c0 = 0;
            for (int j = 1; j < R; ++j) {
                c0 = lam[j - 1] - lam[j] <= ortol ? c0 : j;
                if (c0 == j) continue;
                // slot q holds element lane + 64 q (zero past J; the load
                // itself is clamped to the vector)
                auto ld = [&](int v, int q) {
                    const int t = lane + 64 * q;
                    const double x = XL[(size_t)v * J + min(t, J - 1)];
                    return t < J ? x : 0.0;
                };
                double xj[kGsSlots];
#pragma unroll
                for (int q = 0; q < kGsSlots; ++q) xj[q] = q < nslot ? ld(j, q) : 0.0;
                for (int pass = 0; pass < 2; ++pass) {
                    for (int i = c0; i < j; ++i) {
                        double xi[kGsSlots];
                        double s = 0.0;
#pragma unroll
                        for (int q = 0; q < kGsSlots; ++q) {
                            xi[q] = q < nslot ? ld(i, q) : 0.0;
                            s += xi[q] * xj[q];
                        }
                        s = wave_sum(s);
#pragma unroll
                        for (int q = 0; q < kGsSlots; ++q) xj[q] -= s * xi[q];
                    }
                }
                double n2 = 0.0;
#pragma unroll
                for (int q = 0; q < kGsSlots; ++q) n2 += xj[q] * xj[q];
                n2 = wave_sum(n2);
                const double inv = n2 > 0.0 ? 1.0 / sqrt(n2) : 0.0;
#pragma unroll
                for (int q = 0; q < kGsSlots; ++q) {
                    const int t = lane + 64 * q;
                    if (q < nslot && t < J) XL[(size_t)j * J + t] = xj[q] * inv;
                }
                if (!in_lds) __threadfence_block();  // later iterations read column j
            }
        }
        __syncthreads();
        if (in_lds)
            for (int idx = tid; idx < R * J; idx += kEigThreads) X[idx] = XL[idx];
    }
    __syncthreads();

    // ---- 5. back-transformation X <- Q X, Q = H_0 H_1 ... H_{J-3} -------
    // Sign rule for every vector: the largest |entry| (lowest index on ties)
    // is positive.
    {
        // A in registers (J <= JP): the LDS region, free again, takes the
        // reflectors in one coalesced pass at pitch JP with zeros outside
        // k < t < J (Hz[k JP + t] = v_t of reflector k).  Each vector is held
        // by 16 lanes, element t = 32 p + 2 l + h at lane l, pair p, half h,
        // so that a dot product ends in four row-local lane exchanges; a wave
        // carries four vectors through the J - 2 reflectors without barriers.
        constexpr int NP = JP / 32;
        double* Hz = reg;
        for (int idx = tid; idx < (J - 2) * JP; idx += kEigThreads) {
            const int k = idx / JP, t = idx - k * JP;
            Hz[idx] = (t > k && t < J) ? H[(size_t)k * J + (t - k - 1)] : 0.0;
        }
        __syncthreads();
        const int g = lane >> 4, l16 = lane & 15;
        for (int jw = 4 * wave; jw < R; jw += 4 * kEigWaves) {  // uniform over the wave
            const int j = jw + g;
            const bool jok = j < R;
            double2 xr[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int t = 32 * p + 2 * l16;
                xr[p].x = (jok && t < J) ? X[(size_t)j * J + t] : 0.0;
                xr[p].y = (jok && t + 1 < J) ? X[(size_t)j * J + t + 1] : 0.0;
            }
            // reflector k and beta_k are loaded one reflector ahead of their use
            auto hload = [&](int k, double2 (&h)[NP], double& b) {
                b = beta[k];
                const double2* hk = reinterpret_cast<const double2*>(Hz + (size_t)k * JP);
#pragma unroll
                for (int p = 0; p < NP; ++p) h[p] = hk[16 * p + l16];
            };
            auto apply = [&](const double2 (&h)[NP], double b) {
                if (b == 0.0) return;  // uniform: the identity
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    s0 = fma(h[p].x, xr[p].x, s0);
                    s1 = fma(h[p].y, xr[p].y, s1);
                }
                const double sk = b * row16_sum(s0 + s1);
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    xr[p].x -= sk * h[p].x;
                    xr[p].y -= sk * h[p].y;
                }
            };
            if (J >= 3) {
                double2 hA[NP], hB[NP];
                double bA, bB;
                hload(J - 3, hA, bA);
                for (int k = J - 3;; k -= 2) {
                    hload(max(k - 1, 0), hB, bB);
                    apply(hA, bA);
                    if (k == 0) break;
                    hload(max(k - 2, 0), hA, bA);
                    apply(hB, bB);
                    if (k == 1) break;
                }
            }
            signed_store<NP>(X, J, j, jok, l16, xr);
        }
    }
    }
}

// Steps 4 (second half) and 5 of a solve whose vectors fill more than one
// workgroup of inverse iteration, in launches of their own.
//
// c0[i] of every vector i < R: the first vector of its cluster (eigenvalues
// no further apart than 1e-3 of T's norm, one to the next).  All threads of
// the workgroup; R <= TK_MAX_MODE_DIM <= its size.
__device__ __forceinline__ void cluster_starts(const double* lam, double ortol, int R, int* c0) {
    const int i = threadIdx.x;
    int b = 0;
    if (i < R) {
        b = i >= 1 && lam[i - 1] - lam[i] <= ortol ? 0 : i;
        c0[i] = b;
    }
    __syncthreads();
    for (int o = 1; o < R; o *= 2) {  // running maximum
        const int t = i < R && i >= o ? c0[i - o] : 0;
        __syncthreads();
        b = max(b, t);
        if (i < R) c0[i] = b;
        __syncthreads();
    }
}

// Modified Gram-Schmidt inside the clusters, two sweeps, by one workgroup:
// vector j, normalised, is taken out of every later vector of its cluster.
// One workgroup doing all vectors, batch after batch, with a single wave for
// the Gram-Schmidt, spent 1.79 ms on J = 250, R = 100; spread out, inverse
// iteration takes 99 us (10 workgroups), this 67 us and eig_back 55 us
// (J = 128, R = 64: 298 -> 132 us).  Here 16 waves own R / 16 vectors each,
// in registers, and a step costs one barrier; what bounds it is the wave
// sums.  NS = ceil(J / 64) slots per lane, at most 16 NV vectors.
template <int NS, int NV>
__global__ __launch_bounds__(kEigThreads) void eig_gs_regs(const double* __restrict__ ho,
                                                           double* __restrict__ X, int J, int R) {
    __shared__ double xs[2][64 * NS];
    __shared__ int c0[TK_MAX_MODE_DIM];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    cluster_starts(ho + 5 * J + 4, 1e-3 * ho[5 * J + 3], R, c0);
    double x[NV][NS];
#pragma unroll
    for (int m = 0; m < NV; ++m)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int i = wave + 16 * m, t = lane + 64 * s;
            x[m][s] = i < R && t < J ? X[(size_t)i * J + t] : 0.0;
        }
    int use = 0;  // slots alternate by use, and every use has a barrier
    for (int sweep = 0; sweep < 2; ++sweep) {
        static_for<0, NV>([&](auto mc) {
            constexpr int M = decltype(mc)::value;
            for (int ow = 0; ow < 16; ++ow) {
                const int j = 16 * M + ow;
                if (j >= R) break;  // uniform
                const int cj = c0[j];
                const bool next = j + 1 < R && c0[j + 1] <= j;
                double* slot = xs[use & 1];
                if (wave == ow) {  // uniform over the wave
                    if (cj < j) {
                        double n2 = 0.0;
#pragma unroll
                        for (int s = 0; s < NS; ++s) n2 = fma(x[M][s], x[M][s], n2);
                        n2 = wave_sum(n2);
                        const double inv = n2 > 0.0 ? 1.0 / sqrt(n2) : 0.0;
#pragma unroll
                        for (int s = 0; s < NS; ++s) x[M][s] *= inv;
                    }
                    if (next) {
#pragma unroll
                        for (int s = 0; s < NS; ++s) slot[lane + 64 * s] = x[M][s];
                    }
                }
                if (!next) continue;  // uniform over the workgroup
                // the slot was last read two uses ago, before the barrier of
                // the use in between
                __syncthreads();
                ++use;
                double xj[NS];
#pragma unroll
                for (int s = 0; s < NS; ++s) xj[s] = slot[lane + 64 * s];
                double dt[NV];
#pragma unroll
                for (int m = M; m < NV; ++m) {
                    const int i = wave + 16 * m;
                    dt[m] = 0.0;
                    if (i > j && i < R && c0[i] <= j) {  // uniform over the wave
                        double t = 0.0;
#pragma unroll
                        for (int s = 0; s < NS; ++s) t = fma(x[m][s], xj[s], t);
                        dt[m] = wave_sum(t);
                    }
                }
#pragma unroll
                for (int m = M; m < NV; ++m)
#pragma unroll
                    for (int s = 0; s < NS; ++s) x[m][s] = fma(-dt[m], xj[s], x[m][s]);
            }
        });
    }
#pragma unroll
    for (int m = 0; m < NV; ++m)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int i = wave + 16 * m, t = lane + 64 * s;
            if (i < R && t < J) X[(size_t)i * J + t] = x[m][s];
        }
}

// The same with the vectors in global memory, for ranks whose vectors do not
// fit one workgroup's registers.  A wave rewrites only its own vectors, and
// vector j is read by all between two barriers.
__global__ __launch_bounds__(kEigThreads) void eig_gs_mem(const double* __restrict__ ho,
                                                          double* X, int J, int R) {
    __shared__ double xs[2][TK_MAX_MODE_DIM];
    __shared__ int c0[TK_MAX_MODE_DIM];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    cluster_starts(ho + 5 * J + 4, 1e-3 * ho[5 * J + 3], R, c0);
    int use = 0;
    for (int sweep = 0; sweep < 2; ++sweep)
        for (int j = 0; j < R; ++j) {
            const bool next = j + 1 < R && c0[j + 1] <= j;
            double* slot = xs[use & 1];
            if (wave == (j & 15)) {
                double* xv = X + (size_t)j * J;
                double inv = 1.0;
                if (c0[j] < j) {
                    double n2 = 0.0;
                    for (int t = lane; t < J; t += 64) n2 = fma(xv[t], xv[t], n2);
                    n2 = wave_sum(n2);
                    inv = n2 > 0.0 ? 1.0 / sqrt(n2) : 0.0;
                }
                for (int t = lane; t < J; t += 64) {
                    const double v = xv[t] * inv;
                    xv[t] = v;
                    if (next) slot[t] = v;
                }
            }
            if (!next) continue;  // uniform over the workgroup
            __syncthreads();
            ++use;
            for (int i = wave + 16 * ((j + 16 - wave) / 16); i < R && c0[i] <= j; i += 16) {
                double* xi = X + (size_t)i * J;
                double t0 = 0.0;
                for (int t = lane; t < J; t += 64) t0 = fma(xi[t], slot[t], t0);
                t0 = wave_sum(t0);
                for (int t = lane; t < J; t += 64) xi[t] = fma(-t0, slot[t], xi[t]);
            }
        }
}

// Back-transformation and sign rule, 16 vectors per workgroup of 4 waves,
// each vector held by 16 lanes as in the one-workgroup solver: element
// t = 32 p + 2 l + h at lane l.  The reflectors pass through LDS in chunks of
// eight, the next chunk's loads in flight while one is applied.  (Reading each
// reflector from L2 when it was due cost about 0.6 us per reflector.)
constexpr int kBackThreads = 256;
constexpr int kBackChunk = 8;

template <int NP>
__global__ __launch_bounds__(kBackThreads) void eig_back(const double* __restrict__ scratch,
                                                         double* __restrict__ X, int J, int R) {
    constexpr int W = 32 * NP;  // padded vector length
    constexpr int NL = kBackChunk * W / kBackThreads;
    extern __shared__ double hs[];  // [2][kBackChunk][W], then [2][kBackChunk] betas
    double* sb = hs + 2 * kBackChunk * W;
    const double* H = scratch + (size_t)J * J;
    const double* beta = eig_handoff(const_cast<double*>(scratch), J) + 2 * J;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, l16 = lane & 15;
    const int j = 16 * (int)blockIdx.x + 4 * wave + g;
    const bool jok = j < R;
    double2 xr[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int t = 32 * p + 2 * l16;
        xr[p].x = (jok && t < J) ? X[(size_t)j * J + t] : 0.0;
        xr[p].y = (jok && t + 1 < J) ? X[(size_t)j * J + t + 1] : 0.0;
    }
    double hv[NL], bv = 0.0;
    auto load = [&](int c) {  // chunk c: reflectors J - 3 - 8 c downward
        const int k0 = J - 3 - kBackChunk * c;
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            const int idx = tid + kBackThreads * n;
            const int k = k0 - idx / W, t = idx % W;
            hv[n] = (k >= 0 && t > k && t < J) ? H[(size_t)k * J + (t - k - 1)] : 0.0;
        }
        if (tid < kBackChunk) bv = k0 - tid >= 0 ? beta[k0 - tid] : 0.0;
    };
    auto store = [&](int b) {
#pragma unroll
        for (int n = 0; n < NL; ++n) hs[b * kBackChunk * W + tid + kBackThreads * n] = hv[n];
        if (tid < kBackChunk) sb[b * kBackChunk + tid] = bv;
    };
    const int nc = (J - 2 + kBackChunk - 1) / kBackChunk;
    load(0);
    store(0);
    __syncthreads();
    for (int c = 0; c < nc; ++c) {
        if (c + 1 < nc) load(c + 1);
        const double* hb = hs + (c & 1) * kBackChunk * W;
#pragma unroll
        for (int u = 0; u < kBackChunk; ++u) {
            const double b = sb[(c & 1) * kBackChunk + u];
            const double2* hk = reinterpret_cast<const double2*>(hb + u * W);
            double2 h[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) h[p] = hk[16 * p + l16];
            double s0 = 0.0, s1 = 0.0;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                s0 = fma(h[p].x, xr[p].x, s0);
                s1 = fma(h[p].y, xr[p].y, s1);
            }
            const double sk = b * row16_sum(s0 + s1);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                xr[p].x = fma(-sk, h[p].x, xr[p].x);
                xr[p].y = fma(-sk, h[p].y, xr[p].y);
            }
        }
        if (c + 1 < nc) store((c + 1) & 1);
        __syncthreads();
    }
    signed_store<NP>(X, J, j, jok, l16, xr);
}

template <int JP, int PH>
__global__ __launch_bounds__(kEigThreads) void eig_kernel(EigArgs a, int region) {
    eig_body<JP, PH, PH == 3>(a, region);
}

// Step 2 of a split solve by multisection on the scaled T in the hand-off
// area: each group of TPE lanes of a wave finds one eigenvalue k (k-th
// smallest) with TPE sample points per round (TPE + 1 sub-intervals), the
// same Sturm counts and stopping rule as the one-launch solver, and stores
// it, unscaled, at position J - 1 - k of the descending list.  TPE = 64 (one
// eigenvalue per wave, six bits per round) suits a single solve, whose few
// waves are latency-bound: more waves per eigenvalue (four: eight bits, 7
// rounds instead of 9) gave J = 128 27 -> 25 us and J = 301 46 -> 57.
template <int TPE>
__device__ __forceinline__ void multisect_group(double* __restrict__ ho, int J, int k,
                                                bool active) {
    const ScalarRows ts(ho + 3 * J);
    const double d0 = ho[3 * J];
    const int lane = threadIdx.x;
    if (!active) return;  // the whole group (k is the same in its lanes)
    const int s = lane % TPE, gofs = lane - s;
    const uint64_t gmask = TPE == 64 ? ~0ull : (((1ull << (TPE & 63)) - 1ull) << gofs);
    double lo = ho[5 * J], hi = ho[5 * J + 1];
    const double sc = ho[5 * J + 2];
    for (int it = 0; it < 160; ++it) {
        const double tol = fmax(kSectTol, kSectTol * fmax(fabs(lo), fabs(hi)));
        if (hi - lo <= tol) break;  // lo, hi are the same in every lane of the group
        const double h = (hi - lo) / (double)(TPE + 1);
        const int c = sturm_count(ts, d0, J, lo + h * (double)(s + 1));
        const uint64_t bal = __ballot(c > k) & gmask;
        const int sstar = bal ? (__ffsll((long long)bal) - gofs) : TPE + 1;  // 1-based point
        const double nlo = sstar == 1 ? lo : lo + h * (double)(sstar - 1);
        const double nhi = sstar == TPE + 1 ? hi : lo + h * (double)sstar;
        lo = nlo;
        hi = nhi;
    }
    if (s == 0) ho[5 * J + 4 + (J - 1 - k)] = 0.5 * (lo + hi) / sc;
}

__global__ __launch_bounds__(64) void eig_multisect(double* __restrict__ scratch, int J) {
    multisect_group<64>(eig_handoff(scratch, J), J, (int)blockIdx.x, true);
}

// The same for a batch, four eigenvalues per workgroup: workgroup w takes
// eigenvalues 4 q .. 4 q + 3 of problem w / nq, q = w % nq, nq = ceil(jmax / 4)
// (groups beyond that problem's J do nothing).  A large batch is issue-bound
// and 16 points per round do less work in all: 60 problems of 96 rows 30 us
// against 47 with a wave per eigenvalue, 24 problems 24 against 27; 12
// problems, 23 against 19, do not carry a variant of their own.
constexpr int kBatchTpe = 16;
constexpr int kBatchGroups = 64 / kBatchTpe;

__global__ __launch_bounds__(64) void eig_multisect_batched(const EigArgs* __restrict__ args,
                                                            int nq, int conditional) {
    const int p = blockIdx.x / nq, q = blockIdx.x - p * nq;
    const int J = args[p].J;
    if (kBatchGroups * q >= J) return;  // uniform over the workgroup
    if (conditional && !(args[p].flags[0] & 4)) return;  // the redo pass: bit 4 only
    const int k = kBatchGroups * q + (int)threadIdx.x / kBatchTpe;
    multisect_group<kBatchTpe>(eig_handoff(uni_global(args[p].scratch), J), J, k, k < J);
}

// One workgroup per problem of a batch, as PH = 1, eig_multisect_batched,
// PH = 3.  A problem whose status word has the FP64-only mark (8) took the
// FP64 Gram: the plain rank rule applies, and the pass's last launch clears
// the mark.  conditional != 0: only problems whose status word has the guard
// bit (4) run, on their FP64 Gram and without the guard; afterwards the bit is
// cleared and `mode_bit` is recorded in the problem's second status word.
template <int JP, int PH>
__global__ __launch_bounds__(kEigThreads) void eig_batched(const EigArgs* __restrict__ args,
                                                           int region, int conditional,
                                                           int mode_bit) {
    EigArgs a = args[blockIdx.x];
    // table pointers as global ones (global, not flat, accesses)
    a.s = uni_global(a.s);
    a.nu = uni_global(a.nu);
    a.lambda = uni_global(a.lambda);
    a.u = uni_global(a.u);
    a.rank_out = uni_global(a.rank_out);
    a.disc_out = uni_global(a.disc_out);
    a.flags = uni_global(a.flags);
    a.scratch = uni_global(a.scratch);
    a.split_stats = uni_global(a.split_stats);
    a.tail_bound = uni_global(a.tail_bound);
    const int f0 = a.flags ? a.flags[0] : 0;
    if (conditional && !(f0 & 4)) return;  // uniform over the workgroup
    if (conditional || (f0 & 8)) {
        a.guard = 0.0;  // an FP64 Gram: plain rank rule
        a.split_stats = nullptr;
    }
    eig_body<JP, PH, false>(a, region);
    if (PH != 1 && (conditional || (f0 & 8))) {  // the pass's last launch
        __syncthreads();
        if (threadIdx.x == 0) {
            if (conditional) {
                a.flags[0] &= ~4;
                a.flags[1] |= mode_bit;
            } else {
                a.flags[0] &= ~8;
            }
        }
    }
}

// The register path (J <= JP) keeps reflector k at row k, pitch JP, of the
// region: at least JP * J doubles (<= 16384 for JP <= 128).
static size_t eig_region_doubles_jp(int J, int JP) {
    const size_t r = eig_region_doubles(J), hs = (size_t)JP * J;
    return r < hs ? hs : r;
}

// Register layouts: 32, 64, 96 and 128 rows (16 lanes per two rows, columns in
// blocks of 16); larger extents (0) are brought to 128 rows first.
static int eig_jp(int J) { return J <= 32 ? 32 : J <= 64 ? 64 : J <= 96 ? 96 : J <= 128 ? 128 : 0; }

size_t eig_lds_bytes(int J) {
    const int JP = eig_jp(J);
    return ((size_t)eig_region_doubles_jp(J, JP) + eig_small_doubles(J)) * sizeof(double);
}

int launch_eig_batched(const EigArgs* args_dev, int count, int jmax, int conditional,
                       int mode_bit, hipStream_t st) {
    if (jmax > 128) return fail(TK_ERR_UNSUPPORTED, "batched eigensolver: extent %d > 128", jmax);
    // every problem uses the register layout of the largest extent (96 rows
    // up to 96, else 128); the LDS partition follows each problem's own J
    // (region computed per J <= jmax)
    const int jp = jmax <= 96 ? 96 : 128;
    const int region = (int)eig_region_doubles_jp(jmax, jp);
    const size_t lds = ((size_t)region + eig_small_doubles(jmax)) * sizeof(double);
    auto launch = [&](auto fn) -> int {
        TK_HIP(hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds));
        hipLaunchKernelGGL(fn, dim3(count), dim3(kEigThreads), lds, st, args_dev, region,
                           conditional, mode_bit);
        TK_HIP(hipGetLastError());
        return TK_OK;
    };
    TK_TRY(jp == 96 ? launch(eig_batched<96, 1>) : launch(eig_batched<128, 1>));
    const int nq = (jmax + kBatchGroups - 1) / kBatchGroups;
    hipLaunchKernelGGL(eig_multisect_batched, dim3(count * nq), dim3(64), 0, st, args_dev, nq,
                       conditional);
    TK_HIP(hipGetLastError());
    return jp == 96 ? launch(eig_batched<96, 3>) : launch(eig_batched<128, 3>);
}

// Extents of at least kSplitEig take three launches (reduction, multisection
// over J workgroups, vectors): the multisection then runs on the whole GPU.
constexpr int kSplitEig = 64;

// Vectors of inverse iteration that one workgroup's LDS region holds.
static int eig_batch(int J) {
    const size_t region = eig_region_doubles_jp(J, eig_jp(J));
    return (int)(region / ((size_t)2 * eig_record_doubles(J) + 2));
}

template <int JP, int PH>
static int launch_eig_phase(const EigArgs& a, int region, size_t lds, int wgs, hipStream_t st) {
    auto fn = eig_kernel<JP, PH>;
    TK_HIP(hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds));
    hipLaunchKernelGGL(fn, dim3(wgs), dim3(kEigThreads), lds, st, a, region);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

template <int NS>
static int launch_reduce_grid(const double* s, int J, double* scratch, int* flags, int polls,
                              hipStream_t st) {
    hipLaunchKernelGGL(eig_reduce_grid<NS>, dim3(kGridWaves), dim3(64), 0, st, s, J, scratch, flags,
                       polls);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

int launch_eig_reduce(const double* s, int J, double* scratch, int* flags, int polls,
                      hipStream_t st) {
    if (J <= 128 || J > TK_MAX_MODE_DIM)
        return fail(TK_ERR_UNSUPPORTED, "eigensolver's reduction: extent %d", J);
    const size_t jj = (size_t)J * J;
    const double* src = s;
    int n = J;
    if (J > kMidRows) {
        const int slots = (J - kMidRows) * J;  // of each kind
        hipLaunchKernelGGL(eig_slots_fill, dim3((slots + 255) / 256), dim3(256), 0, st,
                           (unsigned long long*)scratch, (unsigned long long*)(scratch + 2 * jj),
                           slots);
        TK_HIP(hipGetLastError());
        switch ((J + 63) / 64) {
            case 4: TK_TRY(launch_reduce_grid<4>(s, J, scratch, flags, polls, st)); break;
            case 5: TK_TRY(launch_reduce_grid<5>(s, J, scratch, flags, polls, st)); break;
            case 6: TK_TRY(launch_reduce_grid<6>(s, J, scratch, flags, polls, st)); break;
            case 7: TK_TRY(launch_reduce_grid<7>(s, J, scratch, flags, polls, st)); break;
            default: TK_TRY(launch_reduce_grid<8>(s, J, scratch, flags, polls, st)); break;
        }
        src = scratch + jj + (size_t)(J - kMidRows) * J;
        n = kMidRows;
    }
    const bool grid = J > kMidRows;
    TK_HIP(hipFuncSetAttribute((const void*)eig_reduce_mid,
                               hipFuncAttributeMaxDynamicSharedMemorySize, kMidLds));
    hipLaunchKernelGGL(eig_reduce_mid, dim3(1), dim3(kEigThreads), kMidLds, st, src, n, n, J,
                       scratch, grid ? s : nullptr, grid ? flags : nullptr);
    TK_HIP(hipGetLastError());
    const size_t lds = eig_tail_lds_bytes(J);
    TK_HIP(hipFuncSetAttribute((const void*)eig_reduce_tail,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(eig_reduce_tail, dim3(1), dim3(kEigThreads), lds, st, scratch, J);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

template <int JP>
static int launch_eig_jp(const EigArgs& a, int region, size_t lds, hipStream_t st) {
    if constexpr (JP > 0) {
        if constexpr (JP <= kSplitEig)  // the extents of 96 and 128 rows all split
            if (a.J < kSplitEig) return launch_eig_phase<JP, 0>(a, region, lds, 1, st);
        TK_TRY((launch_eig_phase<JP, 1>(a, region, lds, 1, st)));
    } else {
        TK_TRY(launch_eig_reduce(a.s, a.J, a.scratch, a.flags, kGridPolls, st));
    }
    hipLaunchKernelGGL(eig_multisect, dim3(a.J), dim3(64), 0, st, a.scratch, a.J);
    TK_HIP(hipGetLastError());
    // a workgroup per batch of vectors up to the largest rank there can be
    const int jv = a.aug ? a.J / 2 : a.J;
    int cap = a.fixed_rank > 0 && a.fixed_rank < jv ? a.fixed_rank : jv;
    if (a.max_rank < cap) cap = a.max_rank;
    const int nb = eig_batch(a.J);
    return launch_eig_phase<JP, 3>(a, region, lds, (cap + nb - 1) / nb, st);
}

int launch_eig(const EigArgs& a, hipStream_t st) {
    const int JP = eig_jp(a.J);
    const int region = (int)eig_region_doubles_jp(a.J, JP);
    const size_t lds = ((size_t)region + eig_small_doubles(a.J)) * sizeof(double);
    switch (JP) {
        case 32: return launch_eig_phase<32, 0>(a, region, lds, 1, st);  // below kSplitEig
        case 64: return launch_eig_jp<64>(a, region, lds, st);
        case 96: return launch_eig_jp<96>(a, region, lds, st);
        case 128: return launch_eig_jp<128>(a, region, lds, st);
        default: return launch_eig_jp<0>(a, region, lds, st);
    }
}

template <int NS, int NV>
static int launch_gs_t(const EigArgs& a, int R, hipStream_t st) {
    const double* ho = eig_handoff(a.scratch, a.J);
    if (R <= 16 * NV)
        hipLaunchKernelGGL((eig_gs_regs<NS, NV>), dim3(1), dim3(kEigThreads), 0, st, ho, a.u, a.J,
                           R);
    else
        hipLaunchKernelGGL(eig_gs_mem, dim3(1), dim3(kEigThreads), 0, st, ho, a.u, a.J, R);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

template <int NP>
static int launch_back_t(const EigArgs& a, int R, hipStream_t st) {
    const size_t lds = (size_t)2 * kBackChunk * (32 * NP + 1) * sizeof(double);
    auto fn = eig_back<NP>;
    TK_HIP(hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds));
    hipLaunchKernelGGL(fn, dim3((R + 15) / 16), dim3(kBackThreads), lds, st, a.scratch, a.u, a.J,
                       R);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

int launch_eig_finish(const EigArgs& a, int R, hipStream_t st) {
    // the solver itself ends what one launch (J < 64) or one batch holds
    if (a.J < kSplitEig || (a.J <= 128 && R <= eig_batch(a.J))) return TK_OK;
    // vectors per wave of the register version: at most 40 doubles per lane
    switch ((a.J + 63) / 64) {
        case 1: TK_TRY((launch_gs_t<1, 4>(a, R, st))); break;
        case 2: TK_TRY((launch_gs_t<2, 8>(a, R, st))); break;
        case 3: TK_TRY((launch_gs_t<3, 12>(a, R, st))); break;
        case 4: TK_TRY((launch_gs_t<4, 10>(a, R, st))); break;
        case 5: TK_TRY((launch_gs_t<5, 8>(a, R, st))); break;
        case 6: TK_TRY((launch_gs_t<6, 6>(a, R, st))); break;
        case 7: TK_TRY((launch_gs_t<7, 5>(a, R, st))); break;
        default: TK_TRY((launch_gs_t<8, 5>(a, R, st))); break;
    }
    if (a.J <= 128) return launch_back_t<4>(a, R, st);
    if (a.J <= 192) return launch_back_t<6>(a, R, st);
    if (a.J <= 256) return launch_back_t<8>(a, R, st);
    if (a.J <= 384) return launch_back_t<12>(a, R, st);
    return launch_back_t<16>(a, R, st);
}

}  // namespace tk
