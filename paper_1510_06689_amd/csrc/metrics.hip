// Error metrics of a reconstruction (Table II: normalized RMS and maximum
// absolute element error): ||X - X~||^2, max |X - X~| and ||X||^2, in FP64,
// reduced in two fixed-order stages so the result is reproducible.
#include "tk_common.hpp"

namespace tk {

constexpr int kMetThreads = 256;

// Tree over a workgroup's threads, in a fixed order; totals in entry 0.
__device__ __forceinline__ void fold_metrics(double* s0, double* s1, double* s2, double e2,
                                             double mx, double n2) {
    s0[threadIdx.x] = e2;
    s1[threadIdx.x] = mx;
    s2[threadIdx.x] = n2;
    __syncthreads();
    for (int w = kMetThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            s0[threadIdx.x] += s0[threadIdx.x + w];
            s1[threadIdx.x] = fmax(s1[threadIdx.x], s1[threadIdx.x + w]);
            s2[threadIdx.x] += s2[threadIdx.x + w];
        }
        __syncthreads();
    }
}

template <typename T>
__global__ __launch_bounds__(kMetThreads) void metrics_partial(const T* __restrict__ x,
                                                               const T* __restrict__ xh,
                                                               int64_t n,
                                                               double* __restrict__ part) {
    __shared__ double s0[kMetThreads], s1[kMetThreads], s2[kMetThreads];
    double e2 = 0.0, mx = 0.0, n2 = 0.0;
    const int64_t stride = (int64_t)gridDim.x * kMetThreads;
    auto add = [&](T xv, T hv) {
        const double a = (double)xv, b = (double)hv;
        const double dlt = a - b;
        e2 += dlt * dlt;
        mx = fmax(mx, fabs(dlt));
        n2 += a * a;
    };
    // four strides per trip: eight loads in flight per thread, added in order
    int64_t i = (int64_t)blockIdx.x * kMetThreads + threadIdx.x;
    for (; i + 3 * stride < n; i += 4 * stride) {
        T xv[4], hv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            xv[u] = x[i + u * stride];
            hv[u] = xh[i + u * stride];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) add(xv[u], hv[u]);
    }
    for (; i < n; i += stride) add(x[i], xh[i]);
    fold_metrics(s0, s1, s2, e2, mx, n2);
    if (threadIdx.x == 0) {
        part[3 * blockIdx.x + 0] = s0[0];
        part[3 * blockIdx.x + 1] = s1[0];
        part[3 * blockIdx.x + 2] = s2[0];
    }
}

// One workgroup folds the partials: thread t takes blocks t, t + 256, ... in
// order, then a tree over the threads, so the order is fixed.  (One thread
// walking 1024 blocks took 110 us, all of it load latency; this takes 6 us.)
__global__ __launch_bounds__(kMetThreads) void metrics_final(const double* __restrict__ part,
                                                             int nb, double* __restrict__ out) {
    __shared__ double s0[kMetThreads], s1[kMetThreads], s2[kMetThreads];
    const int tid = threadIdx.x;
    double e2 = 0.0, mx = 0.0, n2 = 0.0;
#pragma unroll 4
    for (int b = tid; b < nb; b += kMetThreads) {
        e2 += part[3 * b];
        mx = fmax(mx, part[3 * b + 1]);
        n2 += part[3 * b + 2];
    }
    fold_metrics(s0, s1, s2, e2, mx, n2);
    if (tid == 0) {
        out[0] = s0[0];
        out[1] = s1[0];
        out[2] = s2[0];
    }
}

int error_metrics_blocks(int64_t n) {
    int64_t b = (n + kMetThreads * 16 - 1) / (kMetThreads * 16);
    int cap = 4 * device_cu_count();
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (int)b;
}

int launch_error_metrics(const void* x, const void* xh, int dtype, int64_t n, double* partial,
                         int nblocks, double* out3, hipStream_t st) {
    if (dtype == TK_F64)
        hipLaunchKernelGGL(metrics_partial<double>, dim3(nblocks), dim3(kMetThreads), 0, st,
                           (const double*)x, (const double*)xh, n, partial);
    else
        hipLaunchKernelGGL(metrics_partial<float>, dim3(nblocks), dim3(kMetThreads), 0, st,
                           (const float*)x, (const float*)xh, n, partial);
    TK_HIP(hipGetLastError());
    hipLaunchKernelGGL(metrics_final, dim3(1), dim3(kMetThreads), 0, st, partial, nblocks,
                       out3);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

}  // namespace tk
