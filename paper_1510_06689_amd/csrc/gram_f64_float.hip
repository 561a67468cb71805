// Tiled FP64 Gram of FP32 tensors, one at a time and in batches.
#include "gram_f64.hpp"

namespace tk {

int launch_gram_f64(const float* y, const ModeView& v, const GramPlan& pl, double* partial,
                    hipStream_t st) {
    return launch_gram_f64_t(y, v, pl, partial, st);
}

// FP64 Gram of every problem of a batch (the guard's recomputation when
// `conditional`).  The partials use the split kernel's layout -- 16-blocks of
// the padded extent JB, pairs in pair_of order -- so the same reduction
// tasks apply; pairs in the padding come out zero.
template <int JB>
__global__ __launch_bounds__(GramSched<JB / 16>::T, 2) void gram_f64_batched(
    const BatchGramTask* __restrict__ tasks, int ntasks, int conditional) {
    extern __shared__ double lds[];
    typedef GramSched<JB / 16> S;
    const int ti = find_task_wg(&tasks[0].v, sizeof(BatchGramTask), ntasks, blockIdx.x);
    BatchGramTask tk = tasks[ti];
    tk.y = uni_global(tk.y);  // global, not flat, accesses
    tk.partial = uni_global(tk.partial);
    // uniform over the workgroup: 1 = the redo of uncertain ranks (bit 4),
    // 2 = the problems marked FP64-only (bit 8)
    if (conditional && !(*tk.status & (conditional == 2 ? 8 : 4))) return;
    const int w = blockIdx.x - tk.v.wg_begin;
    const TileMap tm = make_tiles(batch_mode_view(tk.v), S::KT);
    const int active = (int)(tm.ntiles < tk.v.nwg ? tm.ntiles : tk.v.nwg);
    if (w == 0 && threadIdx.x == 0) *tk.nparts = active;
    if (w >= active) return;  // uniform over the workgroup
    const int64_t t0 = tm.ntiles * (int64_t)w / active;
    const int64_t t1 = tm.ntiles * (int64_t)(w + 1) / active;
    gram_f64_body<float, JB / 16, false, true>(tk.y, tm, t0, t1,
                                               tk.partial + (int64_t)w * S::NP * 256, lds);
}

template <int JB>
static int launch_f64_batched_t(const BatchGramTask* tasks, int ntasks, int total_wg,
                                int conditional, hipStream_t st) {
    const size_t lds = GramSched<JB / 16>::kLds * sizeof(double);
    auto fn = gram_f64_batched<JB>;
    TK_HIP(hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds));
    hipLaunchKernelGGL(fn, dim3(total_wg), dim3(GramSched<JB / 16>::T), lds, st, tasks, ntasks,
                       conditional);
    TK_HIP(hipGetLastError());
    return TK_OK;
}

int launch_gram_f64_batched(const BatchGramTask* tasks_dev, int ntasks, int total_wg, int jb,
                            int conditional, hipStream_t st) {
    switch (jb) {
        case 32: return launch_f64_batched_t<32>(tasks_dev, ntasks, total_wg, conditional, st);
        case 64: return launch_f64_batched_t<64>(tasks_dev, ntasks, total_wg, conditional, st);
        case 128: return launch_f64_batched_t<128>(tasks_dev, ntasks, total_wg, conditional, st);
        default: return fail(TK_ERR_UNSUPPORTED, "batched FP64 Gram: extent class %d", jb);
    }
}

}  // namespace tk
