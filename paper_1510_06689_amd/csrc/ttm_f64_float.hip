// FP64 TTM with the operator in registers, FP32 tensors.
#include "ttm_f64.hpp"

namespace tk {

int launch_ttm_reg(const float* y, const ModeView& v, const double* m, int64_t ldm, int K,
                   int transpose, float* z, hipStream_t st) {
    return launch_ttm_reg_any(y, v, m, ldm, K, transpose, z, st);
}

}  // namespace tk
