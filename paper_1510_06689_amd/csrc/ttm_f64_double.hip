// FP64 TTM with the operator in registers, FP64 tensors.
#include "ttm_f64.hpp"

namespace tk {

int launch_ttm_reg(const double* y, const ModeView& v, const double* m, int64_t ldm, int K,
                   int transpose, double* z, hipStream_t st) {
    return launch_ttm_reg_any(y, v, m, ldm, K, transpose, z, st);
}

}  // namespace tk
