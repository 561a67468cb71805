// Tiled FP64 Gram of FP64 tensors.
#include "gram_f64.hpp"

namespace tk {

int launch_gram_f64(const double* y, const ModeView& v, const GramPlan& pl, double* partial,
                    hipStream_t st) {
    return launch_gram_f64_t(y, v, pl, partial, st);
}

}  // namespace tk
