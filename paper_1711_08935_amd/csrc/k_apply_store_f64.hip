// Apply kernels that overwrite their rows, grouped work list, FP64 state storage
// (FP64 sums).
#include "k_apply.h"

hipError_t launch_store_grouped_f64(const ApplyArgs& a, int nchunks, int nq, int cplx, int cpl, int waves, int cls,
                                   hipStream_t st) {
    return launch_store_grouped_prec<double>(a, nchunks, nq, cplx, cpl, waves, cls, st);
}
