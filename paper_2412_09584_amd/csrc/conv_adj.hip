// Direct convolutions of the adjoint and of the forward pass (kernels in conv_kernels.h).
#include "conv_kernels.h"

namespace bp {

hipError_t direct_adj(const GeomSet &gs, const float *A, long n_img, const AdjParams &p,
                        hipStream_t st, int cc, int mode, bool *used) {
    return try_direct(gs, A, n_img, EpiAdj{p}, st, cc, mode, used);
}

hipError_t direct_fwd(const GeomSet &gs, const float *A, long n_img, const FwdParams &p,
                        hipStream_t st, int cc, int mode, bool *used) {
    return try_direct(gs, A, n_img, EpiFwd{p}, st, cc, mode, used);
}

}  // namespace bp
