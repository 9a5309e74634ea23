// Implicit GEMMs of the adjoint and of the forward pass (kernel in gemm_kernels.h).
#include "gemm_kernels.h"

namespace bp {

hipError_t gemm_adj_cfg(const GeomSet &gs, const float *A, long n_img, const AdjParams &p,
                        hipStream_t st, int cfg) {
    return dispatch(gs, A, n_img, dev::EpiAdj{p}, st, cfg);
}
hipError_t gemm_fwd_cfg(const GeomSet &gs, const float *A, long n_img, const FwdParams &p,
                        hipStream_t st, int cfg) {
    return dispatch(gs, A, n_img, dev::EpiFwd{p}, st, cfg);
}

}  // namespace bp
