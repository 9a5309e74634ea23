// Implicit GEMMs of the backward pass (relaxation and concretising epilogues), the tile
// candidates and the choice between the product kernels; the adjoint's and the forward
// pass's are in gemm_adj.hip, the kernel in gemm_kernels.h.
#include "gemm_kernels.h"

namespace bp {

// whether a dense kernel adds in the order of the general GEMM's default tiles, which are
// 32x32x2 from 32 columns on
static bool keeps_order(int cfg, int N) {
    return N < 32 ? cfg == DENSE_W16 : cfg == DENSE_W32 || cfg == DENSE_W16O || cfg == DENSE_F32;
}

int gemm_candidates(const GeomSet &gs, bool keep, int *cfgs, int cap) {
    // a tile wider than the padded N only repeats zero columns
    const int N = gs.g[0].N;
    int n = 0;
    const Geom &g = gs.g[0];
    const bool dma = is_dense(gs) && g.C % 4 == 0 && g.K % BK == 0 && dma_fits(g);
    for (int c = 0; c < kGemmCfgs && n < cap; ++c) {
        if (c >= 9 && !dma) continue;
        if (kCfgBN[c] <= 16 * ((N + 15) / 16) || c == default_cfg(N)) cfgs[n++] = c;
    }
    // the wave-per-tile kernels (they never repeat padding columns past a tile)
    for (int c = DENSE_W32; c <= DENSE_F32 && n < cap && is_dense(gs); ++c)
        if ((c != DENSE_W16K16 || g.K >= 256) && (c != DENSE_SPLIT || g.Bs) && (c < DENSE_SPLIT || dma_fits(g)) &&
            (!keep || keeps_order(c, N)))
            cfgs[n++] = c;
    return n;
}

hipError_t gemm_relax_cfg(const GeomSet &gs, const float *A, long n_img, const RelaxParams &p,
                          hipStream_t st, int cfg) {
    return dispatch(gs, A, n_img, dev::EpiRelax{p}, st, cfg);
}
hipError_t gemm_conc_cfg(const GeomSet &gs, const float *A, long n_img, const ConcParams &p,
                         hipStream_t st, int cfg) {
    return dispatch(gs, A, n_img, dev::EpiConc{p}, st, cfg);
}
int plan_candidates(const GeomSet &gs, bool keep, Plan *out, int cap) {
    int n = 0;
    int cc[kMaxCandidates], mode[kMaxCandidates];
    const int nd = direct_candidates(gs, cc, mode, kMaxCandidates);
    for (int i = 0; i < nd && n < cap; ++i) {
        out[n].path = 1;
        out[n].cfg = mode[i];
        out[n].cc = cc[i];
        ++n;
    }
    int cf[kMaxCandidates];
    const int ng = gemm_candidates(gs, keep, cf, kMaxCandidates);
    for (int i = 0; i < ng && n < cap; ++i) {
        out[n].path = 2;
        out[n].cfg = cf[i];
        out[n].cc = 0;
        ++n;
    }
    if (!keep && n < cap) out[n++] = Plan{};       // conv_split.hip's kernels have no plan of their own
    return n;
}

static hipError_t relax_general(const GeomSet &gs, const float *A, long n_img, const RelaxParams &p,
                                hipStream_t st, const Plan &plan);
hipError_t gemm_relax(const GeomSet &gs, const float *A, long n_img, const RelaxParams &p,
                      hipStream_t st, const Plan &plan) {
    if (plan.path == 0 && plan.cfg != 1 && !plan.keep && !p.save && conv_split_fits(gs, n_img, false))
        return conv_split_relax(gs, A, n_img, p, st);
    return relax_general(gs, A, n_img, p, st, plan);
}

#define BOUND_PRODUCT(NAME, PARAMS, DIRECT, CFG, DENSE)                                      \
    hipError_t NAME(const GeomSet &gs, const float *A, long n_img, const PARAMS &p,          \
                    hipStream_t st, const Plan &plan) {                                      \
        if (plan.path != 2) {                                                                \
            bool used = false;                                                               \
            const hipError_t e = DIRECT(gs, A, n_img, p, st, plan.path == 1 ? plan.cc : 0,   \
                                        plan.path == 1 || plan.cfg == 1 ? plan.cfg : DIRECT_AUTO, \
                                        &used);                                              \
            if (used || e != hipSuccess) return e;                                           \
            const int d = plan.path == 0 ? dense_auto(gs, n_img, plan.keep) : -1;            \
            if (d >= 0) return DENSE(gs, A, n_img, p, st, d);                                \
        } else if (plan.cfg >= DENSE_W32 && is_dense(gs) &&                                  \
                   (plan.cfg != DENSE_SPLIT || gs.g[0].Bs) &&                                \
                   (plan.cfg < DENSE_SPLIT || dma_fits(gs.g[0]))) {                          \
            return DENSE(gs, A, n_img, p, st, plan.cfg);                                     \
        }                                                                                    \
        return CFG(gs, A, n_img, p, st, plan.path == 2 ? plan.cfg : -1);                     \
    }
BOUND_PRODUCT(relax_general, RelaxParams, direct_relax, gemm_relax_cfg, dense_relax)
BOUND_PRODUCT(gemm_conc, ConcParams, direct_conc, gemm_conc_cfg, dense_conc)
BOUND_PRODUCT(gemm_adj, AdjParams, direct_adj, gemm_adj_cfg, dense_adj)
BOUND_PRODUCT(gemm_fwd, FwdParams, direct_fwd, gemm_fwd_cfg, dense_fwd)
#undef BOUND_PRODUCT

}  // namespace bp
