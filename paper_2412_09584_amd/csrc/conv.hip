// Direct convolutions of the backward pass (relaxation and concretising epilogues) and the
// direct kernels' candidates for the autotuner; the adjoint's and the forward pass's are in
// conv_adj.hip, the kernels in conv_kernels.h.
#include "conv_kernels.h"

namespace bp {

hipError_t direct_relax(const GeomSet &gs, const float *A, long n_img, const RelaxParams &p,
                        hipStream_t st, int cc, int mode, bool *used) {
    return try_direct(gs, A, n_img, EpiRelax{p}, st, cc, mode, used);
}
hipError_t direct_conc(const GeomSet &gs, const float *A, long n_img, const ConcParams &p,
                        hipStream_t st, int cc, int mode, bool *used) {
    return try_direct(gs, A, n_img, EpiConc{p}, st, cc, mode, used);
}
int direct_candidates(const GeomSet &gs, int *cc, int *mode, int cap) {
    const Geom &g = gs.g[0];
    if (g.H == 1 && g.W == 1 && g.kh == 1 && g.kw == 1) return 0;
    if (!same_shape(gs)) return 0;
    ConvTile ct{};
    if (!plan_tile(g, ct)) return 0;
    if (g.N <= 4) {
        if (g.C % 4 != 0) return 0;
        int n = 0;
        for (int m = -1; m <= 3 && n < cap; m += 2) {   // registers, DMA, DMA unpadded
            cc[n] = 0;
            mode[n++] = m;
        }
        return n;
    }
    const int BN = bn_for(g.N);
    if (!BN) return 0;
    const int KPL = BN == 16 ? Mma<16>::KPL : Mma<32>::KPL;
    if (g.C < 4) {
        if (!plan_chunk(g, BN, KPL, ct)) return 0;
        cc[0] = 0;
        mode[0] = -1;
        return cap > 0 ? 1 : 0;
    }
    // each channel chunk with register staging (mode -1) and with LDS DMA staging (1);
    // 32-output products also with 16x16 MFMA tiles (modes 2, 3), which allow chunks of
    // 4 channels
    int n = 0;
    const int modes[4] = {-1, 1, 2, 3};
    for (int c = 64; c >= 4; c >>= 1) {
        for (int mi = 0; mi < (BN == 32 ? 4 : 2) && n < cap; ++mi) {
            const int m = modes[mi];
            const int kpl = m >= 2 ? Mma<16>::KPL : KPL;
            ConvTile t = ct;
            if (c >= kpl && g.C % c == 0 && plan_chunk(g, BN, kpl, t, c, m == 1 || m == 3)) {
                cc[n] = c;
                mode[n] = m;
                ++n;
            }
        }
    }
    return n;
}

}  // namespace bp
