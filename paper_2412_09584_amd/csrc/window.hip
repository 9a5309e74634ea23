// Products of the window passes: a row that bounds one neuron of a convolutional layer has
// non-zero coefficients only in that neuron's receptive field, so its coefficients are
// kept, multiplied and concretised on a small window of each layer (WinMap) instead of on
// whole layers.  The kernels are the DMA-staged direct convolutions of conv_kernels.h with
// the window epilogues; a window of 8 x 8 output pixels per phase is one wave's tile, of 4
// x 4 one 16-row MFMA fragment's.
//
// Full CROWN of 64 inputs of the 3x32x32 CNN (conv 16@3x3, 32@4x4/2, 32@3x3, 64@4x4/2, FC
// 512, 10): 278 ms over whole layers, 46 ms with windows on the FP32 kernels here, 34.8 ms
// with the larger relaxing products on conv_split.hip's (one input: 4.93, 0.97, 0.85 ms).  23
// to 44 % of a window's pixels pad it to 4, 8 or 16 a side.
#include "conv_kernels.h"

namespace bp {
namespace {

int win_bn(int N) { return N <= 16 ? 16 : (N <= 32 ? 32 : 64); }

// Tile of an MFMA product: whole images of 16, 64 or 256 pixels per phase.
bool tile_mfma(const GeomSet &gs, ConvTile &ct, int &mf, size_t &lds) {
    const Geom &g = gs.g[0];
    if (g.C % 4 != 0 || g.OW % 4 != 0 || !same_shape(gs) || !plan_tile(g, ct)) return false;
    const int px = g.OH * g.OW, BN = win_bn(g.N);
    if (px % 16 != 0 || px > 256) return false;
    // 32 columns: 32x32 MFMA tiles unless an image is a single 16-row fragment
    mf = BN == 16 || (BN == 32 && px % 32 != 0) ? 16 : 32;
    if (px % mf != 0) return false;
    lds = plan_chunk(g, BN, mf == 16 ? Mma<16>::KPL : Mma<32>::KPL, ct, 0, true);
    if (lds) set_tile_recips(g, ct);
    return lds != 0;
}

// Tile of the narrow-output concretising product: bands of TR rows, each image's threads
// rounded up to whole waves, as many images as fill the block.
bool tile_valu(const GeomSet &gs, ConvTile &ct, size_t &lds) {
    const Geom &g = gs.g[0];
    if (g.N > 4 || g.C % 4 != 0 || g.OW > 256 || !same_shape(gs)) return false;
    for (int bands = 1; bands <= g.OH; ++bands) {
        ct = ConvTile{};
        ct.TR = (g.OH + bands - 1) / bands;
        ct.tiles_y = (g.OH + ct.TR - 1) / ct.TR;
        ct.pxp = (ct.TR * g.OW + 63) / 64 * 64;
        if (ct.pxp > 256) continue;
        ct.G = 256 / ct.pxp;
        ct.IH = (ct.TR - 1) * g.stride + g.kh;
        ct.IW = (g.OW - 1) * g.stride + g.kw;
        ct.T = g.kh * g.kw;
        ct.CC = g.C;
        ct.CS = g.C;
        ct.in_floats = ct.G * ct.IH * ct.IW * ct.CS;
        lds = (size_t)ct.in_floats * 4;
        if (lds > LDS_BUDGET / 2 || ct.in_floats / 4 > 256 * VALU_DMA_IN4) continue;
        set_tile_recips(g, ct);
        const int spp = ct.CS / 4, rs = ct.IW * spp;
        ct.rowdma = (spp & (spp - 1)) == 0 && rs >= 64 && rs <= 64 * DMA_ROW_SEG;
        return true;
    }
    return false;
}

}  // namespace

bool window_fits(const GeomSet &gs, bool conc) {
    ConvTile ct{};
    int mf = 0;
    size_t lds = 0;
    return conc && gs.g[0].N <= 4 ? tile_valu(gs, ct, lds) : tile_mfma(gs, ct, mf, lds);
}

template <class Epi>
static hipError_t window_launch(const GeomSet &gs, const float *A, long n_img, const Epi &epi, hipStream_t st,
                                const ConvTile &ct, int mf, size_t lds) {
    const int BN = win_bn(gs.g[0].N);
    if (BN == 16) return launch_mfma_dma<Epi, 16, 16>(gs, ct, lds, A, n_img, epi, st);
    if (BN == 32 && mf == 16) return launch_mfma_dma<Epi, 16, 32>(gs, ct, lds, A, n_img, epi, st);
    if (BN == 32) return launch_mfma_dma<Epi, 32, 32>(gs, ct, lds, A, n_img, epi, st);
    return launch_mfma_dma<Epi, 32, 64>(gs, ct, lds, A, n_img, epi, st);
}

hipError_t window_relax(const GeomSet &gs, const GeomSet &pair, const float *A, long n_img, const RelaxParams &p,
                        const WinMap &w, hipStream_t st) {
    if (conv_split_pair_fits(pair, n_img)) return conv_split_relax_win(pair, true, A, n_img, p, w, st);
    if (conv_split_fits(gs, n_img, true)) return conv_split_relax_win(gs, false, A, n_img, p, w, st);
    ConvTile ct{};
    int mf = 0;
    size_t lds = 0;
    if (!tile_mfma(gs, ct, mf, lds)) return hipErrorInvalidValue;
    return window_launch(gs, A, n_img, EpiRelaxWin{p, w}, st, ct, mf, lds);
}

hipError_t window_conc(const GeomSet &gs, const float *A, long n_img, const ConcParams &p,
                       const WinMap &w, hipStream_t st) {
    ConvTile ct{};
    int mf = 0;
    size_t lds = 0;
    const EpiConcWin epi{p, w};
    if (gs.g[0].N > 4) {
        if (!tile_mfma(gs, ct, mf, lds)) return hipErrorInvalidValue;
        return window_launch(gs, A, n_img, epi, st, ct, mf, lds);
    }
    if (!tile_valu(gs, ct, lds)) return hipErrorInvalidValue;
    const long groups = (n_img + ct.G - 1) / ct.G;
    const dim3 grid((unsigned)(groups * ct.tiles_y * gs.n));
    if (gs.g[0].N == 3) {
        static const hipError_t ok = allow_lds(k_conv_valu<EpiConcWin, 3, true>);
        if (ok != hipSuccess) return ok;
        hipLaunchKernelGGL((k_conv_valu<EpiConcWin, 3, true>), grid, dim3(256), lds, st, gs, ct, A, n_img, epi);
    } else {
        static const hipError_t ok = allow_lds(k_conv_valu<EpiConcWin, 4, true>);
        if (ok != hipSuccess) return ok;
        hipLaunchKernelGGL((k_conv_valu<EpiConcWin, 4, true>), grid, dim3(256), lds, st, gs, ct, A, n_img, epi);
    }
    return hipGetLastError();
}

}  // namespace bp
