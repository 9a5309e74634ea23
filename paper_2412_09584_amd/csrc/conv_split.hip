// Direct convolutions of the relaxing products on the bf16 matrix cores at FP32 precision,
// for passes that save nothing (whole layers and receptive-field windows).  An FP32 value is
// the sum of three bf16 values, and six of the nine products of their parts stay above
// 2^-24 of a term, as in the dense products of split.hip; v_mfma_f32_32x32x16_bf16 does
// those in 3/8 of the time of v_mfma_f32_32x32x2f32 and, unlike it, leaves the VALU to the
// other waves.
//
// Tile: 256 output pixels (whole images, or a band of rows) of one output phase and 32
// columns, four waves of 64 pixels.  A chunk is 16 channels of the input tile with its halo.
// They come through registers, one chunk ahead, and are split on their way into LDS: every
// value is read once per tap and wave from there, so splitting it at the read would cost
// as much as the matrix instructions save.  A pixel takes 96 bytes, [part][channel], and 16
// of padding, which spreads 16 neighbouring pixels over all banks.  The weights are split
// once at bound_init, in the order of the matrix instructions' operands, and reach LDS by
// DMA.  A step is one tap.
//
// Pairs (windows): a stride-2 layer of at most 16 input channels has four phases of at most 16
// columns, which would fill half of a tile.  The two phases that write neighbouring pixels
// of a row have the same taps in a window, and are one product of 32 columns here, phase h's
// channels from column 16 h on.  On whole layers their taps are a pixel apart; a product over
// the taps of both, a third of them with zero weights, took 3.8 ms where the FP32 kernel
// takes 3.6, so such layers stay with that one.
//
// Infinite operands, and images whose parts leave bf16's range: see launch_pack_split.  Finding
// them by their results takes a maximum per result (no time at 64 inputs of the CNN below).
//
// The bf16 instructions round toward minus infinity.  Odd steps' weights are stored negated
// and go to accumulators of their own, which are subtracted at the end: their bias has the
// other sign.
//
// The 3x32x32 CNN (conv 16@3x3, 32@4x4/2, 32@3x3, 64@4x4/2, FC 512, 10), error against FP64:
// coefficients of 576 spec rows 4.7e-7, with the FP32 kernels 5.1e-7; full CROWN's intermediate
// bounds 1.5e-7, with FP32 kernels on whole layers 1.6e-7.  64 inputs, FP32 kernels -> these: windows on the stride-2 layer 12.6 -> 9.2 ms, on the 3x3 layer 6.1 -> 4.1;
// whole 3x3 and 64-channel layers 6.1 -> 4.5.  Nor do few blocks favour the FP32 kernels: whole
// 3x3 layer, 18 images 21 -> 18 us, 144 images 24 -> 20, 576 images 39 -> 38.
#include "conv_kernels.h"

namespace bp {
namespace {

typedef unsigned u2 __attribute__((ext_vector_type(2)));

constexpr int CK = 16;               // channels per chunk
constexpr int PXB = 3 * 2 * CK + 16; // LDS bytes per pixel
constexpr int SBN = 32;              // columns of a tile
constexpr int SPLIT_IN4 = 7;         // float4s of the input tile per thread
constexpr int SPLIT_W4 = 8;          // 16-byte slots of a chunk's weights per thread
// bits of 2^-80: below it a result's operands (weights of up to 2^20) may lie below SPLIT_MIN
constexpr unsigned RESULT_MIN = 0x17800000u;

// LDS tile of a split product; false where the kernel does not take it.
bool tile_split(const GeomSet &gs, ConvTile &ct, size_t &lds, bool window) {
    const Geom &g = gs.g[0];
    if (g.C % CK != 0 || g.stride != 1 || g.OW % 4 != 0 || !same_shape(gs) || !plan_tile(g, ct)) return false;
    for (int i = 0; i < gs.n; ++i)
        if (!gs.g[i].Bs) return false;
    const int px = g.OH * g.OW;
    if (px < 256 ? px % (window ? 16 : 32) != 0 : px % 256 != 0) return false;
    ct.CC = CK;
    ct.lcc = 4;
    ct.CS = PXB / 4;
    ct.nchunk = g.C / CK;
    ct.KB = ct.T * CK;
    ct.WS = 4;
    ct.in_floats = ct.G * ct.IH * ct.IW * ct.CS;
    set_tile_recips(g, ct);
    lds = (size_t)ct.in_floats * 4 + (size_t)ct.KB / 8 * 3 * SBN * 16;
    return ct.G * ct.IH * ct.IW * 4 <= 256 * SPLIT_IN4 && ct.KB / 8 * 3 * SBN <= 256 * SPLIT_W4 &&
           lds <= LDS_BUDGET && (size_t)ct.G * g.H * g.W * g.C * 4 < (1u << 30);
}

__device__ inline void split4(const float4 v, u2 &hi, u2 &mid, u2 &lo) {
    const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        unsigned hp, mp, lp;
        split_pair(x[2 * i], x[2 * i + 1], hp, mp, lp);
        hi[i] = hp;
        mid[i] = mp;
        lo[i] = lp;
    }
}

template <class Epi, bool PAIR>
__global__ __launch_bounds__(256, 2) void k_conv_split(const GeomSet gs, const ConvTile ct,
                                                       const float *__restrict__ X, const long n_img,
                                                       const Epi epi) {
    constexpr int BN = SBN, MF = 32, FM = 2, FN = 1, NIN = SPLIT_IN4;
    using MM = Mma<MF>;
    using acc_t = typename MM::acc_t;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    char *In = (char *)smem;
    float *Wl = smem + ct.in_floats;

    const TileIdx ti = xcd_tile((gs.g[0].N + BN - 1) / BN, gs.n);
    const Geom &g = gs.g[ti.z];
    const int tid = threadIdx.x, lane0 = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // window passes: several groups of images in turn, as in k_conv
    constexpr bool LOOP = Epi::WIN;
    const int loop = LOOP ? ct.loop : 1;
    const long grp = ldiv_by(ti.x, ct.tiles_y, ct.rTY);
    const int band = (int)(ti.x - grp * ct.tiles_y);
    long img0 = grp * loop * ct.G;
    if (img0 >= n_img) return;
    const int oyb = band * ct.TR, n0 = ti.y * BN, tile_px = ct.TR * g.OW, N = PAIR ? g.N >> 1 : g.N;

    // staging: float4 e = tid + 256 i of the tile, pixel e / 4; out of the layer reads 0
    const int total = ct.G * ct.IH * ct.IW * 4;
    int gin[NIN];
#pragma unroll
    for (int i = 0; i < NIN; ++i) {
        const int e = tid + i * 256, p = e >> 2;
        const int row = qdiv(p, ct.rIW), ix = p - row * ct.IW;
        const int gi = qdiv(row, ct.rIH), iy = row - gi * ct.IH;
        const int y = oyb - g.pad_y + iy, x = ix - g.pad_x;
        gin[i] = e < total && (unsigned)y < (unsigned)g.H && (unsigned)x < (unsigned)g.W
                     ? (((gi * g.H + y) * g.W + x) * g.C + (e & 3) * 4) * 4
                     : 1 << 30;
    }
    char *dst0 = In + (tid >> 2) * PXB + (tid & 3) * 8;
    float4 rin[NIN];
    auto load = [&](long i0, int ch) {
        const int bytes = (int)((n_img - i0 < ct.G ? n_img - i0 : ct.G) * g.H * g.W * g.C * 4);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(X + i0 * (long)g.H * g.W * g.C), (short)0, bytes, BUF_FLAGS);
#pragma unroll
        for (int i = 0; i < NIN; ++i) {
            typedef unsigned u4 __attribute__((ext_vector_type(4)));
            const u4 v = __builtin_amdgcn_raw_buffer_load_b128(r, gin[i] + ch * (CK * 4), 0, 0);
            rin[i] = make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]),
                                 __uint_as_float(v[3]));
        }
    };
    const int wslots = ct.KB / 8 * 3 * BN;                 // 16-byte slots of a chunk's weights
    const float *Wg = (const float *)(g.Bs + (long)ti.y * ct.nchunk * wslots * 8);
    auto stage = [&](int ch) {
#pragma unroll
        for (int i = 0; i < SPLIT_W4; ++i)
            if (i * 256 + wv * 64 < wslots)
                lds_dma16(Wg + (long)ch * wslots * 4, wslots * 16, Wl + (i * 256 + wv * 64) * 4, (i * 256 + tid) * 16);
#pragma unroll
        for (int i = 0; i < NIN; ++i)
            if (tid + i * 256 < total) {
                u2 h, m, l;
                split4(rin[i], h, m, l);
                char *d = dst0 + i * (64 * PXB);
                *(u2 *)d = h;
                *(u2 *)(d + 2 * CK) = m;
                *(u2 *)(d + 4 * CK) = l;
            }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };

    // this lane's operands: pixel idx of each fragment, 8 channels of a tap
    int abase[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int lr = wv * 64 + i * MF + MM::idx(lane0);
        const int gi = qdiv(lr, ct.rTP), q = lr - gi * tile_px;
        const int py = qdiv(q, g.rOW), px = q - py * g.OW;
        abase[i] = ((gi * ct.IH + py) * ct.IW + px) * PXB + MM::grp(lane0) * 16;
    }
    const float *wlane = Wl + (MM::grp(lane0) * 3 * BN + MM::idx(lane0)) * 4;
    load(img0, 0);
    for (int it = 0;; ++it) {
        acc_t acc[FM][FN], neg[FM][FN];
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int v = 0; v < MM::NACC; ++v) acc[i][j][v] = neg[i][j][v] = 0.f;
        const bool next = LOOP && it + 1 < loop && img0 + ct.G < n_img;
        int odd = 0;
        for (int ch = 0; ch < ct.nchunk; ++ch) {
            if (it > 0 || ch > 0) __syncthreads();          // every wave is done with the tile
            stage(ch);
            __syncthreads();
            if (ch + 1 < ct.nchunk) load(img0, ch + 1);
            else if (next) load(img0 + ct.G, 0);
            for (int ty = 0, s = 0; ty < g.kh; ++ty)
            for (int tx = 0; tx < g.kw; ++tx, ++s) {
                const int o = (ty * ct.IW + tx) * PXB;
                bf8 a[FM][3], b[FN][3];
#pragma unroll
                for (int p = 2; p >= 0; --p) {
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        b[j][p] = *(const bf8 *)(wlane + ((s * 2 * 3 + p) * BN + j * MF) * 4);
#pragma unroll
                    for (int i = 0; i < FM; ++i) a[i][p] = *(const bf8 *)(In + abase[i] + o + p * (2 * CK));
                }
                auto six = [&](acc_t (&c)[FM][FN]) {
                    constexpr int pa[6] = {0, 1, 2, 0, 1, 0}, pb[6] = {2, 1, 0, 1, 0, 0};
#pragma unroll
                    for (int q = 0; q < 6; ++q)
#pragma unroll
                        for (int i = 0; i < FM; ++i)
#pragma unroll
                            for (int j = 0; j < FN; ++j) 
                                c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][pa[q]], b[j][pb[q]], c[i][j], 0, 0, 0);
                };
                if (odd) six(neg);
                else six(acc);
                odd ^= 1;
            }
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] -= neg[i][j];

        // results that operands outside the range of the three parts may have formed (one that is
        // not finite, or all so small that their operands' last parts were flushed): the wave's
        // tile by FP32 instructions
        float big = 0.f;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int v = 0; v < MM::NACC; v += 2)   // NaN stays
                big = __builtin_elementwise_maximum(__builtin_elementwise_maximum(big, fabsf(acc[i][0][v])),
                                                    fabsf(acc[i][0][v + 1]));
        const unsigned ub = __float_as_uint(big);
        const bool tiny = ub < RESULT_MIN && __any(ub != 0) && !__any(ub >= RESULT_MIN);
        if (__builtin_expect(__any(ub > 0x7f7fffffu) || tiny, 0)) {
            const int n = n0 + MM::col(lane0), nr = PAIR ? n & 15 : n;
            const float *w = (PAIR && n >= 16 ? g.Bt2 : g.Bt) + (long)(nr < N ? nr : 0) * g.Kp;
#pragma unroll 1
            for (int e = 0; e < FM * MM::NACC; ++e) {
                const int lr = wv * 64 + e / MM::NACC * MF + MM::row(e % MM::NACC, lane0);
                const int gi = qdiv(lr, ct.rTP), q = lr - gi * tile_px;
                const int py = qdiv(q, g.rOW), px = q - py * g.OW;
                float x = 0.f;
                if (nr < N && img0 + gi < n_img)
                    for (int ty = 0; ty < g.kh; ++ty)
                        for (int tx = 0; tx < g.kw; ++tx) {
                            const int y = oyb + py - g.pad_y + ty, xx = px - g.pad_x + tx;
                            if ((unsigned)y >= (unsigned)g.H || (unsigned)xx >= (unsigned)g.W) continue;
                            const float *p = X + (((img0 + gi) * g.H + y) * (long)g.W + xx) * g.C;
                            for (int c = 0; c < g.C; ++c) x = fmaf(p[c], w[(ty * g.kw + tx) * g.C + c], x);
                        }
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int v = 0; v < MM::NACC; ++v) acc[i][0][v] = e == i * MM::NACC + v ? x : acc[i][0][v];
            }
        }

        int lane = lane0;
        if (LOOP) asm volatile("" : "+v"(lane));            // row indices anew, as in k_conv
        int ncol[FN];
        float bcol[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            // a pair's column 16 h + n is channel n of the pixel h further on
            ncol[j] = n0 + j * MF + MM::col(lane);
            const int n = PAIR ? ncol[j] & 15 : ncol[j];
            bcol[j] = n < N ? epi.colv(n) : 0.f;
        }
        if constexpr (Epi::WIN) {
            tile_epilogue_win<Epi, MF, FM, FN, PAIR>(epi, acc, ncol, bcol, g, tile_px, lane, wv * 64, img0, n_img);
        } else {
            // groups of four rows are neighbouring pixels of one output row (OW % 4 == 0)
            auto rowfn4 = [&](int i, int vg, int (&img)[4], int (&dp)[4]) -> bool {
                const int lr = wv * 64 + i * MF + MM::row(4 * vg, lane);
                const int gi = qdiv(lr, ct.rTP), r = lr - gi * tile_px;
                const int py = qdiv(r, g.rOW), px = r - py * g.OW;
                img[0] = img0 + gi < n_img ? (int)(img0 + gi) : -1;
                dp[0] = ((oyb + py) * g.ostr + g.oy0) * g.DW + (px * g.ostr + g.ox0);
#pragma unroll
                for (int q = 1; q < 4; ++q) {
                    img[q] = img[0];
                    dp[q] = dp[0] + q * g.ostr;
                }
                return true;
            };
            const int gfirst = qdiv(wv * 64, ct.rTP), glast = qdiv(wv * 64 + 63, ct.rTP);
            tile_epilogue<Epi, MF, FM, FN, true>(epi, acc, ncol, bcol, g.N, rowfn4, lane,
                                                 gfirst == glast && img0 + gfirst < n_img, (int)(img0 + gfirst));
        }
        if (!next) return;
        img0 += ct.G;
    }
}

// Weights [Np][Kp] of a product, or of a pair's two, -> [column tile][chunk][octet of 8
// channels of a tap][part][32][8], negated in odd steps; zero past the columns.
__global__ void k_pack_conv(const float *B0, const float *B1, int N, int Kp, int C, int T, long total,
                            unsigned short *out, int32_t *flags) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int nch = C / CK;
    int q = (int)(e >> 3);
    const int i = (int)(e & 7), n = q % SBN;
    q /= SBN;
    const int oct = q % (2 * T);
    q /= 2 * T;
    const int ch = q % nch, y = q / nch, t = oct >> 1;
    const int row = B1 ? n & 15 : y * SBN + n;
    const float *Bt = B1 && n >= 16 ? B1 : B0;
    float x = row < N ? Bt[(long)row * Kp + t * C + ch * CK + (oct & 1) * 8 + i] : 0.f;
    flag_range(x, flags);
    if ((ch * T + t) & 1) x = -x;
    unsigned short *o = out + ((((long)y * nch + ch) * (2 * T) + oct) * 3 * SBN + n) * 8 + i;
    split_one(x, o[0], o[SBN * 8], o[2 * SBN * 8]);
}

template <class Epi, bool PAIR>
hipError_t launch(const GeomSet &gs, const float *A, long n_img, const Epi &epi, hipStream_t st) {
    ConvTile ct{};
    size_t lds = 0;
    if (!tile_split(gs, ct, lds, Epi::WIN)) return hipErrorInvalidValue;
    const long groups = (n_img + ct.G - 1) / ct.G, per = (long)ct.tiles_y * ((gs.g[0].N + SBN - 1) / SBN) * gs.n;
    ct.loop = Epi::WIN ? group_loop(ct, groups * per) : 1;
    const long blocks = (groups + ct.loop - 1) / ct.loop * per;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    static const hipError_t ok = allow_lds(k_conv_split<Epi, PAIR>);
    if (ok != hipSuccess) return ok;
    hipLaunchKernelGGL((k_conv_split<Epi, PAIR>), dim3((unsigned)blocks), dim3(256), lds, st, gs, ct, A, n_img, epi);
    return hipGetLastError();
}

bool fits(const GeomSet &gs, long n_img, bool window) {
    ConvTile ct{};
    size_t lds = 0;
    if (gs.n <= 0 || n_img <= 0 || !tile_split(gs, ct, lds, window)) return false;
    const long blocks = (n_img + ct.G - 1) / ct.G * ct.tiles_y * ((gs.g[0].N + SBN - 1) / SBN) * gs.n;
    return blocks <= 0x7fffffffL;
}

}  // namespace

bool conv_split_fits(const GeomSet &gs, long n_img, bool window) {
    const int N = gs.g[0].N;
    return N > 16 && (window || N % SBN == 0) && fits(gs, n_img, window);
}
bool conv_split_pair_fits(const GeomSet &pair, long n_img) { return fits(pair, n_img, true); }
hipError_t conv_split_relax(const GeomSet &gs, const float *A, long n_img, const RelaxParams &p, hipStream_t st) {
    return launch<EpiRelax, false>(gs, A, n_img, EpiRelax{p}, st);
}
hipError_t conv_split_relax_win(const GeomSet &gs, bool pair, const float *A, long n_img, const RelaxParams &p,
                                const WinMap &w, hipStream_t st) {
    return pair ? launch<EpiRelaxWin, true>(gs, A, n_img, EpiRelaxWin{p, w}, st)
                : launch<EpiRelaxWin, false>(gs, A, n_img, EpiRelaxWin{p, w}, st);
}

long conv_split_size(const Geom &g) {
    const int T = g.kh * g.kw;
    if (T == 0 || g.C % CK != 0 || g.stride != 1 || g.N <= 4 || (T == 1 && g.H == 1 && g.W == 1)) return 0;
    return (long)((g.N + SBN - 1) / SBN) * (g.C / CK) * T * 2 * 3 * SBN * 8;
}
hipError_t launch_pack_conv(const Geom &g, const Geom *pair, unsigned short *out, int32_t *flags, hipStream_t st) {
    const long total = conv_split_size(g) / 3;
    if (total > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_pack_conv, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, g.Bt,
                       pair ? pair->Bt : nullptr, pair ? g.N / 2 : g.N, g.Kp, g.C, g.kh * g.kw, total, out,
                       flags);
    return hipGetLastError();
}

}  // namespace bp
