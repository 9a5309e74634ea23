// Dense products (Linear layers) with few output tiles: one wave per 16x16 or 32x32 tile.
//
// The LDS-tiled GEMM of gemm_kernels.h needs hundreds of 128-wide tiles to fill the chip;
// with fewer, each of its blocks walks all of K in 16-wide chunks behind two barriers and a
// memory latency each (a product of 64 rows through a 296x296 layer: 75 us).  Here every
// wave loads its own A and B operands straight from global memory (L2) into registers,
// several chunks ahead, so there is no barrier and the chain is MFMA latency: 8 cycles per k
// with 16x16x4 tiles, 32 with 32x32x2.  Where that chain is long and tiles are few, the KS
// waves of a block split K and add their tiles through LDS in a fixed order.
//
// An FP32 MFMA adds its products one fused multiply-add after the other, k ascending over
// the lane groups (measured: bitwise equal to a chain of fmaf), so a 16x16x4 tile whose
// groups are fed k = s, 8 + s, s + 1, 9 + s (ORD) repeats the 32x32x2 kernels' sums bitwise
// at a quarter of their latency.
//
// 82 layers of 128 to 296 columns, 64 rows, pass and gradient: 9.84 -> 1.4 ms; adj_L5 of the
// CNN (K = 4096, 576 rows): 365 -> 79 us.
#include "device_common.h"

namespace bp {
namespace {

using namespace dev;

constexpr int BK = 16;

// 16 bytes at 4-byte alignment (rows of a width that is no multiple of 4)
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// (x0 | y0), (x1 | y1), ... of the lower | upper 32 lanes become (x0 | x1), (y0 | y1), ...
__device__ inline void swap32(f32x4v &v) {
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 1]), false, false);
        v[i] = __uint_as_float(r[0]);
        v[i + 1] = __uint_as_float(r[1]);
    }
}

template <class Epi, int MF, int KS, bool ORD>
__global__ __launch_bounds__(KS > 4 ? 64 * KS : 256) void k_dense_wave(const Geom g,
                                                                      const float *__restrict__ A,
                                                                      const long M, const Epi epi) {
    using MM = Mma<MF>;
    using acc_t = typename MM::acc_t;
    static_assert(!ORD || MF == 16, "the 32x32x2 order on 16x16x4 tiles");
    constexpr int KPL = MM::KPL, NACC = MM::NACC, Q = KPL / 4;
    constexpr int D = KPL == 4 ? 8 : 6;          // chunks in flight (16: no faster)
    __shared__ float red[KS > 1 ? (KS - 1) * 64 * NACC : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K = g.K, nt = (g.N + MF - 1) / MF;
    const TileIdx ti = xcd_tile(KS > 1 ? nt : (nt + 3) / 4, 1);
    const long m0 = ti.x * MF;
    const int n0 = (KS > 1 ? ti.y : ti.y * 4 + wave) * MF;
    if (m0 >= M) return;
    const bool live = n0 < g.N;                  // KS = 1: the block's last waves may have no tile
    const int nch = (K + BK - 1) / BK;
    const int c0 = KS > 1 ? nch * wave / KS : 0, c1 = KS > 1 ? nch * (wave + 1) / KS : nch;
    const long row = m0 + MM::idx(lane);
    const int grp = MM::grp(lane);
    // this lane's first k inside a chunk; ORD: groups 0 and 2 hold k 0..3 and 4..7, groups 1
    // and 3 the same of the upper half
    const int kl = ORD ? (grp & 1) * 8 + (grp >> 1) * 4 : grp * KPL;
    const float *a = A + (row < M ? row : M - 1) * (long)K + kl;      // rows past M: dropped
    const float *b = g.Bt + (long)(n0 + MM::idx(lane)) * g.Kp + kl;   // N is padded to 128 rows
    __shared__ float sums[Epi::NRED > 0 && KS == 1 ? 4 * MF * 2 : 1];
    // The full chunks [c0, cf) of this wave run through D register slots without a branch
    // around a load, so the loads stay in flight (past the end they repeat the last
    // chunk); the ragged chunk, if it is this wave's, has registers of its own.
    const int nf = K / BK, cf = c1 < nf ? c1 : nf;
    f32x4v ra[D][Q], rb[D][Q], xa[Q], xb[Q];
    const bool ragged = live && c1 > nf;
    if (ragged) {
#pragma unroll
        for (int q = 0; q < KPL; ++q) {
            const int k = nf * BK + q;
            xb[q >> 2][q & 3] = b[k];
            xa[q >> 2][q & 3] = k + kl < K ? a[k] : 0.f;
        }
    }
    auto load = [&](int s, int c) {
        const int k0 = (c < cf ? c : cf - 1) * BK;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            ra[s][q] = *(const f4u *)(a + k0 + 4 * q);
            rb[s][q] = *(const f32x4v *)(b + k0 + 4 * q);
        }
    };
    acc_t acc[1][1];
#pragma unroll
    for (int v = 0; v < NACC; ++v) acc[0][0][v] = 0.f;
    auto mul = [&](f32x4v (&x)[Q], f32x4v (&y)[Q]) {
        if constexpr (ORD) {
            // step t multiplies k = 2t and 2t + 1 (groups 0 and 2) and 8 more: the half
            // waves swap their odd and even registers
            swap32(x[0]);
            swap32(y[0]);
            constexpr int at[4] = {0, 2, 1, 3};
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[0][0] = MM::mma(x[0][at[t]], y[0][at[t]], acc[0][0]);
        } else {
#pragma unroll
            for (int k = 0; k < KPL; ++k) acc[0][0] = MM::mma(x[k >> 2][k & 3], y[k >> 2][k & 3], acc[0][0]);
        }
    };
    if (live && c0 < cf) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            load(s, c0 + s);
            __builtin_amdgcn_sched_barrier(0);       // in order: the first one is waited for first
        }
        int c = c0;
        for (; c + D <= cf; c += D) {
#pragma unroll
            for (int s = 0; s < D; ++s) {
                mul(ra[s], rb[s]);
                load(s, c + s + D);
                __builtin_amdgcn_sched_barrier(0);   // the loads go out here, not after the MFMAs
            }
        }
#pragma unroll
        for (int s = 0; s < D; ++s)
            if (c + s < cf) mul(ra[s], rb[s]);
    }
    if (ragged) mul(xa, xb);
    if constexpr (KS > 1) {
        if (wave > 0) {
#pragma unroll
            for (int v = 0; v < NACC; ++v) red[((wave - 1) * NACC + v) * 64 + lane] = acc[0][0][v];
        }
        __syncthreads();
        if (wave > 0) return;
        for (int w = 0; w < KS - 1; ++w)
#pragma unroll
            for (int v = 0; v < NACC; ++v) acc[0][0][v] += red[(w * NACC + v) * 64 + lane];
    }
    float x = 0.f, y = 0.f;
    int r = 0;
    bool own = false;
    if (live) dense_tile_epilogue<Epi, MF>(epi, acc[0][0], m0, M, n0, g.N, lane, x, y, r, own);
    if constexpr (Epi::NRED > 0 && KS == 1) {
        // one pair of sums per row and block: fewer roundings of the row's running sum
        if (own) {
            sums[(wave * MF + r) * 2] = x;
            sums[(wave * MF + r) * 2 + 1] = y;
        }
        __syncthreads();
        const int nw = (g.N - (n0 - wave * MF) + MF - 1) / MF < 4 ? (g.N - (n0 - wave * MF) + MF - 1) / MF : 4;
        if (threadIdx.x < MF && m0 + threadIdx.x < M) {
            x = y = 0.f;
            for (int w = 0; w < nw; ++w) {
                x += sums[(w * MF + threadIdx.x) * 2];
                y += sums[(w * MF + threadIdx.x) * 2 + 1];
            }
            put_row_sums(epi, m0 + threadIdx.x, 0, n0, x, y);
        }
    } else if (own && m0 + r < M) {
        put_row_sums(epi, m0 + r, 0, n0, x, y);
    }
}

template <class Epi, int MF, int KS, bool ORD = false>
hipError_t launch_wave(const Geom &g, const float *A, long M, const Epi &epi, hipStream_t st) {
    const long nt = (g.N + MF - 1) / MF, tiles = (M + MF - 1) / MF * (KS > 1 ? nt : (nt + 3) / 4);
    if (tiles > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_dense_wave<Epi, MF, KS, ORD>), dim3((unsigned)tiles), dim3(KS > 1 ? 64 * KS : 256), 0, st,
                       g, A, M, epi);
    return hipGetLastError();
}

template <class Epi>
hipError_t run(const GeomSet &gs, const float *A, long M, const Epi &epi, hipStream_t st, int cfg) {
    const Geom &g = gs.g[0];
    switch (cfg) {
    case DENSE_W32: return launch_wave<Epi, 32, 1>(g, A, M, epi, st);
    case DENSE_W16: return launch_wave<Epi, 16, 1>(g, A, M, epi, st);
    case DENSE_W16O: return launch_wave<Epi, 16, 1, true>(g, A, M, epi, st);
    case DENSE_W16K4: return launch_wave<Epi, 16, 4>(g, A, M, epi, st);
    default: return launch_wave<Epi, 16, 16>(g, A, M, epi, st);
    }
}

}  // namespace

// The lines were drawn by relaxing products of K x N = 10 x 512 .. 4096 x 512 and 64 .. 36864
// rows (us, one side / the other):
//  - one 128 x 128 tile per CU: below, the wave kernels are faster than the LDS-tiled GEMM (4096 x
//    512, 4608 rows: 360 W32, 364 GEMM; 256 x 256, 4608: 29, 57), above they re-read A and B too
//    often (296 x 296, 16384: 50, 40).
//  - up to K = 128 a tile is loads and epilogue: 32 x 32 from 96 of them on (64 x 64: 576 rows 11
//    on both, 4608 rows 11, 16 x 16 21; 100 x 100: 576 rows 14, 12; 16384 rows 22, 32).
//  - longer chains: four waves share one of 16 x 16 while tiles are few (4096 x 512: 576 rows,
//    1152 tiles, 86, 32 x 32 123; 1152 rows, 2304 tiles, 148, 125; 512 x 4096, 200 rows, 3328
//    tiles, 54, 27); sixteen waves were slower from the first tile on (4096 x 512, 1 row: 19 by
//    four, 22).  Where a quarter of the 32-wide tiles' columns or more would be padding, 16 x 16
//    stay: 1000 x 40, 9216 rows 31 shared by four, 44; past 2048 tiles one wave each (16384 rows
//    42, shared 51).
//  - products that keep the general order: see the head of the file (W32 from 4096 tiles on:
//    576 rows of 512 x 4096 62, 16 x 16 87).
int dense_auto(const GeomSet &gs, long M, bool keep) {
    const Geom &g = gs.g[0];
    if (!is_dense(gs) || M <= 0) return -1;
    const long big = (M + 127) / 128 * ((g.N + 127) / 128);       // tiles of the LDS-tiled GEMM
    // (a 1x1 convolution on one pixel has no bf16 weights)
    if (big >= 256 && !dma_fits(g)) return -1;
    if (big >= 256) return !keep && g.Bs ? DENSE_SPLIT : (g.N >= 32 ? DENSE_F32 : -1);
    const long small = (M + 15) / 16 * ((g.N + 15) / 16), n32 = (g.N + 31) / 32;
    // the general GEMM's default tiles are 32x32x2 from 32 columns on
    if (keep) return g.N < 32 ? DENSE_W16 : (small <= 4096 ? DENSE_W16O : DENSE_W32);
    if (g.K <= 128) return (M + 31) / 32 * n32 >= 96 ? DENSE_W32 : DENSE_W16;
    const bool padded = n32 * 128 > 5L * g.N;
    if (small > 1152 && !padded) return DENSE_W32;
    return small <= 2048 ? DENSE_W16K4 : DENSE_W16;
}

hipError_t dense_relax(const GeomSet &gs, const float *A, long M, const RelaxParams &p, hipStream_t st, int cfg) {
    if (cfg >= DENSE_SPLIT) return tall_relax(gs, A, M, p, st, cfg == DENSE_SPLIT);
    return run(gs, A, M, EpiRelax{p}, st, cfg);
}
hipError_t dense_conc(const GeomSet &gs, const float *A, long M, const ConcParams &p, hipStream_t st, int cfg) {
    if (cfg >= DENSE_SPLIT) return tall_conc(gs, A, M, p, st, cfg == DENSE_SPLIT);
    return run(gs, A, M, EpiConc{p}, st, cfg);
}
// the adjoint and the forward pass keep the FP32 order (no bf16 weights are packed for them)
hipError_t dense_adj(const GeomSet &gs, const float *A, long M, const AdjParams &p, hipStream_t st, int cfg) {
    if (cfg >= DENSE_SPLIT) return tall_adj(gs, A, M, p, st);
    return run(gs, A, M, EpiAdj{p}, st, cfg);
}
hipError_t dense_fwd(const GeomSet &gs, const float *A, long M, const FwdParams &p, hipStream_t st, int cfg) {
    if (cfg >= DENSE_SPLIT) return tall_fwd(gs, A, M, p, st);
    return run(gs, A, M, EpiFwd{p}, st, cfg);
}

}  // namespace bp
