// Large dense products (Linear layers) on the bf16 matrix cores at FP32 precision.
//
// An FP32 value is the sum of three bf16 values (each the rounded remainder of the one
// before: 8 + 8 + 8 significant bits), so a product of two FP32 matrices is nine products
// of bf16 matrices accumulated in FP32; the three smallest (mid*lo, lo*mid, lo*lo, below
// 2^-24 of a term) are left out.  v_mfma_f32_32x32x16_bf16 runs at 16 times the rate of
// v_mfma_f32_32x32x2f32, so the six remaining ones cost 3/8 of the FP32 MFMAs, and unlike
// those they leave the VALU free for the epilogue and the splitting.
//
// An instruction aligns its terms with the sum it continues and cuts them off there, toward
// minus infinity.  Continuing one sum over all of K would cut the small products at the size of
// the whole sum: error 1.06 times the FP32 kernels'.  So a column's six products of 16 k start
// a sum of their own, which one FP32 fused multiply-add takes into the column's: 0.39 times
// (MLP 784-256x6-10, 16384 rows, coefficients against FP64 5.0e-7 FP32, 5.3e-7, now 2.0e-7).
//
// Tile: 256 threads = 4 waves of 32 rows x 32 FN columns.  The weights are split once at
// bound_init, laid out in 32-wide k chunks ([n][chunk][part][32]), and reach LDS by DMA, two
// buffers deep; their 16-byte k octets are stored in the order q ^ ((r >> 1) & 3) ^ ((r >> 3)
// & 1) of row r, which spreads 16 consecutive rows over the banks.  A wave's own rows of A
// go straight from global memory to registers, one chunk ahead, and are split there: no
// other wave needs them.  One barrier per chunk.  Three waves a SIMD (168 registers) hide the
// chains of products; with two, MLP 784-256x6-10, 256 inputs: 3.87 -> 4.27 ms.
//
// 131072 rows, K = 256: N = 784 with the box 0.59 -> 0.39 ms (135 TFLOP/s of FP32 products),
// N = 256 with the relaxation 0.22 -> 0.12 ms.
//
// The same tile with v_mfma_f32_32x32x2f32 (SPLIT = false) repeats the general GEMM's sums
// bitwise for the passes that have to keep them (Plan::keep): it needs a tenth of the LDS
// reads per MFMA cycle and one barrier per 32 k.
//
// The columns' records (or box) are the same for all rows of an instance, so a wave whose
// rows belong to one instance loads them once instead of once per row.
#include "device_common.h"

namespace bp {
namespace {

using namespace dev;

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // rows of any width
typedef unsigned u4 __attribute__((ext_vector_type(4)));

constexpr int SK = 32;           // k per chunk
constexpr int SBM = 128;         // rows per block

// x = hi + mid + lo, eight values at a time
__device__ inline void split8(const float *x, bf8 &hi, bf8 &mid, bf8 &lo) {
    u4 h, m, l;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned hp, mp, lp;
        split_pair(x[2 * i], x[2 * i + 1], hp, mp, lp);
        h[i] = hp;
        m[i] = mp;
        l[i] = lp;
    }
    hi = __builtin_bit_cast(bf8, h);
    mid = __builtin_bit_cast(bf8, m);
    lo = __builtin_bit_cast(bf8, l);
}

// Sign of chunk c's weights in the 32 columns of tile y.
__host__ __device__ inline bool chunk_sign(int c, int y) { return (__builtin_popcount(c) + y) & 1; }

__device__ inline int swz(int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); }
__device__ inline int swz8(int r) { return (r ^ (r >> 3 & 1)) & 7; }

// What the cut leaves of a sum's products is a bias; sums over many columns of one sign (a
// box's centre) would see it.  Half of the chunks' weights (the Thue-Morse sequence, which also
// cancels a trend along K; every other column tile starts with the other sign) are stored
// negated and their sums subtracted, which turns the bias round.
template <class Epi, int FN, bool SPLIT>
__global__ __launch_bounds__(256, SPLIT ? 3 : 1) void k_dense_tall(const Geom g, const float *__restrict__ A,
                                                    const long M, const Epi epi) {
    using MM = Mma<32>;
    constexpr int BN = 32 * FN, SLOTS = SPLIT ? 3 * BN * 4 : BN * 8, NS = (SLOTS + 255) / 256;
    __shared__ __attribute__((aligned(16))) float Bs[2][SLOTS * 4];
    const TileIdx ti = xcd_tile((g.N + BN - 1) / BN, 1);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long m0 = ti.x * SBM + wv * 32;
    const int n0 = ti.y * BN, K = g.K, nch = (K + SK - 1) / SK;
    const int col = lane & 31, h = lane >> 5;

    // weights: slot s of a buffer is, in bf16, part s / (4 BN), row (s / 4) % BN, octet (s &
    // 3) ^ swz, in FP32 row s / 8, quad (s & 7) ^ swz8
    const float *Bb = SPLIT ? (const float *)(g.Bs + (long)n0 * nch * 3 * SK) : g.Bt + (long)n0 * g.Kp;
    const int bbytes = SPLIT ? BN * nch * 3 * SK * 2 : BN * g.Kp * 4, bstep = SPLIT ? 3 * SK * 2 : SK * 4;
    int boff[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int s = i * 256 + tid;
        if (SPLIT) {
            const int p = s / (4 * BN), r = (s >> 2) % BN, q = (s & 3) ^ swz(r);
            boff[i] = r * nch * 3 * SK * 2 + p * SK * 2 + q * 16;
        } else {
            const int r = s >> 3, q = (s & 7) ^ swz8(r);
            boff[i] = r * g.Kp * 4 + q * 16;
        }
    }
    auto dma = [&](int c, int b) {
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (SLOTS % 256 == 0 || i * 256 + wv * 64 < SLOTS)
                lds_dma16(Bb, bbytes, Bs[b] + (i * 256 + wv * 64) * 4, boff[i] + c * bstep);
    };
    // this lane's row of A: k = 16 t + 8 h + 0 .. 7 of a chunk, t = 0, 1
    const long row = m0 + col;
    const float *a = A + (row < M ? row : M - 1) * (long)K + 8 * h;     // rows past M: dropped
    float ra[16], rn[16];
    auto loadA = [&](int c, float (&x)[16]) {
        const int k0 = c * SK;
        if (k0 + SK <= K) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const f4u v = *(const f4u *)(a + k0 + (t >> 1) * 16 + (t & 1) * 4);
                x[4 * t] = v[0]; x[4 * t + 1] = v[1]; x[4 * t + 2] = v[2]; x[4 * t + 3] = v[3];
            }
        } else {
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const int k = k0 + (t >> 3) * 16 + (t & 7);
                x[t] = k + 8 * h < K ? a[k] : 0.f;
            }
        }
    };
    f32x16 acc[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    float big = 0.f;             // largest magnitude of this lane's part of its row

    dma(0, 0);
    loadA(0, ra);
    for (int c = 0; c < nch; ++c) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();          // chunk c has landed, and every wave is done with c - 1
        if (c + 1 < nch) {
            dma(c + 1, (c + 1) & 1);
            if constexpr (!SPLIT) loadA(c + 1, rn);
        }
        const float *B = Bs[c & 1];
        if constexpr (SPLIT) {
            // two columns at a time, so that one's chain of products hides the other's latency
            constexpr int JC = FN < 2 ? 1 : 2;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                bf8 ah, am, al;
                split8(ra + 8 * t, ah, am, al);
#pragma unroll
                for (int i = 0; i < 8; i += 2)
                    big = fmaxf(fmaxf(big, fabsf(ra[8 * t + i])), fabsf(ra[8 * t + i + 1]));
                if (t == 1) {
                    // the next chunk takes these registers; not earlier, or the second half's
                    // split would wait for it
                    __builtin_amdgcn_sched_barrier(0);
                    if (c + 1 < nch) loadA(c + 1, ra);
                }
#pragma unroll
                for (int j0 = 0; j0 < FN; j0 += JC) {
                    f32x16 s[JC];
#pragma unroll
                    for (int j = 0; j < JC; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v) s[j][v] = 0.f;
#pragma unroll
                    for (int p = 2; p >= 0; --p) {
                        bf8 b[JC];
#pragma unroll
                        for (int j = 0; j < JC; ++j) {
                            const int r = (j0 + j) * 32 + col;
                            b[j] = *(const bf8 *)(B + ((p * BN + r) * 4 + ((2 * t + h) ^ swz(r))) * 4);
                        }
                        auto mm = [&](const bf8 &x) {
#pragma unroll
                            for (int j = 0; j < JC; ++j)
                                s[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, b[j], s[j], 0, 0, 0);
                        };
                        if (p == 0) mm(al);
                        if (p <= 1) mm(am);
                        mm(ah);
                    }
#pragma unroll
                    for (int j = 0; j < JC; ++j) {
                        const float sgn = chunk_sign(c, ti.y * FN + j0 + j) ? -1.f : 1.f;
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[j0 + j][v] = fmaf(s[j][v], sgn, acc[j0 + j][v]);
                        asm volatile("" : "+v"(acc[j0 + j]));   // here, not after all columns: registers
                    }
                }
            }
        } else {
            // the order of the general GEMM's 32x32x2 tiles: k = s and 8 + s at step s
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (c * SK + 16 * t >= K) break;
                f32x4v b[FN][2];
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const int r = j * 32 + col;
                        b[j][q] = *(const f32x4v *)(B + (r * 8 + ((4 * t + 2 * h + q) ^ swz8(r))) * 4);
                    }
#pragma unroll
                for (int k = 0; k < 8; ++k)
#pragma unroll
                    for (int j = 0; j < FN; ++j) acc[j] = MM::mma(ra[8 * t + k], b[j][k >> 2][k & 3], acc[j]);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) ra[i] = rn[i];
        }
    }

    if constexpr (SPLIT) {
        // a row that three bf16 parts do not hold: the wave's tile by FP32 instructions (looking
        // for one: full CROWN of 16-256x3-1, 2048 boxes, 2.78 -> 2.83 ms)
        const unsigned u = __float_as_uint(fmaxf(big, __shfl_xor(big, 32, 64)));
        if (__builtin_expect(__any(u > SPLIT_MAX || (u != 0 && u < SPLIT_MIN)), 0)) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
            const float *b = g.Bt + (long)(n0 + col) * g.Kp + 8 * h;
#pragma unroll 1
            for (int k0 = 0; k0 < K; k0 += 16)
#pragma unroll 1
                for (int k = k0; k < k0 + 8; ++k) {
                    const float x = k + 8 * h < K ? a[k] : 0.f;
#pragma unroll
                    for (int j = 0; j < FN; ++j) acc[j] = MM::mma(x, b[(long)j * 32 * g.Kp + k], acc[j]);
                }
        }
    }

    // ---------------------------------------------------------------- epilogue
    if (m0 >= M) return;
    int ncol[FN];
    float bcol[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        ncol[j] = n0 + j * 32 + col;
        bcol[j] = ncol[j] < g.N ? epi.colv(ncol[j]) : 0.f;
    }
    float s0[16], s1[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) s0[v] = s1[v] = 0.f;
    if (m0 + 32 <= M && epi.one_instance((int)m0, 32)) {
        const auto r0 = epi.row((int)m0);
        typename Epi::Pre pre[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j)
            if (ncol[j] < g.N) pre[j] = epi.pre(r0, 0, ncol[j], g.N);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const auto rc = epi.at(r0, MM::row(v, lane));
#pragma unroll
            for (int j = 0; j < FN; ++j)
                if (ncol[j] < g.N) epi.post(pre[j], rc, 0, ncol[j], ncol[j], bcol[j], acc[j][v], s0[v], s1[v]);
        }
    } else {
        // rows of several instances: two rows' records at a time
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
            typename Epi::Row rc[2];
            typename Epi::Pre pre[2][FN];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const long r = m0 + MM::row(v + q, lane);
                if (r < M) {
                    rc[q] = epi.row((int)r);
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        if (ncol[j] < g.N) pre[q][j] = epi.pre(rc[q], 0, ncol[j], g.N);
                }
            }
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    if (ncol[j] < g.N && m0 + MM::row(v + q, lane) < M) epi.pre2(rc[q], pre[q][j]);
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (m0 + MM::row(v + q, lane) < M)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        if (ncol[j] < g.N)
                            epi.post(pre[q][j], rc[q], 0, ncol[j], ncol[j], bcol[j], acc[j][v + q], s0[v + q],
                                     s1[v + q]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (Epi::NRED > 0) {
        int v;
        const float x = sum_rows<32, 16>(s0, lane, v), y = sum_rows<32, 16>(s1, lane, v);
        const long r = m0 + MM::row(v, lane);
        if ((lane & 1) == 0 && r < M) put_row_sums(epi, r, 0, n0, x, y);
    }
}

// Bt [Np][Kp] FP32 -> [Np][Kc][3][32] bf16 (zero past K, as Bt's padding is)
__global__ void k_pack_split(const float *Bt, int Kp, int Kc, long total, unsigned short *out, int32_t *flags) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const long n = e / (Kc * SK);
    const int k = (int)(e - n * Kc * SK), c = k / SK, i = k - c * SK;
    float x = k < Kp ? Bt[n * Kp + k] : 0.f;
    flag_range(x, flags);
    if (chunk_sign(c, (int)(n >> 5))) x = -x;
    unsigned short *o = out + ((n * Kc + c) * 3) * SK + i;
    split_one(x, o[0], o[SK], o[2 * SK]);
}

template <class Epi, int FN, bool SPLIT>
hipError_t launch(const Geom &g, const float *A, long M, const Epi &epi, hipStream_t st) {
    const long tiles = (M + SBM - 1) / SBM * ((g.N + 32 * FN - 1) / (32 * FN));
    if (tiles > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_dense_tall<Epi, FN, SPLIT>), dim3((unsigned)tiles), dim3(256), 0, st, g, A, M, epi);
    return hipGetLastError();
}

template <class Epi, bool SPLIT>
hipError_t run(const GeomSet &gs, const float *A, long M, const Epi &epi, hipStream_t st) {
    const Geom &g = gs.g[0];
    if (!is_dense(gs) || (SPLIT && !g.Bs) || !dma_fits(g)) return hipErrorInvalidValue;   // no weights it can read
    const int rem = g.N % 128;
    if (g.N <= 32) return launch<Epi, 1, SPLIT>(g, A, M, epi, st);
    // 64 columns where 128 would pad half a tile, and where 128 leave CUs without one of the
    // blocks that hide its chains: 128 / 64 columns, 256 x 256, 24576 rows (384 tiles) 41 / 36 us,
    // 49152 rows (768) 56 / 61; 512 x 512, 9216 rows (288) 56 / 50, 16384 rows (512) 64 / 68 (in
    // FP32 92 / 99); 256 x 784, 131072 rows (padding) 460 / 429
    const long tiles = (M + SBM - 1) / SBM * ((g.N + 127) / 128);
    if ((rem > 0 && rem <= 64) || tiles < 512) return launch<Epi, 2, SPLIT>(g, A, M, epi, st);
    return launch<Epi, 4, SPLIT>(g, A, M, epi, st);
}

}  // namespace

hipError_t tall_relax(const GeomSet &gs, const float *A, long M, const RelaxParams &p, hipStream_t st, bool split) {
    return split ? run<EpiRelax, true>(gs, A, M, EpiRelax{p}, st) : run<EpiRelax, false>(gs, A, M, EpiRelax{p}, st);
}
hipError_t tall_conc(const GeomSet &gs, const float *A, long M, const ConcParams &p, hipStream_t st, bool split) {
    return split ? run<EpiConc, true>(gs, A, M, EpiConc{p}, st) : run<EpiConc, false>(gs, A, M, EpiConc{p}, st);
}
hipError_t tall_adj(const GeomSet &gs, const float *A, long M, const AdjParams &p, hipStream_t st) {
    return run<EpiAdj, false>(gs, A, M, EpiAdj{p}, st);
}
hipError_t tall_fwd(const GeomSet &gs, const float *A, long M, const FwdParams &p, hipStream_t st) {
    return run<EpiFwd, false>(gs, A, M, EpiFwd{p}, st);
}

hipError_t launch_pack_split(const float *Bt, int Np, int Kp, int Kc, unsigned short *out, int32_t *flags,
                             hipStream_t st) {
    const long total = (long)Np * Kc * SK;
    hipLaunchKernelGGL(k_pack_split, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, Bt, Kp, Kc, total, out,
                       flags);
    return hipGetLastError();
}

}  // namespace bp
