// Branch and bound over input boxes on the GPU: the per-iteration steps of the planning
// loop (Algorithms 1-2) around the bound pass -- subdomain pick-out and split (the
// branching heuristics of Section 3.1, Eq. lf_pick), the search's sampling and summary
// (Section 3.3), the best-solution update and the pruner (Section 3).
//
// Large selections (pick-out over the whole candidate set, pruning) use device-wide radix
// sort / flagged selection (hipCUB over rocPRIM): stable, so equal keys keep index
// order.  Per-subdomain work (sorting a subdomain's samples, choosing its split
// dimension) runs one block per subdomain in LDS.
#include <hipcub/hipcub.hpp>

#include <cfloat>
#include <cmath>
#include <mutex>
#include <string>

#include "bound.h"
#include "bound_internal.h"

namespace bp {
bound_status set_error(bound_status s, const std::string &msg);   // api.hip
}

// Scratch of the allocation-free pruner (bound_bab_prune_noalloc): the per-block counts,
// then offsets, of up to 4096 blocks of 1024 subdomains (16 KiB).  Every GPU the library
// runs on holds its own copy until the process ends.  Host code passes the address that
// hipGetSymbolAddress returned for the current device, never the symbol itself (that is
// a host-side stand-in, not a device address).
static __device__ __align__(256) int32_t scratch[4096];

struct bound_bab {
    int max_dom = 0, dim = 0, max_samples = 0;
    float *keys = nullptr, *keys_out = nullptr;
    int32_t *vals = nullptr, *vals_out = nullptr;
    uint8_t *flag = nullptr;
    int32_t *count = nullptr;     // device scratch: selection count
    float *mm = nullptr;          // device scratch: min / max of the scaled keys
    void *tmp = nullptr;
    size_t tmp_bytes = 0;
    ~bound_bab() {
        for (void *p : {(void *)keys, (void *)keys_out, (void *)vals, (void *)vals_out,
                        (void *)flag, (void *)count, (void *)mm, tmp})
            if (p) (void)hipFree(p);
    }
};

namespace bp {
namespace {

constexpr int TPB = 256;
constexpr int MAX_SAMPLES = 2048;
inline unsigned blocks(long n) { return (unsigned)((n + TPB - 1) / TPB); }

// comparison key: -0 -> +0, NaN -> +inf
__device__ inline float canon(float x) { return x != x ? INFINITY : x + 0.0f; }

__global__ void k_iota_keys(int n, const float *src, float *keys, int32_t *vals) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        keys[i] = canon(src[i]);
        vals[i] = i;
    }
}

__global__ void k_fill_u8(int n, uint8_t *p, uint8_t v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// picked[off + t] = sorted[t], t < cnt; those subdomains are marked taken (flag = 0)
__global__ void k_take(int cnt, const int32_t *sorted, int32_t *picked, int off, uint8_t *flag) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < cnt) {
        const int i = sorted[t];
        picked[off + t] = i;
        flag[i] = 0;
    }
}

// min / max of the finite f_lo of the subdomains still available (one block)
__global__ void k_minmax(int n, const float *f_lo, const uint8_t *avail, float *mm) {
    __shared__ float smin[TPB], smax[TPB];
    float lo = INFINITY, hi = -INFINITY;
    for (int i = threadIdx.x; i < n; i += TPB) {
        const float v = f_lo[i];
        if (avail[i] && isfinite(v)) {
            lo = fminf(lo, v);
            hi = fmaxf(hi, v);
        }
    }
    smin[threadIdx.x] = lo;
    smax[threadIdx.x] = hi;
    __syncthreads();
    for (int s = TPB / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            smin[threadIdx.x] = fminf(smin[threadIdx.x], smin[threadIdx.x + s]);
            smax[threadIdx.x] = fmaxf(smax[threadIdx.x], smax[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        mm[0] = smin[0];
        mm[1] = smax[0];
    }
}

// Sort key of the softmax draw (ascending = pick first): s * fl(1/T) - g, each operation
// rounded in FP32, for available subdomains with finite f_lo; FLT_MAX for non-finite
// f_lo, +inf for taken ones.
__global__ void k_gumbel_keys(int n, const float *f_lo, const float *gum, const uint8_t *avail,
                              const float *mm, float inv_t, float *keys, int32_t *vals) {
#pragma clang fp contract(off)   // s * inv_t and the subtraction rounded separately
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    vals[i] = i;
    const float v = f_lo[i];
    if (!avail[i]) {
        keys[i] = INFINITY;
        return;
    }
    if (!isfinite(v)) {
        keys[i] = FLT_MAX;
        return;
    }
    const float lo = mm[0], hi = mm[1];
    const float s = hi > lo ? (v - lo) / (hi - lo) : 0.f;
    keys[i] = canon(s * inv_t - gum[i]);
}

__global__ void k_samples(long total, int M, int d, const float *lo, const float *hi,
                          const float *U, float *S) {
#pragma clang fp contract(off)   // three separately rounded operations, no fused multiply-add
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const long i = e / ((long)M * d);
    const int j = (int)(e % d);
    const float a = lo[i * d + j], b = hi[i * d + j];
    S[e] = a + (b - a) * U[e];
}

// Bitonic sort, by the whole block, of the (canonical value, index) pairs of v[0 .. M)
// in LDS (P2 = M rounded up to a power of two; the padding sorts last): ascending
// value, equal values by index.
__device__ void block_sort(const float *v, int M, int P2, float *sv, int *si) {
    for (int t = threadIdx.x; t < P2; t += TPB) {
        sv[t] = t < M ? canon(v[t]) : INFINITY;
        si[t] = t;
    }
    __syncthreads();
    for (int size = 2; size <= P2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = threadIdx.x; t < P2; t += TPB) {
                const int o = t ^ stride;
                if (o > t) {
                    const bool up = (t & size) == 0;
                    const float va = sv[t], vb = sv[o];
                    const int ia = si[t], ib = si[o];
                    const bool a_gt_b = va > vb || (va == vb && ia > ib);
                    if (a_gt_b == up) {
                        sv[t] = vb; sv[o] = va;
                        si[t] = ib; si[o] = ia;
                    }
                }
            }
            __syncthreads();
        }
    }
}

// One block per subdomain: its M samples sorted by value, then f_hi and the k best
// samples.
__global__ void k_search_summary(int M, int P2, int d, const float *values, const float *S, int k,
                                 float *f_hi, float *top) {
    __shared__ float sv[MAX_SAMPLES];
    __shared__ int si[MAX_SAMPLES];
    const long b = blockIdx.x;
    block_sort(values + b * M, M, P2, sv, si);
    if (threadIdx.x == 0) f_hi[b] = values[b * M + si[0]];
    for (long e = threadIdx.x; e < (long)k * d; e += TPB) {
        const int t = (int)(e / d), j = (int)(e - (long)t * d);
        top[(b * k + t) * d + j] = S[(b * M + si[t]) * d + j];
    }
}

// CEM start of box i: mu = u[i / u_div] if it lies in the box, else the centre;
// sigma = half the width.  One thread per box.
__global__ void k_cem_start(int n, int d, const float *lo, const float *hi, const float *u,
                            int u_div, float *mu, float *sigma) {
#pragma clang fp contract(off)
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float *p = u ? u + (long)(i / u_div) * d : nullptr;
    bool in = p != nullptr;
    for (int j = 0; j < d && in; ++j) in = p[j] >= lo[(long)i * d + j] && p[j] <= hi[(long)i * d + j];
    for (int j = 0; j < d; ++j) {
        const float a = lo[(long)i * d + j], c = hi[(long)i * d + j];
        mu[(long)i * d + j] = in ? p[j] : (a + c) * 0.5f;
        sigma[(long)i * d + j] = (c - a) * 0.5f;
    }
}

// One CEM round's samples (and their copy into the round's slice of the archive).
__global__ void k_cem_samples(long total, int M, int d, const float *lo, const float *hi,
                              const float *mu, const float *sigma, const float *Z, float *S,
                              float *arch, int ld, int a0) {
#pragma clang fp contract(off)   // the product and the sum rounded separately (plain
                                 // operators: the header's __fmul_rn / __fadd_rn may fuse)
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const long i = e / ((long)M * d);
    const int r = (int)(e - i * M * d), m = r / d, j = r - m * d;
    const long o = i * d + j;
    const float u = mu[o] + sigma[o] * Z[e];
    const float v = fminf(fmaxf(u, lo[o]), hi[o]);
    S[e] = v;
    if (arch) arch[((i * ld) + a0 + m) * d + j] = v;
}

// One block per box: the round's values sorted, then mean and deviation of the n_elite
// best samples per coordinate, summed in elite order.
__global__ void k_cem_refit(int M, int P2, int d, const float *values, const float *S, int E,
                            float jitter, float *mu, float *sigma, float *arch_v, int ld, int a0) {
#pragma clang fp contract(off)
    __shared__ float sv[MAX_SAMPLES];
    __shared__ int si[MAX_SAMPLES];
    const long b = blockIdx.x;
    block_sort(values + b * M, M, P2, sv, si);
    const float rE = (float)E;
    for (int j = threadIdx.x; j < d; j += TPB) {
        float s = 0.f;
        for (int r = 0; r < E; ++r) s += S[(b * M + si[r]) * d + j];
        const float m = s / rE;
        float q = 0.f;
        for (int r = 0; r < E; ++r) {
            const float dv = S[(b * M + si[r]) * d + j] - m;
            q += dv * dv;
        }
        mu[b * d + j] = m;
        sigma[b * d + j] = sqrtf(q / rE) + jitter;
    }
    if (arch_v)
        for (int t = threadIdx.x; t < M; t += TPB) arch_v[b * ld + a0 + t] = values[b * M + t];
}

// One block per subdomain: split dimension and the two children.
__global__ void k_split(int d, const float *lo, const float *hi, const float *top, int k,
                        float *clo, float *chi, int32_t *dim_out) {
    __shared__ float sbest[TPB], wbest[TPB];
    __shared__ int jbest[TPB], jw[TPB];
    const long b = blockIdx.x;
    float bs = -1.f, bw = -1.f;
    int bj = 0x7fffffff, bjw = 0x7fffffff;
    for (int j = threadIdx.x; j < d; j += TPB) {
        const float a = lo[b * d + j], c = hi[b * d + j];
        const float mid = __fmul_rn(__fadd_rn(a, c), 0.5f);
        int nlo = 0;
        for (int t = 0; t < k; ++t) nlo += top[(b * k + t) * d + j] <= mid ? 1 : 0;
        const int diff = nlo - (k - nlo);
        const float width = __fsub_rn(c, a);
        const float score = __fmul_rn(width, (float)(diff < 0 ? -diff : diff));
        if (score > bs) { bs = score; bj = j; }          // j ascending per thread
        if (width > bw) { bw = width; bjw = j; }
    }
    sbest[threadIdx.x] = bs; jbest[threadIdx.x] = bj;
    wbest[threadIdx.x] = bw; jw[threadIdx.x] = bjw;
    __syncthreads();
    for (int s = TPB / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            const int o = threadIdx.x + s;
            if (sbest[o] > sbest[threadIdx.x] ||
                (sbest[o] == sbest[threadIdx.x] && jbest[o] < jbest[threadIdx.x])) {
                sbest[threadIdx.x] = sbest[o];
                jbest[threadIdx.x] = jbest[o];
            }
            if (wbest[o] > wbest[threadIdx.x] ||
                (wbest[o] == wbest[threadIdx.x] && jw[o] < jw[threadIdx.x])) {
                wbest[threadIdx.x] = wbest[o];
                jw[threadIdx.x] = jw[o];
            }
        }
        __syncthreads();
    }
    const int js = sbest[0] > 0.f ? jbest[0] : jw[0];
    for (int j = threadIdx.x; j < d; j += TPB) {
        const float a = lo[b * d + j], c = hi[b * d + j];
        const float mid = __fmul_rn(__fadd_rn(a, c), 0.5f);
        clo[(2 * b) * d + j] = a;
        chi[(2 * b) * d + j] = j == js ? mid : c;
        clo[(2 * b + 1) * d + j] = j == js ? mid : a;
        chi[(2 * b + 1) * d + j] = c;
    }
    if (threadIdx.x == 0 && dim_out) dim_out[b] = js;
}

// one block: argmin of f_hi (ties: lower index); strict improvement updates the best
__global__ void k_update_best(int n, const float *f_hi, const float *top, int k, int d, float *best,
                              float *u_best) {
    __shared__ float sv[TPB];
    __shared__ int si[TPB];
    float v = INFINITY;
    int idx = 0x7fffffff;
    for (int i = threadIdx.x; i < n; i += TPB) {
        const float x = canon(f_hi[i]);
        if (x < v) { v = x; idx = i; }
    }
    sv[threadIdx.x] = v;
    si[threadIdx.x] = idx;
    __syncthreads();
    for (int s = TPB / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            const int o = threadIdx.x + s;
            if (sv[o] < sv[threadIdx.x] || (sv[o] == sv[threadIdx.x] && si[o] < si[threadIdx.x])) {
                sv[threadIdx.x] = sv[o];
                si[threadIdx.x] = si[o];
            }
        }
        __syncthreads();
    }
    const bool better = si[0] < n && sv[0] < canon(*best);
    __syncthreads();
    if (!better) return;
    const int i = si[0];
    for (int j = threadIdx.x; j < d; j += TPB) u_best[j] = top[((long)i * k) * d + j];
    if (threadIdx.x == 0) *best = f_hi[i];
}

__global__ void k_zero_i32(int32_t *p) { *p = 0; }

__global__ void k_prune_flags(int n, const float *f_lo, const float *best, uint8_t *flag) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) flag[i] = canon(f_lo[i]) <= canon(*best) ? 1 : 0;
}

// ---- pruner without allocation: stable compaction through per-block counts.
// Block b of the count and scatter kernels covers subdomains [b * PRUNE_TILE, ...);
// the scan kernel turns the block counts into block offsets and writes the total.
constexpr int PRUNE_TILE = 1024;                  // subdomains per block (4 per thread)
constexpr int PRUNE_MAX_BLOCKS = 4096;
constexpr long PRUNE_MAX_N = (long)PRUNE_TILE * PRUNE_MAX_BLOCKS;
static_assert(PRUNE_MAX_BLOCKS == sizeof(::scratch) / sizeof(int32_t), "scratch holds the block counts");

__device__ inline bool kept(const float *f_lo, int i, float b) { return canon(f_lo[i]) <= b; }

__global__ __launch_bounds__(TPB) void k_prune_count(int n, const float *f_lo, const float *best,
                                                     int32_t *counts) {
    __shared__ int wsum[TPB / 64];
    const float b = canon(*best);
    const int i0 = blockIdx.x * PRUNE_TILE;
    int c = 0;
    for (int t = threadIdx.x; t < PRUNE_TILE; t += TPB) {
        const int i = i0 + t;
        c += (i < n && kept(f_lo, i, b)) ? 1 : 0;
    }
    for (int m = 1; m < 64; m <<= 1) c += __shfl_xor(c, m, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int s = 0;
        for (int w = 0; w < TPB / 64; ++w) s += wsum[w];
        counts[blockIdx.x] = s;
    }
}

// One block: exclusive scan of nb block counts in place, total to *n_keep.
__global__ __launch_bounds__(TPB) void k_prune_scan(int nb, int32_t *counts, int32_t *n_keep) {
    __shared__ int part[TPB];
    const int per = (nb + TPB - 1) / TPB, a = threadIdx.x * per;
    int s = 0;
    for (int k = 0; k < per && a + k < nb; ++k) s += counts[a + k];
    part[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int t = 0; t < TPB; ++t) {
            const int v = part[t];
            part[t] = run;
            run += v;
        }
        *n_keep = run;
    }
    __syncthreads();
    int run = part[threadIdx.x];
    for (int k = 0; k < per && a + k < nb; ++k) {
        const int v = counts[a + k];
        counts[a + k] = run;
        run += v;
    }
}

// Block b writes its kept subdomains, in index order, from offset counts[b] on: the
// rank of a kept subdomain inside the block is the number of kept ones before it (wave
// ballots, then the waves' and rounds' totals through LDS).
__global__ __launch_bounds__(TPB) void k_prune_scatter(int n, const float *f_lo, const float *best,
                                                       const int32_t *offsets, int32_t *keep) {
    __shared__ int wcnt[PRUNE_TILE / 64];
    const float b = canon(*best);
    const int i0 = blockIdx.x * PRUNE_TILE, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    bool f[PRUNE_TILE / TPB];
    uint64_t m[PRUNE_TILE / TPB];
#pragma unroll
    for (int r = 0; r < PRUNE_TILE / TPB; ++r) {   // round r covers [r * TPB, (r + 1) * TPB)
        const int i = i0 + r * TPB + threadIdx.x;
        f[r] = i < n && kept(f_lo, i, b);
        m[r] = __ballot(f[r]);
        if (lane == 0) wcnt[r * (TPB / 64) + w] = __popcll(m[r]);
    }
    __syncthreads();
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int base = offsets[blockIdx.x];
#pragma unroll
    for (int r = 0; r < PRUNE_TILE / TPB; ++r) {
        // kept subdomains of the (round, wave) segments before this one
        int before = base;
        for (int s = 0; s < r * (TPB / 64) + w; ++s) before += wcnt[s];
        if (f[r]) keep[before + __popcll(m[r] & below)] = i0 + r * TPB + threadIdx.x;
    }
}

// ---- pick-out and pruning of up to ONE_MAX subdomains by one block.  Wave w holds the
// subdomains from w * 64 * rounds on, round it's lane l the one at 64 it + l; flags of them
// are bits of a word per lane, and their keys stay in registers over the whole selection: a
// device-wide sort of 60000 pairs takes a dozen dependent launches for the same picks.  What
// bounds it is the one unit's instruction rate, and its LDS in the histograms, where every
// lane has 16-bit counters of its own: the leading byte of FP32 keys takes few values, and a
// shared bin would serialise the wave.  Pick-out of 1024 from 60000, split, best and pruner:
// 223 -> 148 us (keys in memory and one histogram: 200 us).  Larger sets and picks keep the
// device-wide sort: see pick_one_fits.
constexpr int ONE_T = 1024, ONE_PER = 64, ONE_MAX = ONE_T * ONE_PER, ONE_SORT = 2048;

// order-preserving bits of a comparison key
__device__ inline unsigned order_bits(float x) {
    const unsigned u = __float_as_uint(canon(x));
    return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}

struct OneShared {
    union {
        unsigned hist[128 * 64];                // [bin / 2][lane], two 16-bit counters (<= 1024)
        unsigned long long sort[ONE_SORT];
    };
    int wave[ONE_T / 64];
    float fmin[ONE_T / 64], fmax[ONE_T / 64];
    int bin, less, n;
};

// Exclusive scan over the block of one value per thread.
__device__ inline int block_scan(OneShared &sh, int v, int &total) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    if (lane == 63) sh.wave[wv] = incl;
    __syncthreads();
    int before = 0;
    total = 0;
    for (int w = 0; w < ONE_T / 64; ++w) {
        if (w < wv) before += sh.wave[w];
        total += sh.wave[w];
    }
    __syncthreads();
    return before + incl - v;
}

// A wave's first subdomain, of n in rounds of 64 a wave.
__device__ inline int one_first(int rounds) { return (int)(threadIdx.x >> 6) * 64 * rounds + (threadIdx.x & 63); }

// Positions, in index order, of the flagged subdomains (bit `it` of flags): calls
// put(it, position) for each; returns how many there are.
template <class Put> __device__ inline int ordered(OneShared &sh, unsigned long long flags, Put put) {
    const int lane = threadIdx.x & 63;
    int total, pos = block_scan(sh, __popcll(flags), total);
    pos = __builtin_amdgcn_readfirstlane(pos);                  // the wave's first position
    unsigned lo = (unsigned)flags, hi = (unsigned)(flags >> 32);
    for (int m = 1; m < 64; m <<= 1) {
        lo |= __shfl_xor(lo, m, 64);
        hi |= __shfl_xor(hi, m, 64);
    }
    const unsigned long long below = lane ? (~0ull >> (64 - lane)) : 0ull;
    // the rounds in which any lane has a flag
    unsigned long long any = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(hi) << 32) |
                             (unsigned)__builtin_amdgcn_readfirstlane(lo);
    for (; any; any &= any - 1) {
        const int it = __builtin_ctzll(any);
        const bool f = (flags >> it) & 1;
        const unsigned long long m = __ballot(f);
        if (f) put(it, pos + __popcll(m & below));
        pos += __popcll(m);
    }
    return total;
}

// The want (<= ONE_SORT) smallest (key, index) pairs, ascending, to out; taken gets their
// bits.  At least want keys are below ONE_NONE, which stands for no subdomain (comparison
// keys end at +inf).  Radix selection of the want-th key, a byte a pass, then a bitonic sort
// of the selected.
constexpr unsigned ONE_NONE = 0xffffffffu;
template <int PER>
__device__ void one_select(OneShared &sh, const unsigned (&key)[PER], int rounds, int want, int32_t *out,
                           unsigned long long &taken) {
    const int tid = threadIdx.x, lane = tid & 63;
    unsigned prefix = 0, mask = 0;
    int need = want;
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int q = tid; q < 128 * 64; q += ONE_T) sh.hist[q] = 0;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < PER; ++it)
            if ((key[it] & mask) == prefix) {
                const unsigned bin = (key[it] >> shift) & 255;
                atomicAdd(&sh.hist[(bin >> 1) * 64 + lane], bin & 1 ? 1u << 16 : 1u);
            }
        __syncthreads();
        // eight threads a pair of bins; the rotation spreads a wave's eight pairs over the banks
        const int pair = tid >> 3;
        int h0 = 0, h1 = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const unsigned c = sh.hist[pair * 64 + (tid & 7) * 8 + ((i + pair) & 7)];
            h0 += c & 0xffff;
            h1 += c >> 16;
        }
#pragma unroll
        for (int m = 1; m < 8; m <<= 1) {
            h0 += __shfl_xor(h0, m, 64);
            h1 += __shfl_xor(h1, m, 64);
        }
        int total;
        const int before = block_scan(sh, tid & 7 ? 0 : h0 + h1, total);
        if ((tid & 7) == 0 && before < need && need <= before + h0 + h1) {
            const bool second = need > before + h0;
            sh.bin = 2 * pair + (second ? 1 : 0);
            sh.less = before + (second ? h0 : 0);
        }
        __syncthreads();
        prefix |= (unsigned)sh.bin << shift;
        mask |= 255u << shift;
        need -= sh.less;
    }
    // keys below the want-th, and the first `need` in index order of those equal to it
    unsigned long long sel = 0, eq = 0;
#pragma unroll
    for (int it = 0; it < PER; ++it) {
        sel |= key[it] < prefix ? 1ull << it : 0;
        eq |= key[it] == prefix ? 1ull << it : 0;
    }
    ordered(sh, eq, [&](int it, int pos) {
        if (pos < need) sel |= 1ull << it;
    });
    int P2 = 1;
    while (P2 < want) P2 <<= 1;
    for (int q = want + tid; q < P2; q += ONE_T) sh.sort[q] = ~0ull;
    if (tid == 0) sh.n = 0;
    __syncthreads();
    // one atomic a thread reserves its places; the sort puts them in order
    int at = sel ? atomicAdd(&sh.n, __popcll(sel)) : 0;
#pragma unroll
    for (int it = 0; it < PER; ++it)
        if ((sel >> it) & 1) sh.sort[at++] = ((unsigned long long)key[it] << 32) | (unsigned)(one_first(rounds) + it * 64);
    __syncthreads();
    if (P2 <= ONE_T) {
        // an element a thread: strides inside a wave are register exchanges
        unsigned long long x = tid < P2 ? sh.sort[tid] : ~0ull;
        for (int size = 2; size <= P2; size <<= 1)
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                unsigned long long y;
                if (stride >= 64) {
                    if (tid < P2) sh.sort[tid] = x;
                    __syncthreads();
                    y = tid < P2 ? sh.sort[tid ^ stride] : x;
                    __syncthreads();
                } else {
                    y = __shfl_xor(x, stride, 64);
                }
                const bool up = (tid & size) == 0, lower = (tid & stride) == 0;
                if ((x > y) == (up == lower)) x = y;
            }
        if (tid < want) out[tid] = (int32_t)(unsigned)x;
    } else {
        for (int size = 2; size <= P2; size <<= 1)
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int q = tid; q < P2 / 2; q += ONE_T) {
                    const int a = 2 * q - (q & (stride - 1)), c = a + stride;
                    const unsigned long long x = sh.sort[a], y = sh.sort[c];
                    if ((x > y) == ((a & size) == 0)) {
                        sh.sort[a] = y;
                        sh.sort[c] = x;
                    }
                }
                __syncthreads();
            }
        for (int q = tid; q < want; q += ONE_T) out[q] = (int32_t)(unsigned)sh.sort[q];
    }
    __syncthreads();
    taken |= sel;
}

template <int PER>
__global__ __launch_bounds__(ONE_T) void k_pick_one(int n_dom, int n1, int n, const float *f_lo,
                                                    const float *f_hi, const float *gum, float inv_t,
                                                    int32_t *picked, int32_t *rest) {
#pragma clang fp contract(off)   // s * inv_t and the subtraction rounded separately
    __shared__ OneShared sh;
    const int tid = threadIdx.x, rounds = (n_dom + ONE_T - 1) / ONE_T;   // <= PER
    unsigned long long all = 0, taken = 0;
    const int i0 = one_first(rounds);
    for (int it = 0; it < rounds; ++it)
        if (i0 + it * 64 < n_dom) all |= 1ull << it;
    // clamped loads in batches, so that no branch and no wait stands between those of a batch
    auto at = [&](int it, int i) { return (unsigned)(i + it * 64 < n_dom ? i + it * 64 : n_dom - 1); };
    // a value anew for each batch: indices and masks kept from one use to the next would push
    // the keys out of the registers
    auto fresh = [](auto v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    constexpr int NB = PER < 16 ? PER : 16;
    unsigned key[PER];
    if (n1 > 0) {
#pragma unroll
        for (int r0 = 0; r0 < PER; r0 += NB) {
            const int i = fresh(i0);
            const unsigned long long avail = fresh(all);
            float v[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q) v[q] = f_hi[at(r0 + q, i)];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < NB; ++q) key[r0 + q] = (avail >> (r0 + q)) & 1 ? order_bits(v[q]) : ONE_NONE;
        }
        one_select(sh, key, rounds, n1, picked, taken);
    }
    if (n > n1) {
        float lo = INFINITY, hi = -INFINITY;
#pragma unroll
        for (int r0 = 0; r0 < PER; r0 += NB) {
            const int i = fresh(i0);
            const unsigned long long avail = fresh(all & ~taken);
#pragma unroll
            for (int q = 0; q < NB; ++q) key[r0 + q] = __float_as_uint(f_lo[at(r0 + q, i)]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const float v = __uint_as_float(key[r0 + q]);
                if (isfinite(v) && ((avail >> (r0 + q)) & 1)) {
                    lo = fminf(lo, v);
                    hi = fmaxf(hi, v);
                }
            }
        }
        for (int m = 1; m < 64; m <<= 1) {
            lo = fminf(lo, __shfl_xor(lo, m, 64));
            hi = fmaxf(hi, __shfl_xor(hi, m, 64));
        }
        if ((tid & 63) == 0) {
            sh.fmin[tid >> 6] = lo;
            sh.fmax[tid >> 6] = hi;
        }
        __syncthreads();
        for (int w = 0; w < ONE_T / 64; ++w) {
            lo = fminf(lo, sh.fmin[w]);
            hi = fmaxf(hi, sh.fmax[w]);
        }
#pragma unroll
        for (int r0 = 0; r0 < PER; r0 += NB) {
            const int i = fresh(i0);
            const unsigned long long avail = fresh(all & ~taken);
            float gv[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q) gv[q] = gum[at(r0 + q, i)];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const float v = __uint_as_float(key[r0 + q]);
                float k = FLT_MAX;                       // non-finite f_lo comes last
                if (isfinite(v)) {
                    const float s = hi > lo ? (v - lo) / (hi - lo) : 0.f;
                    k = canon(s * inv_t - gv[q]);
                }
                key[r0 + q] = (avail >> (r0 + q)) & 1 ? order_bits(k) : ONE_NONE;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        one_select(sh, key, rounds, n - n1, picked + n1, taken);
    }
    if (n_dom > n) ordered(sh, all & ~taken, [&](int it, int pos) { rest[pos] = i0 + it * 64; });
}

__global__ __launch_bounds__(ONE_T) void k_prune_one(int n, const float *f_lo, const float *best, int32_t *keep,
                                                     int32_t *n_keep) {
    __shared__ OneShared sh;
    const int tid = threadIdx.x, rounds = (n + ONE_T - 1) / ONE_T, i0 = one_first(rounds);
    const float b = canon(*best);
    unsigned long long f = 0;
#pragma unroll 8
    for (int it = 0; it < rounds; ++it) {
        const int i = i0 + it * 64;
        if (i < n && kept(f_lo, i, b)) f |= 1ull << it;
    }
    const int total = ordered(sh, f, [&](int it, int pos) { keep[pos] = i0 + it * 64; });
    if (tid == 0) *n_keep = total;
}

std::mutex g_scratch_mu;
int32_t *g_scratch_ptr[64] = {};   // per device: the address of `scratch` on that GPU

hipError_t sort_pairs(bound_bab *b, int n, hipStream_t st) {
    size_t bytes = b->tmp_bytes;
    return hipcub::DeviceRadixSort::SortPairs(b->tmp, bytes, b->keys, b->keys_out, b->vals,
                                              b->vals_out, n, 0, 32, st);
}

hipError_t select_flagged(bound_bab *b, int n, int32_t *out, int32_t *n_out, hipStream_t st) {
    size_t bytes = b->tmp_bytes;
    hipcub::CountingInputIterator<int32_t> it(0);
    return hipcub::DeviceSelect::Flagged(b->tmp, bytes, it, b->flag, out, n_out, n, st);
}

}  // namespace

// One block or the device-wide sort (which takes a dozen launches, but is bound by no single
// unit).  us, device-wide / one block, eta = 0.75 and 1: 60000 subdomains, 1024 picks 205 / 134;
// 8192, 2048 90 / 54 and 44 / 35; 8192, 6000 90 / 100; 8193, 5461 90 / 101 -- a phase of more than
// 2048 picks sorts in LDS behind a barrier a stride.  Few or very many subdomains leave less to
// gain: 4096, 3072 63 / 70; 32769, 3072 149 / 158.  With all picked the device-wide path has no
// rest to list (1000, 1000 30 / 38), and with phase 1 alone it has one sort: 32768, 2048 54 / 45,
// 32769, 2048 55 / 78.
bool pick_one_fits(int n_dom, int n, int n1) {
    return n_dom <= ONE_MAX && n < n_dom && n1 <= ONE_SORT && n - n1 <= ONE_SORT &&
           (n <= ONE_SORT || (n_dom > 4096 && n_dom <= 32768)) && (n_dom <= 32768 || n > n1);
}
}  // namespace bp

using bp::set_error;

#define BCHK(x)                                                                         \
    do {                                                                                \
        hipError_t e_ = (x);                                                            \
        if (e_ != hipSuccess) return set_error(BOUND_E_HIP, std::string(#x ": ") + hipGetErrorString(e_)); \
    } while (0)

extern "C" {

bound_status bound_bab_init(int32_t max_dom, int32_t dim, int32_t max_samples, bound_bab **out) {
    if (!out || max_dom < 1 || dim < 1 || max_samples < 1 || max_samples > bp::MAX_SAMPLES)
        return set_error(BOUND_E_ARG, "bound_bab_init: need max_dom, dim >= 1 and 1 <= max_samples <= 2048");
    *out = nullptr;
    bound_bab *b = new bound_bab();
    b->max_dom = max_dom;
    b->dim = dim;
    b->max_samples = max_samples;
    size_t s1 = 0, s2 = 0;
    hipcub::CountingInputIterator<int32_t> it(0);
    bool ok = hipcub::DeviceRadixSort::SortPairs(nullptr, s1, b->keys, b->keys_out, b->vals,
                                                 b->vals_out, max_dom, 0, 32) == hipSuccess &&
              hipcub::DeviceSelect::Flagged(nullptr, s2, it, b->flag, b->vals, b->count,
                                            max_dom) == hipSuccess;
    b->tmp_bytes = s1 > s2 ? s1 : s2;
    ok = ok && hipMalloc(&b->keys, sizeof(float) * max_dom) == hipSuccess &&
         hipMalloc(&b->keys_out, sizeof(float) * max_dom) == hipSuccess &&
         hipMalloc(&b->vals, sizeof(int32_t) * max_dom) == hipSuccess &&
         hipMalloc(&b->vals_out, sizeof(int32_t) * max_dom) == hipSuccess &&
         hipMalloc(&b->flag, max_dom) == hipSuccess &&
         hipMalloc(&b->count, sizeof(int32_t)) == hipSuccess &&
         hipMalloc(&b->mm, 2 * sizeof(float)) == hipSuccess &&
         hipMalloc(&b->tmp, b->tmp_bytes > 0 ? b->tmp_bytes : 1) == hipSuccess;
    if (!ok) {
        delete b;
        return set_error(BOUND_E_NOMEM, "bound_bab_init: device allocation");
    }
    *out = b;
    return BOUND_OK;
}

void bound_bab_destroy(bound_bab *b) { delete b; }

bound_status bound_bab_pick_out(bound_bab *b, int32_t n_dom, const float *f_lo, const float *f_hi,
                                const float *g, int32_t n_pick, float eta, float temperature,
                                int32_t *picked, int32_t *rest, void *stream) {
    if (!b || n_dom < 0 || n_dom > b->max_dom || n_pick < 0 || !(eta >= 0.f && eta <= 1.f) ||
        !(temperature > 0.f) || !(1.0f / temperature < FLT_MAX) ||
        (n_dom > 0 && (!f_lo || !f_hi || !g || !picked || !rest)))
        return set_error(BOUND_E_ARG, "bound_bab_pick_out: bad arguments");
    if (n_dom == 0) return BOUND_OK;
    hipStream_t st = (hipStream_t)stream;
    const int n = n_pick < n_dom ? n_pick : n_dom;
    const int n1 = (int)std::floor((double)eta * (double)n);
    if (bp::pick_one_fits(n_dom, n, n1)) {
        const auto f = n_dom <= 8 * bp::ONE_T    ? bp::k_pick_one<8>
                       : n_dom <= 32 * bp::ONE_T ? bp::k_pick_one<32>
                                                 : bp::k_pick_one<bp::ONE_PER>;
        hipLaunchKernelGGL(f, dim3(1), dim3(bp::ONE_T), 0, st, n_dom, n1, n, f_lo, f_hi, g, 1.0f / temperature,
                           picked, rest);
        BCHK(hipGetLastError());
        return BOUND_OK;
    }
    hipLaunchKernelGGL(bp::k_fill_u8, dim3(bp::blocks(n_dom)), dim3(bp::TPB), 0, st, n_dom, b->flag,
                       (uint8_t)1);
    if (n1 > 0) {
        hipLaunchKernelGGL(bp::k_iota_keys, dim3(bp::blocks(n_dom)), dim3(bp::TPB), 0, st, n_dom, f_hi,
                           b->keys, b->vals);
        BCHK(bp::sort_pairs(b, n_dom, st));
        hipLaunchKernelGGL(bp::k_take, dim3(bp::blocks(n1)), dim3(bp::TPB), 0, st, n1, b->vals_out,
                           picked, 0, b->flag);
    }
    if (n - n1 > 0) {
        hipLaunchKernelGGL(bp::k_minmax, dim3(1), dim3(bp::TPB), 0, st, n_dom, f_lo, b->flag, b->mm);
        hipLaunchKernelGGL(bp::k_gumbel_keys, dim3(bp::blocks(n_dom)), dim3(bp::TPB), 0, st, n_dom,
                           f_lo, g, b->flag, b->mm, 1.0f / temperature, b->keys, b->vals);
        BCHK(bp::sort_pairs(b, n_dom, st));
        hipLaunchKernelGGL(bp::k_take, dim3(bp::blocks(n - n1)), dim3(bp::TPB), 0, st, n - n1,
                           b->vals_out, picked, n1, b->flag);
    }
    if (n_dom - n > 0) BCHK(bp::select_flagged(b, n_dom, rest, b->count, st));
    BCHK(hipGetLastError());
    return BOUND_OK;
}

bound_status bound_bab_samples(bound_bab *b, int32_t n, int32_t M, const float *lo, const float *hi,
                               const float *U, float *samples, void *stream) {
    if (!b || n < 0 || M < 1 || (n > 0 && (!lo || !hi || !U || !samples)))
        return set_error(BOUND_E_ARG, "bound_bab_samples: bad arguments");
    const long total = (long)n * M * b->dim;
    if (total == 0) return BOUND_OK;
    hipLaunchKernelGGL(bp::k_samples, dim3(bp::blocks(total)), dim3(bp::TPB), 0, (hipStream_t)stream,
                       total, M, b->dim, lo, hi, U, samples);
    BCHK(hipGetLastError());
    return BOUND_OK;
}

bound_status bound_bab_search_summary(bound_bab *b, int32_t n, int32_t M, const float *values,
                                      const float *samples, int32_t k, float *f_hi, float *top,
                                      void *stream) {
    if (!b || n < 0 || M < 1 || M > b->max_samples || k < 1 || k > M ||
        (n > 0 && (!values || !samples || !f_hi || !top)))
        return set_error(BOUND_E_ARG, "bound_bab_search_summary: bad arguments");
    if (n == 0) return BOUND_OK;
    int P2 = 1;
    while (P2 < M) P2 <<= 1;
    hipLaunchKernelGGL(bp::k_search_summary, dim3(n), dim3(bp::TPB), 0, (hipStream_t)stream, M, P2,
                       b->dim, values, samples, k, f_hi, top);
    BCHK(hipGetLastError());
    return BOUND_OK;
}

bound_status bound_bab_split(bound_bab *b, int32_t n, const float *lo, const float *hi,
                             const float *top, int32_t k, float *child_lo, float *child_hi,
                             int32_t *split_dim, void *stream) {
    if (!b || n < 0 || k < 1 || (n > 0 && (!lo || !hi || !top || !child_lo || !child_hi)))
        return set_error(BOUND_E_ARG, "bound_bab_split: bad arguments");
    if (n == 0) return BOUND_OK;
    hipLaunchKernelGGL(bp::k_split, dim3(n), dim3(bp::TPB), 0, (hipStream_t)stream, b->dim, lo, hi,
                       top, k, child_lo, child_hi, split_dim);
    BCHK(hipGetLastError());
    return BOUND_OK;
}

bound_status bound_bab_cem_start(bound_bab *b, int32_t n, const float *lo, const float *hi,
                                 const float *u, int32_t u_div, float *mu, float *sigma, void *stream) {
    if (!b || n < 0 || u_div < 1 || (n > 0 && (!lo || !hi || !mu || !sigma)))
        return set_error(BOUND_E_ARG, "bound_bab_cem_start: bad arguments");
    if (n == 0) return BOUND_OK;
    hipLaunchKernelGGL(bp::k_cem_start, dim3(bp::blocks(n)), dim3(bp::TPB), 0, (hipStream_t)stream,
                       n, b->dim, lo, hi, u, u_div, mu, sigma);
    BCHK(hipGetLastError());
    return BOUND_OK;
}

bound_status bound_bab_cem_samples(bound_bab *b, int32_t n, int32_t M, const float *lo, const float *hi,
                                   const float *mu, const float *sigma, const float *Z, float *samples,
                                   float *archive, int32_t ld, int32_t a0, void *stream) {
    if (!b || n < 0 || M < 1 || (archive && (a0 < 0 || (long)a0 + M > ld)) ||
        (n > 0 && (!lo || !hi || !mu || !sigma || !Z || !samples)))
        return set_error(BOUND_E_ARG, "bound_bab_cem_samples: bad arguments");
    const long total = (long)n * M * b->dim;
    if (total == 0) return BOUND_OK;
    hipLaunchKernelGGL(bp::k_cem_samples, dim3(bp::blocks(total)), dim3(bp::TPB), 0, (hipStream_t)stream,
                       total, M, b->dim, lo, hi, mu, sigma, Z, samples, archive, ld, a0);
    BCHK(hipGetLastError());
    return BOUND_OK;
}

bound_status bound_bab_cem_refit(bound_bab *b, int32_t n, int32_t M, const float *values,
                                 const float *samples, int32_t n_elite, float jitter, float *mu,
                                 float *sigma, float *archive_values, int32_t ld, int32_t a0,
                                 void *stream) {
    if (!b || n < 0 || M < 1 || M > b->max_samples || n_elite < 1 || n_elite > M ||
        !(jitter >= 0.f) || (archive_values && (a0 < 0 || (long)a0 + M > ld)) ||
        (n > 0 && (!values || !samples || !mu || !sigma)))
        return set_error(BOUND_E_ARG, "bound_bab_cem_refit: bad arguments");
    if (n == 0) return BOUND_OK;
    int P2 = 1;
    while (P2 < M) P2 <<= 1;
    hipLaunchKernelGGL(bp::k_cem_refit, dim3(n), dim3(bp::TPB), 0, (hipStream_t)stream, M, P2, b->dim,
                       values, samples, n_elite, jitter, mu, sigma, archive_values, ld, a0);
    BCHK(hipGetLastError());
    return BOUND_OK;
}

bound_status bound_bab_update_best(bound_bab *b, int32_t n, const float *f_hi, const float *top,
                                   int32_t k, float *best, float *u_best, void *stream) {
    if (!b || n < 0 || k < 1 || !best || !u_best || (n > 0 && (!f_hi || !top)))
        return set_error(BOUND_E_ARG, "bound_bab_update_best: bad arguments");
    if (n == 0) return BOUND_OK;
    hipLaunchKernelGGL(bp::k_update_best, dim3(1), dim3(bp::TPB), 0, (hipStream_t)stream, n, f_hi,
                       top, k, b->dim, best, u_best);
    BCHK(hipGetLastError());
    return BOUND_OK;
}

bound_status bound_bab_prune_noalloc(int32_t n, const float *f_lo, const float *best, int32_t *keep,
                                     int32_t *n_keep, void *stream) {
    if (n < 0 || (long)n > bp::PRUNE_MAX_N || !best || !n_keep || (n > 0 && (!f_lo || !keep)))
        return set_error(BOUND_E_ARG, "bound_bab_prune_noalloc: bad arguments (need 0 <= n <= " +
                                          std::to_string(bp::PRUNE_MAX_N) + ")");
    int dev = 0;
    BCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return set_error(BOUND_E_ARG, "bound_bab_prune_noalloc: device id");
    int32_t *scr;
    {
        std::lock_guard<std::mutex> lk(bp::g_scratch_mu);
        if (!bp::g_scratch_ptr[dev]) {
            void *p = nullptr;
            BCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
            bp::g_scratch_ptr[dev] = (int32_t *)p;
        }
        scr = bp::g_scratch_ptr[dev];
    }
    hipStream_t st = (hipStream_t)stream;
    if (n == 0) {
        hipLaunchKernelGGL(bp::k_zero_i32, dim3(1), dim3(1), 0, st, n_keep);
        BCHK(hipGetLastError());
        return BOUND_OK;
    }
    const int nb = (int)((n + bp::PRUNE_TILE - 1) / bp::PRUNE_TILE);
    hipLaunchKernelGGL(bp::k_prune_count, dim3(nb), dim3(bp::TPB), 0, st, n, f_lo, best, scr);
    hipLaunchKernelGGL(bp::k_prune_scan, dim3(1), dim3(bp::TPB), 0, st, nb, scr, n_keep);
    hipLaunchKernelGGL(bp::k_prune_scatter, dim3(nb), dim3(bp::TPB), 0, st, n, f_lo, best, scr, keep);
    BCHK(hipGetLastError());
    return BOUND_OK;
}

bound_status bound_bab_prune(bound_bab *b, int32_t n, const float *f_lo, const float *best,
                             int32_t *keep, int32_t *n_keep, void *stream) {
    if (!b || n < 0 || n > b->max_dom || !best || !n_keep || (n > 0 && (!f_lo || !keep)))
        return set_error(BOUND_E_ARG, "bound_bab_prune: bad arguments");
    hipStream_t st = (hipStream_t)stream;
    if (n == 0) {
        hipLaunchKernelGGL(bp::k_zero_i32, dim3(1), dim3(1), 0, st, n_keep);
        BCHK(hipGetLastError());
        return BOUND_OK;
    }
    if (n <= bp::ONE_MAX) {
        hipLaunchKernelGGL(bp::k_prune_one, dim3(1), dim3(bp::ONE_T), 0, st, n, f_lo, best, keep, n_keep);
        BCHK(hipGetLastError());
        return BOUND_OK;
    }
    hipLaunchKernelGGL(bp::k_prune_flags, dim3(bp::blocks(n)), dim3(bp::TPB), 0, st, n, f_lo, best,
                       b->flag);
    BCHK(bp::select_flagged(b, n, keep, n_keep, st));
    BCHK(hipGetLastError());
    return BOUND_OK;
}

}  // extern "C"
