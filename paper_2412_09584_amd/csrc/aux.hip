// Element-wise and small kernels around the MFMA products: relaxation tables (Lemma 1),
// split clamping, box centre / radius, start of a backward pass, split-multiplier
// injection and gradient, final assembly of the bound, the adjoint's start, the
// standalone box concretisation (Theorem 2), Adam, and weight packing.
#include "device_common.h"

namespace bp {
namespace {

constexpr int TPB = 256;

inline unsigned blocks_for(long n, int per = TPB) { return (unsigned)((n + per - 1) / per); }

__device__ inline float wave_sum(float x) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) x += __shfl_xor(x, m, 64);
    return x;
}

// Block-wide sum of two values (256 threads); result valid in thread 0.
__device__ inline void block_sum2(float &a, float &b) {
    __shared__ float sa[4], sb[4];
    a = wave_sum(a);
    b = wave_sum(b);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0) { sa[w] = a; sb[w] = b; }
    __syncthreads();
    if (threadIdx.x == 0) {
        a = sa[0] + sa[1] + sa[2] + sa[3];
        b = sb[0] + sb[1] + sb[2] + sb[3];
    }
}

// ReLU layer (0-based, < used) holding global ReLU index jg: the last layer whose offset
// is <= jg (binary search over the layers' offsets).
__device__ inline int layer_of(const LayerShape *ls, int used, long jg) {
    int a = 0, b = used - 1;
    while (a < b) {
        const int mid = (a + b + 1) >> 1;
        if (ls[mid].off <= jg) a = mid;
        else b = mid - 1;
    }
    return a;
}

// Row of lo/hi used by an instance; out-of-range indices are clamped so a bad index can
// never read outside the caller's arrays.
__device__ inline long bound_row(const int32_t *bound_of, long inst, int n_bounds) {
    long b = bound_of ? (long)bound_of[inst] : inst;
    return b < 0 ? 0 : (b >= n_bounds ? n_bounds - 1 : b);
}

// internal (y, x, c) index -> C-major index within a layer of C channels, HW pixels
__device__ inline long to_cmajor(long j, int C, int HW) { return (j % C) * HW + j / C; }
__device__ inline long to_internal(long jn, int C, int HW) { return (jn % HW) * C + jn / HW; }

// Lemma 1 for one neuron (boundary reading: active iff l >= 0, else inactive iff u <= 0);
// an unstable neuron's record carries w = k + 1, k its slot in the compact rows of saved
// coefficients (see k_prep_slots).
__device__ inline Relax relax_of(float l, float u, float a, int k) {
    if (l >= 0.f) return make_float4(1.f, 1.f, 0.f, 0.f);
    if (u <= 0.f) return make_float4(0.f, 0.f, 0.f, 0.f);
    const float su = u / (u - l);
    return make_float4(a, su, -l * su, (float)(k + 1));
}

// Slots of the unstable neurons of one ReLU layer under one bound row: the unstable
// neurons in internal order get 0, 1, 2, ... (stable: -1).  The adjoint needs a saved
// coefficient only where the neuron is unstable, so a pass saves G at these slots only.
// Block (row r, layer m): the bounds are read contiguously (C-major) and leave one bit per
// neuron, in internal order, in LDS; a scan over the 64-bit words' counts gives every
// neuron's slot, written contiguously.  64 bound rows of the 3x32x32 CNN's five layers: 31
// -> 21 us (threads walked strided segments, one thread scanned).  A sweep reads its own pixels
// of every channel: one row of 2^20 neurons 2.8 -> 0.9 ms (11.5 with each sweep over the layer).
constexpr int SLOT_TPB = 1024, SLOT_RANGE = 65536;   // most threads; neurons per sweep (8 KB of bits)
__global__ __launch_bounds__(SLOT_TPB) void k_prep_slots(const LayerShape *ls, long n_relu, const float *lo,
                                                         const float *hi, const int32_t *bound_of,
                                                         int n_bounds, int per_inst, int layer0,
                                                         int32_t *slot, int32_t *inv, int32_t *count) {
    __shared__ unsigned long long bits[SLOT_RANGE / 64];
    __shared__ int base[SLOT_RANGE / 64], wtot[SLOT_TPB / 64];
    const long r = blockIdx.x;
    const int nt = blockDim.x;
    const int layer = layer0 + (int)blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const LayerShape L = ls[layer];
    const long b = per_inst ? bound_row(bound_of, r, n_bounds) : r;
    const float *lr = lo + b * n_relu + L.off, *hr = hi + b * n_relu + L.off;
    int32_t *out = slot + r * n_relu + L.off;
    int32_t *back = inv + r * n_relu + L.off;     // slot -> internal index
    int run = 0;                                  // unstable neurons of the sweeps before
    for (long j0 = 0; j0 < L.d; j0 += SLOT_RANGE) {
        const int n = (int)(L.d - j0 < SLOT_RANGE ? L.d - j0 : SLOT_RANGE), nw = (n + 63) / 64;
        for (int w = tid; w < nw; w += nt) bits[w] = 0;
        __syncthreads();
        // the sweep's pixels of every channel; a Linear layer's neurons are channels of one pixel
        const bool dense = L.HW == 1;
        const long p0 = dense ? 0 : j0 / L.C;
        const unsigned np = dense ? 1 : (unsigned)((j0 + n - 1) / L.C - p0 + 1);
        const unsigned c0 = dense ? (unsigned)j0 : 0, ne = dense ? n : (unsigned)L.C * np;
        for (unsigned e = tid; e < ne; e += nt) {
            const unsigned q = dense ? e : e / np, c = c0 + q;
            const long p = p0 + (dense ? 0 : e - q * np), jn = (long)c * L.HW + p;
            if (lr[jn] >= 0.f || hr[jn] <= 0.f) continue;
            const long j = p * L.C + c - j0;
            if (j >= 0 && j < n) atomicOr(&bits[j >> 6], 1ull << (j & 63));
        }
        __syncthreads();
        // exclusive scan of the words' counts: a contiguous run of words per thread
        const int per = (nw + nt - 1) / nt, w0 = tid * per;
        int c = 0;
        for (int w = w0; w < w0 + per && w < nw; ++w) c += __popcll(bits[w]);
        int incl = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        if (lane == 63) wtot[wv] = incl;
        __syncthreads();
        int before = run + incl - c, total = 0;
        for (int w = 0; w < nt / 64; ++w) {
            if (w < wv) before += wtot[w];
            total += wtot[w];
        }
        for (int w = w0; w < w0 + per && w < nw; ++w) {
            base[w] = before;
            before += __popcll(bits[w]);
        }
        __syncthreads();
        for (int j = tid; j < n; j += nt) {
            const unsigned long long w = bits[j >> 6];
            const int bit = j & 63;
            int k = -1;
            if ((w >> bit) & 1) {
                k = base[j >> 6] + __popcll(w & ((1ull << bit) - 1));
                back[k] = (int32_t)(j0 + j);
            }
            out[j0 + j] = k;
        }
        run += total;
        __syncthreads();
    }
    if (tid == 0) count[r * MAX_RELU_LAYERS + layer] = run;
}

// alpha-gradient of ReLU layer L: the adjoint product left each img's contributions
// [G >= 0] G Lambda_bar at the compact slots of its unstable neurons (gc, row stride D);
// one block per instance walks its slots, sums the instance's rows and stores the
// result at the neuron's C-major index.  Slots of split neurons (w = 0) are skipped.
__global__ void k_alpha_grad(int rows, const LayerShape *ls, int layer0, long gc_rows, long n_relu,
                             const int32_t *srow, const int32_t *count, const int32_t *inv,
                             const float *gc, float *galpha, long ga_ld) {
    const long inst = blockIdx.x;
    const long r = srow[inst];
    const int layer = layer0 + (int)blockIdx.y;
    const LayerShape L = ls[layer];
    const long D = L.d, ga_off = L.off;
    gc += gc_rows * (L.off - ls[layer0].off);
    const int cnt = count[r * MAX_RELU_LAYERS + layer];
    const int32_t *iv = inv + r * n_relu + L.off;
    const float *g = gc + inst * rows * D;
    float *ga = galpha + inst * ga_ld + ga_off;
    for (int k = threadIdx.x; k < cnt; k += TPB) {
        const int j = iv[k];
        float acc = 0.f;
        int q = 0;
        // eight rows' loads in flight at once; the sum keeps the row order
        for (; q + 8 <= rows; q += 8) {
            float a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = g[(q + u) * D + k];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += a[u];
        }
        for (; q < rows; ++q) acc += g[q * D + k];
        // a split neuron's slot holds no contribution of this pass: its entry is
        // overwritten with 0 by k_alpha_split_zero (no per-slot record read here)
        const int c = j % L.C, p = j / L.C;
        ga[(long)c * L.HW + p] = acc;
    }
}

// The alpha-gradient of a split neuron is 0 (its relaxation has no alpha): one thread per
// split entry of the layer.
__global__ void k_alpha_split_zero(int nnz, int layer0, int layers, const LayerShape *ls, const int32_t *sp_inst,
                                   const int32_t *sp_layer, const int32_t *sp_j, float *galpha,
                                   long ga_ld) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nnz || sp_layer[q] < layer0 || sp_layer[q] >= layer0 + layers) return;
    const LayerShape L = ls[sp_layer[q]];
    const int j = sp_j[q], c = j % L.C, p = j / L.C;
    galpha[(long)sp_inst[q] * ga_ld + L.off + (long)c * L.HW + p] = 0.f;
}

template <class T>
__global__ void k_count_nonfinite(const T *p, long n, int32_t *cnt) {
    int a = 0, b = 0;
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        const float v = (float)p[i];
        a += v != v;
        b += isinf(v);
    }
    if (a) atomicAdd(cnt, a);
    if (b) atomicAdd(cnt + 1, b);
}

__global__ void k_fill(float *p, long n, float v) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Four values per thread through 16-byte stores (16-byte aligned p, n4 = n / 4).
__global__ void k_fill4(float4 *p, long n4, float v) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n4) p[i] = make_float4(v, v, v, v);
}

// Centre and radius of input element e (internal order); without a box 0, as the
// coefficient form needs; infeas is cleared along where no tables are built.
__device__ inline void prep_box(const BoxParams &b, long e) {
    if (b.infeas && e < b.n_inst) b.infeas[e] = 0;
    if (e >= b.total) return;
    if (!b.x_lo) {
        b.cen[e] = b.rad[e] = 0.f;
        return;
    }
    // 32-bit quotients whenever the launch has fewer than 2^31 elements
    long inst, j;
    if (b.total < 0x7fffffffL) {
        inst = (unsigned)e / (unsigned)b.d0;
        j = (unsigned)e - (unsigned)inst * (unsigned)b.d0;
    } else {
        inst = e / b.d0;
        j = e - inst * b.d0;
    }
    const unsigned p = (unsigned)j / (unsigned)b.C0, c = (unsigned)j - p * (unsigned)b.C0;
    const long jn = (long)c * b.HW0 + p;
    const float lo = b.x_lo[inst * b.d0 + jn], hi = b.x_hi[inst * b.d0 + jn];
    b.cen[e] = 0.5f * (lo + hi);
    b.rad[e] = 0.5f * (hi - lo);
}

// Relaxation records of one instance: a block covers a tile of one ReLU layer -- P
// pixels x all C channels of a convolutional layer (C <= PREP_TILE), or PREP_TILE
// consecutive neurons of a dense one -- and moves the bounds and alpha, stored C-major,
// into the records, stored pixel-major, through LDS: both the reads and the 16-byte
// record writes are contiguous across the block.  Layers with more channels than a tile
// take one pixel's channels per block with direct (strided) reads.
constexpr int PREP_SH = PREP_TILE + PREP_TILE / 8;  // room for one pad per pixel when C >= 8

template <bool SAVE>
__global__ __launch_bounds__(256) void k_prep_tables(const LayerShape *ls, const int32_t *tile0,
                                                     int used, long n_relu,
                                                     const float *lo, const float *hi,
                                                     const int32_t *bound_of, const float *alpha,
                                                     Relax *tab, int32_t *infeas, int n_bounds,
                                                     const int32_t *slot, int per_inst,
                                                     int32_t *srow, int tiles, int tile_first,
                                                     long n_tab, const BoxParams bx) {
    __shared__ float sh[3 * PREP_SH];
    // the blocks past the tables' form the input boxes' centres and radii
    if (blockIdx.x >= n_tab) {
        prep_box(bx, ((long)blockIdx.x - n_tab) * 256 + threadIdx.x);
        return;
    }
    // consecutive blocks take consecutive tiles of one instance, so the blocks in flight
    // write one contiguous stretch of the record table (and share one bounds row)
    const long inst = blockIdx.x / (unsigned)tiles;
    const int t0 = tile_first + (int)(blockIdx.x - inst * tiles);
    if (t0 >= tile0[used]) return;
    // the tile's layer: the last m < used with tile0[m] <= t0
    int m = 0, mb = used - 1;
    while (m < mb) {
        const int mid = (m + mb + 1) >> 1;
        if (tile0[mid] <= t0) m = mid;
        else mb = mid - 1;
    }
    const int t = t0 - tile0[m];
    const LayerShape L = ls[m];
    const long b = bound_row(bound_of, inst, n_bounds);
    if (t0 == tile_first && threadIdx.x == 0) {
        infeas[inst] = 0;
        srow[inst] = per_inst ? (int32_t)inst : (int32_t)b;
    }
    const float *lr = lo + b * n_relu + L.off, *hr = hi + b * n_relu + L.off;
    const float *ar = alpha ? alpha + inst * n_relu + L.off : nullptr;
    // without slots (a pass that saves nothing) an unstable record carries w = 1
    const int32_t *kr = SAVE ? slot + (per_inst ? inst : b) * n_relu + L.off : nullptr;
    Relax *tr = tab + inst * n_relu + L.off;
    auto record = [&](long j, float l, float u, float a, int32_t k) {
        if (!ar) a = u >= -l ? 1.f : 0.f;
        const Relax r = relax_of(l, u, a, k);
        // streaming store: the table is far larger than the caches and read back later
        typedef float f4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store((f4){r.x, r.y, r.z, r.w}, (f4 *)(tr + j));
    };
    if (L.HW == 1) {                        // dense: the two orders coincide
        const long j0 = (long)t * PREP_TILE;
        for (int e = threadIdx.x; e < PREP_TILE; e += 256) {
            const long j = j0 + e;
            if (j < L.d) record(j, lr[j], hr[j], ar ? ar[j] : 0.f, SAVE ? kr[j] : 0);
        }
        return;
    }
    if (L.C > PREP_TILE) {                  // one pixel, a chunk of its channels
        const int nch = (L.C + PREP_TILE - 1) / PREP_TILE;
        const int p = t / nch, c0 = (t - p * nch) * PREP_TILE;
        for (int e = threadIdx.x; e < PREP_TILE && c0 + e < L.C; e += 256) {
            const long jn = (long)(c0 + e) * L.HW + p;
            record((long)p * L.C + c0 + e, lr[jn], hr[jn], ar ? ar[jn] : 0.f,
                   SAVE ? kr[(long)p * L.C + c0 + e] : 0);
        }
        return;
    }
    const int C = L.C, P = PREP_TILE / C, p0 = t * P;
    const int np = L.HW - p0 < P ? L.HW - p0 : P;     // pixels of this tile
    const int CS = C >= 8 ? C + 1 : C;                // LDS pixel stride, odd when padded
    const float rP = 1.0f / (float)P, rC = 1.0f / (float)C;
    constexpr int PER = PREP_TILE / 256;
    const float *av = ar ? ar : lr;                   // record() ignores it without alpha
    // C-major reads: e -> (c, pixel p0 + q), contiguous in q; all of a thread's loads are
    // issued before the first LDS store
    float vl[PER], vh[PER], va[PER];
    int vs[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = threadIdx.x + k * 256;
        // e / P through one FP32 multiply by fl(1 / P): exact for e < 2^21
        const int c = (int)(((float)e + 0.5f) * rP), q = e - c * P;
        vs[k] = e < C * P && q < np ? q * CS + c : -1;
        // clamped rather than guarded, so that no branch stands between the loads
        const long jn = (long)(c < C ? c : C - 1) * L.HW + p0 + (q < np ? q : np - 1);
        vl[k] = lr[jn];
        vh[k] = hr[jn];
        va[k] = av[jn];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (vs[k] >= 0) {
            sh[vs[k]] = vl[k];
            sh[PREP_SH + vs[k]] = vh[k];
            sh[2 * PREP_SH + vs[k]] = va[k];
        }
    __syncthreads();
    // pixel-major writes: record p0 * C + e, slot entries loaded first
    int ks[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = threadIdx.x + k * 256;
        ks[k] = SAVE ? kr[(long)p0 * C + (e < np * C ? e : np * C - 1)] : 0;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = threadIdx.x + k * 256;
        if (e < np * C) {
            const int q = (int)(((float)e + 0.5f) * rC), o = e + q * (CS - C);
            record((long)p0 * C + e, sh[o], sh[PREP_SH + o], sh[2 * PREP_SH + o], ks[k]);
        }
    }
}

// One wave per instance, a lane per split entry; lists of up to 64 entries compare their
// neurons through the lanes' registers instead of reading the list once per entry.
__global__ void k_prep_splits(const LayerShape *ls, int used, long T, int n_inst, long n_relu,
                              const float *lo, const float *hi, const int32_t *bound_of,
                              const int32_t *off, const int32_t *idx, const int8_t *sign,
                              Relax *tab, int32_t *infeas, int32_t *sp_inst, int32_t *sp_layer,
                              int32_t *sp_j, int32_t *sp_dup, int n_bounds, int stop_m,
                              int stop_relu, float *stop_cen, float *stop_rad) {
    const int i = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= n_inst) return;
    const long b = bound_row(bound_of, i, n_bounds);
    const int q0 = off[i], q1 = off[i + 1];
    const bool small = q1 - q0 <= 64;
    const int myi = small && q0 + lane < q1 ? idx[q0 + lane] : -1;
    const int mys = small && q0 + lane < q1 ? sign[q0 + lane] : 0;
    for (int q = q0 + lane; q - lane < q1; q += 64) {       // whole wave: lanes past q1 only lend registers
        const long g = small ? myi : (q < q1 ? idx[q] : -1);
        int first = q, pos = 0, neg = 0;
        for (int q2 = q0; q2 < q1; ++q2) {
            const int gi = small ? __shfl(myi, q2 - q0, 64) : idx[q2];
            const int sg = small ? __shfl(mys, q2 - q0, 64) : sign[q2];
            if (gi != g) continue;
            if (q2 < first) first = q2;
            pos |= sg > 0;
            neg |= sg <= 0;
        }
        if (q >= q1) continue;
        sp_inst[q] = i;
        sp_layer[q] = -1;
        sp_j[q] = 0;
        sp_dup[q] = 0;
        if (g < 0 || g >= T) continue;  // not a layer this pass relaxes
        const int m = layer_of(ls, used, g);
        const LayerShape L = ls[m];
        const long jn = g - L.off;
        float l = lo[b * n_relu + g], u = hi[b * n_relu + g];
        if (pos) l = fmaxf(l, 0.f);
        if (neg) u = fminf(u, 0.f);
        if (l > u) infeas[i] = 1;
        const long j = to_internal(jn, L.C, L.HW);
        // a split neuron's record carries w = -(q + 1), q its first entry in the
        // instance's list, and that entry's sign in the sign bit of z: the adjoint
        // epilogue writes the entry's beta-gradient -sign * Lambda_bar
        const float wq = -(float)(first + 1);
        const float zs = sign[first] < 0 ? -0.0f : 0.0f;
        tab[(long)i * n_relu + L.off + j] = l >= 0.f ? make_float4(1.f, 1.f, zs, wq)
                                                     : make_float4(0.f, 0.f, zs, wq);
        sp_dup[q] = first != q;   // a repeated entry: k_beta_repeat copies its gradient
        if (m == stop_m && stop_cen) {  // the early-stop node's box sees the clamp too
            const float a = stop_relu ? fmaxf(l, 0.f) : l, c = stop_relu ? fmaxf(u, 0.f) : u;
            stop_cen[(long)i * L.d + j] = 0.5f * (a + c);
            stop_rad[(long)i * L.d + j] = 0.5f * (c - a);
        }
        sp_layer[q] = m;
        sp_j[q] = (int32_t)j;
    }
}

// Box of the early-stop node of ReLU layer `L` (internal order): [l, u] of z_s, or
// [ReLU(l), ReLU(u)] of h_s when relu != 0.
__global__ void k_prep_stop_box(long total, LayerShape L, long n_relu, const float *lo,
                                const float *hi, const int32_t *bound_of, int n_bounds, int relu,
                                float *cen, float *rad) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const long inst = e / L.d, j = e - inst * L.d;
    const long b = bound_row(bound_of, inst, n_bounds);
    const long jn = to_cmajor(j, L.C, L.HW);
    float l = lo[b * n_relu + L.off + jn], u = hi[b * n_relu + L.off + jn];
    if (relu) {
        l = fmaxf(l, 0.f);
        u = fmaxf(u, 0.f);
    }
    cen[e] = 0.5f * (l + u);
    rad[e] = 0.5f * (u - l);
}

__global__ void k_prep_box(const BoxParams bx) {
    prep_box(bx, (long)blockIdx.x * blockDim.x + threadIdx.x);
}

// Spec rows: coefficients in internal order and the target's bias terms; TPI threads an img
// (a wave, or a block where the target is wide).
template <int TPI>
__global__ __launch_bounds__(256) void k_init_spec(long img0, long n_img, int rows, int rpi, const float *spec,
                                                   long dk, int Ck, int HWk, const float *bias_k, float *lam,
                                                   double *s, double *mag, double *low) {
    const long li = (long)blockIdx.x * (256 / TPI) + threadIdx.x / TPI;
    const int t0 = threadIdx.x & (TPI - 1);
    if (li >= n_img) return;
    const long gimg = img0 + li;
    const long inst = gimg / rpi;
    const int rr = (int)(gimg - inst * rpi);
    const float sg = rr < rows ? 1.f : -1.f;
    const float *row = spec + (inst * rows + (rr < rows ? rr : rr - rows)) * dk;
    float a = 0.f, b = 0.f;
    for (long j = t0; j < dk; j += TPI) {
        const unsigned p = (unsigned)j / (unsigned)Ck, c = (unsigned)j - p * (unsigned)Ck;
        const float w = row[(long)c * HWk + p], t = w * bias_k[c];
        lam[li * dk + j] = sg * w;
        a += t;
        b += fabsf(t);
    }
    if (TPI == 256) {
        block_sum2(a, b);
    } else {
        a = wave_sum(a);
        b = wave_sum(b);
    }
    if (t0 == 0) {
        s[li] = sg * a;
        mag[li] = b;
        low[li] = 0.f;
    }
}

template <bool CONC>
__global__ void k_init_identity(const IdentityParams p, long n_img) {
    const long li = blockIdx.x;
    if (li >= n_img) return;
    const long gimg = p.img0 + li;
    const long inst = gimg / p.rpi;
    const long rr = gimg - inst * p.rpi;
    const float sg = rr < p.dk ? 1.f : -1.f;
    const long nr = rr < p.dk ? rr : rr - p.dk;  // C-major neuron of z_k
    int co = 0, oy = 0, ox = 0;
    if (p.kind == 1) {
        const int hw = p.ho * p.wo;
        co = (int)(nr / hw);
        const int q = (int)(nr - (long)co * hw);
        oy = q / p.wo;
        ox = q - oy * p.wo;
    }
    const int hwin = p.hi_ * p.wi;
    float a = 0.f, b = 0.f;
    for (long j = threadIdx.x; j < p.din; j += blockDim.x) {
        const long pix = j / p.ci;
        const int c = (int)(j - pix * p.ci);
        float gval = 0.f;
        if (p.kind == 0) {
            gval = p.W[nr * p.din + (long)c * hwin + pix];
        } else {
            const int iy = (int)(pix / p.wi), ix = (int)(pix - (long)(pix / p.wi) * p.wi);
            const int ky = iy - (oy * p.stride - p.pad), kx = ix - (ox * p.stride - p.pad);
            if (ky >= 0 && ky < p.kh && kx >= 0 && kx < p.kw)
                gval = p.W[(((long)co * p.ci + c) * p.kh + ky) * p.kw + kx];
        }
        gval *= sg;
        if (CONC) {
            const float cc = p.cen[inst * p.din + j], rad = p.rad[inst * p.din + j];
            a += gval * cc - fabsf(gval) * rad;
            b += fabsf(gval) * (fabsf(cc) + rad);
            if (p.emit) p.emit[li * p.din + (long)c * hwin + pix] = gval;
        } else {
            const Relax t = p.tab[inst * p.tab_ld + j];
            float lam = gval >= 0.f ? gval * t.x : gval * t.y;
            // split neuron: the multipliers' term of its first entry (rows = rpi here)
            if (p.bsum && t.w < 0.f) lam -= p.bsum[(long)(-(int)t.w - 1) * p.rpi + rr];
            const float off = gval < 0.f ? gval * t.z : 0.f;
            const float bt = lam * p.bias_m[j % p.chan_m];
            a += bt + off;
            b += fabsf(bt) + fabsf(off);
            p.out[li * p.din + j] = lam;
        }
    }
    block_sum2(a, b);
    if (threadIdx.x == 0) {
        const float bk = sg * p.bias_k[p.kind == 1 ? co : nr];
        if (CONC) {
            p.s[li] = bk;
            p.low[li] = a;
        } else {
            p.s[li] = (double)bk + a;
            p.low[li] = 0.f;
        }
        p.mag[li] = (double)fabsf(bk) + b;
    }
}

// Identity rows of a Linear target: one wave takes ID_ROWS neurons of one instance, both
// sides, and walks their columns 64 at a time, so a column's record (or box) is loaded once
// for all of them and the sums of all rows are reduced together.  W: the layer's rows in
// internal order (stride ldw).  2048 instances of 256 neurons and columns, both sides (1 GB
// written): 1.25 -> 0.54 ms (a block per row); the box bounds of z_1, 256 inputs, 784 ->
// 256: 0.17 -> 0.03 ms.
constexpr int ID_ROWS = 8, ID_COLS = 4;

__global__ __launch_bounds__(256) void k_init_dense(const IdentityParams p, const float *W, int ldw,
                                                    long inst0, long n_wave, long n_img) {
    const long wid = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (wid >= n_wave) return;
    const int tiles = (int)((p.dk + ID_ROWS - 1) / ID_ROWS);
    const unsigned ii = (unsigned)wid / (unsigned)tiles;     // the launch keeps wid below 2^31
    const long inst = inst0 + ii;
    const int r0 = (int)((unsigned)wid - ii * (unsigned)tiles) * ID_ROWS;
    const bool both = p.rpi > p.dk;
    const long up = inst * p.rpi + r0 - p.img0, dn = up + p.dk;    // local imgs of row r0
    const Relax *tb = p.tab + inst * p.tab_ld;
    float sp[ID_ROWS], mp[ID_ROWS], sn[ID_ROWS], mn[ID_ROWS];
#pragma unroll
    for (int q = 0; q < ID_ROWS; ++q) sp[q] = mp[q] = sn[q] = mn[q] = 0.f;
    for (long c0 = 0; c0 < p.din; c0 += 64 * ID_COLS) {
        Relax t[ID_COLS];
        float bm[ID_COLS];
#pragma unroll
        for (int u = 0; u < ID_COLS; ++u) {
            const long j = c0 + u * 64 + lane;
            t[u] = j < p.din ? tb[j] : make_float4(0.f, 0.f, 0.f, 0.f);
            bm[u] = j < p.din ? p.bias_m[(unsigned)j % (unsigned)p.chan_m] : 0.f;
        }
        float w[ID_ROWS][ID_COLS];      // all rows' loads before the first store
#pragma unroll
        for (int q = 0; q < ID_ROWS; ++q)
#pragma unroll
            for (int u = 0; u < ID_COLS; ++u) {
                const long j = c0 + u * 64 + lane;
                w[q][u] = r0 + q < p.dk && j < p.din ? W[(long)(r0 + q) * ldw + j] : 0.f;
            }
#pragma unroll
        for (int q = 0; q < ID_ROWS; ++q) {
            if (r0 + q >= p.dk) break;
            const bool wp = up + q >= 0 && up + q < n_img, wn = both && dn + q >= 0 && dn + q < n_img;
#pragma unroll
            for (int u = 0; u < ID_COLS; ++u) {
                const long j = c0 + u * 64 + lane;
                if (j >= p.din) continue;
                const float g = w[q][u];
                auto side = [&](float gv, long li, int rr, float &s, float &m) {
                    float lam = gv >= 0.f ? gv * t[u].x : gv * t[u].y;
                    // split neuron: the multipliers' term of its first entry
                    if (p.bsum && t[u].w < 0.f) lam -= p.bsum[(long)(-(int)t[u].w - 1) * p.rpi + rr];
                    const float off = gv < 0.f ? gv * t[u].z : 0.f, bt = lam * bm[u];
                    s += bt + off;
                    m += fabsf(bt) + fabsf(off);
                    p.out[li * p.din + j] = lam;
                };
                if (wp) side(g, up + q, r0 + q, sp[q], mp[q]);
                if (wn) side(-g, dn + q, (int)(r0 + q + p.dk), sn[q], mn[q]);
            }
        }
    }
    int q;
    const float a = dev::sum_rows<64, ID_ROWS>(sp, lane, q), b = dev::sum_rows<64, ID_ROWS>(mp, lane, q);
    const float c = dev::sum_rows<64, ID_ROWS>(sn, lane, q), d = dev::sum_rows<64, ID_ROWS>(mn, lane, q);
    if ((lane & (64 / ID_ROWS - 1)) != 0 || r0 + q >= p.dk) return;
    const float bk = p.bias_k[r0 + q];
    if (up + q >= 0 && up + q < n_img) {
        p.s[up + q] = (double)bk + a;
        p.mag[up + q] = (double)fabsf(bk) + b;
        p.low[up + q] = 0.f;
    }
    if (both && dn + q >= 0 && dn + q < n_img) {
        p.s[dn + q] = c - (double)bk;
        p.mag[dn + q] = (double)fabsf(bk) + d;
        p.low[dn + q] = 0.f;
    }
}

// Bounds of z_1 behind a Linear layer (Theorem 2), both sides from one sum.
__global__ __launch_bounds__(256) void k_dense1_bounds(const IdentityParams p, const float *W, int ldw,
                                                       long n_wave, int slack, float *lower,
                                                       float *upper, long ld, float *best,
                                                       float *best_upper) {
    const long wid = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (wid >= n_wave) return;
    const int tiles = (int)((p.dk + ID_ROWS - 1) / ID_ROWS);
    const long inst = (unsigned)wid / (unsigned)tiles;       // the launch keeps wid below 2^31
    const int r0 = (int)(wid - inst * tiles) * ID_ROWS;
    const float *cen = p.cen + inst * p.din, *rad = p.rad + inst * p.din;
    float gc[ID_ROWS], gr[ID_ROWS], gm[ID_ROWS];
#pragma unroll
    for (int q = 0; q < ID_ROWS; ++q) gc[q] = gr[q] = gm[q] = 0.f;
    for (long j = lane; j < p.din; j += 64) {
        const float cc = cen[j], rr = rad[j], m = fabsf(cc) + rr;
        float w[ID_ROWS];
#pragma unroll
        for (int q = 0; q < ID_ROWS; ++q) w[q] = r0 + q < p.dk ? W[(long)(r0 + q) * ldw + j] : 0.f;
#pragma unroll
        for (int q = 0; q < ID_ROWS; ++q) {
            gc[q] += w[q] * cc;
            gr[q] += fabsf(w[q]) * rr;
            gm[q] += fabsf(w[q]) * m;
        }
    }
    int q;
    const float a = dev::sum_rows<64, ID_ROWS>(gc, lane, q), b = dev::sum_rows<64, ID_ROWS>(gr, lane, q);
    const float m = dev::sum_rows<64, ID_ROWS>(gm, lane, q);
    if ((lane & (64 / ID_ROWS - 1)) != 0 || r0 + q >= p.dk) return;
    const float bk = p.bias_k[r0 + q], sl = slack ? KAPPA_U * (fabsf(bk) + m) : 0.f;
    const float lo = bk + (a - b) - sl, hi = bk + (a + b) + sl;
    const long o = inst * ld + r0 + q;
    lower[o] = lo;
    if (best) best[o] = fmaxf(best[o], lo);
    if (upper) {
        upper[o] = hi;
        if (best_upper) best_upper[o] = fminf(best_upper[o], hi);
    }
}

// Identity rows of a convolutional target in window form: img r (pixel-major order, see
// WinMap) starts with row r of W_k, kh x kw x ci coefficients, relaxed at the layer below.
// One wave per img.
__global__ __launch_bounds__(256) void k_init_window(const IdentityParams p, const WinMap w, long n_img) {
    const long li = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (li >= n_img) return;
    const long gi = w.img0 + li, inst = gi / w.rpi;
    int r = (int)(gi - inst * w.rpi);
    const float sg = r < w.dk ? 1.f : -1.f;
    r = r < w.dk ? r : r - w.dk;
    const int pix = r / p.co, co = r - pix * p.co;
    const int oy = pix / w.ow, ox = pix - oy * w.ow;
    const int y0 = oy * w.S - w.P, x0 = ox * w.S - w.P, E = p.kh * p.kw * p.ci;
    const Relax *tb = p.tab + inst * p.tab_ld;
    float a = 0.f, b = 0.f;
    for (int e = lane; e < E; e += 64) {
        const int t = e / p.ci, c = e - t * p.ci, ky = t / p.kw, kx = t - ky * p.kw;
        const int y = y0 + ky, x = x0 + kx;
        float lam = 0.f;
        if ((unsigned)y < (unsigned)w.H && (unsigned)x < (unsigned)w.W) {
            const float g = sg * p.W[(((long)co * p.ci + c) * p.kh + ky) * p.kw + kx];
            const Relax q = tb[(y * w.W + x) * p.ci + c];
            lam = g >= 0.f ? g * q.x : g * q.y;
            const float off = g < 0.f ? g * q.z : 0.f, bt = lam * p.bias_m[c];
            a += bt + off;
            b += fabsf(bt) + fabsf(off);
        }
        p.out[li * E + e] = lam;
    }
    a = wave_sum(a);
    b = wave_sum(b);
    if (lane == 0) {
        const float bk = sg * p.bias_k[co];
        p.s[li] = (double)bk + a;
        p.mag[li] = (double)fabsf(bk) + b;
        p.low[li] = 0.f;
    }
}

// Bounds of z_1 behind a convolution: Theorem 2 over each neuron's own window of the
// input, both sides from one sum.  One thread per (instance, neuron), C-major, so the
// bounds and the box rows are read and written contiguously.  64 inputs of 3x32x32 with 16
// channels: 0.04 ms (block per row over the whole input: 9.4 ms).
__global__ __launch_bounds__(256) void k_conv1_bounds(const IdentityParams p, long total, int slack,
                                                      float *lower, float *upper, long ld, float *best,
                                                      float *best_upper) {
    const long e = (long)blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    const long inst = e / p.dk;
    const int nr = (int)(e - inst * p.dk), hw = p.ho * p.wo;
    const int co = nr / hw, q = nr - co * hw, oy = q / p.wo, ox = q - oy * p.wo;
    const float *W = p.W + (long)co * p.ci * p.kh * p.kw;
    const float *cen = p.cen + inst * p.din, *rad = p.rad + inst * p.din;
    float gc = 0.f, gr = 0.f, m = 0.f;
    for (int ky = 0; ky < p.kh; ++ky) {
        const int y = oy * p.stride - p.pad + ky;
        if ((unsigned)y >= (unsigned)p.hi_) continue;
        for (int kx = 0; kx < p.kw; ++kx) {
            const int x = ox * p.stride - p.pad + kx;
            if ((unsigned)x >= (unsigned)p.wi) continue;
            const long j = ((long)y * p.wi + x) * p.ci;
            for (int c = 0; c < p.ci; ++c) {
                const float g = W[(c * p.kh + ky) * p.kw + kx], cc = cen[j + c], r = rad[j + c];
                gc += g * cc;
                gr += fabsf(g) * r;
                m += fabsf(g) * (fabsf(cc) + r);
            }
        }
    }
    const float bk = p.bias_k[co], sl = slack ? KAPPA_U * (fabsf(bk) + m) : 0.f;
    const float lo = bk + (gc - gr) - sl, hi = bk + (gc + gr) + sl;
    const long o = inst * ld + nr;
    lower[o] = lo;
    if (best) best[o] = fmaxf(best[o], lo);
    if (upper) {
        upper[o] = hi;
        if (best_upper) best_upper[o] = fminf(best_upper[o], hi);
    }
}

__global__ void k_beta_sum(int nnz, int rows, const int32_t *off, const int32_t *idx,
                           const int8_t *sign, const int32_t *sp_inst, const int32_t *sp_layer,
                           const int32_t *sp_dup, const float *beta, float *bsum) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)nnz * rows) return;
    const int q = (int)(e / rows), r = (int)(e - (long)q * rows);
    // entries this pass does not relax, and repeats (their term is in the first entry's)
    if (sp_layer[q] < 0 || sp_dup[q]) return;
    const int i = sp_inst[q], g = idx[q];
    float s = 0.f;
    for (int q2 = off[i]; q2 < off[i + 1]; ++q2)
        if (idx[q2] == g) s += (float)sign[q2] * beta[(long)q2 * rows + r];
    bsum[e] = s;
}

__global__ void k_finalize(long img0, long n_img, int rows, int rpi, const double *s,
                           const double *low, const double *mag, const int32_t *infeas, int slack,
                           float *lower, float *upper, long ld, float *offset, float *offset_mag,
                           float *best, float *best_upper, int pC, int pHW) {
    const long li = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (li >= n_img) return;
    const long gimg = img0 + li;
    const long inst = gimg / rpi;
    int rr = (int)(gimg - inst * rpi);
    if (pC > 0) {   // rows of a window pass: pixel-major neurons -> C-major
        const int nr = rr < rows ? rr : rr - rows, pix = nr / pC;
        rr += (nr - pix * pC) * pHW + pix - nr;
    }
    if (offset) offset[gimg] = (float)s[li];
    if (offset_mag) offset_mag[gimg] = (float)mag[li];
    if (!lower) return;
    double sum = s[li] + low[li];
    if (slack) sum -= KAPPA_U * mag[li];
    float v = (float)sum;
    if (infeas[inst]) v = INFINITY;
    if (rr < rows) {
        lower[inst * ld + rr] = v;
        if (best) best[inst * ld + rr] = fmaxf(best[inst * ld + rr], v);
    } else if (upper) {
        upper[inst * ld + rr - rows] = -v;
        if (best_upper)
            best_upper[inst * ld + rr - rows] = fminf(best_upper[inst * ld + rr - rows], -v);
    }
}

__global__ void k_adj_init(long n_img, int rows, long d0, const float *gl, const float *g1,
                           const float *cen, const float *rad, const int32_t *infeas,
                           float *gbar, float *sbar) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_img * d0) return;
    const long img = e / d0, j = e - img * d0;
    const long inst = img / rows;
    const float w = infeas[inst] ? 0.f : gl[img];
    if (j == 0) sbar[img] = w;
    const float g = g1[e];
    const float sg = g > 0.f ? 1.f : (g < 0.f ? -1.f : 0.f);
    gbar[e] = w * (cen[inst * d0 + j] - sg * rad[inst * d0 + j]);
}

// The same, four consecutive inputs per thread (d0 % 4 == 0): 16-byte loads and stores.
__global__ void k_adj_init4(long n_img, int rows, long d0, const float *gl, const float *g1,
                            const float *cen, const float *rad, const int32_t *infeas,
                            float *gbar, float *sbar) {
    // 32-bit quotients: the launch keeps n_img * d0 / 4 below 2^31
    const unsigned e4 = blockIdx.x * blockDim.x + threadIdx.x;
    const unsigned q = (unsigned)(d0 >> 2);
    if (e4 >= (unsigned)n_img * q) return;
    const long img = e4 / q, j = (long)(e4 - (unsigned)img * q) * 4;
    const long inst = (unsigned)img / (unsigned)rows;
    // every load issued before the first use
    const int bad = infeas[inst];
    const float glv = gl[img];
    const float4 g = *(const float4 *)(g1 + img * d0 + j);
    const float4 c = *(const float4 *)(cen + inst * d0 + j);
    const float4 r = *(const float4 *)(rad + inst * d0 + j);
    const float w = bad ? 0.f : glv;
    if (j == 0) sbar[img] = w;
    auto one = [&](float gv, float cv, float rv) {
        const float sg = gv > 0.f ? 1.f : (gv < 0.f ? -1.f : 0.f);
        return w * (cv - sg * rv);
    };
    *(float4 *)(gbar + img * d0 + j) =
        make_float4(one(g.x, c.x, r.x), one(g.y, c.y, r.y), one(g.z, c.z, r.z), one(g.w, c.w, r.w));
}

// beta-gradient of repeated split entries: their neuron's first entry holds -sign *
// Lambda_bar already (the adjoint's epilogue wrote it), so a repeat takes it with the two
// signs' product.  One thread per entry and row; most leave at once.
__global__ void k_beta_repeat(int nnz, int rows, const int32_t *sp_inst, const int32_t *sp_layer,
                              const int32_t *sp_j, const int32_t *sp_dup, const int8_t *sign, float *gbeta) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)nnz * rows) return;
    const int q = (int)(e / rows), r = (int)(e - (long)q * rows);
    if (sp_layer[q] < 0 || !sp_dup[q]) return;
    for (int f = q - 1; f >= 0 && sp_inst[f] == sp_inst[q]; --f)
        if (!sp_dup[f] && sp_layer[f] == sp_layer[q] && sp_j[f] == sp_j[q]) {
            const float g = gbeta[(long)f * rows + r];
            gbeta[e] = (sign[f] < 0) == (sign[q] < 0) ? g : -g;
            return;
        }
}

// lower/mag[img] += sum_j lam c - |lam| r, sum_j |lam| (|c| + r) over one row of internal-order
// coefficients, c / r the per-instance box (early stop over a pre-activation box).
__global__ void k_box_conc(long img0, int rpi, long D, const float *lam, const float *cen,
                           const float *rad, double *low, double *mag, float *save) {
    const long li = blockIdx.x;
    const long inst = (img0 + li) / rpi;
    const float *row = lam + li * D;
    const float *c = cen + inst * D, *r = rad + inst * D;
    float a = 0.f, b = 0.f;
    for (long j = threadIdx.x; j < D; j += blockDim.x) {
        const float w = row[j];
        a += w * c[j] - fabsf(w) * r[j];
        b += fabsf(w) * (fabsf(c[j]) + r[j]);
        if (save) save[li * D + j] = w;
    }
    block_sum2(a, b);
    if (threadIdx.x == 0) {
        low[li] += a;
        mag[li] += b;
    }
}

// Adjoint at an early stop over the pre-activation box of layer m: lam_bar = s_bar (c -
// sign(lam) r), then the reverse of the relaxation of layer m (G_bar_{m+1}, alpha-grad).
__global__ void k_adj_stop_linear(long n_img, int rows, long D, const float *lam, const float *g,
                                  const float *cen, const float *rad, const float *gl,
                                  const int32_t *infeas, float *sbar, const Relax *tab, long tab_ld,
                                  float *gout, float *gc, int C, int HW) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_img * D) return;
    const long img = e / D, j = e - img * D;
    const long inst = img / rows;
    const float sb = infeas[inst] ? 0.f : gl[img];
    if (j == 0) sbar[img] = sb;
    const float l = lam[e];
    const float sg = l > 0.f ? 1.f : (l < 0.f ? -1.f : 0.f);
    const float v = sb * (cen[inst * D + j] - sg * rad[inst * D + j]);
    const Relax t = tab[inst * tab_ld + j];
    // saved coefficients exist at the unstable neurons only (slot w - 1); elsewhere the
    // record has equal slopes and no intercept, so the sign of G does not matter
    const float gv = t.w > 0.f ? g[img * D + (int)t.w - 1] : 0.f;
    if (gout) gout[e] = v * (gv >= 0.f ? t.x : t.y) + (gv < 0.f ? sb * t.z : 0.f);
    if (t.w > 0.f) gc[img * D + (int)t.w - 1] = gv >= 0.f ? gv * v : 0.f;   // see k_alpha_grad
}

__global__ void k_beta_grad_stop(int nnz, int rows, int layer, long D, const int32_t *sp_inst,
                                 const int32_t *sp_layer, const int32_t *sp_j, const int8_t *sign,
                                 const float *lam, const float *cen, const float *rad,
                                 const float *sbar, float *gbeta) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)nnz * rows) return;
    const int q = (int)(e / rows), r = (int)(e - (long)q * rows);
    if (sp_layer[q] != layer) return;
    const long inst = sp_inst[q];
    const long img = inst * rows + r;
    const long j = sp_j[q];
    const float l = lam[img * D + j];
    const float sg = l > 0.f ? 1.f : (l < 0.f ? -1.f : 0.f);
    const float lam_bar = sbar[img] * (cen[inst * D + j] - sg * rad[inst * D + j]);
    gbeta[(long)q * rows + r] = -(float)sign[q] * lam_bar;
}

// C-major rows -> internal (channels-last) rows.
__global__ void k_to_internal(long total, long D, int C, int HW, const float *x, float *y) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const long img = e / D, j = e - img * D;
    y[e] = x[img * D + to_cmajor(j, C, HW)];
}

// Per subdomain and neuron: min / max of z over its per_sub sample rows (written C-major
// at lo/hi[sub*ld + j], merged with the values there when `merge`); then z <- ReLU(z) in
// place for the next layer, or a copy of the last layer's output to `out` (C-major).
// MM_ROWS samples' loads go out together, ahead of their stores, and the samples of a
// subdomain are split over `parts` threads whose results meet in LDS: 256 x 64 samples of
// 296 neurons (39 MB moved): 25 -> 13 us.
constexpr int MM_ROWS = 8;
__global__ __launch_bounds__(256) void k_sample_minmax(long n_sub, int per_sub, long D, int C, int HW,
                                                       float *z, float *lo, float *hi, long ld, int relu,
                                                       float *out, int merge, int parts) {
    __shared__ float smn[256], smx[256];
    const int cols = 256 / parts;                       // (subdomain, neuron) pairs of this block
    const int part = threadIdx.x / cols;
    const long e = (long)blockIdx.x * cols + (threadIdx.x - part * cols);
    const bool live = e < n_sub * D;
    const long sub = live ? e / D : 0, j = live ? e - sub * D : 0;
    const int per = (per_sub + parts - 1) / parts, s1 = min(per_sub, (part + 1) * per);
    float mn = INFINITY, mx = -INFINITY;
    const long oj = to_cmajor(j, C, HW);
    for (int s = part * per; live && s < s1; s += MM_ROWS) {
        float v[MM_ROWS];
        float *zp = z + (sub * per_sub + s) * D + j;
#pragma unroll
        for (int u = 0; u < MM_ROWS; ++u) v[u] = zp[(s + u < s1 ? u : 0) * D];
#pragma unroll
        for (int u = 0; u < MM_ROWS; ++u) {
            mn = fminf(mn, v[u]);
            mx = fmaxf(mx, v[u]);
            if (relu && s + u < s1) zp[u * D] = fmaxf(v[u], 0.f);
            if (out && s + u < s1) out[(sub * per_sub + s + u) * D + oj] = v[u];
        }
    }
    if (!lo) return;
    smn[threadIdx.x] = mn;
    smx[threadIdx.x] = mx;
    __syncthreads();
    if (part != 0 || !live) return;
    for (int q = 1; q < parts; ++q) {
        mn = fminf(mn, smn[q * cols + threadIdx.x]);
        mx = fmaxf(mx, smx[q * cols + threadIdx.x]);
    }
    const long o = sub * ld + oj;
    lo[o] = merge ? fminf(lo[o], mn) : mn;
    hi[o] = merge ? fmaxf(hi[o], mx) : mx;
}

// One projected Adam step of one parameter p with gradient g (moments m, v updated in
// place); shared by the dense step and the fused alpha step, so both round alike.
__device__ inline float adam_elem(float p, float g, float &m, float &v, const AdamArgs &a) {
    const float gr = a.gs * g;
    m = a.b1 * m + (1.f - a.b1) * gr;
    v = a.b2 * v + (1.f - a.b2) * gr * gr;
    const float x = p - (a.lr / a.bc1) * m / (sqrtf(v) / a.bc2s + a.eps);
    return fminf(fmaxf(x, a.lo), a.hi);
}

__global__ void k_adam(long n, float *p, const float *g, float *m, float *v, const AdamArgs a) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float pi = p[i];   // loaded with the others, ahead of the moment stores
    float mi = m[i], vi = v[i];
    const float x = adam_elem(pi, g[i], mi, vi, a);
    m[i] = mi;
    v[i] = vi;
    p[i] = x;
}

// Split neurons keep the slot they have as unstable neurons but take no alpha: their
// slots' row contributions are cleared, so the fused step below sees a zero gradient
// there, as the dense gradient has.  One thread per (split entry, row).
__global__ void k_split_gc_zero(int nnz, int rows, int layer0, int layers, const LayerShape *ls, long gc_rows,
                                long n_relu, const int32_t *sp_inst, const int32_t *sp_layer,
                                const int32_t *sp_j, const int32_t *srow, const int32_t *slot,
                                float *gc) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long)nnz * rows) return;
    const int q = (int)(t / rows), r = (int)(t - (long)q * rows);
    if (sp_layer[q] < layer0 || sp_layer[q] >= layer0 + layers) return;
    const LayerShape L = ls[sp_layer[q]];
    const long inst = sp_inst[q];
    const int s = slot[(long)srow[inst] * n_relu + L.off + sp_j[q]];
    if (s >= 0) gc[gc_rows * (L.off - ls[layer0].off) + (inst * rows + r) * L.d + s] = 0.f;
}

// alpha-gradient of ReLU layer L fused with the Adam step on alpha: as k_alpha_grad, the
// block of an instance sums its rows' contributions at each slot (in the same order),
// then steps the neuron's alpha (C-major index) with moments kept at the slot's index.
__global__ void k_alpha_adam(int rows, const LayerShape *ls, int layer0, long gc_rows, long n_relu,
                             const int32_t *srow, const int32_t *count, const int32_t *inv,
                             const float *gc, float *alpha, float *m, float *v, long ld,
                             const AdamArgs a) {
    const long inst = blockIdx.x;
    const long r = srow[inst];
    const int layer = layer0 + (int)blockIdx.y;
    const LayerShape L = ls[layer];
    const long D = L.d, aoff = L.off;
    gc += gc_rows * (L.off - ls[layer0].off);
    const int cnt = count[r * MAX_RELU_LAYERS + layer];
    const int32_t *iv = inv + r * n_relu + L.off;
    const float *g = gc + inst * rows * D;
    float *al = alpha + inst * ld + aoff, *mm = m + inst * ld + aoff, *vv = v + inst * ld + aoff;
    for (int k = threadIdx.x; k < cnt; k += TPB) {
        const int j = iv[k];
        const int c = j % L.C, p = j / L.C;
        const long ai = (long)c * L.HW + p;
        const float pi = al[ai];        // issued ahead of the row loads
        float mi = mm[k], vi = vv[k];
        float acc = 0.f;
        int q = 0;
        for (; q + 8 <= rows; q += 8) {
            float t8[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t8[u] = g[(q + u) * D + k];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += t8[u];
        }
        for (; q < rows; ++q) acc += g[q * D + k];
        const float x = adam_elem(pi, acc, mi, vi, a);
        mm[k] = mi;
        vv[k] = vi;
        al[ai] = x;
    }
}

// One block per (instance, row): reads the row once, coalesced.
// One block per instance: the box (centre, radius) of each of the thread's input
// elements is formed once and serves all the instance's rows, CROWS rows at a time, whose
// coefficient loads are all in flight together; the rows' two sums are then reduced over
// the block.
constexpr int CROWS = 12;
__global__ __launch_bounds__(256) void k_concretize(int rows, long d0, const float *coeff,
                                                   const float *offset, const float *offset_mag,
                                                   const float *x_lo, const float *x_hi, int slack,
                                                   float *lower) {
    __shared__ float red[4][2 * CROWS];
    const long inst = blockIdx.x;
    const float *lo = x_lo + inst * d0, *hi = x_hi + inst * d0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int r0 = 0; r0 < rows; r0 += CROWS) {
        const int nr = rows - r0 < CROWS ? rows - r0 : CROWS;
        const float *cr = coeff + (inst * rows + r0) * d0;
        float a[CROWS], b[CROWS];
#pragma unroll
        for (int q = 0; q < CROWS; ++q) a[q] = b[q] = 0.f;
        for (long j = threadIdx.x; j < d0; j += TPB) {
            const float l = lo[j], h = hi[j];
            float w[CROWS];
#pragma unroll
            for (int q = 0; q < CROWS; ++q) w[q] = q < nr ? cr[q * d0 + j] : 0.f;
            const float c = 0.5f * (l + h), r = 0.5f * (h - l), m = fabsf(c) + r;
#pragma unroll
            for (int q = 0; q < CROWS; ++q) {
                a[q] += w[q] * c - fabsf(w[q]) * r;
                b[q] += fabsf(w[q]) * m;
            }
        }
#pragma unroll
        for (int q = 0; q < CROWS; ++q) {
            a[q] = wave_sum(a[q]);
            b[q] = wave_sum(b[q]);
        }
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < CROWS; ++q) {
                red[wave][q] = a[q];
                red[wave][CROWS + q] = b[q];
            }
        }
        __syncthreads();
        if (threadIdx.x < nr) {
            const int q = threadIdx.x;
            const float A = red[0][q] + red[1][q] + red[2][q] + red[3][q];
            const float M = red[0][CROWS + q] + red[1][CROWS + q] + red[2][CROWS + q] + red[3][CROWS + q];
            const long row = inst * rows + r0 + q;
            float v = A + offset[row];
            if (slack) v -= KAPPA_U * (M + (offset_mag ? offset_mag[row] : 0.f));
            lower[row] = v;
        }
        __syncthreads();
    }
}

__global__ void k_pack_T(const float *W, int kind, int ci, int hwin, int co, int kh, int kw,
                         int stride, int ky0, int kx0, int Ty, int Tx, int N, int K, int Kp,
                         long total, float *Bt) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const long n = e / Kp;
    const int k = (int)(e - n * Kp);
    float v = 0.f;
    if (n < N && k < K) {
        if (kind == 0) {  // Bt[n][k] = W[k][cmajor(n)]
            const long pix = n / ci;
            const int c = (int)(n - pix * ci);
            v = W[(long)k * N + (long)c * hwin + pix];
        } else {          // k = (t'y * Tx + t'x) * co + o
            const int o = k % co, tt = k / co;
            const int ty = tt / Tx, tx = tt - ty * Tx;
            const int ky = ky0 + stride * (Ty - 1 - ty), kx = kx0 + stride * (Tx - 1 - tx);
            if (ky < kh && kx < kw) v = W[(((long)o * ci + n) * kh + ky) * kw + kx];
        }
    }
    Bt[e] = v;
}

__global__ void k_pack_F(const float *W, int kind, int ci, int hwin, int kh, int kw, int N, int K,
                         int Kp, long total, float *Bt) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const long n = e / Kp;
    const int k = (int)(e - n * Kp);
    float v = 0.f;
    if (n < N && k < K) {
        if (kind == 0) {  // Bt[n][k] = W[n][cmajor(k)]
            const long pix = k / ci;
            const int c = (int)(k - pix * ci);
            v = W[n * K + (long)c * hwin + pix];
        } else {          // k = (ky * kw + kx) * ci + c
            const int c = k % ci, tt = k / ci;
            const int ky = tt / kw, kx = tt - ky * kw;
            v = W[((n * ci + c) * kh + ky) * kw + kx];
        }
    }
    Bt[e] = v;
}

}  // namespace

template <class T>
static hipError_t count_nonfinite(const T *p, long n, int32_t *cnt, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const long nb = blocks_for(n) < 4096 ? blocks_for(n) : 4096;
    hipLaunchKernelGGL(k_count_nonfinite<T>, dim3((unsigned)nb), dim3(TPB), 0, st, p, n, cnt);
    return hipGetLastError();
}
hipError_t launch_count_nonfinite(const float *p, long n, int32_t *cnt, hipStream_t st) {
    return count_nonfinite(p, n, cnt, st);
}
hipError_t launch_count_nonfinite(const double *p, long n, int32_t *cnt, hipStream_t st) {
    return count_nonfinite(p, n, cnt, st);
}

// One wave per img: lane l sums slots l, l + 64, ... in order, then a fixed xor tree.
__global__ void k_det_reduce(long n_img, long nslot, const float *part, double *s, double *mag) {
    const long img = (long)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
    const int lane = threadIdx.x & 63;
    if (img >= n_img) return;
    const float *p = part + img * nslot * 2;
    double a = 0.0, b = 0.0;
    for (long k = lane; k < nslot; k += 64) {
        a += p[2 * k];
        b += p[2 * k + 1];
    }
#pragma unroll
    for (int mk = 32; mk > 0; mk >>= 1) {
        a += __shfl_xor(a, mk, 64);
        b += __shfl_xor(b, mk, 64);
    }
    if (lane == 0) {
        s[img] += a;
        mag[img] += b;
    }
}

hipError_t launch_det_reduce(long n_img, long nslot, const float *part, double *s, double *mag,
                             hipStream_t st) {
    if (n_img <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_det_reduce, dim3((unsigned)((n_img + 3) / 4)), dim3(256), 0, st, n_img,
                       nslot, part, s, mag);
    return hipGetLastError();
}

hipError_t launch_fill(float *p, long n, float v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (n % 4 == 0 && ((uintptr_t)p & 15) == 0)
        hipLaunchKernelGGL(k_fill4, dim3(blocks_for(n / 4)), dim3(TPB), 0, st, (float4 *)p, n / 4, v);
    else
        hipLaunchKernelGGL(k_fill, dim3(blocks_for(n)), dim3(TPB), 0, st, p, n, v);
    return hipGetLastError();
}

hipError_t launch_prep_tables(const NetShapes &ns, int first, int used, int n_inst, long n_relu,
                              const float *lo, const float *hi, const int32_t *bound_of,
                              const float *alpha, Relax *tab, int32_t *infeas, int n_bounds,
                              int32_t *slot, int32_t *slot_inv, int32_t *slot_count,
                              int32_t *srow, int max_rows, bool save, const BoxParams &box, hipStream_t st) {
    // slots per bound row when the rows fit the slot table, else per instance
    const bool per_inst = bound_of == nullptr || n_bounds > max_rows;
    const int rows = per_inst ? n_inst : n_bounds;
    long dmax = 0;
    for (int m = first; m < used; ++m) dmax = ns.l[m].d > dmax ? ns.l[m].d : dmax;
    if (save)
        hipLaunchKernelGGL(k_prep_slots, dim3((unsigned)rows, (unsigned)(used - first)),
                           dim3(dmax > 4096 ? SLOT_TPB : 256), 0, st,
                           ns.dev, n_relu, lo, hi, bound_of, n_bounds, per_inst ? 1 : 0, first, slot, slot_inv,
                           slot_count);
    long tiles = 0, tile_first = 0;
    for (int m = 0; m < used; ++m) (m < first ? tile_first : tiles) += prep_tiles(ns.l[m]);
    const long n_tab = tiles * n_inst;
    long n_box = (box.total + TPB - 1) / TPB;
    if (n_tab > 0x7fffffffL) return hipErrorInvalidValue;
    if (n_tab + n_box >= (1L << 32) / TPB) {      // more than HIP launches at once: the box by itself
        const hipError_t e = launch_prep_box(box, st);
        if (e != hipSuccess) return e;
        n_box = 0;
    }
    const auto f = save ? k_prep_tables<true> : k_prep_tables<false>;
    hipLaunchKernelGGL(f, dim3((unsigned)(n_tab + n_box)), dim3(256), 0, st, ns.dev, ns.tile0, used, n_relu, lo, hi,
                       bound_of, alpha, tab, infeas, n_bounds, slot, per_inst ? 1 : 0, srow, (int)tiles,
                       (int)tile_first, n_tab, box);
    return hipGetLastError();
}

hipError_t launch_alpha_grad(int n_inst, int rows, const NetShapes &ns, int layer0, int layers, long gc_rows,
                             long n_relu, const int32_t *srow, const int32_t *slot_count,
                             const int32_t *slot_inv, const float *gc, float *galpha, long ga_ld, int nnz,
                             const int32_t *sp_inst, const int32_t *sp_layer, const int32_t *sp_j,
                             hipStream_t st) {
    if (n_inst <= 0 || layers <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_alpha_grad, dim3((unsigned)n_inst, (unsigned)layers), dim3(TPB), 0, st, rows, ns.dev,
                       layer0, gc_rows, n_relu, srow, slot_count, slot_inv, gc, galpha, ga_ld);
    if (nnz > 0)
        hipLaunchKernelGGL(k_alpha_split_zero, dim3(blocks_for(nnz)), dim3(TPB), 0, st, nnz, layer0, layers,
                           ns.dev, sp_inst, sp_layer, sp_j, galpha, ga_ld);
    return hipGetLastError();
}

hipError_t launch_prep_splits(const NetShapes &ns, int used, int n_inst, long n_relu,
                              const float *lo, const float *hi, const int32_t *bound_of,
                              const int32_t *off, const int32_t *idx, const int8_t *sign,
                              Relax *tab, int32_t *infeas, int32_t *sp_inst, int32_t *sp_layer,
                              int32_t *sp_j, int32_t *sp_dup, int n_bounds, int stop_m,
                              int stop_relu, float *stop_cen, float *stop_rad, hipStream_t st) {
    const long T = used > 0 ? ns.l[used - 1].off + ns.l[used - 1].d : 0;
    hipLaunchKernelGGL(k_prep_splits, dim3(blocks_for(n_inst, 4)), dim3(TPB), 0, st, ns.dev, used, T,
                       n_inst, n_relu, lo, hi, bound_of, off, idx, sign, tab, infeas, sp_inst,
                       sp_layer, sp_j, sp_dup, n_bounds, stop_m, stop_relu, stop_cen, stop_rad);
    return hipGetLastError();
}

hipError_t launch_prep_box(const BoxParams &box, hipStream_t st) {
    const long n = box.total > box.n_inst ? box.total : box.n_inst;
    hipLaunchKernelGGL(k_prep_box, dim3(blocks_for(n)), dim3(TPB), 0, st, box);
    return hipGetLastError();
}

hipError_t launch_init_spec(long img0, long n_img, int rows, int rpi, const float *spec, long dk,
                            int Ck, int HWk, const float *bias_k, float *lam, double *s,
                            double *mag, double *low, hipStream_t st) {
    if (dk > 256)
        hipLaunchKernelGGL(k_init_spec<256>, dim3((unsigned)n_img), dim3(TPB), 0, st, img0, n_img, rows, rpi,
                           spec, dk, Ck, HWk, bias_k, lam, s, mag, low);
    else
        hipLaunchKernelGGL(k_init_spec<64>, dim3(blocks_for(n_img, 4)), dim3(TPB), 0, st, img0, n_img, rows, rpi,
                           spec, dk, Ck, HWk, bias_k, lam, s, mag, low);
    return hipGetLastError();
}

hipError_t launch_init_identity(const IdentityParams &p, long n_img, bool conc, hipStream_t st) {
    if (conc)
        hipLaunchKernelGGL(k_init_identity<true>, dim3((unsigned)n_img), dim3(TPB), 0, st, p, n_img);
    else
        hipLaunchKernelGGL(k_init_identity<false>, dim3((unsigned)n_img), dim3(TPB), 0, st, p, n_img);
    return hipGetLastError();
}

hipError_t launch_init_dense(const IdentityParams &p, const float *W, int ldw, long n_img, hipStream_t st) {
    const long i0 = p.img0 / p.rpi, i1 = (p.img0 + n_img - 1) / p.rpi;
    const long n_wave = (i1 - i0 + 1) * ((p.dk + ID_ROWS - 1) / ID_ROWS);
    if (n_wave > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_init_dense, dim3(blocks_for(n_wave, 4)), dim3(TPB), 0, st, p, W, ldw, i0, n_wave, n_img);
    return hipGetLastError();
}

// The bounds of z_1 take one launch for as many instances as 2^31 threads cover (HIP refuses
// 2^32): launch(params, instances, outputs) for each such part.
template <class F>
static hipError_t in_launches(const IdentityParams &p, int n_inst, long threads, long ld, float *lower, float *upper,
                              float *best, float *best_upper, F launch) {
    const long per = threads < (1L << 31) ? (1L << 31) / threads : 1;
    for (long i = 0; i < n_inst; i += per) {
        IdentityParams q = p;
        q.cen += i * p.din;
        q.rad += i * p.din;
        auto at = [&](float *x) { return x ? x + i * ld : nullptr; };
        launch(q, (int)(n_inst - i < per ? n_inst - i : per), at(lower), at(upper), at(best), at(best_upper));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_dense1_bounds(const IdentityParams &p, const float *W, int ldw, int n_inst, bool slack,
                                float *lower, float *upper, long ld, float *best, float *best_upper,
                                hipStream_t st) {
    const long tiles = (p.dk + ID_ROWS - 1) / ID_ROWS;
    return in_launches(p, n_inst, tiles * 64, ld, lower, upper, best, best_upper,
                       [&](const IdentityParams &q, int n, float *lo, float *up, float *b, float *bu) {
        hipLaunchKernelGGL(k_dense1_bounds, dim3(blocks_for(n * tiles, 4)), dim3(TPB), 0, st, q, W, ldw, n * tiles,
                           slack ? 1 : 0, lo, up, ld, b, bu);
    });
}

hipError_t launch_init_window(const IdentityParams &p, const WinMap &w, long n_img, hipStream_t st) {
    hipLaunchKernelGGL(k_init_window, dim3(blocks_for(n_img, 4)), dim3(TPB), 0, st, p, w, n_img);
    return hipGetLastError();
}

hipError_t launch_conv1_bounds(const IdentityParams &p, int n_inst, bool slack, float *lower, float *upper,
                               long ld, float *best, float *best_upper, hipStream_t st) {
    return in_launches(p, n_inst, p.dk, ld, lower, upper, best, best_upper,
                       [&](const IdentityParams &q, int n, float *lo, float *up, float *b, float *bu) {
        hipLaunchKernelGGL(k_conv1_bounds, dim3(blocks_for(n * p.dk)), dim3(TPB), 0, st, q, n * p.dk, slack ? 1 : 0,
                           lo, up, ld, b, bu);
    });
}

hipError_t launch_beta_sum(int nnz, int rows, const int32_t *off, const int32_t *idx,
                           const int8_t *sign, const int32_t *sp_inst, const int32_t *sp_layer,
                           const int32_t *sp_dup, const float *beta, float *bsum, hipStream_t st) {
    const long total = (long)nnz * rows;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_beta_sum, dim3(blocks_for(total)), dim3(TPB), 0, st, nnz, rows, off, idx,
                       sign, sp_inst, sp_layer, sp_dup, beta, bsum);
    return hipGetLastError();
}

hipError_t launch_finalize(long img0, long n_img, int rows, int rpi, const double *s,
                           const double *low, const double *mag, const int32_t *infeas, bool slack,
                           float *lower, float *upper, long ld, float *offset, float *offset_mag,
                           float *best, float *best_upper, hipStream_t st, int pC, int pHW) {
    hipLaunchKernelGGL(k_finalize, dim3(blocks_for(n_img)), dim3(TPB), 0, st, img0, n_img, rows,
                       rpi, s, low, mag, infeas, slack ? 1 : 0, lower, upper, ld, offset,
                       offset_mag, best, best_upper, pC, pHW);
    return hipGetLastError();
}

hipError_t launch_adj_init(long n_img, int rows, long d0, const float *gl, const float *g1,
                           const float *cen, const float *rad, const int32_t *infeas, float *gbar,
                           float *sbar, hipStream_t st) {
    const long total = n_img * d0;
    const bool al16 = (((uintptr_t)g1 | (uintptr_t)cen | (uintptr_t)rad | (uintptr_t)gbar) & 15) == 0;
    if (d0 % 4 == 0 && al16 && total / 4 < 0x7fffffffL)
        hipLaunchKernelGGL(k_adj_init4, dim3(blocks_for(total / 4)), dim3(TPB), 0, st, n_img, rows,
                           d0, gl, g1, cen, rad, infeas, gbar, sbar);
    else
        hipLaunchKernelGGL(k_adj_init, dim3(blocks_for(total)), dim3(TPB), 0, st, n_img, rows, d0,
                           gl, g1, cen, rad, infeas, gbar, sbar);
    return hipGetLastError();
}

hipError_t launch_beta_repeat(int nnz, int rows, const int32_t *sp_inst, const int32_t *sp_layer,
                              const int32_t *sp_j, const int32_t *sp_dup, const int8_t *sign, float *gbeta,
                              hipStream_t st) {
    const long total = (long)nnz * rows;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_beta_repeat, dim3(blocks_for(total)), dim3(TPB), 0, st, nnz, rows, sp_inst, sp_layer,
                       sp_j, sp_dup, sign, gbeta);
    return hipGetLastError();
}

hipError_t launch_prep_stop_box(int n_inst, const LayerShape &L, long n_relu, const float *lo,
                                const float *hi, const int32_t *bound_of, int n_bounds, bool relu,
                                float *cen, float *rad, hipStream_t st) {
    const long total = (long)n_inst * L.d;
    hipLaunchKernelGGL(k_prep_stop_box, dim3(blocks_for(total)), dim3(TPB), 0, st, total, L, n_relu,
                       lo, hi, bound_of, n_bounds, relu ? 1 : 0, cen, rad);
    return hipGetLastError();
}

hipError_t launch_box_conc(long img0, long n_img, int rpi, long D, const float *lam, const float *cen,
                           const float *rad, double *low, double *mag, float *save, hipStream_t st) {
    if (n_img <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_box_conc, dim3((unsigned)n_img), dim3(TPB), 0, st, img0, rpi, D, lam, cen,
                       rad, low, mag, save);
    return hipGetLastError();
}

hipError_t launch_adj_stop_linear(long n_img, int rows, long D, const float *lam, const float *g,
                                  const float *cen, const float *rad, const float *gl,
                                  const int32_t *infeas, float *sbar, const Relax *tab, long tab_ld,
                                  float *gout, float *gc, int C, int HW, hipStream_t st) {
    const long total = n_img * D;
    hipLaunchKernelGGL(k_adj_stop_linear, dim3(blocks_for(total)), dim3(TPB), 0, st, n_img, rows, D,
                       lam, g, cen, rad, gl, infeas, sbar, tab, tab_ld, gout, gc, C, HW);
    return hipGetLastError();
}

hipError_t launch_beta_grad_stop(int nnz, int rows, int layer, long D, const int32_t *sp_inst,
                                 const int32_t *sp_layer, const int32_t *sp_j, const int8_t *sign,
                                 const float *lam, const float *cen, const float *rad,
                                 const float *sbar, float *gbeta, hipStream_t st) {
    const long total = (long)nnz * rows;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_beta_grad_stop, dim3(blocks_for(total)), dim3(TPB), 0, st, nnz, rows, layer,
                       D, sp_inst, sp_layer, sp_j, sign, lam, cen, rad, sbar, gbeta);
    return hipGetLastError();
}

hipError_t launch_to_internal(long n_img, int C, int HW, const float *x, float *y, hipStream_t st) {
    const long D = (long)C * HW, total = n_img * D;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_to_internal, dim3(blocks_for(total)), dim3(TPB), 0, st, total, D, C, HW, x, y);
    return hipGetLastError();
}

hipError_t launch_sample_minmax(long n_sub, int per_sub, long D, int C, int HW, float *z, float *lo,
                                float *hi, long ld, bool relu, float *out, bool merge, hipStream_t st) {
    const long total = n_sub * D;
    if (total == 0) return hipSuccess;
    // four threads a (subdomain, neuron) from 32 samples on: they stay above one batch of loads
    const int parts = per_sub >= 4 * MM_ROWS ? 4 : 1;
    hipLaunchKernelGGL(k_sample_minmax, dim3(blocks_for(total, TPB / parts)), dim3(TPB), 0, st, n_sub, per_sub,
                       D, C, HW, z, lo, hi, ld, relu ? 1 : 0, out, merge ? 1 : 0, parts);
    return hipGetLastError();
}

AdamArgs adam_args(int step, float lr, float b1, float b2, float eps, float gs, float lo, float hi) {
    AdamArgs a;
    a.b1 = b1;
    a.b2 = b2;
    a.bc1 = 1.f - powf(b1, (float)step);
    a.bc2s = sqrtf(1.f - powf(b2, (float)step));
    a.lr = lr;
    a.eps = eps;
    a.gs = gs;
    a.lo = lo;
    a.hi = hi;
    return a;
}

hipError_t launch_adam(long n, float *p, const float *g, float *m, float *v, int step, float lr,
                       float b1, float b2, float eps, float gs, float lo, float hi, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(n)), dim3(TPB), 0, st, n, p, g, m, v,
                       adam_args(step, lr, b1, b2, eps, gs, lo, hi));
    return hipGetLastError();
}

hipError_t launch_alpha_adam(int n_inst, int rows, const NetShapes &ns, int layer0, int layers, long gc_rows,
                             long n_relu, const int32_t *srow, const int32_t *slot_count,
                             const int32_t *slot_inv, const int32_t *slot, float *gc, float *alpha,
                             float *m, float *v, long ld, int nnz, const int32_t *sp_inst,
                             const int32_t *sp_layer, const int32_t *sp_j, const AdamArgs &a, hipStream_t st) {
    if (n_inst <= 0 || layers <= 0) return hipSuccess;
    if (nnz > 0) {
        const long nt = (long)nnz * rows;
        hipLaunchKernelGGL(k_split_gc_zero, dim3(blocks_for(nt)), dim3(TPB), 0, st, nnz, rows, layer0, layers,
                           ns.dev, gc_rows, n_relu, sp_inst, sp_layer, sp_j, srow, slot, gc);
    }
    hipLaunchKernelGGL(k_alpha_adam, dim3((unsigned)n_inst, (unsigned)layers), dim3(TPB), 0, st, rows, ns.dev,
                       layer0, gc_rows, n_relu, srow, slot_count, slot_inv, gc, alpha, m, v, ld, a);
    return hipGetLastError();
}

hipError_t launch_concretize(int n_inst, int rows, long d0, const float *coeff,
                             const float *offset, const float *offset_mag, const float *x_lo,
                             const float *x_hi, bool slack, float *lower, hipStream_t st) {
    const long nrow = (long)n_inst * rows;
    if (nrow == 0) return hipSuccess;
    hipLaunchKernelGGL(k_concretize, dim3((unsigned)n_inst), dim3(TPB), 0, st, rows, d0, coeff,
                       offset, offset_mag, x_lo, x_hi, slack ? 1 : 0, lower);
    return hipGetLastError();
}

hipError_t launch_pack_T(const float *W, int kind, int ci, int hi_, int wi, int co, int ho, int wo,
                         int kh, int kw, int stride, int pad, int py, int px, int ky0, int kx0,
                         int Ty, int Tx, int N, int K, int Kp, int Np, float *Bt, hipStream_t st) {
    (void)ho; (void)wo; (void)pad; (void)py; (void)px;
    const long total = (long)Np * Kp;
    hipLaunchKernelGGL(k_pack_T, dim3(blocks_for(total)), dim3(TPB), 0, st, W, kind, ci, hi_ * wi,
                       co, kh, kw, stride, ky0, kx0, Ty, Tx, N, K, Kp, total, Bt);
    return hipGetLastError();
}

hipError_t launch_pack_F(const float *W, int kind, int ci, int hi_, int wi, int co, int kh, int kw,
                         int N, int K, int Kp, int Np, float *Bt, hipStream_t st) {
    (void)co;
    const long total = (long)Np * Kp;
    hipLaunchKernelGGL(k_pack_F, dim3(blocks_for(total)), dim3(TPB), 0, st, W, kind, ci, hi_ * wi,
                       kh, kw, N, K, Kp, total, Bt);
    return hipGetLastError();
}

}  // namespace bp
