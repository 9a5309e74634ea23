// Device code shared by the gfx950 product kernels: MFMA lane layouts and the fused
// epilogues of the bound pass (Lemma 1 relaxation, Theorem 2 concretisation) and of
// its adjoint.
#pragma once
#include "bound_internal.h"

namespace bp {
namespace dev {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4v __attribute__((ext_vector_type(4)));

template <int MF> struct Mma;
template <> struct Mma<32> {
    using acc_t = f32x16;
    static constexpr int NACC = 16;
    static constexpr int KPL = 8;  // k values per lane per chunk (2 lane groups)
    static __device__ inline acc_t mma(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }
    static __device__ inline int col(int lane) { return lane & 31; }
    static __device__ inline int grp(int lane) { return lane >> 5; }
    static __device__ inline int idx(int lane) { return lane & 31; }
};
template <> struct Mma<16> {
    using acc_t = f32x4v;
    static constexpr int NACC = 4;
    static constexpr int KPL = 4;  // 4 lane groups
    static __device__ inline acc_t mma(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int v, int lane) { return 4 * (lane >> 4) + v; }
    static __device__ inline int col(int lane) { return lane & 15; }
    static __device__ inline int grp(int lane) { return lane >> 4; }
    static __device__ inline int idx(int lane) { return lane & 15; }
};

// ---------------------------------------------------------------------- tile order
// Logical tile (x, y, z) of this workgroup in an [nx][ny][nz] tile grid launched as a
// one-dimensional grid of nx * ny * nz workgroups.  Workgroups are dispatched to the 8
// XCDs round-robin (workgroup b to XCD b mod 8) and every XCD has its own L2, so the
// renumbering hands XCD k the k-th contiguous range of logical tiles, z (the output
// phase of a transposed convolution) fastest and y (the column tile) next: tiles that
// gather the same input rows, and the rows of one instance, which share its relaxation
// records, then meet in one L2 at about the same time.
struct TileIdx {
    long x;
    int y, z;
};
__device__ inline TileIdx xcd_tile(int ny, int nz) {
    const unsigned T = gridDim.x, b = blockIdx.x;
    const unsigned q = T >> 3, r = T & 7, xcd = b & 7, slot = b >> 3;
    unsigned t = xcd < r ? xcd * (q + 1) + slot : r * (q + 1) + (xcd - r) * q + slot;
    TileIdx ti;
    ti.z = (int)(t % (unsigned)nz);
    t /= (unsigned)nz;
    ti.y = (int)(t % (unsigned)ny);
    ti.x = (long)(t / (unsigned)ny);
    return ti;
}

// ---------------------------------------------------------------------- index helpers
// n / d for 0 <= n < 2^21 through one FP32 multiply by rd = fl(1/d): (n + 0.5) / d lies
// at least 0.5/d away from an integer, and the two roundings move the product by less
// than (n + 0.5)/d * 2^-23 < 0.5/d, so truncation gives the exact quotient.
__device__ inline int qdiv(int n, float rd) { return (int)(((float)n + 0.5f) * rd); }
__device__ inline long ldiv_by(long n, int d, float rd) {
    // past 2^21 an FP64 quotient of the same form: exact for n < 2^50, and a tenth of the
    // instructions of a 64-bit integer division
    return n < (1L << 21) ? (long)qdiv((int)n, rd) : (long)(((double)n + 0.5) / (double)d);
}
// The same in FP64 with rd = fl64(1 / d): exact for 0 <= n < 2^50 by the argument above
// with 2^-52 in place of 2^-23.
__device__ inline long ldiv64(long n, double rd) { return (long)(((double)n + 0.5) * rd); }

// Element i of one img's row segment starting at base.  Every epilogue offset stays inside
// such a segment (i * sizeof(T) < 2^32, layer widths are validated on the host), so the
// byte offset is formed in 32 bits; the access goes through a global-address-space
// pointer, so that with a wave-uniform base it takes the scalar-base global form (a
// generic pointer that the compiler cannot place would give a flat access with 64-bit
// address arithmetic per element).
template <class T> __device__ inline T ld(const T *base, int i) {
    using G = const __attribute__((address_space(1))) T;
    return *(G *)((const char *)base + (unsigned)i * (unsigned)sizeof(T));
}
// float4 records through the compiler's native vector type (HIP's float4 class has no
// copy from another address space)
__device__ inline float4 ld(const float4 *base, int i) {
    using V = float __attribute__((ext_vector_type(4)));
    using G = const __attribute__((address_space(1))) V;
    const V v = *(G *)((const char *)base + (unsigned)i * 16u);
    return make_float4(v.x, v.y, v.z, v.w);
}
template <class T> __device__ inline void st(T *base, int i, T v) {
    using G = __attribute__((address_space(1))) T;
    *(G *)((char *)base + (unsigned)i * (unsigned)sizeof(T)) = v;
}

// ---------------------------------------------------------------------- bf16 parts
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// An FP32 value as three bf16 values, each the rounded remainder of the one before: of a pair,
// packed, and of one (weights, on packing).
__device__ inline void split_pair(float a, float b, unsigned &hi, unsigned &mid, unsigned &lo) {
    hi = __builtin_bit_cast(unsigned, __builtin_convertvector((f2){a, b}, bf2));
    const float ra = a - __uint_as_float(hi << 16), rb = b - __uint_as_float(hi & 0xffff0000u);
    mid = __builtin_bit_cast(unsigned, __builtin_convertvector((f2){ra, rb}, bf2));
    const float qa = ra - __uint_as_float(mid << 16), qb = rb - __uint_as_float(mid & 0xffff0000u);
    lo = __builtin_bit_cast(unsigned, __builtin_convertvector((f2){qa, qb}, bf2));
}
__device__ inline void split_one(float x, unsigned short &hi, unsigned short &mid, unsigned short &lo) {
    const __bf16 h = (__bf16)x;
    const float r = x - (float)h;
    const __bf16 m = (__bf16)r, l = (__bf16)(r - (float)m);
    hi = __builtin_bit_cast(unsigned short, h);
    mid = __builtin_bit_cast(unsigned short, m);
    lo = __builtin_bit_cast(unsigned short, l);
}
// Packed weights' range (SPLIT_MAX, SPLIT_MIN): see launch_pack_split.
__device__ inline void flag_range(float x, int32_t *flags) {
    const unsigned u = __float_as_uint(x) & 0x7fffffffu;
    const int i = u > SPLIT_MAX ? 0 : (u < SPLIT_MIN ? 1 : 2);
    if (u != 0 && !flags[i]) flags[i] = 1;
}

// ---------------------------------------------------------------------- LDS DMA
// dword 3 of a raw buffer resource (32-bit data format; no swizzle, no index stride)
constexpr int BUF_FLAGS = 0x00020000;

// 16 bytes per lane from base + voff (bytes) into LDS at lds + 16 * lane (lds uniform
// across the wave); offsets at or past nbytes read nothing.
__device__ inline void lds_dma16(const float *base, int nbytes, float *lds, int voff) {
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, nbytes, BUF_FLAGS);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds, 16,
                                             voff, 0, 0, 0);
}

// ---------------------------------------------------------------------- epilogues
// Each epilogue splits its per-element work into pre() -- the global loads it needs
// (relaxation record, box) --, pre2() -- loads whose address depends on pre()'s result
// (the saved coefficient of the adjoint) -- and post() -- arithmetic, stores and
// atomics -- so that tile_epilogue can issue loads ahead of earlier groups' stores.
// Row(img) resolves the per-img pointers once per row group; j is the element's offset
// inside its img (dpix * N + n), dpix the destination pixel.
struct EpiRelax {
    RelaxParams p;
    static constexpr int NRED = 2;
    static constexpr bool WIN = false;
    using Pre = Relax;
    struct Row { const Relax *tb; float *out, *save; };
    __device__ Row row(int img) const {
        const long inst = ldiv_by(p.img0 + img, p.rpi, p.rrpi);
        const long o = (long)img * p.D;
        return Row{p.tab + inst * p.tab_ld, p.out + o, p.save ? p.save + o : nullptr};
    }
    // whether n rows from img on share their columns' records
    __device__ bool one_instance(int img, int n) const {
        return ldiv_by(p.img0 + img, p.rpi, p.rrpi) == ldiv_by(p.img0 + img + n - 1, p.rpi, p.rrpi);
    }
    // the img k after r's, of the same instance
    __device__ Row at(const Row &r, int k) const {
        return Row{r.tb, r.out + (long)k * p.D, r.save ? r.save + (long)k * p.D : nullptr};
    }
    // split multipliers' term of row rc at first split entry q: the row within its
    // instance is recovered from the row's output pointer (only on this rare path, so the
    // common path keeps no extra register per row)
    __device__ float split_term(const Row &rc, int q) const {
        // (host reciprocals: a division here costs 12 registers in every tile's epilogue, two
        // waves per SIMD of the 16-channel relaxing product: 2.05 -> 2.15 ms on 4096 subdomains)
        const long gi = p.img0 + ldiv64(rc.out - p.out, p.rDd);   // exact multiple of D
        const long r = gi - ldiv64(gi, p.rrpid) * p.rpi;
        return p.bsum[(long)q * p.rpi + r];
    }
    __device__ float colv(int n) const { return p.bias[n % p.chan]; }
    __device__ double *red0() const { return p.s; }
    __device__ double *red1() const { return p.mag; }
    __device__ const DetSums *det() const { return &p.det; }
    __device__ Pre pre(const Row &rc, int dp, int n, int N) const { return ld(rc.tb, dp * N + n); }
    __device__ void pre2(const Row &, Pre &) const {}
    __device__ void post(const Pre &t, const Row &rc, int, int, int j, float bcol, float g,
                         float &r0, float &r1) const {
        // Lemma 1's line by the sign of G, then -sum(beta sign) of the split entries at a
        // split neuron (first entry q = -w - 1); split neurons are a few per instance, so
        // their term is loaded here, in a branch most waves skip, rather than carried in
        // registers with every element's record.  The bias term takes the coefficient with
        // the split term included.
        float lam = g >= 0.f ? g * t.x : g * t.y;
        if (t.w < 0.f && p.bsum) lam -= split_term(rc, -(int)t.w - 1);
        const float off = g < 0.f ? g * t.z : 0.f;
        const float bt = lam * bcol;
        r0 += bt + off;
        r1 += fabsf(bt) + fabsf(off);
        // the sums are formed in order; without this the compiler defers them past the
        // tile's stores and keeps every lam and offset of the tile live in registers
        asm volatile("" : "+v"(r0), "+v"(r1));
        st(rc.out, j, lam);
        if (rc.save && t.w > 0.f) st(rc.save, (int)t.w - 1, g);    // unstable: compact slot
    }
};

struct EpiConc {
    ConcParams p;
    static constexpr int NRED = 2;
    static constexpr bool WIN = false;
    using Pre = float2;
    struct Row { const float *cen, *rad; float *save, *emit; };
    __device__ Row row(int img) const {
        const long inst = ldiv_by(p.img0 + img, p.rpi, p.rrpi);
        const long o = (long)img * p.D;
        return Row{p.cen + inst * p.D, p.rad + inst * p.D, p.save ? p.save + o : nullptr,
                   p.emit ? p.emit + o : nullptr};
    }
    __device__ bool one_instance(int img, int n) const {
        return ldiv_by(p.img0 + img, p.rpi, p.rrpi) == ldiv_by(p.img0 + img + n - 1, p.rpi, p.rrpi);
    }
    __device__ Row at(const Row &r, int k) const {
        return Row{r.cen, r.rad, r.save ? r.save + (long)k * p.D : nullptr, r.emit ? r.emit + (long)k * p.D : nullptr};
    }
    __device__ float colv(int) const { return 0.f; }
    __device__ double *red0() const { return p.low; }
    __device__ double *red1() const { return p.mag; }
    __device__ const DetSums *det() const { return &p.det; }
    __device__ Pre pre(const Row &rc, int dp, int n, int N) const {
        return make_float2(ld(rc.cen, dp * N + n), ld(rc.rad, dp * N + n));
    }
    __device__ void pre2(const Row &, Pre &) const {}
    __device__ void post(const Pre &cr, const Row &rc, int dpix, int n, int j, float, float g,
                         float &r0, float &r1) const {
        r0 += g * cr.x - fabsf(g) * cr.y;
        r1 += fabsf(g) * (fabsf(cr.x) + cr.y);
        asm volatile("" : "+v"(r0), "+v"(r1));   // in order, as in EpiRelax
        if (rc.save) st(rc.save, j, g);
        if (rc.emit) st(rc.emit, n * p.hw + dpix, g);
    }
};

struct EpiAdj {
    AdjParams p;
    static constexpr int NRED = 0;
    static constexpr bool WIN = false;
    struct Pre { Relax t; float g; };
    struct Row { const Relax *tb; const float *gs; float *go; float *gc; float *gb; float sb; };
    __device__ Row row(int img) const {
        const long inst = ldiv_by(img, p.rpi, p.rrpi);
        const long o = (long)img * p.D;
        return Row{p.tab + inst * p.tab_ld, p.gsave + o, p.gout ? p.gout + o : nullptr,
                   p.gc + o, p.gbeta ? p.gbeta + (img - inst * p.rpi) : nullptr, p.sbar[img]};
    }
    __device__ bool one_instance(int, int) const { return false; }   // saved rows differ
    __device__ Row at(const Row &r, int) const { return r; }
    __device__ float colv(int n) const { return p.bias[n]; }
    __device__ double *red0() const { return nullptr; }
    __device__ double *red1() const { return nullptr; }
    __device__ const DetSums *det() const { return nullptr; }
    // G is saved at the unstable neurons only (slot w - 1), a load that depends on the
    // record: pre() fetches the record, pre2() the saved coefficient.  Elsewhere x = y
    // and z = 0, so the sign of G does not matter.
    __device__ Pre pre(const Row &rc, int dp, int n, int N) const { return Pre{ld(rc.tb, dp * N + n), 0.f}; }
    __device__ void pre2(const Row &rc, Pre &q) const {
        if (q.t.w > 0.f) q.g = ld(rc.gs, (int)q.t.w - 1);
    }
    __device__ void post(const Pre &q, const Row &rc, int dpix, int n, int j, float bcol, float acc,
                         float &, float &) const {
        const float v = acc + rc.sb * bcol;           // Lambda_bar_m[img, j]
        const float g = q.g;                          // G_{m+1}[img, j]
        const Relax &t = q.t;
        if (rc.go) st(rc.go, j, v * (g >= 0.f ? t.x : t.y) + (g < 0.f ? rc.sb * t.z : 0.f));
        // alpha-gradient contribution of this row at the neuron's slot (summed over the
        // instance's rows by k_alpha_grad)
        if (t.w > 0.f) st(rc.gc, (int)t.w - 1, g >= 0.f ? g * v : 0.f);
        // split neuron (first entry q of the instance's list): d lower / d beta_{q,r} =
        // -sign_q * Lambda_bar, sign_q carried in the sign bit of the record's z
        if (t.w < 0.f && rc.gb) rc.gb[(long)(-(int)t.w - 1) * p.rpi] = signbit(t.z) ? v : -v;
    }
};

// Forward pass of sample rows (search-integrated bounds): z = W h + b.
struct EpiFwd {
    FwdParams p;
    static constexpr int NRED = 0;
    static constexpr bool WIN = false;
    struct Pre {};
    struct Row { float *out; };
    __device__ Row row(int img) const { return Row{p.out + (long)img * p.D}; }
    __device__ bool one_instance(int, int) const { return true; }
    __device__ Row at(const Row &r, int k) const { return Row{r.out + (long)k * p.D}; }
    __device__ float colv(int n) const { return p.bias[n]; }
    __device__ double *red0() const { return nullptr; }
    __device__ double *red1() const { return nullptr; }
    __device__ const DetSums *det() const { return nullptr; }
    __device__ Pre pre(const Row &, int, int, int) const { return Pre{}; }
    __device__ void pre2(const Row &, Pre &) const {}
    __device__ void post(const Pre &, const Row &rc, int, int, int j, float bcol, float acc,
                         float &, float &) const {
        st(rc.out, j, acc + bcol);
    }
};

// Origin and records of an img's receptive-field window (WinMap): the img's target pixel
// (oy, ox) puts window pixel (0, 0) at layer pixel (oy * S - P, ox * S - P).
struct WinOrg { long inst; int y0, x0; };
__device__ inline WinOrg win_origin(const WinMap &w, int img) {
    const long gi = w.img0 + img, inst = ldiv_by(gi, w.rpi, w.rrpi);
    int r = (int)(gi - inst * w.rpi);
    r = r >= w.dk ? r - w.dk : r;
    const int pix = qdiv(r, w.rC), oy = qdiv(pix, w.rOw), ox = pix - oy * w.ow;
    return WinOrg{inst, oy * w.S - w.P, ox * w.S - w.P};
}
// Layer pixel of window pixel dp, -1 outside the layer.
__device__ inline int win_pixel(const WinMap &w, int y0, int x0, int dp) {
    const int wy = qdiv(dp, w.rDW), y = y0 + wy, x = x0 + dp - wy * w.DW;
    return (unsigned)y < (unsigned)w.H && (unsigned)x < (unsigned)w.W ? y * w.W + x : -1;
}

// Lemma 1 on a window: as EpiRelax without split terms and saved coefficients.  Window
// pixels outside the layer (and columns past N) take a zero record, so their
// coefficient is 0 and they add nothing to the sums.
struct EpiRelaxWin {
    RelaxParams p;
    WinMap w;
    static constexpr int NRED = 2;
    static constexpr bool WIN = true;
    using Pre = Relax;
    struct Row { const Relax *tb; float *out; int y0, x0; };
    __device__ Row row(int img) const {
        const WinOrg o = win_origin(w, img);
        return Row{p.tab + o.inst * p.tab_ld, p.out + (long)img * p.D, o.y0, o.x0};
    }
    __device__ float colv(int n) const { return p.bias[n % p.chan]; }
    __device__ double *red0() const { return p.s; }
    __device__ double *red1() const { return p.mag; }
    __device__ const DetSums *det() const { return nullptr; }
    __device__ void post(const Pre &t, const Row &rc, int, int, int j, float bcol, float g,
                         float &r0, float &r1) const {
        const float lam = g >= 0.f ? g * t.x : g * t.y;
        const float off = g < 0.f ? g * t.z : 0.f;
        const float bt = lam * bcol;
        r0 += bt + off;
        r1 += fabsf(bt) + fabsf(off);
        asm volatile("" : "+v"(r0), "+v"(r1));   // in order, as in EpiRelax
        st(rc.out, j, lam);
    }
    // record i of row rc, zero where !ok
    __device__ Pre at(const Row &rc, int i, bool ok) const {
        const Relax t = ld(rc.tb, ok ? i : 0);
        return make_float4(ok ? t.x : 0.f, ok ? t.y : 0.f, ok ? t.z : 0.f, 0.f);
    }
};

// Theorem 2 on a window of the input.
struct EpiConcWin {
    ConcParams p;
    WinMap w;
    static constexpr int NRED = 2;
    static constexpr bool WIN = true;
    using Pre = float2;
    struct Row { const float *cen, *rad; int y0, x0; };
    __device__ Row row(int img) const {
        const WinOrg o = win_origin(w, img);
        return Row{p.cen + o.inst * p.D, p.rad + o.inst * p.D, o.y0, o.x0};
    }
    __device__ float colv(int) const { return 0.f; }
    __device__ double *red0() const { return p.low; }
    __device__ double *red1() const { return p.mag; }
    __device__ const DetSums *det() const { return nullptr; }
    __device__ Pre pre(const Row &rc, int dp, int n, int N) const {
        const int px = win_pixel(w, rc.y0, rc.x0, dp);
        return px >= 0 && n < N ? make_float2(ld(rc.cen, px * N + n), ld(rc.rad, px * N + n))
                                : make_float2(0.f, 0.f);
    }
    __device__ void pre2(const Row &, Pre &) const {}
    __device__ void post(const Pre &cr, const Row &, int, int, int, float, float g, float &r0,
                         float &r1) const {
        r0 += g * cr.x - fabsf(g) * cr.y;
        r1 += fabsf(g) * (fabsf(cr.x) + cr.y);
        asm volatile("" : "+v"(r0), "+v"(r1));
    }
    __device__ Pre at(const Row &rc, int i, bool ok) const {
        const float c = ld(rc.cen, ok ? i : 0), r = ld(rc.rad, ok ? i : 0);
        return make_float2(ok ? c : 0.f, ok ? r : 0.f);
    }
};

// One row sum pair of a tile: an FP64 atomic per accumulator, or with deterministic sums
// a store to the tile's own slot (dp: destination pixel of the tile's first row, n0: its
// first column).
template <class Epi>
__device__ inline void put_row_sums(const Epi &epi, long img, int dp, int n0, float r0, float r1) {
    const DetSums *d = epi.det();
    if (d && d->part) {
        float *q = d->part + (img * d->nslot + (long)dp * d->ncu + (n0 >> 4)) * 2;
        q[0] = r0;
        q[1] = r1;
    } else {
        atomicAdd(epi.red0() + img, (double)r0);
        atomicAdd(epi.red1() + img, (double)r1);
    }
}

// Sum of r0 / r1 over the lanes that hold the same output row (they differ only in the
// column bits of the lane id), then one sum pair per row from the column-0 lane.
// img < 0: none; so for a wave whose columns all lie past the last one, which has no slot.
template <int MF, class Epi>
__device__ inline void reduce_row(const Epi &epi, float r0, float r1, int img, int dp, int n0,
                                  int lane) {
#pragma unroll
    for (int mk = 1; mk < MF; mk <<= 1) {
        r0 += __shfl_xor(r0, mk, 64);
        r1 += __shfl_xor(r1, mk, 64);
    }
    if ((lane & (MF - 1)) == 0 && img >= 0) put_row_sums(epi, img, dp, n0, r0, r1);
}

// The sums of a whole wave (one img), then one pair from lane 0 (which holds the wave's
// first row and its tile's first column).
template <class Epi>
__device__ inline void reduce_wave(const Epi &epi, float u0, float u1, long img, int dp, int n0,
                                   int lane) {
#pragma unroll
    for (int mk = 1; mk < 64; mk <<= 1) {
        u0 += __shfl_xor(u0, mk, 64);
        u1 += __shfl_xor(u1, mk, 64);
    }
    if (lane == 0) put_row_sums(epi, img, dp, n0, u0, u1);
}

// Epilogue of one wave's accumulator tile.  The accumulator rows of a lane come in
// groups of four consecutive tile rows (MFMA row groups); rowfn4(i, vg, img, dp) maps
// group vg of fragment i to the local img of each row (-1 if out of range) and its
// destination pixel, and returns true when all four rows lie in one img (then the
// per-img pointers are resolved once).  A group's loads are issued before its stores.
// FAST: every row of the wave lies in img uimg and every column is in range (the
// common case of a convolution tile), so the pointers are resolved once per wave, no
// element is masked and the row sums collapse into one atomic pair per wave.
template <bool FAST, bool LEAN, class Epi, int MF, int FM, int FN, class Acc, class RowFn>
__device__ inline void tile_epilogue_impl(const Epi &epi, Acc (&acc)[FM][FN], const int (&ncol)[FN],
                                          const float (&bcol)[FN], int N, const RowFn &rowfn4,
                                          int lane, int uimg) {
    constexpr int NACC = Mma<MF>::NACC;
    constexpr int NR = Epi::NRED;
    float u0 = 0.f, u1 = 0.f;
    typename Epi::Row rw;
    if (FAST) {
        // Pipeline over the row groups: the first loads of group g + 2 and the dependent
        // loads of group g + 1 are issued before the stores of group g (records and saved
        // coefficients never alias the outputs), so about one memory latency is exposed
        // per tile rather than one or two per group -- when three groups' loads fit in
        // about 64 registers (else two stages, or none).
        rw = epi.row(__builtin_amdgcn_readfirstlane(uimg));
        constexpr int NG = FM * (NACC / 4);
        constexpr int GREG = FN * 4 * (int)sizeof(typename Epi::Pre) / 4;
        constexpr int DEPTH = 2 * GREG <= 48 ? 1 : 0;
        using PreG = typename Epi::Pre[FN][4];
        auto load1 = [&](int g, int (&dp)[4], PreG &pre) {
            int img[4];
            rowfn4(g / (NACC / 4), g % (NACC / 4), img, dp);
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) pre[j][q] = epi.pre(rw, dp[q], ncol[j], N);
        };
        auto load2 = [&](PreG &pre) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) epi.pre2(rw, pre[j][q]);
        };
        auto copy = [&](int (&dd)[4], PreG &pd, const int (&ds)[4], const PreG &ps) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                dd[q] = ds[q];
#pragma unroll
                for (int j = 0; j < FN; ++j) pd[j][q] = ps[j][q];
            }
        };
        int dpA[4], dpB[4];
        PreG preA, preB;
        load1(0, dpA, preA);
        load2(preA);
        const int dp0 = dpA[0];           // lane 0: the wave's first row
        if (DEPTH == 2 && NG > 1) load1(1, dpB, preB);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            int dpC[4];
            PreG preC;
            if (DEPTH == 2) {
                if (g + 2 < NG) load1(g + 2, dpC, preC);
                if (g + 1 < NG) load2(preB);
            } else if (DEPTH == 1 && g + 1 < NG) {
                load1(g + 1, dpB, preB);
                load2(preB);
            }
            const int i = g / (NACC / 4), vg = g % (NACC / 4);
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    epi.post(preA[j][q], rw, dpA[q], ncol[j], dpA[q] * N + ncol[j], bcol[j],
                             acc[i][j][vg * 4 + q], u0, u1);
            if (DEPTH == 0 && g + 1 < NG) {
                load1(g + 1, dpB, preB);
                load2(preB);
            }
            if (g + 1 < NG) copy(dpA, preA, dpB, preB);
            if (DEPTH == 2 && g + 2 < NG) copy(dpB, preB, dpC, preC);
        }
        if (NR > 0) reduce_wave(epi, u0, u1, uimg, dp0, ncol[0], lane);
        return;
    }
    if (LEAN) {
        // one element at a time: the rare tiles of a convolution that straddle images
        // or the end of the batch; few registers, so the common path keeps its occupancy
#pragma unroll
        for (int i = 0; i < FM; ++i) {
#pragma unroll
            for (int vg = 0; vg < NACC / 4; ++vg) {
                int img[4], dp[4];
                rowfn4(i, vg, img, dp);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float r0 = 0.f, r1 = 0.f;
                    if (img[q] >= 0) {
                        const typename Epi::Row rc = epi.row(img[q]);
#pragma unroll
                        for (int j = 0; j < FN; ++j)
                            if (ncol[j] < N) {
                                typename Epi::Pre pr = epi.pre(rc, dp[q], ncol[j], N);
                                epi.pre2(rc, pr);
                                epi.post(pr, rc, dp[q], ncol[j], dp[q] * N + ncol[j], bcol[j],
                                         acc[i][j][vg * 4 + q], r0, r1);
                            }
                    }
                    if (NR > 0) reduce_row<MF>(epi, r0, r1, ncol[0] < N ? img[q] : -1, dp[q], ncol[0], lane);
                }
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int vg = 0; vg < NACC / 4; ++vg) {
            int img[4], dp[4];
            typename Epi::Row rc[4];
            const bool one = rowfn4(i, vg, img, dp);
            if (FAST) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    img[q] = uimg;
                    rc[q] = rw;
                }
            } else if (one) {
                if (img[0] >= 0) rc[0] = epi.row(img[0]);
                rc[1] = rc[2] = rc[3] = rc[0];
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (img[q] >= 0) rc[q] = epi.row(img[q]);
            }
            float r0[4] = {0.f, 0.f, 0.f, 0.f}, r1[4] = {0.f, 0.f, 0.f, 0.f};
            typename Epi::Pre pre[FN][4];
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (FAST || (img[q] >= 0 && ncol[j] < N)) {
                        pre[j][q] = epi.pre(rc[q], dp[q], ncol[j], N);
                        epi.pre2(rc[q], pre[j][q]);
                    }
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (FAST || (img[q] >= 0 && ncol[j] < N))
                        epi.post(pre[j][q], rc[q], dp[q], ncol[j], dp[q] * N + ncol[j], bcol[j],
                                 acc[i][j][vg * 4 + q], FAST ? u0 : r0[q], FAST ? u1 : r1[q]);
            if (NR > 0 && !FAST) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    reduce_row<MF>(epi, r0[q], r1[q], ncol[0] < N ? img[q] : -1, dp[q], ncol[0], lane);
            }
        }
    }
}

// Sums over the MF lanes that share output rows, for the NV = 4 or 16 rows v of a lane at
// once: each step halves the rows a lane carries by exchanging the other half with its
// partner, so 16 rows over 32 lanes take 16 shuffles instead of 80.  Returns the sum of the
// lane's row `r`; lanes of one MF group whose index bits past log2(NV) differ hold the same.
template <int MF, int NV> __device__ inline float sum_rows(float (&v)[NV], int lane, int &r) {
    r = 0;
    int n = NV;
#pragma unroll
    for (int mk = MF / 2; mk > 0; mk >>= 1) {
        if (n > 1) {
            n >>= 1;
            const bool up = (lane & mk) != 0;
            r += up ? n : 0;
#pragma unroll
            for (int k = 0; k < NV / 2; ++k)
                if (k < n) {
                    const float mine = up ? v[k + n] : v[k], other = up ? v[k] : v[k + n];
                    v[k] = mine + __shfl_xor(other, mk, 64);
                }
        } else {
            v[0] += __shfl_xor(v[0], mk, 64);
        }
    }
    return v[0];
}

// Epilogue of a wave's 64 rows in a window pass: whole images of tile_px (a power of two, >=
// 16) pixels, rows of ow = 2^low pixels, low >= 2.  A lane's four consecutive rows are
// neighbouring pixels of one row; their window coordinates depend on the lane alone, so a
// record's index and its validity take an add and a compare per pixel instead of the
// divisions and 32-bit multiplications of win_pixel.  Sixteen rows i lie in one image, img0 +
// its number in the block; those past the batch load the last image's records and write
// nothing.  PAIR: columns 16 h + n are channel n of the pixel h further on, g.N / 2 channels.
template <class Epi, int MF, int FM, int FN, bool PAIR = false, class Acc>
__device__ inline void tile_epilogue_win(const Epi &epi, Acc (&acc)[FM][FN], const int (&ncol)[FN],
                                         const float (&bcol)[FN], const Geom &g, int tile_px, int lane,
                                         int row0, long img0, long n_img) {
    constexpr int NGF = Mma<MF>::NACC / 4, NG = FM * NGF, DEPTH = NG < 3 ? NG : 3, NI = FM * MF / 16;
    const int lpx = __builtin_ctz(tile_px), low = __builtin_ctz(g.OW);
    const int N = PAIR ? g.N >> 1 : g.N, step = g.ostr * N;
    const WinMap &w = epi.w;
    const bool one = tile_px >= 64;          // the wave's rows lie in one image
    long img[NI];
    typename Epi::Row rw[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        if (i > 0 && one) {
            img[i] = img[0];
            rw[i] = rw[0];
            continue;
        }
        img[i] = img0 + ((row0 + i * 16) >> lpx);
        rw[i] = epi.row((int)(img[i] < n_img ? img[i] : n_img - 1));
    }
    float sums[2 * NI];
#pragma unroll
    for (int i = 0; i < 2 * NI; ++i) sums[i] = 0.f;
#pragma unroll
    for (int j = 0; j < FN; ++j)
        if (const int n = PAIR ? ncol[j] & 15 : ncol[j], h = PAIR ? ncol[j] >> 4 : 0; n < N) {
            typename Epi::Pre t[NG][4];
            int oi[NG];
            // rows 8 vg + .. of a 32-row fragment, 4 .. of a 16-row one
            auto im = [](int gi) { return MF == 32 ? gi / NGF * 2 + (gi % NGF) / 2 : gi; };
            auto load = [&](int gi) {
                const int i = im(gi);
                const int q = (row0 + gi / NGF * MF + Mma<MF>::row(4 * (gi % NGF), lane)) & (tile_px - 1);
                const int py = q >> low, px = q & (g.OW - 1);
                const int wy = __mul24(py, g.ostr) + g.oy0, wx = __mul24(px, g.ostr) + g.ox0 + h;
                const int y = rw[i].y0 + wy, x = rw[i].x0 + wx;
                const int ri = __mul24(__mul24(y, w.W) + x, N) + n;
                oi[gi] = __mul24(__mul24(wy, w.DW) + wx, N) + n;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    t[gi][e] = epi.at(rw[i], ri + e * step, (unsigned)y < (unsigned)w.H &&
                                                                (unsigned)(x + e * g.ostr) < (unsigned)w.W);
            };
#pragma unroll
            for (int gi = 0; gi < DEPTH - 1; ++gi) load(gi);
#pragma unroll
            for (int gi = 0; gi < NG; ++gi) {
                if (gi + DEPTH - 1 < NG) load(gi + DEPTH - 1);
                __builtin_amdgcn_sched_barrier(0);
                const int i = im(gi);
                if (img[i] < n_img)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        epi.post(t[gi][e], rw[i], 0, n, oi[gi] + e * step, bcol[j],
                                 acc[gi / NGF][j][(gi % NGF) * 4 + e], sums[2 * i], sums[2 * i + 1]);
            }
        }
    if (one) {
        float u0 = sums[0], u1 = sums[1];
#pragma unroll
        for (int i = 1; i < NI; ++i) {
            u0 += sums[2 * i];
            u1 += sums[2 * i + 1];
        }
        if (img[0] < n_img) reduce_wave(epi, u0, u1, img[0], 0, 0, lane);
        return;
    }
    int v;
    const float x = sum_rows<64, 2 * NI>(sums, lane, v);
    const long im = img0 + ((row0 + (v >> 1) * 16) >> lpx);
    if ((lane & (64 / (2 * NI) - 1)) == 0 && im < n_img) atomicAdd((v & 1 ? epi.red1() : epi.red0()) + im, (double)x);
}

// Epilogue of a wave that holds one MF x MF tile of a dense product (rows m0 .., M rows in
// all): every row's records are loaded before the first is used, so the tile pays one memory
// latency (two for the adjoint's dependent loads) instead of one per group of four rows.
// The two sums of a row over the tile's columns go to `a` / `b`, of tile row `r` (each held
// by several lanes; `own` marks one of them).
template <class Epi, int MF, class Acc>
__device__ inline void dense_tile_epilogue(const Epi &epi, const Acc &acc, long m0, long M, int n0,
                                           int N, int lane, float &a, float &b, int &r, bool &own) {
    using MM = Mma<MF>;
    constexpr int NACC = MM::NACC;
    const int n = n0 + MM::col(lane);
    const bool col = n < N;
    const float bcol = col ? epi.colv(n) : 0.f;
    typename Epi::Row rc[NACC];
    typename Epi::Pre pre[NACC];
#pragma unroll
    for (int v = 0; v < NACC; ++v) {
        const long r = m0 + MM::row(v, lane);
        if (r < M) {
            rc[v] = epi.row((int)r);
            if (col) pre[v] = epi.pre(rc[v], 0, n, N);
        }
    }
#pragma unroll
    for (int v = 0; v < NACC; ++v)
        if (col && m0 + MM::row(v, lane) < M) epi.pre2(rc[v], pre[v]);
    float s0[NACC], s1[NACC];
#pragma unroll
    for (int v = 0; v < NACC; ++v) {
        s0[v] = s1[v] = 0.f;
        if (col && m0 + MM::row(v, lane) < M)
            epi.post(pre[v], rc[v], 0, n, n, bcol, acc[v], s0[v], s1[v]);
    }
    own = false;
    if constexpr (Epi::NRED > 0) {
        int v;
        a = sum_rows<MF, NACC>(s0, lane, v);
        b = sum_rows<MF, NACC>(s1, lane, v);
        r = MM::row(v, lane);
        own = (lane & (MF / NACC - 1)) == 0;
    }
}

// fast: see tile_epilogue_impl (wave-uniform).
// LEAN: the other tiles take the one-element-at-a-time path (convolution tiles, where
// they are rare) instead of the batched one (dense products, where every tile is such).
template <class Epi, int MF, int FM, int FN, bool LEAN = false, class Acc, class RowFn>
__device__ inline void tile_epilogue(const Epi &epi, Acc (&acc)[FM][FN], const int (&ncol)[FN],
                                     const float (&bcol)[FN], int N, const RowFn &rowfn4, int lane,
                                     bool fast, int uimg) {
    if (fast)
        tile_epilogue_impl<true, false, Epi, MF, FM, FN>(epi, acc, ncol, bcol, N, rowfn4, lane, uimg);
    else
        tile_epilogue_impl<false, LEAN, Epi, MF, FM, FN>(epi, acc, ncol, bcol, N, rowfn4, lane, -1);
}

}  // namespace dev
}  // namespace bp
