// Internal declarations shared by the gfx950 kernels and the host side of the library.
//
// Layout inside the library: every coefficient tensor is [img][H][W][C] (channels last),
// where img enumerates (instance, spec row) pairs; Linear layers are the 1x1 case.
// Neuron index j inside a layer is therefore (y * W + x) * C + c ("internal order");
// the C ABI uses the C-major order c * H * W + y * W + x.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace bp {

// Implicit-GEMM geometry.  Row m of the GEMM is (img, oy, ox) over an OH x OW grid; the
// A operand gathers A[img][y][x][c] at y = oy*stride - pad_y + ky, x = ox*stride - pad_x
// + kx for k = (ky*kw + kx)*C + c (zero outside the source); B is packed as Bt[N][Kp];
// the result element (m, n) goes to destination pixel (oy*ostr + oy0, ox*ostr + ox0)
// of a [img][DH][DW][N] tensor.
struct Geom {
    int H, W, C;
    int OH, OW;
    int kh, kw, stride, pad_y, pad_x;
    int K, N, Kp;
    int DH, DW, ostr, oy0, ox0;
    float rOW, rM;             // fl(1 / OW), fl(1 / (OH * OW)) for the quotients of qdiv
    float rC, rKW;             // fl(1 / C), fl(1 / kw)
    double rMd;                // 1 / (OH * OW) in FP64 for row indices beyond 2^21
    const float *Bt;
    // Bt in three bf16 parts: dense layers [n][Kc][3][32] (split.hip), transposed
    // convolutions as conv_split.hip packs them (null where it does not take them)
    const unsigned short *Bs;
    int Kc;                    // its 32-wide k chunks
    const float *Bt2;          // a pair's second phase (conv_split.hip)
};

// Reciprocals of a geometry's divisors, taken once on the host (the same correctly
// rounded FP32 quotients a kernel would form).
inline void set_recips(Geom &g) {
    const int m = g.OH * g.OW > 0 ? g.OH * g.OW : 1;
    g.rOW = 1.0f / (float)(g.OW > 0 ? g.OW : 1);
    g.rM = 1.0f / (float)m;
    g.rC = 1.0f / (float)(g.C > 0 ? g.C : 1);
    g.rKW = 1.0f / (float)(g.kw > 0 ? g.kw : 1);
    g.rMd = 1.0 / (double)m;
}

struct GeomSet {
    Geom g[4];
    int n;
};

// Per-neuron relaxation record (Lemma 1) for one instance:
// x = lower slope, y = upper slope, z = upper intercept; w = 0 for a stable neuron,
// -(q + 1) for a split neuron whose first entry in the instance's split list is q, and
// k + 1 for an unstable one, k its slot in the compact rows of saved coefficients (alpha
// free).  Records with w <= 0 have x = y and z = +-0: a split record carries the sign of
// its first entry's constraint in the sign bit of z (-0 for sign -1), which the adjoint
// needs for that entry's beta-gradient (the slope cannot tell it when l = u = 0).
typedef float4 Relax;

// ----- epilogue parameter blocks -----------------------------------------------------
// A row's sums are accumulated in FP64: a tile adds its FP32 partial sums, and with an FP32
// running sum each of these additions rounds at the size of the whole sum, the more often the
// narrower the tiles are.  Error of the spec bounds against FP64 (root mean square, relative)
// with FP32 sums over 64-column tiles / over 16- and 32-column tiles / with FP64 sums: one
// 3x32x32 CNN input 2.8e-7 / 4.6e-7 / 4.0e-8, three inputs of an MLP 784-252-190-158-57-11
// 1.0e-7 / 1.6e-7 / 5.1e-8, 256 of 784-256x6-10 1.1e-7 / 1.1e-7 / 3.7e-8.
// Deterministic row sums: each tile's partial sums of a row go to their own slot
// part[(img * nslot + dp * ncu + n0 / 16) * 2 + {0, 1}] (dp the destination pixel of the
// tile's first row, n0 its first column, ncu = ceil(N / 16)) of a zeroed workspace, and
// launch_det_reduce adds the slots to the accumulators in slot order.
struct DetSums {
    float *part;
    long nslot;
    int ncu;
};

struct RelaxParams {       // G_m = Lambda_m W_m  ->  Lambda_{m-1} = relax(G_m)
    float *out;            // Lambda_{m-1}  [img][D]
    float *save;           // G_m kept for the gradient (nullable): per img, the unstable
                           // neurons only, at slot w - 1 of their record
    const Relax *tab;      // relaxation table of layer m-1, row stride tab_ld
    long tab_ld;
    const float *bias;     // b_{m-1} per channel
    int chan;              // channels of layer m-1 (bias index = j % chan)
    long D;                // width of layer m-1
    double *s, *mag;       // per-img offset accumulator and |term| accumulator
    long img0;             // global img index of local img 0
    int rpi;               // imgs per instance
    float rrpi;            // fl(1 / rpi)
    double rDd, rrpid;     // 1 / D and 1 / rpi in FP64, set with bsum
    const float *bsum;     // [nnz][rpi] split-multiplier term per first split entry and
                           // row, subtracted at the split neuron (nullable: no beta)
    DetSums det;           // deterministic row sums (det.part null: FP64 atomics)
};

struct ConcParams {        // G_1 = Lambda_1 W_1  ->  concretise over the box
    const float *cen, *rad;  // [n_inst][d0] internal order
    long D;                // d0
    double *low, *mag;     // per-img accumulators
    float *save;           // G_1 kept (nullable)
    float *emit;           // coefficient output in C-major order (nullable)
    int chan, hw;          // input shape for the C-major index
    long img0;
    int rpi;
    float rrpi;
    DetSums det;
};

struct AdjParams {         // Lambda_bar_m = G_bar_m W_m^T + s_bar b_m  -> G_bar_{m+1}
    const float *sbar;     // per img: gradient of the offset (0 for infeasible instances)
    const float *bias;     // b_m per channel
    int chan;
    long D;                // width of layer m
    const float *gsave;    // saved G_{m+1} [img][D], compact (slot w - 1 of the record)
    const Relax *tab;
    long tab_ld;
    float *gout;           // G_bar_{m+1} (nullable at the last layer)
    float *gc;             // [img][D] compact: alpha-gradient contributions (k_alpha_grad)
    float *gbeta;          // [nnz][rpi] beta-gradient of first split entries (nullable)
    int hw;                // H*W of layer m (C-major index)
    int rpi;
    float rrpi;
};

struct FwdParams {         // z_m = W_m h_{m-1} + b_m for sample rows
    float *out;            // z_m [img][D]
    const float *bias;     // b_m per channel
    long D;
};

// Receptive-field windows.  A row that bounds one neuron of a convolutional layer has
// non-zero coefficients only inside a window of every layer below, so such passes keep
// [img][window][C] tensors: img r of an instance is the target's neuron r (pixel-major,
// channel fastest; dk further imgs hold the negated rows), whose window at this layer
// starts at (oy * S - P, ox * S - P) for its target pixel (oy, ox).
struct WinMap {
    int H, W;                // the layer's own extent; window pixels outside it hold 0
    int N;                   // its channels
    int DW;                  // pixels per window row
    int S, P;
    int ow, dk;              // target layer: pixels per row, width
    int rpi;                 // imgs per instance
    long img0;
    float rDW, rC, rOw, rrpi;   // fl(1 / .) of DW, the target's channels, ow, rpi
};

// Whether the window epilogues' indices hold for a layer of H x W pixels and windows of `store`
// a side: they form y * W + x by 24-bit multiplications, y and x up to a window outside the
// layer on either side.
inline bool win_index_fits(long H, long W, long store) {
    return (H + 2 * store) * W + 2 * store < (1L << 23) && H + 2 * store < (1L << 23) && W < (1L << 23);
}

// ----- product launchers ---------------------------------------------------------
// A plan picks the kernel of one product: path 0 = automatic (direct convolution when
// the geometry fits, else the implicit GEMM with the default tile), 1 = direct
// convolution with channel chunk cc (0 = largest that fits), 2 = implicit GEMM with tile
// configuration cfg (see gemm_candidates).  Path 0 with cfg 1 (BOUND_OPT_DIRECT_DMA): direct
// convolutions as in path 1 with cfg 1, dense products automatic.
struct Plan {
    int path = 0;
    int cfg = -1;
    int cc = 0;
    // Plans keep the order in which the general kernels add a row's terms: the saved
    // coefficients' signs pick the branch of the adjoint, and some of them are within rounding
    // of 0, so an automatic SAVE_FOR_GRAD pass takes only kernels that give bitwise the same
    // coefficients, and the adjoint, whose gradients move the next step's slopes, the same.  A
    // tuned one takes the general FP32 kernels (whose tiles and channel chunks have orders of
    // their own) and those that repeat such an order, never the bf16 matrix cores.
    bool keep = false;
};
constexpr int kMaxCandidates = 32;

hipError_t gemm_relax(const GeomSet &gs, const float *A, long n_img, const RelaxParams &p,
                      hipStream_t st, const Plan &plan);
hipError_t gemm_conc(const GeomSet &gs, const float *A, long n_img, const ConcParams &p,
                     hipStream_t st, const Plan &plan);
hipError_t gemm_adj(const GeomSet &gs, const float *A, long n_img, const AdjParams &p,
                    hipStream_t st, const Plan &plan);
hipError_t gemm_fwd(const GeomSet &gs, const float *A, long n_img, const FwdParams &p,
                    hipStream_t st, const Plan &plan);
// Valid plans for a product (direct variants first, then GEMM tiles, then, unless it keeps the
// order, the automatic choice); returns the count.
int plan_candidates(const GeomSet &gs, bool keep, Plan *out, int cap);
// gemm.hip: implicit GEMM with an explicit tile configuration (cfg < 0: default)
hipError_t gemm_relax_cfg(const GeomSet &gs, const float *A, long n_img, const RelaxParams &p,
                          hipStream_t st, int cfg);
hipError_t gemm_conc_cfg(const GeomSet &gs, const float *A, long n_img, const ConcParams &p,
                         hipStream_t st, int cfg);
hipError_t gemm_adj_cfg(const GeomSet &gs, const float *A, long n_img, const AdjParams &p,
                        hipStream_t st, int cfg);
hipError_t gemm_fwd_cfg(const GeomSet &gs, const float *A, long n_img, const FwdParams &p,
                        hipStream_t st, int cfg);
int gemm_candidates(const GeomSet &gs, bool keep, int *cfgs, int cap);
// dense.hip: wave-per-tile kernels for dense products with few tiles (configurations that
// follow the GEMM's); dense_auto picks one, or -1 where the LDS-tiled GEMM serves better
//
// Dense means that row m of the product is img m and its columns are all of the result: one
// geometry, one source pixel, one tap on it, one result pixel.  A convolution with one source
// pixel and tap can fall short of that (a stride-2 2x2 layer onto one pixel has four phases,
// a padded 1x1 layer several result pixels) and takes the implicit GEMM's gather.
inline bool is_dense(const GeomSet &gs) {
    const Geom &g = gs.g[0];
    return gs.n == 1 && g.H == 1 && g.W == 1 && g.OH == 1 && g.OW == 1 && g.DH == 1 && g.DW == 1 &&
           g.kh == 1 && g.kw == 1 && g.pad_y == 0 && g.pad_x == 0;
}
// Whether 128 packed rows of K weights (6 bytes each on the bf16 tile) lie within the 32-bit byte
// offsets of the LDS DMA
inline bool dma_fits(const Geom &g) { return 128L * 6 * (g.K + 32L) < (1L << 31); }
enum { DENSE_W32 = 11, DENSE_W16 = 12, DENSE_W16K4 = 13, DENSE_W16K16 = 14, DENSE_W16O = 15, DENSE_SPLIT = 16, DENSE_F32 = 17 };
int dense_auto(const GeomSet &gs, long M, bool keep);
hipError_t dense_relax(const GeomSet &gs, const float *A, long M, const RelaxParams &p, hipStream_t st, int cfg);
hipError_t dense_conc(const GeomSet &gs, const float *A, long M, const ConcParams &p, hipStream_t st, int cfg);
hipError_t dense_adj(const GeomSet &gs, const float *A, long M, const AdjParams &p, hipStream_t st, int cfg);
hipError_t dense_fwd(const GeomSet &gs, const float *A, long M, const FwdParams &p, hipStream_t st, int cfg);
// split.hip: large dense products, on the bf16 matrix cores at FP32 precision (DENSE_SPLIT) or
// by FP32 MFMAs in the general GEMM's order (DENSE_F32)
hipError_t tall_relax(const GeomSet &gs, const float *A, long M, const RelaxParams &p, hipStream_t st, bool split);
hipError_t tall_conc(const GeomSet &gs, const float *A, long M, const ConcParams &p, hipStream_t st, bool split);
hipError_t tall_adj(const GeomSet &gs, const float *A, long M, const AdjParams &p, hipStream_t st);
hipError_t tall_fwd(const GeomSet &gs, const float *A, long M, const FwdParams &p, hipStream_t st);
// Three bf16 parts hold an FP32 value's 24 bits where no part leaves the range of normal bf16
// values: from SPLIT_MAX on the first one rounds to infinity, below SPLIT_MIN the last ones are
// flushed to 0.  Rows outside are formed again by FP32 instructions, and a layer of such
// weights stays with the FP32 kernels: `flags` [3] gets 1 where there are weights past SPLIT_MAX,
// non-zero ones below SPLIT_MIN, and others.
constexpr unsigned SPLIT_MAX = 0x7f7f0000u, SPLIT_MIN = 0x0d800000u;   // bits of 3.39e38, 2^-100
hipError_t launch_pack_split(const float *Bt, int Np, int Kp, int Kc, unsigned short *out, int32_t *flags,
                             hipStream_t st);
// conv.hip: direct convolution (cc = 0: largest chunk that fits; mode 1 or 3: tiles staged
// by LDS DMA, else through registers; mode 2 or 3: 16x16 MFMA tiles for 32 output
// channels); *used = false when the geometry does not fit
hipError_t direct_relax(const GeomSet &gs, const float *A, long n_img, const RelaxParams &p,
                        hipStream_t st, int cc, int mode, bool *used);
hipError_t direct_conc(const GeomSet &gs, const float *A, long n_img, const ConcParams &p,
                       hipStream_t st, int cc, int mode, bool *used);
hipError_t direct_adj(const GeomSet &gs, const float *A, long n_img, const AdjParams &p,
                      hipStream_t st, int cc, int mode, bool *used);
hipError_t direct_fwd(const GeomSet &gs, const float *A, long n_img, const FwdParams &p,
                      hipStream_t st, int cc, int mode, bool *used);
constexpr int DIRECT_AUTO = 4;      // the direct kernels' own choice of staging
int direct_candidates(const GeomSet &gs, int *cc, int *mode, int cap);
// conv_split.hip: relaxing direct convolutions on the bf16 matrix cores at FP32 precision, for
// passes that save nothing; the launchers take what conv_split_fits accepts.  conv_split_size:
// elements of a geometry's packed weights (0: not taken); launch_pack_conv packs them, a
// pair's with the second phase's geometry
bool conv_split_fits(const GeomSet &gs, long n_img, bool window);
bool conv_split_pair_fits(const GeomSet &pair, long n_img);
hipError_t conv_split_relax(const GeomSet &gs, const float *A, long n_img, const RelaxParams &p, hipStream_t st);
hipError_t conv_split_relax_win(const GeomSet &gs, bool pair, const float *A, long n_img, const RelaxParams &p,
                                const WinMap &w, hipStream_t st);
long conv_split_size(const Geom &g);
hipError_t launch_pack_conv(const Geom &g, const Geom *pair, unsigned short *out, int32_t *flags, hipStream_t st);
// window.hip: the products of a window pass (direct convolution, DMA-staged); window_fits
// tells whether the kernels cover a geometry (conc: the concretising step)
bool window_fits(const GeomSet &gs, bool conc);
hipError_t window_relax(const GeomSet &gs, const GeomSet &pair, const float *A, long n_img, const RelaxParams &p,
                        const WinMap &w, hipStream_t st);
hipError_t window_conc(const GeomSet &gs, const float *A, long n_img, const ConcParams &p,
                       const WinMap &w, hipStream_t st);

// ----- auxiliary kernels (aux.hip) ---------------------------------------------------
struct LayerShape {        // output shape of a ReLU layer (for index maps)
    int C, HW;             // channels, pixels
    long off;              // offset in the flat ReLU index
    long d;
};

constexpr int MAX_RELU_LAYERS = 128;

// The ReLU layers' shapes on the host (l) and in device memory (dev), with the device
// prefix sums of the relaxation-table tiles per layer (tile0[m] = tiles of layers < m).
struct NetShapes {
    int n;                 // number of ReLU layers described
    LayerShape l[MAX_RELU_LAYERS];
    const LayerShape *dev;
    const int32_t *tile0;
};
// Tiles of the relaxation-table kernel for one ReLU layer (host and device).
constexpr int PREP_TILE = 1024;
__host__ __device__ inline int prep_tiles(const LayerShape &L) {
    if (L.HW == 1) return (int)((L.d + PREP_TILE - 1) / PREP_TILE);
    if (L.C > PREP_TILE) return L.HW * ((L.C + PREP_TILE - 1) / PREP_TILE);
    const int P = PREP_TILE / L.C;
    return (L.HW + P - 1) / P;
}

hipError_t launch_fill(float *p, long n, float v, hipStream_t st);
// deterministic row sums: s[img] += the slots' first values, mag[img] += their second
// values, each summed in slot order (one wave per img, a fixed shuffle tree)
hipError_t launch_det_reduce(long n_img, long nslot, const float *part, double *s, double *mag,
                             hipStream_t st);
// cnt[0] += NaN count, cnt[1] += Inf count of p[0 .. n) (debug checks)
hipError_t launch_count_nonfinite(const float *p, long n, int32_t *cnt, hipStream_t st);
hipError_t launch_count_nonfinite(const double *p, long n, int32_t *cnt, hipStream_t st);   // as FP32
// input boxes -> centre / radius in internal order (x_lo null: zeros); infeas (nullable):
// cleared for n_inst instances
struct BoxParams {
    long total, d0;          // n_inst * d0 elements
    int n_inst, C0, HW0;
    const float *x_lo, *x_hi;
    float *cen, *rad;
    int32_t *infeas;
};
// relaxation tables of ReLU layers [first, used), their slots when the pass saves, and the box
hipError_t launch_prep_tables(const NetShapes &ns, int first, int used, int n_inst,
                              long n_relu, const float *lo, const float *hi,
                              const int32_t *bound_of, const float *alpha, Relax *tab,
                              int32_t *infeas, int n_bounds, int32_t *slot, int32_t *slot_inv,
                              int32_t *slot_count, int32_t *srow, int max_rows, bool save,
                              const BoxParams &box, hipStream_t st);
hipError_t launch_prep_box(const BoxParams &box, hipStream_t st);
// alpha-gradient of the ReLU layers [layer0, layer0 + layers) from the compact per-row
// contributions gc (sum over an instance's rows per slot, written C-major), then 0 at the
// layers' split neurons; layer l's rows start at gc + gc_rows * (off_l - off_layer0)
hipError_t launch_alpha_grad(int n_inst, int rows, const NetShapes &ns, int layer0, int layers, long gc_rows,
                             long n_relu, const int32_t *srow, const int32_t *slot_count,
                             const int32_t *slot_inv, const float *gc, float *galpha, long ga_ld, int nnz,
                             const int32_t *sp_inst, const int32_t *sp_layer, const int32_t *sp_j,
                             hipStream_t st);
hipError_t launch_prep_splits(const NetShapes &ns, int n_layers_used, int n_inst, long n_relu,
                              const float *lo, const float *hi, const int32_t *bound_of,
                              const int32_t *off, const int32_t *idx, const int8_t *sign,
                              Relax *tab, int32_t *infeas, int32_t *sp_inst,
                              int32_t *sp_layer, int32_t *sp_j, int32_t *sp_dup, int n_bounds,
                              int stop_m, int stop_relu, float *stop_cen, float *stop_rad,
                              hipStream_t st);
hipError_t launch_prep_stop_box(int n_inst, const LayerShape &L, long n_relu, const float *lo,
                                const float *hi, const int32_t *bound_of, int n_bounds, bool relu,
                                float *cen, float *rad, hipStream_t st);
hipError_t launch_box_conc(long img0, long n_img, int rpi, long D, const float *lam, const float *cen,
                           const float *rad, double *low, double *mag, float *save, hipStream_t st);
hipError_t launch_adj_stop_linear(long n_img, int rows, long D, const float *lam, const float *g,
                                  const float *cen, const float *rad, const float *gl,
                                  const int32_t *infeas, float *sbar, const Relax *tab, long tab_ld,
                                  float *gout, float *gc, int C, int HW, hipStream_t st);
hipError_t launch_beta_grad_stop(int nnz, int rows, int layer, long D, const int32_t *sp_inst,
                                 const int32_t *sp_layer, const int32_t *sp_j, const int8_t *sign,
                                 const float *lam, const float *cen, const float *rad,
                                 const float *sbar, float *gbeta, hipStream_t st);
hipError_t launch_init_spec(long img0, long n_img, int rows, int rpi, const float *spec,
                            long dk, int Ck, int HWk, const float *bias_k, float *lam,
                            double *s, double *mag, double *low, hipStream_t st);

struct IdentityParams {
    // target layer k
    int kind;                  // 0 linear, 1 conv
    const float *W;            // user weight of layer k (C-major)
    const float *bias_k;
    int ci, hi_, wi;           // input shape of layer k
    int co, ho, wo;            // output shape of layer k
    int kh, kw, stride, pad;
    long dk, din;              // widths of z_k and of the layer's input
    int rpi;                   // 2*dk (both sides) or dk
    long img0;
    // relax mode (k > 1): table and bias of layer k-1
    const Relax *tab;
    long tab_ld;
    const float *bias_m;
    int chan_m;
    float *out;                // Lambda_{k-1} [img][din]
    const float *bsum;         // split-multiplier terms (see RelaxParams), nullable
    // concretise mode (k == 1)
    const float *cen, *rad;
    float *emit;
    // accumulators
    double *s, *mag, *low;
};
hipError_t launch_init_identity(const IdentityParams &p, long n_img, bool conc, hipStream_t st);
// identity rows of a Linear target (relaxed), W its rows in internal order with stride ldw
hipError_t launch_init_dense(const IdentityParams &p, const float *W, int ldw, long n_img, hipStream_t st);
// lower / upper bounds of z_1 = W x + b over the box (both or lower only)
hipError_t launch_dense1_bounds(const IdentityParams &p, const float *W, int ldw, int n_inst, bool slack,
                                float *lower, float *upper, long ld, float *best, float *best_upper,
                                hipStream_t st);
// identity rows of a convolutional target as windows of layer k-1 (w: that layer's map)
hipError_t launch_init_window(const IdentityParams &p, const WinMap &w, long n_img, hipStream_t st);
// lower / upper bounds of z_1 = conv(x) over the box (both or lower only)
hipError_t launch_conv1_bounds(const IdentityParams &p, int n_inst, bool slack, float *lower, float *upper,
                               long ld, float *best, float *best_upper, hipStream_t st);

// Per first split entry q and row r: sum over the instance's entries on the same neuron
// of sign * beta (the term the relaxation epilogue subtracts at the split neuron).
hipError_t launch_beta_sum(int nnz, int rows, const int32_t *off, const int32_t *idx,
                           const int8_t *sign, const int32_t *sp_inst, const int32_t *sp_layer,
                           const int32_t *sp_dup, const float *beta, float *bsum, hipStream_t st);
hipError_t launch_finalize(long img0, long n_img, int rows, int rpi, const double *s,
                           const double *low, const double *mag, const int32_t *infeas,
                           bool slack, float *lower, float *upper, long ld, float *offset,
                           float *offset_mag, float *best, float *best_upper, hipStream_t st,
                           int pC = 0, int pHW = 0);   // pC: window pass, the target's channels
hipError_t launch_adj_init(long n_img, int rows, long d0, const float *gl, const float *g1,
                           const float *cen, const float *rad, const int32_t *infeas,
                           float *gbar, float *sbar, hipStream_t st);

// beta-gradient of repeated split entries from their neurons' first entries
hipError_t launch_beta_repeat(int nnz, int rows, const int32_t *sp_inst, const int32_t *sp_layer,
                              const int32_t *sp_j, const int32_t *sp_dup, const int8_t *sign, float *gbeta,
                              hipStream_t st);
hipError_t launch_to_internal(long n_img, int C, int HW, const float *x, float *y, hipStream_t st);
hipError_t launch_sample_minmax(long n_sub, int per_sub, long D, int C, int HW, float *z,
                                float *lo, float *hi, long ld, bool relu, float *out, bool merge,
                                hipStream_t st);
hipError_t launch_adam(long n, float *p, const float *g, float *m, float *v, int step,
                       float lr, float b1, float b2, float eps, float gs, float lo, float hi,
                       hipStream_t st);
// Adam constants of one step (bias corrections folded in on the host)
struct AdamArgs {
    float b1, b2, bc1, bc2s, lr, eps, gs, lo, hi;
};
AdamArgs adam_args(int step, float lr, float b1, float b2, float eps, float gs, float lo, float hi);
// alpha-gradient of ReLU layers (as launch_alpha_grad) fused with the Adam step on alpha
// (moments in slot order); clears split neurons' slots of gc first
hipError_t launch_alpha_adam(int n_inst, int rows, const NetShapes &ns, int layer0, int layers, long gc_rows,
                             long n_relu, const int32_t *srow, const int32_t *slot_count,
                             const int32_t *slot_inv, const int32_t *slot, float *gc, float *alpha,
                             float *m, float *v, long ld, int nnz, const int32_t *sp_inst,
                             const int32_t *sp_layer, const int32_t *sp_j, const AdamArgs &a, hipStream_t st);
hipError_t launch_concretize(int n_inst, int rows, long d0, const float *coeff,
                             const float *offset, const float *offset_mag, const float *x_lo,
                             const float *x_hi, bool slack, float *lower, hipStream_t st);

// bab.hip: whether one block picks n of n_dom subdomains, n1 of them in phase 1
bool pick_one_fits(int n_dom, int n, int n1);

// Packing helpers (aux.hip)
hipError_t launch_pack_T(const float *W, int kind, int ci, int hi_, int wi, int co, int ho,
                         int wo, int kh, int kw, int stride, int pad, int py, int px, int ky0,
                         int kx0, int Ty, int Tx, int N, int K, int Kp, int Np, float *Bt,
                         hipStream_t st);
hipError_t launch_pack_F(const float *W, int kind, int ci, int hi_, int wi, int co, int kh,
                         int kw, int N, int K, int Kp, int Np, float *Bt, hipStream_t st);

constexpr float KAPPA_U = 64.0f / 16777216.0f;   // slack factor: 64 * 2^-24

}  // namespace bp
