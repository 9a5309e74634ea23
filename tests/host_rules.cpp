// Checks of the library's host rules (see test_host_rules.py): exits with 1 and a message
// where one does not hold.  The program defines the HIP runtime calls that the library makes,
// so its passes run here without a GPU: allocations are host memory, and a launch is recorded
// by its kernel's name and grid instead of run.
#include "bound.h"
#include "bound_internal.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <cxxabi.h>
#include <functional>
#include <map>
#include <string>
#include <vector>

using namespace bp;

// ---- a HIP runtime that records launches --------------------------------------------
struct Launch { const std::string &name; dim3 grid, block; };
// filled by the library's initialisers, before this program's run
static std::map<const void *, std::string> &kernels() {
    static auto *m = new std::map<const void *, std::string>;
    return *m;
}
static std::vector<Launch> launches;
static std::function<float()> elapsed = [] { return 1.f; };   // of the launches since the last event
static hipError_t last = hipSuccess;
static struct { dim3 grid, block; size_t lds; hipStream_t st; } config;

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *) {
    int st = 0;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    kernels()[host] = d ? d : name;
    std::free(d);
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) {
    config = {g, b, lds, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *st) {
    *g = config.grid; *b = config.block; *lds = config.lds; *st = config.st;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t, hipStream_t) {
    if ((unsigned long)g.x * b.x > 0xffffffffUL) return last = hipErrorInvalidConfiguration;   // as HIP does
    launches.push_back({kernels()[f], g, b});
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
hipError_t hipMalloc(void **p, size_t n) { *p = std::calloc(n, 1); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = elapsed(); return hipSuccess; }
}

// launches whose kernel's name holds every one of `parts`
static int count(std::initializer_list<const char *> parts) {
    int n = 0;
    for (const auto &l : launches) {
        bool all = true;
        for (const char *p : parts) all = all && l.name.find(p) != std::string::npos;
        n += all;
    }
    return n;
}

// ---- networks and passes -------------------------------------------------------------
static std::vector<float> memory(1 << 22);        // stands in for every tensor that no host code reads

static bound_layer conv(int ci, int hw, int co, int k, int s, int p) {
    const int o = (hw + 2 * p - k) / s + 1;
    return bound_layer{BOUND_CONV2D, ci, hw, hw, co, o, o, k, k, s, p, memory.data(), memory.data()};
}
static bound_layer linear(int ci, int hw, int co) {
    return bound_layer{BOUND_LINEAR, ci, hw, hw, co, 1, 1, 1, 1, 1, 0, memory.data(), memory.data()};
}

struct Net {
    bound_net *h = nullptr;
    std::vector<bound_layer> layers;
    Net(std::vector<bound_layer> l, int inst, long rows, long save = 0) : layers(std::move(l)) {
        if (bound_init(layers.data(), (int)layers.size(), inst, rows, save, nullptr, &h) != BOUND_OK) {
            std::printf("bound_init: %s\n", bound_last_error());
            std::exit(1);
        }
    }
    ~Net() { bound_destroy(h); }
    // rows [n, rows] of z_target (rows = 0: the identity) with `flags`; runs f on them
    template <class F> void pass(int target, int n, int rows, int flags, F f) {
        float *m = memory.data();
        const bound_layer &T = layers[target - 1];
        bound_pass p{};
        bound_out o{};
        p.n_inst = n;
        p.rows = rows > 0 ? rows : T.out_c * T.out_h * T.out_w;
        p.target = target;
        p.n_bounds = n;
        p.spec = rows > 0 ? m : nullptr;
        p.lo = p.hi = p.x_lo = p.x_hi = m;
        p.flags = flags;
        o.lower = o.upper = m;
        launches.clear();
        const bound_status s = f(&p, &o);
        if (s != BOUND_OK) {
            std::printf("pass: %s\n", bound_last_error());
            std::exit(1);
        }
    }
    void backward(int target, int n, int rows, int flags) {
        pass(target, n, rows, flags, [&](bound_pass *p, bound_out *o) { return bound_backward(h, p, o, nullptr); });
    }
};

static int bad = 0;
static void check(bool ok, const char *what, int i = 0) {
    if (!ok) {
        std::printf("%s (%d)\n", what, i);
        bad = 1;
    }
}

// one source pixel, one tap on it, c -> n channels, as a Linear layer's products
static Geom pixel(int c, int n) {
    static const float w = 0.f;
    Geom g{};
    g.H = g.W = g.OH = g.OW = g.DH = g.DW = g.kh = g.kw = g.stride = g.ostr = 1;
    g.C = g.K = c;
    g.N = n;
    g.Kp = (c + 15) / 16 * 16;
    g.Bt = &w;
    set_recips(g);
    return g;
}

static GeomSet one(const Geom &g) {
    GeomSet s{};
    s.g[0] = g;
    s.n = 1;
    return s;
}

static std::vector<int> listed(const GeomSet &gs) {
    int c[kMaxCandidates];
    const int n = gemm_candidates(gs, false, c, kMaxCandidates);
    return std::vector<int>(c, c + n);
}

static void dense() {
    check(dense_auto(one(pixel(64, 128)), 64, true) >= 0, "a Linear layer's kernel");
    std::vector<GeomSet> not_dense;
    // the phases of a 2x2 stride-2 layer from 2x2 onto one pixel
    GeomSet ph{};
    ph.n = 4;
    for (int i = 0; i < 4; ++i) {
        ph.g[i] = pixel(64, 128);
        ph.g[i].DH = ph.g[i].DW = ph.g[i].ostr = 2;
        ph.g[i].oy0 = i / 2;
        ph.g[i].ox0 = i % 2;
    }
    not_dense.push_back(ph);
    // one of its phases alone
    not_dense.push_back(one(ph.g[3]));
    // a 1x1 layer with padding 1 on one pixel: 3x3 result pixels
    Geom pad = pixel(64, 128);
    pad.OH = pad.OW = pad.DH = pad.DW = 3;
    pad.pad_y = pad.pad_x = 1;
    set_recips(pad);
    not_dense.push_back(one(pad));
    for (size_t i = 0; i < not_dense.size(); ++i) {
        for (long m : {1L, 64L, 100000L})
            for (bool keep : {false, true}) check(dense_auto(not_dense[i], m, keep) < 0, "dense kernel", (int)i);
        for (int c : listed(not_dense[i])) check(c < 9, "candidate", c);
    }
}

// The bf16 tile needs the weights packed for it, which a convolution's dense products lack.
static void split_weights() {
    const unsigned short w = 0;
    GeomSet gs = one(pixel(64, 128));
    for (long m : {1L, 100000L}) {
        check(dense_auto(gs, m, false) != DENSE_SPLIT, "chosen without weights");
        gs.g[0].Bs = &w;
        check((dense_auto(gs, m, false) == DENSE_SPLIT) == (m > 1), "chosen with weights");
        gs.g[0].Bs = nullptr;
    }
    for (int c : listed(gs)) check(c != DENSE_SPLIT, "listed without weights");
    check(tall_relax(gs, nullptr, 1, RelaxParams{}, nullptr, true) == hipErrorInvalidValue, "relaxing product");
    check(tall_conc(gs, nullptr, 1, ConcParams{}, nullptr, true) == hipErrorInvalidValue, "concretising product");
    // nor may 128 rows of them pass the DMA's 32-bit offsets
    GeomSet wide = one(pixel(3000000, 4096));
    wide.g[0].Bs = &w;
    for (bool keep : {false, true}) check(dense_auto(wide, 4096, keep) < 0, "chosen for too wide rows");
    for (int c : listed(wide)) check(c != 9 && c != 10 && c < DENSE_SPLIT, "listed for too wide rows", c);
    check(tall_relax(wide, nullptr, 4096, RelaxParams{}, nullptr, false) == hipErrorInvalidValue, "too wide rows");
    gs.g[0].Bs = &w;
    bool found = false;
    for (int c : listed(gs)) found = found || c == DENSE_SPLIT;
    check(found, "listed with weights");
}

// BOUND_OPT_DIRECT_DMA: every direct convolution stages by LDS DMA (k_conv's last template
// argument), also where few blocks would keep the registers, and none is replaced by another
// kernel.
static void direct_dma() {
    Net net({conv(4, 8, 16, 3, 1, 1), conv(16, 8, 32, 3, 1, 1), conv(32, 8, 64, 3, 1, 1), linear(64, 8, 4)}, 2, 64, 64);
    for (int flags : {0, (int)BOUND_SAVE_FOR_GRAD})
        for (int on : {0, 1}) {
            bound_set_options(net.h, on ? BOUND_OPT_DIRECT_DMA : 0);
            net.backward(4, 2, 3, flags);
            check(count({"k_conv<", "EpiRelax", "true>"}) == (on ? 2 : 0), "relaxing products by DMA", flags);
            if (on) check(count({"k_conv_split"}) == 0, "another kernel", flags);
        }
}

// The tuner, when one kernel would win every timing it takes part in: a saving pass and its
// gradient never time the bf16 tile or the kernels that split K, and their plans do not govern
// passes that save nothing, which may choose those and keep the automatic choice among theirs.
static void tuning() {
    const long n = 4096, R = 8;           // 256 tiles of 128 x 128
    for (const char *best : {"k_dense_tall<bp::dev::EpiRelax, 4, true>", "k_conv_split", "16, 4, false>"}) {
        Net net({conv(4, 8, 16, 3, 1, 1), conv(16, 8, 32, 3, 1, 1), conv(32, 8, 32, 3, 1, 1), linear(32, 8, 256),
                 linear(256, 1, 64)}, (int)n, n * R, n * R);
        elapsed = [&] { return launches.back().name.find(best) != std::string::npos ? .5f : 1.f; };
        auto tune = [&](int flags) {
            net.pass(5, n, R, flags, [&](bound_pass *p, bound_out *o) {
                return bound_autotune(net.h, p, o, memory.data(), nullptr);
            });
        };
        tune(BOUND_SAVE_FOR_GRAD);
        check(count({best}) == 0, "timed for a saving pass");
        net.backward(5, n, R, BOUND_SAVE_FOR_GRAD);
        check(count({best}) == 0, "launched by a saving pass");
        check(count({"k_conv<", "EpiRelax"}) + count({"k_gemm<", "EpiRelax"}) >= 2, "its convolutions");
        net.backward(5, n, R, 0);
        check(count({"k_conv_split"}) == 1 && count({"k_dense_tall", "true>"}) >= 1, "a saving pass's plans elsewhere");
        tune(0);
        check(count({best}) > 0, "not timed for a pass that saves nothing");
        net.backward(5, n, R, 0);
        check(count({best}) > 0, "not kept for a pass that saves nothing");
        net.backward(5, n, R, BOUND_SAVE_FOR_GRAD);
        check(count({best}) == 0, "its plans in a saving pass");
        elapsed = [] { return 1.f; };
    }
}

// Passes of more instances than one launch takes threads for: the box bounds of z_1 (z_1's
// values go up to 2^32 and beyond, in chunks), and the tables with the box in one launch.
static void large() {
    Net fc({linear(4, 1, 8192)}, 65537, 1024);
    fc.backward(1, 65537, 0, BOUND_BOTH_SIDES);
    check(count({"k_dense1_bounds"}) >= 2, "dense");
    Net cv({conv(1, 64, 16, 3, 1, 1)}, 65537, 1024);
    cv.backward(1, 65537, 0, BOUND_BOTH_SIDES);
    check(count({"k_conv1_bounds"}) >= 2, "conv");
    const int n = 1 << 21;
    Net deep({linear(1024, 1, 8), linear(8, 1, 8), linear(8, 1, 8), linear(8, 1, 8), linear(8, 1, 8), linear(8, 1, 2)},
             n, 1024);
    deep.backward(6, n, 1, 0);
    check(count({"k_prep_tables"}) == 1 && count({"k_prep_box"}) == 1, "tables and box");
    long rows = 0;      // every instance of the dense pass once: 4 waves a block, 1024 rows of 8 an instance
    fc.backward(1, 65537, 0, BOUND_BOTH_SIDES);
    for (auto &l : launches)
        if (l.name.find("k_dense1_bounds") != std::string::npos) rows += (long)l.grid.x * 4 / 1024;
    check(rows == 65537, "instances", (int)rows);
}

// Window passes form y * W + x by 24-bit multiplications: the rule against these products at
// the corners of every accepted layer, and a pass past it does not run on windows.
static void window_index() {
    auto mul24 = [](long a, long b) { return (int)((unsigned)(int)((a << 40) >> 40) * (unsigned)(int)((b << 40) >> 40)); };
    for (long store : {4L, 32L, 512L})
        for (long H : {1L, 7L, 100L, 2047L, 2868L, 2896L, 4096L, 70000L, 5000000L})
            for (long W : {1L, 3L, 64L, 2048L, 2896L, 4095L, 8191L, 100000L, 8000000L}) {
                if (!win_index_fits(H, W, store)) continue;
                for (long y : {-store, 0L, H - 1, H + store - 1})
                    for (long x : {-store, 0L, W - 1, W + store - 1}) {
                        const long p = y * W + x;
                        check(mul24(y, W) + x == p && (int)mul24(p, 8) == (int)(p * 8), "index", (int)p);
                    }
            }
    check(win_index_fits(2048, 2048, 32), "an ordinary large layer");
    for (int hw : {64, 2904}) {           // 2904 x 2904 pixels are more than 2^23
        Net net({conv(4, hw, 16, 3, 1, 1), conv(16, hw, 16, 2, 2, 0), conv(16, hw / 2, 16, 2, 2, 0),
                 conv(16, hw / 4, 1, 3, 1, 1), linear(1, hw / 4, 1)}, 1, 8);
        // (whole layers of that width are past the implicit GEMM's own limit: the pass is refused)
        net.pass(4, 1, 0, 0, [&](bound_pass *p, bound_out *o) {
            const bound_status s = bound_backward(net.h, p, o, nullptr);
            check((s == BOUND_OK) == (hw == 64), "accepted", hw);
            return BOUND_OK;
        });
        check((count({"k_init_window"}) > 0) == (hw == 64), "windows", hw);
    }
}

// What the passes of test_gpu_window_loops.py reach: blocks of several groups with a ragged end,
// and windows of 16 pixels a side.
static void window_loops() {
    Net net({conv(3, 32, 16, 3, 1, 1), conv(16, 32, 32, 4, 2, 1), conv(32, 16, 32, 3, 1, 1), conv(32, 16, 64, 4, 2, 1),
             linear(64, 8, 2)}, 5, 81901);
    auto grid = [](const char *kernel, const char *epi) {
        for (auto &l : launches)
            if (l.name.find(kernel) != std::string::npos && l.name.find(epi) != std::string::npos) return (long)l.grid.x;
        return 0L;
    };
    net.backward(3, 5, 0, BOUND_BOTH_SIDES);
    // 5119 groups of 16 images, two pairs of phases, two groups a block: 2560 blocks a pair
    check(grid("k_conv_split", "EpiRelaxWin, true>") == 2560 * 2, "pairs", (int)grid("k_conv_split", "EpiRelaxWin, true>"));
    net.backward(4, 5, 0, BOUND_BOTH_SIDES);
    // 40960 rows in groups of 4 images: 10240 tiles, two a block
    check(grid("k_conv_split", "EpiRelaxWin, false>") == 5120, "single phases",
          (int)grid("k_conv_split", "EpiRelaxWin, false>"));
    Net wide({conv(3, 20, 32, 3, 1, 1), conv(32, 20, 32, 3, 1, 1), conv(32, 20, 32, 3, 1, 1), conv(32, 20, 32, 3, 1, 1),
              conv(32, 20, 32, 3, 1, 1), linear(32, 20, 2)}, 1, 25600);
    wide.backward(5, 1, 0, BOUND_BOTH_SIDES);
    // 25600 rows: 256 pixels a window are a tile of one image, six of them a block
    check(count({"k_init_window"}) == 1 && launches[launches.size() - 3].grid.x == (25600 + 5) / 6, "16 a side",
          (int)launches[launches.size() - 3].grid.x);
}

// BOUND_OPT_CHECK checks the window kernels that full CROWN runs without it: the first windows,
// every product and the concretised sums.
static void debug_windows() {
    Net net({conv(4, 16, 16, 3, 1, 1), conv(16, 16, 16, 3, 1, 1), conv(16, 16, 16, 3, 1, 1), linear(16, 16, 2)}, 1, 8192);
    bound_set_options(net.h, BOUND_OPT_CHECK);
    net.backward(3, 1, 0, BOUND_BOTH_SIDES);
    check(count({"k_init_window"}) == 1 && count({"EpiRelaxWin"}) == 1 && count({"EpiConcWin"}) == 1, "windows");
    check(count({"k_count_nonfinite"}) == 3, "checks", count({"k_count_nonfinite"}));
}

// One block picks only where that was measured faster than the device-wide sort.
static void picks() {
    struct { int n_dom, n, n1; bool one; } t[] = {
        {300, 64, 48, true}, {1000, 700, 700, true}, {2048, 1500, 1125, true}, {4096, 2048, 1024, true},
        {60000, 1024, 768, true}, {8192, 2048, 2048, true}, {8192, 4096, 2048, true}, {32768, 2048, 2048, true},
        {65536, 2048, 1536, true}, {1000, 1000, 750, false}, {4096, 3072, 1536, false}, {8192, 6000, 3000, false},
        {8193, 5461, 4095, false}, {12000, 3072, 3072, false}, {32769, 2048, 2048, false}, {32769, 3072, 1536, false},
        {45000, 64, 64, false}, {65537, 64, 48, false}};
    for (auto &q : t) check(pick_one_fits(q.n_dom, q.n, q.n1) == q.one, "one block", q.n_dom);
}

// The dense kernels' lines, on either side.
static void dense_lines() {
    struct { int K, N; long M; int cfg; } t[] = {
        {64, 64, 576, DENSE_W16}, {64, 64, 1536, DENSE_W32}, {64, 16, 4608, DENSE_W32}, {10, 512, 200, DENSE_W32},
        {4096, 512, 1, DENSE_W16K4}, {4096, 512, 576, DENSE_W16K4}, {4096, 512, 1152, DENSE_W32},
        {4096, 512, 4608, DENSE_W32}, {2048, 2048, 1152, DENSE_W32}, {512, 4096, 200, DENSE_W32},
        {1000, 40, 9216, DENSE_W16K4}, {1000, 40, 16384, DENSE_W16}, {1000, 16, 9216, DENSE_W16K4},
        {256, 256, 16384, DENSE_SPLIT}};
    const unsigned short w = 0;
    for (auto &q : t) {
        GeomSet gs = one(pixel(q.K, q.N));
        gs.g[0].Bs = &w;
        check(dense_auto(gs, q.M, false) == q.cfg, "dense kernel", dense_auto(gs, q.M, false));
    }
}

int main(int argc, char **argv) {
    const struct { const char *name; void (*f)(); } tests[] = {{"dense", dense}, {"split_weights", split_weights}, {"direct_dma", direct_dma}, {"tuning", tuning}, {"large", large}, {"window_index", window_index}, {"window_loops", window_loops}, {"debug_windows", debug_windows}, {"picks", picks}, {"dense_lines", dense_lines}};
    for (auto &t : tests)
        if (argc == 2 && !std::strcmp(argv[1], t.name)) {
            t.f();
            return bad;
        }
    std::printf("no such rule\n");
    return 2;
}
