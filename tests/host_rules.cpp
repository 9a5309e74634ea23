// Checks of the library's host rules (see test_host_rules.py): exits with 1 and a message
// where one does not hold.
#include "bound_internal.h"
#include <cstdio>
#include <cstring>
#include <vector>

using namespace bp;

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
    const int n = gemm_candidates(gs, c, kMaxCandidates);
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
    gs.g[0].Bs = &w;
    bool found = false;
    for (int c : listed(gs)) found = found || c == DENSE_SPLIT;
    check(found, "listed with weights");
}

int main(int argc, char **argv) {
    const struct { const char *name; void (*f)(); } tests[] = {{"dense", dense}, {"split_weights", split_weights}};
    for (auto &t : tests)
        if (argc == 2 && !std::strcmp(argv[1], t.name)) {
            t.f();
            return bad;
        }
    std::printf("no such rule\n");
    return 2;
}
