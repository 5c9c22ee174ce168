// Host checks of the single-pass plan (test infrastructure): the runtime is
// included as source, handles are planned without a device (size_only), and
// the block tables and the admission are compared with a node-by-node reading
// of what each block computes.  The kernels' launches come from the library.
//   plan_driver masks   what a block's variant must handle, tile limits, planes
//                       in the event masks, one owner per node
//   plan_driver routes  which kernels AUTO takes, forward and adjoint
//   plan_driver spans   absorber memories, planes and eps rows of admitted
//                       domains within the 31-bit offsets of their descriptors
#include "../../paper_2609_30039_amd/csrc/fdtd_runtime.cpp"

#include <random>

namespace {

int failures = 0;

// the variant that k_pass and k_adj_pass run for a block's mask
int fwd_variant(int m) { return m < kPassMix || m == kPassMix || m == (kPassMix | kPassX) || m == (kPassMix | kPassZ) ? m : (int)kPassAll; }
int adj_variant(int m) { return m < kAdjPer || m == (kAdjPer | kPassZ) || m == kAdjLor ? m : (int)kAdjAll; }

struct Case {
    fdtd_domain_desc d;
    fdtd_options o;
};

Case blank(int nx, int ny, int nz, int dtype, int kernel, int tile_kz) {
    Case c;
    std::memset(&c, 0, sizeof c);
    c.d.n[0] = nx;
    c.d.n[1] = ny;
    c.d.n[2] = nz;
    c.d.courant = 0.99 / std::sqrt(3.0);
    c.d.pml_m = 3;
    c.d.pml_kappa_max = 5;
    c.d.pml_sigma_max = 3;
    c.d.pml_alpha_max = 0.05;
    c.d.eps_bg = 1.0;
    c.d.grad = 1;
    for (int a = 0; a < 3; ++a) c.d.grad_hi[a] = c.d.n[a];
    c.o.dtype = dtype;
    c.o.kernel = kernel;
    c.o.tile_kz = tile_kz;
    c.o.max_steps = 2;
    return c;
}

void periodic(Case& c, int a, int sign) {
    c.d.periodic[a] = 1;
    c.d.bloch_sign[a] = sign;
    c.d.pml[2 * a] = c.d.pml[2 * a + 1] = 0;
}

void box(Case& c, const int lo[3], const int hi[3], int poles) {
    c.d.n_lorentz = 1;
    for (int a = 0; a < 3; ++a) {
        c.d.lorentz.lo[a] = lo[a];
        c.d.lorentz.hi[a] = hi[a];
    }
    c.d.lorentz.n_poles = poles;
    for (int p = 0; p < poles; ++p) c.d.lorentz.poles[p] = {FDTD_POLE_LORENTZ, 1.2, 0.4, 0.02};
}

std::string name(const Case& c) {
    char b[320];
    const auto& d = c.d;
    snprintf(b, sizeof b, "%dx%dx%d %s kernel %d kz %d pml %d %d %d %d %d %d per %d %d box %d %d..%d %d..%d %d..%d", d.n[0], d.n[1],
             d.n[2], c.o.dtype == FDTD_F32 ? "f32" : "f64", c.o.kernel, c.o.tile_kz, d.pml[0], d.pml[1], d.pml[2], d.pml[3], d.pml[4],
             d.pml[5], d.periodic[0], d.periodic[1], d.n_lorentz, d.lorentz.lo[0], d.lorentz.hi[0], d.lorentz.lo[1], d.lorentz.hi[1],
             d.lorentz.lo[2], d.lorentz.hi[2]);
    return b;
}

template <typename T>
bool plan(Handle<T>& h, const Case& c) {
    h.size_only = true;
    if (int rc = h.create(&c.d, 1, &c.o)) {
        std::printf("%s: refused, %d %s\n", name(c).c_str(), rc, h.err.c_str());
        ++failures;
        return false;
    }
    return true;
}

// ADJ: the adjoint's blocks.  Per owned node the E nodes that its H update (or
// its transpose) reads are it and its neighbours one step forward, across a
// seam too; the H terms those take are one step back.
template <typename T, bool ADJ>
void check_blocks(const Handle<T>& h, const Case& c) {
    const DomDev<T>& d = h.dd[0];
    constexpr int V = kPassGroup<T>;
    const std::vector<int4>& tab = ADJ ? h.aptab : h.ptab;
    const int nt = ADJ ? h.cfg.ant : h.cfg.pnt, nq = (d.n[0] + V - 1) / V;
    std::vector<unsigned char> owner((size_t)d.n[0] * d.n[1] * d.n[2], 0);
    auto bad = [&](const char* what, const int4& a, const int4& b) {
        if (failures++ < 20)
            std::printf("%s: %s %s: mask %d, groups %d..%d, rows %d..%d, planes %d..%d\n", name(c).c_str(), ADJ ? "adjoint" : "forward",
                        what, a.y, a.z, a.w, b.x, b.y, b.z, b.w);
    };
    for (size_t q = 0; q + 1 < tab.size(); q += 2) {
        const int4 a = tab[q], b = tab[q + 1];
        if (a.x < 0) continue;
        const int wt = a.w - a.z + (d.per[0] || a.z > 0) + (d.per[0] || a.w < nq);
        const int rt = b.y - b.x + (d.per[1] || b.x > 0) + (d.per[1] || b.y < d.n[1]);
        if (wt * rt > nt || rt > kPassMaxRows || wt > (ADJ ? kAdjMaxGroups : kPassMaxGroups) || b.w - b.z > kPassMaxPlanes ||
            a.w <= a.z || b.y <= b.x || b.w <= b.z)
            bad("tile out of its limits", a, b);
        if (!ADJ && b.w - b.z + 1 > 64)   // the march's planes, halo included, in the event masks
            bad("more planes than the event masks have bits", a, b);
        const int have = ADJ ? adj_variant(a.y) : fwd_variant(a.y), seam = ADJ ? (int)kAdjPer : (int)kPassMix,
                  disp = ADJ ? (int)kAdjLor : (int)kPassMix;
        int need = 0;
        auto slab = [&](int ax, int x) { return x < d.L[ax][0] || x >= d.n[ax] - d.L[ax][1] ? 1 << ax : 0; };
        for (int k = b.z; k < b.w; ++k)
            for (int j = b.x; j < b.y; ++j)
                for (int i = a.z * V; i < std::min(a.w * V, d.n[0]); ++i) {
                    owner[((size_t)k * d.n[1] + j) * d.n[0] + i]++;
                    for (int f = 0; f < 4; ++f) {   // E nodes: this one, one forward along x, y, z
                        int x[3] = {i, j, k};
                        if (f) ++x[f - 1];
                        bool past = false;
                        for (int ax = 0; ax < 3; ++ax)
                            if (x[ax] == d.n[ax]) {
                                x[ax] = 0;
                                if (d.per[ax]) need |= seam;
                                else past = true;
                            }
                        if (past) continue;
                        bool in = d.has_lor;
                        for (int ax = 0; ax < 3; ++ax) in = in && x[ax] >= d.llo[ax] && x[ax] < d.lhi[ax];
                        if (in) need |= disp;
                        for (int ax = 0; ax < 3; ++ax) {
                            need |= slab(ax, x[ax]);
                            if (d.per[ax] && x[ax] == 0) need |= seam;
                            if (ADJ && x[ax] > 0) need |= slab(ax, x[ax] - 1);   // the H term along ax of the node one back
                        }
                    }
                }
        if (need & ~have) bad("variant lacks what a node meets", a, b);
    }
    size_t wrong = 0;
    for (unsigned char o : owner) wrong += o != 1;
    if (wrong && failures++ < 20)
        std::printf("%s: %s: %zu nodes not owned once\n", name(c).c_str(), ADJ ? "adjoint" : "forward", wrong);
}

template <typename T>
int check_masks(const Case& c) {
    Handle<T> h;
    if (!plan(h, c)) return 0;
    if (h.dd[0].pass) check_blocks<T, false>(h, c);
    if (h.dd[0].apass) check_blocks<T, true>(h, c);
    return h.dd[0].pass + h.dd[0].apass;
}

int check_masks(const Case& c) { return c.o.dtype == FDTD_F32 ? check_masks<float>(c) : check_masks<double>(c); }

void masks() {
    std::mt19937 rng(7);
    auto pick = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
    int taken = 0;
    // a box on the low side of a seam, below the last tile
    for (int dtype : {FDTD_F32, FDTD_F64})
        for (int poles : {1, 3})
            for (int a = 0; a < 2; ++a) {
                Case c = blank(a ? 48 : 120, 48, 40, dtype, FDTD_KERNEL_AUTO, 0);
                c.d.pml[4] = c.d.pml[5] = 6;
                periodic(c, 0, 1);
                periodic(c, 1, -1);
                int lo[3] = {0, 0, 15}, hi[3] = {c.d.n[0], c.d.n[1], 25};
                hi[a] = 5;
                box(c, lo, hi, poles);
                taken += check_masks(c);
                std::swap(lo[a], hi[a]);   // on its high side only
                lo[a] = c.d.n[a] - 1;
                hi[a] = c.d.n[a];
                box(c, lo, hi, poles);
                taken += check_masks(c);
            }
    for (int q = 0; q < 400; ++q) {
        const int big = pick(0, 3) == 0;
        Case c = blank(pick(1, big ? 150 : 60), pick(1, 60), pick(1, 70), pick(0, 1) ? FDTD_F64 : FDTD_F32,
                       pick(0, 1) ? FDTD_KERNEL_AUTO : FDTD_KERNEL_ONEPASS, 0);
        if (c.o.kernel == FDTD_KERNEL_ONEPASS && pick(0, 1)) c.o.tile_kz = pick(1, 80);
        for (int a = 0; a < 3; ++a)
            for (int s = 0; s < 2; ++s)
                if (pick(0, 2)) c.d.pml[2 * a + s] = pick(0, c.d.n[a] / 2);
        for (int a = 0; a < 2; ++a)
            if (pick(0, 2) == 0) {
                if (a == 0 && c.d.n[0] % 2) c.d.n[0]++, c.d.grad_hi[0]++;
                periodic(c, a, pick(0, 1) ? 1 : -1);
            }
        if (pick(0, 2)) {
            int lo[3], hi[3];
            for (int a = 0; a < 3; ++a) {
                lo[a] = pick(0, 1) ? 0 : pick(0, c.d.n[a] - 1);
                hi[a] = pick(lo[a] + 1, c.d.n[a]);
            }
            box(c, lo, hi, pick(0, 1) ? 1 : 3);
        }
        taken += check_masks(c);
    }
    // the larger block shapes
    for (int per = 0; per < 2; ++per)
        for (int dtype : {FDTD_F32, FDTD_F64}) {
            Case c = blank(per ? 200 : 203, 170, dtype == FDTD_F32 ? 310 : 170, dtype, FDTD_KERNEL_AUTO, 0);
            for (int f = 0; f < 6; ++f) c.d.pml[f] = 5 + f;
            if (per) {
                periodic(c, 0, -1);
                periodic(c, 1, 1);
            }
            const int lo[3] = {0, 0, 40}, hi[3] = {90, 9, 60};
            box(c, lo, hi, 1);
            taken += check_masks(c);
        }
    Case c = blank(350, 350, 352, FDTD_F32, FDTD_KERNEL_AUTO, 0);
    for (int f = 0; f < 6; ++f) c.d.pml[f] = 10;
    taken += check_masks(c);
    if (taken < 300 && ++failures) std::printf("only %d plans took a single pass\n", taken);
}

// bytes from the first to the end of the last absorber array of an axis (the
// kernels' psi_range), from the pointers that layout gives
template <typename T, typename P>
double span(const DomDev<T>& d, int a, const P& psiE, const P& psiH) {
    double lo = 1e30, hi = 0;
    for (int side = 0; side < 2; ++side) {
        if (!d.L[a][side]) continue;
        const double e0 = (double)(size_t)psiE[a][side][0], h0 = (double)(size_t)psiH[a][side][0];
        if (h0 - e0 != (double)(size_t)psiE[a][side][1] - h0 || h0 - e0 != (double)(size_t)psiH[a][side][1] - (double)(size_t)psiE[a][side][1])
            ++failures, std::printf("axis %d side %d: arrays not at one distance\n", a, side);
        lo = std::min(lo, e0);
        hi = std::max(hi, e0 + 4 * (h0 - e0));
    }
    return hi > lo ? hi - lo : 0;
}

template <typename T>
int check_spans(const Case& c) {
    Handle<T> h;
    if (!plan(h, c)) return 0;
    Arena ar[4];
    for (int q = 0; q < 4; ++q) {
        ar[q].base = (char*)((size_t)(q + 1) << 44);   // never read
        ar[q].assign = true;
    }
    h.layout(ar[0], ar[1], ar[2], ar[3]);
    const DomDev<T>& d = h.dd[0];
    const double lim = 2147483648.0;   // an offset of it must lie outside
    double most = (double)d.plane * sizeof(T);
    for (int a = 0; a < 3; ++a) {
        most = std::max(most, span(d, a, d.psiE, d.psiH));
        if (d.grad) most = std::max(most, span(d, a, d.psiEa, d.psiHa));
    }
    if ((d.pass || d.apass) != (most < lim)) {
        ++failures;
        std::printf("%s: span %.6e, pass %d, adjoint %d\n", name(c).c_str(), most, d.pass, d.apass);
    }
    return 1;
}

void spans() {
    struct S {
        int n[3], L, dtype;
    };
    // odd numbers of cells of x slabs round up to pairs, by two on the high side of an odd nx
    const S set[] = {{{101, 2500, 2500}, 10, FDTD_F32}, {{100, 3000, 3000}, 7, FDTD_F32}, {{101, 1800, 1800}, 10, FDTD_F64},
                     {{100, 2500, 2500}, 10, FDTD_F32}, {{100, 2600, 2600}, 10, FDTD_F32}, {{41, 4000, 4000}, 1, FDTD_F32},
                     {{2501, 81, 2500}, 40, FDTD_F32},  {{3001, 3001, 40}, 7, FDTD_F64},   {{200, 200, 200}, 11, FDTD_F64}};
    for (const S& e : set)
        for (int sides = 1; sides < 4; ++sides) {
            Case c = blank(e.n[0], e.n[1], e.n[2], e.dtype, FDTD_KERNEL_ONEPASS, 0);
            for (int a = 0; a < 3; ++a) {
                if (sides & 1) c.d.pml[2 * a] = e.L;
                if (sides & 2) c.d.pml[2 * a + 1] = e.L;
            }
            if (e.dtype == FDTD_F32) check_spans<float>(c);
            else check_spans<double>(c);
        }
    // sizes a little either side of the limit
    std::mt19937 rng(11);
    auto pick = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
    for (int q = 0; q < 60; ++q) {
        const bool f64 = pick(0, 1);
        const int L = pick(1, 12), M = pick(0, 12), nx = pick(L + M + 4, L + M + 60);
        const double rows = 2147483648.0 / (4.0 * (f64 ? 8 : 4) * (L + M)) * (0.7 + 0.01 * pick(0, 35));
        const int ny = pick(300, 3000), nz = std::max(8, (int)(rows / ny));
        Case c = blank(nx, ny, nz, f64 ? FDTD_F64 : FDTD_F32, FDTD_KERNEL_ONEPASS, 0);
        c.d.pml[0] = L;
        c.d.pml[1] = M;
        if (f64) check_spans<double>(c);
        else check_spans<float>(c);
    }
}

// n^3 cells, pml absorbing cells on walled axes, box lo..hi per axis (hi 0:
// none), periodic x and y; expected: single pass forward, adjoint
void routes() {
    struct R {
        int n, dtype, pml, per, lo, hi, poles, fwd, adj;
        bool diag = false;
        int kernel = FDTD_KERNEL_AUTO, tile_kz = 0;
    };
    const int f = FDTD_F32, d = FDTD_F64;
    const R set[] = {
        {140, f, 10, 0, 0, 0, 0, 1, 1},      {160, f, 10, 0, 0, 0, 0, 0, 1},     {212, f, 10, 0, 0, 0, 0, 1, 1},
        {148, f, 10, 0, 0, 0, 0, 1, 1},      {148, f, 10, 0, 0, 0, 0, 0, 1, true}, {132, f, 30, 0, 0, 0, 0, 0, 1},
        {116, d, 10, 0, 0, 0, 0, 1, 1},      {125, d, 10, 0, 0, 0, 0, 0, 1},     {170, d, 10, 0, 0, 0, 0, 1, 1},
        {150, f, 10, 0, 10, 140, 1, 0, 1},   {100, f, 10, 0, 10, 90, 1, 0, 1},   {100, f, 10, 0, 40, 72, 1, 1, 1},
        {212, f, 10, 0, 10, 202, 1, 1, 1},   {212, f, 10, 0, 10, 202, 3, 0, 1},  {212, f, 10, 0, 10, 202, 16, 1, 1},
        {170, d, 10, 0, 10, 160, 16, 0, 1},  {212, f, 10, 0, 42, 170, 2, 0, 1},  {212, f, 10, 0, 56, 156, 3, 1, 1},
        {128, f, 10, 1, 0, 128, 16, 1, 1},   {128, f, 10, 1, 0, 128, 3, 0, 1},   {256, f, 10, 1, 0, 256, 3, 1, 0},
        {200, f, 10, 1, 11, 189, 1, 0, 1},   {200, f, 10, 1, 11, 189, 16, 0, 0}, {180, d, 10, 1, 11, 169, 3, 1, 0},
        {128, d, 10, 1, 0, 128, 1, 0, 0},    {256, f, 10, 0, 64, 192, 1, 1, 0},  {256, f, 10, 0, 96, 160, 16, 1, 1},
        {300, f, 10, 0, 86, 214, 16, 1, 1},  {250, d, 10, 0, 64, 192, 16, 1, 0}, {250, d, 10, 0, 64, 192, 6, 1, 1},
        {256, f, 10, 0, 64, 192, 16, 1, 1, false, FDTD_KERNEL_ONEPASS},          {256, f, 10, 0, 64, 192, 1, 0, 0, false, FDTD_KERNEL_SPLIT},
        {140, f, 10, 0, 0, 0, 0, 0, 0, false, FDTD_KERNEL_AUTO, 8},
    };
    std::vector<double> eps;
    for (const R& r : set) {
        Case c = blank(r.n, r.n, r.n, r.dtype, r.kernel, r.tile_kz);
        for (int q = 0; q < 6; ++q) c.d.pml[q] = r.pml;
        if (r.per) {
            periodic(c, 0, 1);
            periodic(c, 1, -1);
        }
        const int lo[3] = {r.lo, r.lo, r.per && r.hi == r.n ? 10 : r.lo}, hi[3] = {r.hi, r.hi, r.per && r.hi == r.n ? r.n - 10 : r.hi};
        if (r.hi) box(c, lo, hi, r.poles);
        if (r.diag) {
            c.d.eps_kind = FDTD_EPS_DIAG;
            size_t cells = 1;
            for (int a = 0; a < 3; ++a) {
                c.d.eps_lo[a] = r.pml;
                c.d.eps_hi[a] = r.n - r.pml;
                cells *= (size_t)(r.n - 2 * r.pml);
            }
            eps.assign(3 * cells, 2.0);
            c.d.eps = eps.data();
        }
        auto check = [&](auto& h) {
            if (!plan(h, c)) return;
            if (h.dd[0].pass == r.fwd && h.dd[0].apass == r.adj) return;
            ++failures;
            std::printf("%s, poles %d: forward %d, adjoint %d\n", name(c).c_str(), r.poles, h.dd[0].pass, h.dd[0].apass);
        };
        if (r.dtype == FDTD_F32) {
            Handle<float> h;
            check(h);
        } else {
            Handle<double> h;
            check(h);
        }
    }
}

}  // namespace

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "masks") masks();
    else if (what == "spans") spans();
    else if (what == "routes") routes();
    else return 2;
    std::printf("%s: %s\n", what.c_str(), failures ? "FAILED" : "ok");
    return failures ? 1 : 0;
}
