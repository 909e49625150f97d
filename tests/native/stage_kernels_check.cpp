// The FP64 stage kernels of one (dim, degree) run on the host (hostsim), on
// a forest with hanging faces in both directions:
//  - the result must not depend on the order in which the waves and threads
//    of a workgroup run between barriers, nor on what LDS held before the
//    launch (a slot read before it is written, or two waves' conflicting
//    accesses between two barriers, would make it), and no LDS past the
//    launch's bytes may be written;
//  - the axis-by-axis item must agree with the point-by-point item, and the
//    3-D lane kernel with it too, to the rounding of a stage;
//  - the CFL rate folded into a last stage that stores in place must be the
//    one of the stored state.
// Modes: fused stage with the far side inline and from the guard buffer, the
// residual, the limiter and mortar faces; every slab height the launcher
// takes.  Prints the number of cases and "OK".
#define DG_PART 9
#include "../../paper_2502_12620_amd/csrc/inst.hip"

namespace dgk {
alignas(64) double lds[hostsim::kLds + 64], lds_d[hostsim::kLds + 64], lds_all[hostsim::kLds + 64];
}

using namespace dgk;

constexpr int D = DG_D, P = DG_P, NV = D + 2, NB = Tab<D, P>::NB;
static int cases = 0, bad = 0;
static double worst = 0.0; // largest difference between two forms

struct Setup {
    dgamr::Forest forest;
    std::vector<LeafGeo> geo;
    std::vector<double> us, un, guard;
    int ncell, N;
    double dt = 1e-3;
    StageArgs args(bool conservative) const
    {
        StageArgs a{};
        a.us = us.data();
        a.un = un.data();
        a.guard = guard.data();
        a.geo = geo.data();
        a.links = forest.links().data();
        a.dt = &dt;
        a.gamma = 1.4;
        a.nleaves = forest.n();
        a.N = N;
        a.conservative = conservative;
        a.inv_n = unsigned((65536 + N - 1) / N);
        return a;
    }
};

static dgamr_forest_desc desc(int N, int bc, int rx, int ry, int rz, int levels)
{
    dgamr_forest_desc d{};
    d.dim = D;
    d.degree = P;
    d.n_cell = N;
    const int r[3] = {rx, ry, D == 3 ? rz : 1};
    for (int a = 0; a < 3; ++a) {
        d.roots[a] = r[a];
        d.hi[a] = r[a];
        d.bc[a] = bc;
    }
    d.max_level = levels;
    d.gamma = 1.4;
    return d;
}

// noise: of the coefficients past the mean, relative to a state of order one
static Setup make(int N, int bc, int rx, int ry, int rz, bool refine, double noise)
{
    Setup s{dgamr::Forest(desc(N, bc, rx, ry, rz, refine ? 2 : 1)), {}, {}, {}, {}, 0, N};
    std::string err;
    if (s.forest.build_links(err) != 0) std::exit(3);
    if (refine) {
        std::vector<int8_t> flags(s.forest.n(), 0);
        flags[0] = 1;
        std::vector<dgamr::Inherit> inh;
        if (s.forest.plan(flags.data(), err) != 0 || s.forest.commit(inh, err) != 0) std::exit(3);
    }
    s.geo = s.forest.geometry();
    s.ncell = D == 2 ? N * N : N * N * N;
    std::mt19937_64 rng(N + 10 * P + bc);
    std::uniform_real_distribution<double> u(-1.0, 1.0);
    for (auto *x : {&s.us, &s.un}) {
        x->resize(size_t(s.forest.n()) * NV * NB * s.ncell);
        for (size_t i = 0; i < x->size(); ++i) {
            const int m = int(i / s.ncell) % NB, v = int(i / s.ncell / NB) % NV;
            (*x)[i] = m > 0 ? noise * u(rng) : (v == 0 ? 1.0 : (v <= D ? 0.3 * v : 3.0)) + 0.1 * u(rng);
        }
    }
    // the last leaf is the fastest, and faster in the stage's input than in its
    // base state: a rate taken from an updated base state is too large
    for (int c = 0; c < s.ncell; ++c) {
        double *last = s.us.data() + size_t(s.forest.n() - 1) * NV * NB * s.ncell + c;
        last[size_t(1) * NB * s.ncell] += 8.0;
        last[size_t(D + 1) * NB * s.ncell] += 40.0;
    }
    const int nfc = D == 2 ? N : N * N;
    s.guard.resize(size_t(s.forest.n()) * 2 * D * NV * NB * nfc);
    FillArgs f{s.us.data(), s.guard.data(), s.forest.links().data(), nullptr, nullptr, s.forest.n() * 2 * D, N, 0};
    hostsim::launch(dim3((f.nfaces * nfc + 255) / 256), dim3(256), 0, [&] { k_fill<D, P>(f); });
    return s;
}

// largest difference over the largest value: some hundred terms of one sum's
// rounding leave 1e-13
constexpr double kTol = 1e-13;
static double differ(const std::vector<double> &a, const std::vector<double> &b)
{
    double d = 0.0, big = 0.0;
    for (size_t i = 0; i < a.size(); ++i) {
        if (!std::isfinite(a[i]) || !std::isfinite(b[i])) return 1e300;
        d = std::max(d, std::fabs(a[i] - b[i]));
        big = std::max(big, std::fabs(a[i]));
    }
    worst = std::max(worst, d / big);
    return d / big;
}

static void report(bool ok, const char *what, const std::string &name)
{
    ++cases;
    if (ok) return;
    ++bad;
    std::printf("%s: %s\n", what, name.c_str());
}

// runs launch(args) for every order and LDS fill; the results of all are equal
template <class L>
static std::vector<double> run(const Setup &s, StageArgs a, int om, const std::string &name, L &&launch)
{
    std::vector<double> first, out(s.us.size());
    unsigned long long first_rate = 0;
    // a last stage: in place on its base state, with the rate of what it stores
    const bool last = om == OUT_RK;
    for (int k = 0; k < 3; ++k) {
        hostsim::order = k;
        hostsim::fill = k == 0 ? std::nan("") : 1e3 * k;
        const int errors = hostsim::errors;
        unsigned long long rate = 0;
        if (last) {
            out = s.un;
            a.un = out.data();
            a.rk_a = 1.0 / 3.0;
            a.rk_b = 2.0 / 3.0;
            a.rate_out = &rate;
        } else {
            std::fill(out.begin(), out.end(), std::nan(""));
        }
        a.out64 = out.data();
        if (launch(a) != hipSuccess) {
            report(false, "refused", name);
            return out;
        }
        report(hostsim::errors == errors, "writes past its LDS", name);
        if (k == 0) {
            first = out;
            first_rate = rate;
        }
        report(std::memcmp(first.data(), out.data(), sizeof(double) * out.size()) == 0, "order or LDS fill changes the result", name);
        report(rate == first_rate, "order or LDS fill changes the rate", name);
    }
    if (last) {
        double ref = 0.0;
        for (int l = 0; l < s.forest.n(); ++l)
            for (int c = 0; c < s.ncell; ++c) {
                double U[NV], r = 0.0;
                for (int v = 0; v < NV; ++v) U[v] = first[(size_t(l) * NV + v) * NB * s.ncell + c];
                const double cs = std::sqrt(1.4 * pressure<D>(U, 0.4) / U[0]);
                for (int a2 = 0; a2 < D; ++a2) r += (std::fabs(U[1 + a2] / U[0]) + cs) / s.geo[l].h[a2];
                ref = std::max(ref, r);
            }
        const double got = __longlong_as_double((long long)first_rate);
        report(std::fabs(got - ref) <= 1e-13 * ref, "rate is not that of the stored state", name);
    }
    return first;
}

template <int GM, int OM, bool LIM>
static void forms(const Setup &s, bool conservative, int rows, const std::string &name)
{
    const int layer = D == 2 ? s.N : s.N * s.N, nslab = rows * layer, total = s.forest.n() * (s.N / rows);
    const StageArgs a = s.args(conservative);
    hostsim::skip_lane = nullptr;
    const auto points = run(s, a, OM, name + " points", [&](const StageArgs &g) {
        const size_t n = sizeof(double) * std::max((D + 2) * face_chunk<D, P>() * nslab, nslab);
        hostsim::launch(dim3(total), dim3(nslab), n,
                        [&] { stage_item_points<D, P, GM, OM, LIM, double, EQ_EULER, false>(g, rows, blockIdx.x, total); });
        return hipSuccess;
    });
    const auto axis = run(s, a, OM, name + " axis by axis", [&](const StageArgs &g) {
        const size_t n = sizeof(double) * std::max(stage_lds_values<D, P, NV>(s.N, rows), size_t(nslab));
        hostsim::launch(dim3(total), dim3(nslab), n,
                        [&] { stage_item<D, P, GM, OM, LIM, EQ_EULER>(g, rows, blockIdx.x, total); });
        return hipSuccess;
    });
    report(differ(points, axis) <= kTol, "forms differ", name);
    if constexpr (D == 3 && !LIM) {
        if (conservative || !(rows == s.N || rows == 1 || rows_ok_3v(s.N, rows))) return;
        // (lanes 60 to 63 repeat others' work in lockstep)
        hostsim::skip_lane = [](int lane) { return lane >= 5 * kCells3v; };
        const auto lanes = run(s, a, OM, name + " lanes", [&](const StageArgs &g) {
            return launch_stage_3v<P>(g, GM, OM, nullptr, rows_ok_3v(s.N, rows) ? rows : 0);
        });
        hostsim::skip_lane = nullptr;
        report(differ(points, lanes) <= kTol, "lane kernel differs", name);
    }
}

int main()
{
    hostsim::lds_arrays = {lds, lds_d, lds_all};
    const int sizes[] = DG_SIZES;
    for (int N : sizes)
        for (int bc : {DGAMR_BC_PERIODIC, DGAMR_BC_OUTFLOW}) {
            // one root of 2 x 2 refined: 7 or 15 leaves (3-D: odd counts, so
            // that the lane kernel's groups are partly filled)
            const Setup s = make(N, bc, 2, 2, D == 3 ? 1 : 1, true, 0.01);
            for (int rows = N; rows >= 1; --rows) {
                if (!rows_ok<D, P, double>(N, rows)) continue;
                const std::string name = "N " + std::to_string(N) + " rows " + std::to_string(rows) + (bc ? " outflow" : " periodic");
                forms<GUARD_INLINE, OUT_RK, false>(s, false, rows, name + " inline");
                forms<GUARD_BUFFER, OUT_RES64, false>(s, false, rows, name + " residual");
                forms<GUARD_BUFFER, OUT_RES64, false>(s, true, rows, name + " residual, mortar");
                forms<GUARD_INLINE, OUT_RK, false>(s, true, rows, name + " inline, mortar");
                if (bc) continue;
                forms<GUARD_BUFFER, OUT_RK, false>(s, false, rows, name + " buffer");
                forms<GUARD_INLINE, OUT_RK, true>(s, true, rows, name + " inline, mortar, limiter");
            }
        }
    std::printf("%s %d cases, dim %d degree %d, forms within %.1e\n", bad ? "FAILED" : "OK", cases, D, P, worst);
    return bad != 0;
}
