// HIP kernels of the DG stage for gfx950: guard-cell fill (Sec. 3.5,
// Eq. 15-17) and the residual of the Galerkin weak form (Sec. 2, Eq. 3-5),
// optionally fused with the SSP-RK3 stage update.
//
// One thread per cell.  The thread keeps its cell's coefficients K[var][mode]
// and residual R[var][mode] in registers; the basis tables are compile-time
// constants and every contraction goes one axis at a time.  The flux of each
// face inside a workgroup's slab of cells is computed once: the + trace of
// every cell goes through LDS to its + neighbour, which computes the Rusanov
// flux and sends it back through LDS, both as the face's modes.
#pragma once

#include <type_traits>

#include "kernel_common.hpp"

namespace dgk {

// one cell's coefficients (or residual) per variable and mode
template <int D, int P>
using CellCoef = double[D + 2][Tab<D, P>::NB];

// Full unrolling over the quadrature points makes every table entry an
// immediate.  In 3-D the unrolled code and its live ranges outgrow the
// register file (one cell's state and residual already take 4 NB VGPRs per
// variable), so there the point loops stay loops over tables read with
// scalar loads.
template <int D, int P>
constexpr bool unroll_points() { return D == 2; }

// Whether to apply table entry c taken at a point of such a loop: unrolled,
// c is an immediate and its structural zeros drop out; in a loop, c is a
// runtime value and a multiply by zero costs less than a branch on it.
template <int D, int P>
__device__ __forceinline__ bool use_entry(double c) { return !unroll_points<D, P>() || c != 0.0; }

// The tables of the point loops in the arithmetic's type.  A loop over points
// takes its entries at run time (scalar loads), and an FP64 entry used in FP32
// would be converted again at every point, at a quarter of the vector rate
// (FP32 3-D degree 2, 12^3 roots of 8^3 cells, two steps: 5.85 -> 5.59 ms).
template <int D, int P>
struct PointTab32 {
    static constexpr int NB = Tab<D, P>::NB, NQ = Tab<D, P>::NQ, NF = Tab<D, P>::NF;
    float phi_v[NQ][NB] = {}, dproj[D][NQ][NB] = {}, phi_f[D][NF][NB] = {}, lift_f[D][NF][NB] = {};
    constexpr PointTab32()
    {
        for (int m = 0; m < NB; ++m) {
            for (int q = 0; q < NQ; ++q) {
                phi_v[q][m] = float(kTab<D, P>.phi_v[q][m]);
                for (int a = 0; a < D; ++a) dproj[a][q][m] = float(kTab<D, P>.dproj[a][q][m]);
            }
            for (int f = 0; f < NF; ++f)
                for (int a = 0; a < D; ++a) {
                    phi_f[a][f][m] = float(kTab<D, P>.phi_f[a][f][m]);
                    lift_f[a][f][m] = float(kTab<D, P>.lift_f[a][f][m]);
                }
        }
    }
};
template <int D, int P>
inline constexpr PointTab32<D, P> kPointTab32{};
// whether the loops take those (unrolled, the entries are immediates)
template <int D, int P, typename T>
inline constexpr bool kTake32 = std::is_same<T, float>::value && !unroll_points<D, P>();

// even / odd parts (in the normal mode index) of the trace of K at face
// point f of axis a: the trace at xi_a = +1 is e + o, at xi_a = -1 it is e - o.
template <int D, int P, typename T>
__device__ __forceinline__ void trace_eo(const T *K, int a, int f, T &e, T &o)
{
    e = T(0);
    o = T(0);
#pragma unroll
    for (int m = 0; m < Tab<D, P>::NB; ++m) {
        const double c = kTake32<D, P, T> ? kPointTab32<D, P>.phi_f[a][f][m] : kTab<D, P>.phi_f[a][f][m];
        if (use_entry<D, P>(c)) {
            if (kTab<D, P>.e[m][a] % 2 == 0) e = fma(T(c), K[m], e);
            else o = fma(T(c), K[m], o);
        }
    }
}

// the same for coefficients streamed from memory (coef[m*sm])
template <int D, int P, typename T>
__device__ __forceinline__ void trace_eo_mem(const double *__restrict__ coef, long sm, int a, int f, T &e, T &o)
{
    e = T(0);
    o = T(0);
#pragma unroll
    for (int m = 0; m < Tab<D, P>::NB; ++m) {
        const double c = kTab<D, P>.phi_f[a][f][m];
        if (use_entry<D, P>(c)) {
            const T k = T(coef[m * sm]);
            if (kTab<D, P>.e[m][a] % 2 == 0) e = fma(T(c), k, e);
            else o = fma(T(c), k, o);
        }
    }
}

// Conservative hanging-face flux: the coarse cell integrates the Rusanov
// flux over the 2^(d-1) fine sub-faces at the fine Gauss points, with the
// fine cells' own traces, and lifts it with its own basis evaluated at the
// mapped points (tangential xi = (xi_fine + sigma)/2).  MASS: R is M^-1
// times the weak form's right-hand side; otherwise that right-hand side.
template <int D, int P, int A, int EQ, typename T, bool MASS>
__device__ __forceinline__ void mortar_lift(const StageArgs &g, const T (&K)[nvar<D, EQ>()][Tab<D, P>::NB],
                                            T (&R)[nvar<D, EQ>()][Tab<D, P>::NB], int side, const FaceLink L, int t,
                                            T scale)
{
    constexpr int NV = nvar<D, EQ>(), NB = Tab<D, P>::NB, Q = P + 1, NF = Tab<D, P>::NF;
    constexpr int TA = A == 0 ? 1 : 0, TBX = A == 2 ? 1 : 2; // tangential axes, lower first
    const int N = g.N, ncell = D == 2 ? N * N : N * N * N;
    const long sv = long(NB) * ncell;
    const int fleaf = link_nbr(L, fine_block(t, N, D));
    // the fine cells touching the face: children with the half along A
    // nearest to this block
    const int near = (side > 0 ? 0 : 1) << A;
    const double sub = D == 2 ? 0.5 : 0.25; // fine face Jacobian / coarse face Jacobian
    // runs only on hanging faces: kept as loops (table values computed on
    // the fly) to keep the code small
#pragma unroll 1
    for (int S = 0; S < (1 << (D - 1)); ++S) {
        const int s0 = S & 1, s1 = (S >> 1) & 1;
        const int fcell = fine_cell(A, side, t, near | (s0 << TA) | (s1 << TBX), N, D);
        const double *fk = g.us + long(fleaf) * NV * sv + fcell;
#pragma unroll 1
        for (int F = 0; F < NF; ++F) {
            const int q0 = F % Q, q1 = F / Q;
            const double x0 = 0.5 * (gl_x(Q, q0) + (s0 ? 1.0 : -1.0));
            const double x1 = 0.5 * (gl_x(Q, q1) + (s1 ? 1.0 : -1.0));
            const double w = gl_w(Q, q0) * (D == 3 ? gl_w(Q, q1) : 1.0);
            T Uf[NV], Uc[NV], Phi[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                T e, o;
                trace_eo_mem<D, P, T>(fk + v * sv, ncell, A, F, e, o);
                Uf[v] = side > 0 ? e - o : e + o; // the fine cell touches the face with its -side side
                T ec = T(0), oc = T(0);
#pragma unroll
                for (int m = 0; m < NB; ++m) {
                    const double c = leg(kTab<D, P>.e[m][TA], x0) * (D == 3 ? leg(kTab<D, P>.e[m][TBX], x1) : 1.0);
                    if (c != 0.0) {
                        if (kTab<D, P>.e[m][A] % 2 == 0) ec = fma(T(c), K[v][m], ec);
                        else oc = fma(T(c), K[v][m], oc);
                    }
                }
                Uc[v] = side > 0 ? ec + oc : ec - oc;
            }
            if (side > 0) num_flux<D, A, EQ, T>(g, Uc, Uf, T(g.gamma), Phi);
            else num_flux<D, A, EQ, T>(g, Uf, Uc, T(g.gamma), Phi);
            // +face: -int Phi phi ; -face: +int Phi phi with phi(-1) = (-1)^{m_A} phi(+1)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const T f = scale * T(sub * w) * Phi[v];
#pragma unroll
                for (int m = 0; m < NB; ++m) {
                    const double c = leg(kTab<D, P>.e[m][TA], x0) * (D == 3 ? leg(kTab<D, P>.e[m][TBX], x1) : 1.0) *
                                     (MASS ? kTab<D, P>.inv_mass[m] : 1.0);
                    if (c != 0.0) {
                        const double sg = side > 0 ? -1.0 : ((kTab<D, P>.e[m][A] % 2) ? -1.0 : 1.0);
                        R[v][m] = fma(T(sg * c), f, R[v][m]);
                    }
                }
            }
        }
    }
}

// Coefficients of the split of a coarse cell for child CH (Eq. 11-12):
// g = S_CH k, one variable at a time.
template <int D, int P, int CH, typename T>
__host__ __device__ __forceinline__ void split_coeffs(const T *k, T *gk)
{
    constexpr int NB = Tab<D, P>::NB;
#pragma unroll
    for (int m = 0; m < NB; ++m) {
        T s = T(0);
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const double c = kTab<D, P>.split[CH][m][n];
            if (c != 0.0) s = fma(T(c), k[n], s);
        }
        gk[m] = s;
    }
}

template <int D, int P, typename T>
__host__ __device__ __forceinline__ void split_any(int child, const T *k, T *gk)
{
    switch (child) {
    case 0: split_coeffs<D, P, 0, T>(k, gk); break;
    case 1: split_coeffs<D, P, 1, T>(k, gk); break;
    case 2: split_coeffs<D, P, 2, T>(k, gk); break;
    case 3: split_coeffs<D, P, 3, T>(k, gk); break;
    case 4: if constexpr (D == 3) split_coeffs<D, P, 4, T>(k, gk); break;
    case 5: if constexpr (D == 3) split_coeffs<D, P, 5, T>(k, gk); break;
    case 6: if constexpr (D == 3) split_coeffs<D, P, 6, T>(k, gk); break;
    default: if constexpr (D == 3) split_coeffs<D, P, 7, T>(k, gk); break;
    }
}

// Adds the combine contribution of child CH (Eq. 13-14): gk += C_CH k.
template <int D, int P, int CH>
__device__ __forceinline__ void comb_coeffs(const double *k, double *gk)
{
    constexpr int NB = Tab<D, P>::NB;
#pragma unroll
    for (int m = 0; m < NB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const double c = kTab<D, P>.comb[CH][m][n];
            if (c != 0.0) gk[m] = fma(c, k[n], gk[m]);
        }
}

template <int D, int P>
__device__ __forceinline__ void comb_any(int child, const double *k, double *gk)
{
    switch (child) {
    case 0: comb_coeffs<D, P, 0>(k, gk); break;
    case 1: comb_coeffs<D, P, 1>(k, gk); break;
    case 2: comb_coeffs<D, P, 2>(k, gk); break;
    case 3: comb_coeffs<D, P, 3>(k, gk); break;
    case 4: if constexpr (D == 3) comb_coeffs<D, P, 4>(k, gk); break;
    case 5: if constexpr (D == 3) comb_coeffs<D, P, 5>(k, gk); break;
    case 6: if constexpr (D == 3) comb_coeffs<D, P, 6>(k, gk); break;
    default: if constexpr (D == 3) comb_coeffs<D, P, 7>(k, gk); break;
    }
}

// Far-side polynomial of block face (A, side) for the cell with tangential
// index t, per variable (its traces at the face are taken at -side):
//  - guard-buffer mode: the stored guard cell;
//  - inline mode: the same-level neighbour cell (Eq. 15), the split of the
//    coarser neighbour cell (Eq. 16), the combine of the 2^d finer cells
//    (Eq. 17), or at an outflow boundary the mirror image K_m (-1)^{m_A}.
template <int D, int P, int A, int GM, int NV, typename T>
__host__ __device__ __forceinline__ void far_poly(const StageArgs &g, const T (&K)[NV][Tab<D, P>::NB], int leaf, int side,
                                         int t, const FaceLink &L, T (&Kf)[NV][Tab<D, P>::NB])
{
    constexpr int NB = Tab<D, P>::NB;
    const int N = g.N, ncell = D == 2 ? N * N : N * N * N, nfc = D == 2 ? N : N * N;
    const long sv = long(NB) * ncell;
    const int face = 2 * A + (side > 0);
    if constexpr (GM == GUARD_BUFFER) {
        const double *gk = g.guard + ((long(leaf) * 2 * D + face) * NV * NB) * nfc + t;
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int m = 0; m < NB; ++m) Kf[v][m] = T(gk[(long(v) * NB + m) * nfc]);
        return;
    }
    if (L.type == dgamr::LINK_BOUNDARY) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int m = 0; m < NB; ++m) Kf[v][m] = (kTab<D, P>.e[m][A] % 2) ? -K[v][m] : K[v][m];
    } else if (L.type == dgamr::LINK_SAME) {
        const int c = same_cell(A, side, t, N, D);
        const double *nk = g.us + long(L.nbr[0]) * NV * sv + c;
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int m = 0; m < NB; ++m) Kf[v][m] = T(nk[v * sv + m * ncell]);
    } else if (L.type == dgamr::LINK_COARSE) {
        const int c = coarse_cell(A, side, t, L.off, N, D);
        const int child = coarse_child(A, side, t, N, D);
        const double *ck = g.us + long(L.nbr[0]) * NV * sv + c;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            T kv[NB];
#pragma unroll
            for (int m = 0; m < NB; ++m) kv[m] = T(ck[v * sv + m * ncell]);
            split_any<D, P, T>(child, kv, Kf[v]);
        }
    } else { // LINK_FINE
        const double *fk = g.us + long(link_nbr(L, fine_block(t, N, D))) * NV * sv;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
#pragma unroll
            for (int m = 0; m < NB; ++m) Kf[v][m] = T(0);
#pragma unroll
            for (int ch = 0; ch < (1 << D); ++ch) {
                const int fc = fine_cell(A, side, t, ch, N, D);
                T kv[NB];
#pragma unroll
                for (int n = 0; n < NB; ++n) kv[n] = T(fk[v * sv + n * ncell + fc]);
#pragma unroll
                for (int m = 0; m < NB; ++m)
#pragma unroll
                    for (int n = 0; n < NB; ++n) {
                        const double cc = kTab<D, P>.comb[ch][m][n];
                        if (cc != 0.0) Kf[v][m] = fma(T(cc), kv[n], Kf[v][m]);
                    }
            }
        }
    }
}

// Variable v of the far-side polynomial of a hanging block face (a, side) for
// the cell with tangential index t: the split of the coarser neighbour cell
// (Eq. 16) or the combine of the 2^d finer cells (Eq. 17).
template <int D, int P, int NV>
__device__ __forceinline__ void hanging_var(const StageArgs &g, int v, int a, int side, int t, const FaceLink &L,
                                            double *kf)
{
    constexpr int NB = Tab<D, P>::NB;
    const int N = g.N, ncell = D == 2 ? N * N : N * N * N;
    const long sv = long(NB) * ncell;
    if (L.type == dgamr::LINK_COARSE) {
        const int c = coarse_cell(a, side, t, L.off, N, D);
        const double *ck = g.us + long(L.nbr[0]) * NV * sv + v * sv + c;
        double kv[NB];
#pragma unroll
        for (int m = 0; m < NB; ++m) kv[m] = ck[m * ncell];
        split_any<D, P, double>(coarse_child(a, side, t, N, D), kv, kf);
    } else { // LINK_FINE
        const double *fk = g.us + long(link_nbr(L, fine_block(t, N, D))) * NV * sv + v * sv;
#pragma unroll
        for (int m = 0; m < NB; ++m) kf[m] = 0.0;
#pragma unroll
        for (int ch = 0; ch < (1 << D); ++ch) {
            const int fc = fine_cell(a, side, t, ch, N, D);
            double kv[NB];
#pragma unroll
            for (int n = 0; n < NB; ++n) kv[n] = fk[n * ncell + fc];
            comb_any<D, P>(ch, kv, kf);
        }
    }
}

// ------------------------------------------------------------------ positivity limiter
// Gauss-Lobatto rule of Zhang and Shu's point set: the fewest points L
// (L >= 2) whose rule is exact for degree P (2L - 3 >= P); its nodes are
// -1, +1 and, for L = 3, 0.
template <int P>
constexpr int lobatto_points() { return P <= 1 ? 2 : 3; }

// Interior Lobatto nodes that are not Gauss nodes of the (P+1)-point rule
// (0 for L = 3 with an even number of Gauss points): 1 at degree 3, else 0.
template <int P>
constexpr int lobatto_extra() { return (lobatto_points<P>() == 3 && (P + 1) % 2 == 0) ? 1 : 0; }

// Point set of the limiter: the volume Gauss points, then the face Gauss
// points of every face (basis values with the face side's sign), then for
// every axis a the points with xi_a = 0 and Gauss nodes on the other axes
// when 0 is a Lobatto node but not a Gauss node.  Together these are
// Zhang and Shu's points (Lobatto nodes along one axis, Gauss nodes along
// the others, over all axes) plus the volume Gauss points.
template <int D, int P>
struct LimiterPoints {
    static constexpr int NQ = Tab<D, P>::NQ, NF = Tab<D, P>::NF, NB = Tab<D, P>::NB;
    static constexpr int NPT = NQ + 2 * D * NF + lobatto_extra<P>() * D * NF;
    double phi[NPT][NB] = {};
    constexpr LimiterPoints()
    {
        for (int q = 0; q < NQ; ++q)
            for (int m = 0; m < NB; ++m) phi[q][m] = kTab<D, P>.phi_v[q][m];
        int n = NQ;
        for (int face = 0; face < 2 * D; ++face) {
            const int a = face / 2;
            const bool minus = (face & 1) == 0;
            for (int f = 0; f < NF; ++f, ++n)
                for (int m = 0; m < NB; ++m)
                    phi[n][m] = kTab<D, P>.phi_f[a][f][m] * ((minus && kTab<D, P>.e[m][a] % 2) ? -1.0 : 1.0);
        }
        if (lobatto_extra<P>())
            for (int a = 0; a < D; ++a)
                for (int f = 0; f < NF; ++f, ++n)
                    for (int m = 0; m < NB; ++m) // the face point's tangential values times P_{m_a}(0)
                        phi[n][m] = kTab<D, P>.phi_f[a][f][m] * leg(kTab<D, P>.e[m][a], 0.0);
    }
};
template <int D, int P>
inline constexpr LimiterPoints<D, P> kLimPts{};

// Zhang-Shu scaling limiter (named in Sec. 5.3.2) on one cell, in place,
// with eps = min(1e-13, mean rho, p(mean)):
//   theta1 = min(1, (rho_mean - eps)/(rho_mean - min_S rho)) scales the
//   non-mean density modes; then theta2 = min over S of the chord bound
//   t = (p(mean) - eps)/(p(mean) - p(U)) at the points with p(U) < eps
//   (pressure is concave in the conserved variables where rho > 0, so the
//   scaled state keeps p >= eps there) scales all non-mean modes.  The cell
//   mean is never changed.  MEAN_GIVEN: the cell mean is given (a bilinear /
//   trilinear cell, whose full mass matrix makes the mean differ from the
//   mode-0 coefficient), and the scalings U <- mean + theta (U - mean) move
//   mode 0 as well.
//
// Most cells of a run need no scaling, and the basis shows it without the
// points: every |phi_m| <= 1 in the cell, so each variable stays within the
// sum of its non-mean coefficients' moduli of the mean coefficient, which
// bounds density and pressure from below at all points.  When both bounds
// clear eps by more than the rounding of the point values, both scalings are
// 1 and the points are skipped (a wave skips them when all its cells do; the
// 176-leaf blast of 8^3-cell blocks at degree 2, average stage: 266 -> 210 us).  The margins: density
// above 1e-3 of its terms, so that its rounding (some 20 ulp of them) is
// below 1e-11 of it, and pressure by 1e-11 of its own terms.  NaN and
// infinities fail the comparisons and take the points.
template <int D, int P>
__device__ __forceinline__ bool limiter_idle(const CellCoef<D, P> &K, double gm1, double eps)
{
    constexpr int NV = D + 2, NB = Tab<D, P>::NB;
    double dev[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        dev[v] = 0.0;
#pragma unroll
        for (int m = 1; m < NB; ++m) dev[v] += fabs(K[v][m]);
    }
    const double rho = K[0][0] - dev[0], rho_all = fabs(K[0][0]) + dev[0];
    if (!(rho > eps && rho > 1e-3 * rho_all)) return false;
    double m2 = 0.0;
#pragma unroll
    for (int b = 0; b < D; ++b) {
        const double m = fabs(K[1 + b][0]) + dev[1 + b];
        m2 = fma(m, m, m2);
    }
    const double ke = 0.5 * m2 / rho, e_all = fabs(K[D + 1][0]) + dev[D + 1];
    const double p = gm1 * (K[D + 1][0] - dev[D + 1] - ke);
    return p > eps + 1e-11 * gm1 * (e_all + ke);
}

template <int D, int P, bool MEAN_GIVEN = false>
__device__ __forceinline__ void limit_cell(CellCoef<D, P> &K, double gamma, const double *given_mean = nullptr)
{
    constexpr int NV = D + 2, NB = Tab<D, P>::NB, NPT = LimiterPoints<D, P>::NPT;
    const double gm1 = gamma - 1.0;
    double mean[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) mean[v] = MEAN_GIVEN ? given_mean[v] : K[v][0];
    const double pbar = pressure<D>(mean, gm1);
    double eps = 1e-13;
    eps = mean[0] < eps ? mean[0] : eps;
    eps = pbar < eps ? pbar : eps;
    if (limiter_idle<D, P>(K, gm1, eps)) return;
    double rmin = mean[0];
#pragma unroll 1
    for (int pt = 0; pt < NPT; ++pt) {
        double r = 0.0;
#pragma unroll
        for (int m = 0; m < NB; ++m) r = fma(kLimPts<D, P>.phi[pt][m], K[0][m], r);
        rmin = r < rmin ? r : rmin;
    }
    if (rmin < mean[0]) {
        double th1 = (mean[0] - eps) / (mean[0] - rmin);
        if (th1 < 1.0) {
#pragma unroll
            for (int m = 1; m < NB; ++m) K[0][m] *= th1;
            if constexpr (MEAN_GIVEN) K[0][0] = mean[0] + th1 * (K[0][0] - mean[0]);
        }
    }
    double th2 = 1.0;
#pragma unroll 1
    for (int pt = 0; pt < NPT; ++pt) {
        double U[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            double s = 0.0;
#pragma unroll
            for (int m = 0; m < NB; ++m) s = fma(kLimPts<D, P>.phi[pt][m], K[v][m], s);
            U[v] = s;
        }
        const double pq = pressure<D>(U, gm1);
        if (pq < eps) {
            double tq = (pbar - eps) / (pbar - pq);
            tq = tq > 1.0 ? 1.0 : (tq < 0.0 ? 0.0 : tq);
            th2 = tq < th2 ? tq : th2;
        }
    }
    if (th2 < 1.0)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
#pragma unroll
            for (int m = 1; m < NB; ++m) K[v][m] *= th2;
            if constexpr (MEAN_GIVEN) K[v][0] = mean[v] + th2 * (K[v][0] - mean[v]);
        }
}

// ------------------------------------------------------------------ sum-factorised contractions
// What bounds the stage: memory latency and the instructions of one wave's
// chain, with two or three waves per SIMD.  Contracting one axis at a time
// takes 9 points x 6 modes at 2-D degree 2 from 54 multiply-adds per variable
// to 27, and the faces exchange their modes with two barriers per axis
// instead of four per chunk of face points; the traces from outside the slab
// are gathered densely, one exposed memory latency for all axes.  Measured
// against the contraction point by point (uniform vortex forests, two steps):
// 2-D, degree 1, 128^2 roots of 16^2 cells 1.71 -> 1.49 ms; degree 2, 64^2
// roots 0.98 -> 0.79 ms; 3-D degree 1, 16^3 roots of 8^3 cells 2.75 -> 2.07 ms.

// Coefficients of the trace of one variable's polynomial on the face of
// axis A at xi_A = s (s = +1 or -1) in the face modes: sum_i s^i K_(i, f).
template <int D, int P, int A>
__device__ __forceinline__ void face_trace(const double *K, double s, double *tr)
{
    constexpr int NB = Tab<D, P>::NB, NBF = face_modes<D, P>();
    double odd[NBF];
    // modes come in ascending degree, so the first of a face mode has i = 0
#pragma unroll
    for (int m = 0; m < NB; ++m) {
        const int f = face_mode<D, P>(m, A), i = kTab<D, P>.e[m][A];
        if (i == 0) tr[f] = K[m];
        else if (i == 1) odd[f] = K[m];
        else if (i % 2 == 0) tr[f] += K[m];
        else odd[f] += K[m];
    }
#pragma unroll
    for (int m = 0; m < NB; ++m) // the face modes that have odd terms
        if (kTab<D, P>.e[m][A] == 1) tr[face_mode<D, P>(m, A)] = fma(s, odd[face_mode<D, P>(m, A)], tr[face_mode<D, P>(m, A)]);
}

// Numerical flux in the +e_A direction between the own state Uo and the
// neighbour's Un across the face on the `side` (+1 / -1) of axis A, the
// same value to the last bit from both sides: Rusanov (Eq. 5), or upwind
// for scalar convection (num_flux with left and right ordered by the side).
template <int D, int A, int EQ, class Args>
__device__ __forceinline__ void side_flux(const Args &g, const double *Uo, const double *Un, double side, double gamma, double *Phi)
{
    if constexpr (EQ == EQ_ADVECTION) {
        const double a = g.vel[A];
        Phi[0] = 0.5 * (a * (Uo[0] + Un[0]) - side * (fabs(a) * (Un[0] - Uo[0])));
    } else {
        constexpr int NV = D + 2;
        const double gm1 = gamma - 1.0;
        const double ro = recip(Uo[0]), rn = recip(Un[0]);
        const double po = pressure_r<D>(Uo, gm1, ro), pn = pressure_r<D>(Un, gm1, rn);
        const double uo = Uo[1 + A] * ro, un = Un[1 + A] * rn;
        const double ao = fabs(uo) + sqrt_nn(gamma * po * ro), an = fabs(un) + sqrt_nn(gamma * pn * rn);
        const double alpha = side * (ao > an ? ao : an);
        double Fo[NV], Fn[NV];
        euler_flux<D, A>(Uo, uo, po, Fo);
        euler_flux<D, A>(Un, un, pn, Fn);
#pragma unroll
        for (int v = 0; v < NV; ++v) Phi[v] = 0.5 * ((Fo[v] + Fn[v]) - alpha * (Un[v] - Uo[v]));
    }
}

// Flux of one face in its face modes: both traces evaluated at the face
// points row by row, the numerical flux there, and its projection int Phi
// phi_f.  own(v, tr) gives the own trace's modes of variable v, nbr(v, f) the
// neighbour's mode f.
template <int D, int P, int A, int EQ, class Args, class Own, class Nbr>
__device__ __forceinline__ void face_flux(double side, double gamma, const Args &gv, Own &&own, Nbr &&nbr,
                                          double (&Phi)[nvar<D, EQ>()][face_modes<D, P>()])
{
    constexpr int NV = nvar<D, EQ>(), NBF = face_modes<D, P>(), Q = P + 1;
    // one row of points along the lower tangential axis: ro, rn its
    // coefficients, acc the projection of the flux along the row
    auto row = [&](const double (&ro)[NV][Q], const double (&rn)[NV][Q], double (&acc)[NV][Q]) __attribute__((always_inline)) {
        static_for<0, Q>([&](auto qv) __attribute__((always_inline)) {
            constexpr int q = qv;
            double Uo[NV], Un[NV], F[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                Uo[v] = ro[v][0];
                Un[v] = rn[v][0];
#pragma unroll
                for (int j = 1; j < Q; ++j) {
                    const double c = kRule<P>.val[q][j];
                    if (c != 0.0) {
                        Uo[v] = fma(c, ro[v][j], Uo[v]);
                        Un[v] = fma(c, rn[v][j], Un[v]);
                    }
                }
            }
            side_flux<D, A, EQ>(gv, Uo, Un, side, gamma, F);
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    const double c = kRule<P>.w[q] * kRule<P>.val[q][j];
                    if (c != 0.0) acc[v][j] = q == 0 ? c * F[v] : fma(c, F[v], acc[v][j]);
                    else if (q == 0) acc[v][j] = 0.0;
                }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    double tr[NV][NBF];
#pragma unroll
    for (int v = 0; v < NV; ++v) own(v, tr[v]);
    if constexpr (D == 2) {
        double rn[NV][Q];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int f = 0; f < NBF; ++f) rn[v][f] = nbr(v, f);
        row(tr, rn, Phi);
    } else {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int f = 0; f < NBF; ++f) Phi[v][f] = 0.0;
        static_for<0, Q>([&](auto rv) __attribute__((always_inline)) {
            constexpr int r = decltype(rv)::value;
            double ro[NV][Q], rn[NV][Q], acc[NV][Q];
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    ro[v][j] = tr[v][mode2(j, 0)];
                    rn[v][j] = nbr(v, mode2(j, 0));
#pragma unroll
                    for (int k = 1; j + k < Q; ++k) {
                        const double c = kRule<P>.val[r][k];
                        if (c != 0.0) {
                            ro[v][j] = fma(c, tr[v][mode2(j, k)], ro[v][j]);
                            rn[v][j] = fma(c, nbr(v, mode2(j, k)), rn[v][j]);
                        }
                    }
                }
            row(ro, rn, acc);
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int j = 0; j < Q; ++j)
#pragma unroll
                    for (int k = 0; j + k < Q; ++k) {
                        const double c = kRule<P>.w[r] * kRule<P>.val[r][k];
                        if (c != 0.0) Phi[v][mode2(j, k)] = fma(c, acc[v][j], Phi[v][mode2(j, k)]);
                    }
        });
    }
}

// R_m -= side^(m_A + 1) (2/h_A) Phi_f(m): the face's flux modes lifted onto
// the cell's modes (before M^-1)
template <int D, int P, int A, int EQ>
__device__ __forceinline__ void lift(const double (&Phi)[nvar<D, EQ>()][face_modes<D, P>()], int side, double sc,
                                     double (&R)[nvar<D, EQ>()][Tab<D, P>::NB])
{
    constexpr int NV = nvar<D, EQ>(), NB = Tab<D, P>::NB;
    const double even = side < 0 ? sc : -sc;
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int m = 0; m < NB; ++m)
            R[v][m] = fma(kTab<D, P>.e[m][A] % 2 == 0 ? even : -sc, Phi[v][face_mode<D, P>(m, A)], R[v][m]);
}

// x / N of a cell index x with g.inv_n = ceil(2^16 / N): exact for x < 4096
// and N <= 16
__device__ __forceinline__ int div_n(int x, unsigned inv_n) { return int((unsigned(x) * inv_n) >> 16); }

// Faces normal to axis a between a slab's cells and the cells outside it:
// count(a) on either side, numbered over the slab's other axes; all sides of
// all axes in sequence (the extra LDS slots): first(a) of the lower axes.
template <int D>
struct SlabFaces {
    int N, rows, layer;
    unsigned inv_n;
    __device__ __forceinline__ int side_faces() const { return D == 2 ? rows : rows * N; }
    __device__ __forceinline__ int count(int a) const { return a == D - 1 ? layer : side_faces(); }
    __device__ __forceinline__ int first(int a) const
    {
        return a < D ? a * 2 * side_faces() : 2 * ((D - 1) * side_faces() + layer);
    }
    // slab cell at face b on the given side
    __device__ __forceinline__ int cell(int a, int side, int b) const
    {
        if (a == D - 1) return b + (side < 0 ? 0 : (rows - 1) * layer);
        const int n = side < 0 ? 0 : N - 1;
        if (a == 0) return n + N * b;
        const int k = div_n(b, inv_n);
        return b - N * k + N * n + layer * k;
    }
    // face number of a cell next to either side
    __device__ __forceinline__ int slot(int a, int lc) const
    {
        const int j = div_n(lc, inv_n);
        if (a == 0) return j;
        const int k = D == 3 ? div_n(j, inv_n) : 0;
        return a == D - 1 ? lc - (D == 3 ? k * layer : j * N) : lc - j * N + N * k;
    }
    __device__ __forceinline__ void ijk(int cell, int *x) const
    {
        const int j = div_n(cell, inv_n), k = D == 3 ? div_n(j, inv_n) : 0;
        x[0] = cell - j * N;
        x[1] = D == 3 ? j - k * N : j;
        x[2] = k;
    }
};

// doubles in the dynamic LDS of a slab of `rows` layers
template <int D, int P, int NV>
constexpr size_t stage_lds_values(int N, int rows)
{
    const size_t layer = D == 2 ? N : size_t(N) * N, side = size_t(rows) * (D == 2 ? 1 : N);
    return size_t((NV * face_modes<D, P>()) | 1) * (rows * layer + 2 * ((D - 1) * side + layer));
}

// Volume integral of one cell by sum factorisation: R_m += sum_q w_q
// F_a(U_q) (2/h_a) dphi_m/dxi_a.  The state along a row of points (x) comes
// from the row's coefficients; the row's fluxes are contracted along x
// before they reach the modes.
template <int D, int P, int EQ, class Args>
__device__ __forceinline__ void volume_rows(const double (&K)[nvar<D, EQ>()][Tab<D, P>::NB],
                                            double (&R)[nvar<D, EQ>()][Tab<D, P>::NB], const double *scale, double gm1,
                                            const Args &gv)
{
    constexpr int NV = nvar<D, EQ>(), NB = Tab<D, P>::NB, Q = P + 1, NB2 = Q * (Q + 1) / 2;
    // C: the polynomial in (x, y) on the plane qz; qz = 0 and unit weight in 2-D
    auto plane = [&](const double (&C)[NV][NB2], auto qzv) __attribute__((always_inline)) {
        constexpr int qz = decltype(qzv)::value;
        static_for<0, Q>([&](auto qyv) __attribute__((always_inline)) {
            constexpr int qy = qyv;
            double row[NV][Q], rx[NV][P], ry[NV][P], rz[NV][P];
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    row[v][i] = C[v][mode2(i, 0)];
#pragma unroll
                    for (int j = 1; i + j < Q; ++j) {
                        const double c = kRule<P>.val[qy][j];
                        if (c != 0.0) row[v][i] = fma(c, C[v][mode2(i, j)], row[v][i]);
                    }
                }
            static_for<0, Q>([&](auto qxv) __attribute__((always_inline)) {
                constexpr int qx = qxv;
                double U[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    U[v] = row[v][0];
#pragma unroll
                    for (int i = 1; i < Q; ++i) {
                        const double c = kRule<P>.val[qx][i];
                        if (c != 0.0) U[v] = fma(c, row[v][i], U[v]);
                    }
                }
                double rinv = 0.0, p = 0.0;
                if constexpr (EQ == EQ_EULER) {
                    rinv = recip(U[0]);
                    p = pressure_r<D>(U, gm1, rinv);
                }
                static_for<0, D>([&](auto Ai) __attribute__((always_inline)) {
                    constexpr int A = Ai;
                    double F[NV];
                    if constexpr (EQ == EQ_ADVECTION) {
                        F[0] = (gv.vel[A] * scale[A]) * U[0];
                    } else { // the flux along A times 2/h_A
                        const double us = U[1 + A] * (rinv * scale[A]), ps = p * scale[A];
                        F[0] = U[0] * us;
#pragma unroll
                        for (int b = 0; b < D; ++b) F[1 + b] = U[1 + b] * us;
                        F[1 + A] += ps;
                        F[D + 1] = fma(U[D + 1], us, ps * (U[1 + A] * rinv));
                    }
#pragma unroll
                    for (int i = 0; i < P; ++i) {
                        // x: modes i + 1 through their derivative; y, z: modes
                        // i < P (the other factor has degree >= 1)
                        const double c = kRule<P>.w[qx] * (A == 0 ? kRule<P>.der[qx][i + 1] : kRule<P>.val[qx][i]);
                        double(&r)[NV][P] = A == 0 ? rx : (A == 1 ? ry : rz);
#pragma unroll
                        for (int v = 0; v < NV; ++v) {
                            if (c != 0.0) r[v][i] = qx == 0 ? c * F[v] : fma(c, F[v], r[v][i]);
                            else if (qx == 0) r[v][i] = 0.0;
                        }
                    }
                });
            });
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const int i = kTab<D, P>.e[m][0], j = kTab<D, P>.e[m][1], k = kTab<D, P>.e[m][2];
                const double wz = D == 3 ? kRule<P>.w[qz] : 1.0, vz = wz * (D == 3 ? kRule<P>.val[qz][k] : 1.0);
                const double vy = kRule<P>.w[qy] * kRule<P>.val[qy][j], dy = kRule<P>.w[qy] * kRule<P>.der[qy][j];
                if (i > 0 && vy != 0.0 && vz != 0.0) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) R[v][m] = fma(vy * vz, rx[v][i - 1], R[v][m]);
                }
                if (j > 0 && dy != 0.0 && vz != 0.0) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) R[v][m] = fma(dy * vz, ry[v][i], R[v][m]);
                }
                if (D == 3 && k > 0) {
                    const double dz = wz * kRule<P>.der[qz][k];
                    if (vy != 0.0 && dz != 0.0) {
#pragma unroll
                        for (int v = 0; v < NV; ++v) R[v][m] = fma(vy * dz, rz[v][i], R[v][m]);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    if constexpr (D == 2) {
        plane(K, std::integral_constant<int, 0>{});
    } else {
        static_for<0, Q>([&](auto qzv) __attribute__((always_inline)) {
            constexpr int qz = decltype(qzv)::value;
            double C[NV][NB2];
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const int f = mode2(kTab<D, P>.e[m][0], kTab<D, P>.e[m][1]), k = kTab<D, P>.e[m][2];
                const double c = kRule<P>.val[qz][k];
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    if (k == 0) C[v][f] = K[v][m];
                    else if (c != 0.0) C[v][f] = fma(c, K[v][m], C[v][f]);
                }
            }
            plane(C, qzv);
        });
    }
}

// ------------------------------------------------------------------ stage kernel
// One thread per cell.  A workgroup covers a slab of `rows` layers of the
// leaf along its last axis (in 3-D slabs of at most 256 cells from degree 2,
// so a thread may keep its cell's state and residual in up to 512
// registers); faces on a slab edge inside the leaf read the adjacent layer
// straight from the stage input.
// threads per workgroup: 3-D degree <= 1 keeps whole 512-cell leaves (the
// state fits 256 registers); every other case uses slabs of <= 256 cells
// (3-D degree 2 in FP32 at 512 threads spills ~600 bytes per lane)
template <int D, int P, typename T = double>
constexpr int stage_threads() { return (D == 3 && P <= 1) ? 512 : 256; }
// default slab (cells per workgroup) when the caller does not choose one.
// Axis by axis (FP64, 2-D and 3-D to degree 1): 128 cells, so that several
// workgroups share a compute unit and hide each other's barriers, and one wave
// at 2-D degree 3, which runs one wave per SIMD (40^2 roots of 16^2 cells:
// degree 1 64 / 128 / 256 cells 32.7 / 30.7 / 32.3 us; degree 2 57.7 / 54.7 /
// 60.8; degree 3 124.6 / 136.8 / 152.6; 3-D degree 1, 12^3 roots of 8^3 cells
// 128 / 256 / 512 cells 153 / 150 / 183 us); 2-D degree 0, whose work is the
// smallest against a workgroup's own (the folded rate's atomic), 192 (12^2-cell
// blocks, 150 000 cells, a run of three steps: 144 cells 90 us, 48 118).  Point by point: 3-D degree 2 in
// FP64 128 cells (256: 2.68 -> 2.53 ms on 16^3 roots), in FP32 the whole budget
// (2.18 against 2.21 ms), as at degree 3, and 128 cells for the other FP32
// kernels below.
template <int D, int P, typename T = double>
constexpr int stage_default_cells()
{
    if (D == 2 && P == 3 && sizeof(T) == 8) return 64;
    if (D == 2 && P == 0 && sizeof(T) == 8) return 192;
    return ((D == 3 && P <= 1) || (D == 3 && P == 2 && sizeof(T) == 8) || (D == 2 && (P == 1 || P == 2)))
               ? 128
               : stage_threads<D, P, T>();
}
// waves per SIMD the register budget is cut for, chosen by measurement on
// large forests: 2-D degree 1 in FP32 fits 128 registers (four waves), in FP64
// 160 (three, without a bound); 2-D degree 2 in FP64 fits 255 with 12 bytes per
// lane spilled (two waves; 2-D degree 3 at two waves spills 1 KB); 2-D degree 3
// in FP32 runs two waves with 212 bytes of spills (-18%); 3-D
// degree 1 in FP32 fits 164 registers (three waves; four: 335 -> 550 us on
// 16^3 roots); 3-D degree 2 in FP32 runs two waves with 268 bytes of
// spills (16^3 roots: 3.46 -> 2.17 ms), while three waves (more spills)
// take 7.0 ms and in FP64 two waves spill 936 bytes (2.69 -> 10.0 ms); 2-D
// degree 2 in FP32 fits 227 registers (two waves; three: 159 -> 263 us on
// 64^2 roots)
template <int D, int P, typename T = double>
constexpr int stage_min_waves()
{
    if (D != 2) return (D == 3 && P == 1 && sizeof(T) == 4) ? 3 : ((D == 3 && P == 2 && sizeof(T) == 4) ? 2 : 1);
    if (P == 1) return sizeof(T) == 4 ? 4 : 1;
    if (P == 2) return 2;
    return P == 3 && sizeof(T) == 4 ? 2 : 1;
}

// One work item: slab `item` of the leaf list (all leaves, or the listed
// ones), for the thread's cell.
template <int D, int P, int GM, int OM, bool LIM, int EQ>
__device__ __forceinline__ void stage_item(const StageArgs &g, int rows, int item, int total)
{
    constexpr int NV = nvar<D, EQ>(), NB = Tab<D, P>::NB, NBF = face_modes<D, P>();
    constexpr int PITCH = (NV * NBF) | 1; // values per LDS slot: odd, so that the lanes spread over the banks
    extern __shared__ double lds[];

    const int N = g.N, ncell = D == 2 ? N * N : N * N * N;
    const int layer = D == 2 ? N : N * N; // cells per layer of the last axis
    const int slabs = N / rows;
    const int wg = xcd_leaf(item, total);
    const int li = wg / slabs, k0 = (wg % slabs) * rows;
    const int leaf = g.work ? g.work[li] : li;
    const int lc = threadIdx.x, nslab = rows * layer;
    const int cell = lc + k0 * layer;
    int ijk[3];
    SlabFaces<D>{N, rows, layer, g.inv_n}.ijk(cell, ijk);
    const double scale[3] = {g.geo[leaf].scale[0], g.geo[leaf].scale[1], g.geo[leaf].scale[2]};
    const long sv = long(NB) * ncell;
    const long base = long(leaf) * NV * sv + cell;
    // (v, m) plane of this leaf in array X: a workgroup-uniform address, so
    // the per-lane part of every state access is the one 32-bit cell offset
    const long lbase = long(leaf) * NV * sv;
    const unsigned uc = unsigned(cell);
    auto plane = [&](auto *X, int v, int m) __attribute__((always_inline)) { return X + (lbase + v * sv + long(m) * ncell); };

    double K[NV][NB], R[NV][NB];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int m = 0; m < NB; ++m) {
            K[v][m] = plane(g.us, v, m)[uc];
            R[v][m] = 0.0;
        }

    // ---- volume integral: sum_q w_q F_a(U_q) (2/h_a) dphi_m/dxi_a, one axis
    // contracted at a time: planes (3-D), rows along x, points.  R is the
    // right-hand side of the weak form; M^-1 (diagonal) follows at the end.
    const double gamma = g.gamma, gm1 = g.gamma - 1.0;
    // scalar convection: the velocity along the leaf's local axes, Q^T vel
    // (Sec. 3.1 frames; the identity on aligned roots)
    struct {
        double vel[3];
    } gv;
    if constexpr (EQ == EQ_ADVECTION) {
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            double s = 0.0;
#pragma unroll
            for (int a = 0; a < D; ++a) s += double(g.geo[leaf].q[3 * a + l]) * g.vel[a];
            gv.vel[l] = s;
        }
    } else {
        gv.vel[0] = gv.vel[1] = gv.vel[2] = 0.0;
    }
    // ---- traces from outside the slab (block faces and slab edges) into their
    // extra LDS slots, the faces of all axes dense over the threads and before
    // the volume integral: one exposed memory latency
    {
        const SlabFaces<D> sf{N, rows, layer, g.inv_n};
        const int total_faces = sf.first(D);
        const int layer_faces = D == 2 ? N : N * N; // cells of a block face
#pragma unroll 1
        for (int e = lc; e < total_faces; e += nslab) {
            // extra slot e: axis, side, face number
            const int a = e < sf.first(1) ? 0 : (D == 2 || e < sf.first(2) ? 1 : 2), b = e - sf.first(a);
            const int nE = sf.count(a), side = b < nE ? -1 : 1;
            const int own = sf.cell(a, side, side < 0 ? b : b - nE), cell2 = own + k0 * layer;
            int ijk2[3];
            sf.ijk(cell2, ijk2);
            const int ia2 = a == 0 ? ijk2[0] : (a == 1 ? ijk2[1] : ijk2[2]);
            const bool at_face = ia2 == (side < 0 ? 0 : N - 1);
            const FaceLink L = g.links[leaf * 2 * D + 2 * a + (side > 0)];
            if (g.conservative && at_face && L.type == dgamr::LINK_FINE) continue; // mortar: its flux is not used
            const int stride = a == 0 ? 1 : (a == 1 ? N : N * N);
            const int t = face_t(ijk2, a, N, D);
            double *const out = lds + PITCH * (nslab + e);
            auto emit = [&](const double *kf, int v, double s) __attribute__((always_inline)) {
                static_for<0, D>([&](auto Ai) __attribute__((always_inline)) {
                    if (a == Ai) {
                        double tr[NBF];
                        face_trace<D, P, Ai>(kf, s, tr);
#pragma unroll
                        for (int f = 0; f < NBF; ++f) out[v * NBF + f] = tr[f];
                    }
                });
            };
            if (GM == GUARD_INLINE && at_face && (L.type == dgamr::LINK_COARSE || L.type == dgamr::LINK_FINE)) {
                if constexpr (P == 0) {
                    // one value per variable: the mean of the finer cells, or
                    // the coarser cell's.  The cells are found once (their
                    // indices take divisions by N), and the loads of all
                    // variables go together (3-D, one root in ten
                    // refined, 40 000 cells in 2^3 / 8^3 blocks, a step: 124 / 52
                    // -> 97 / 36 us)
                    double kf[NV];
                    if (L.type == dgamr::LINK_COARSE) {
                        const double *src = g.us + long(L.nbr[0]) * NV * sv + coarse_cell(a, side, t, L.off, N, D);
#pragma unroll
                        for (int v = 0; v < NV; ++v) kf[v] = src[v * sv];
                    } else {
                        const double *src = g.us + long(link_nbr(L, fine_block(t, N, D))) * NV * sv;
#pragma unroll
                        for (int v = 0; v < NV; ++v) kf[v] = 0.0;
#pragma unroll
                        for (int ch = 0; ch < (1 << D); ++ch) {
                            const double *fc = src + fine_cell(a, side, t, ch, N, D);
#pragma unroll
                            for (int v = 0; v < NV; ++v) kf[v] = fma(kTab<D, P>.comb[ch][0][0], fc[v * sv], kf[v]);
                        }
                    }
#pragma unroll
                    for (int v = 0; v < NV; ++v) out[v] = kf[v];
                } else {
                    // hanging faces, one variable at a time
#pragma unroll 1
                    for (int v = 0; v < NV; ++v) {
                        double kf[NB];
                        hanging_var<D, P, NV>(g, v, a, side, t, L, kf);
                        emit(kf, v, double(-side));
                    }
                }
            } else {
                // one source cell, every load issued before the first use: the
                // neighbour cell at a slab edge or in the neighbour leaf, the
                // guard cell, or (outflow) the own cell, whose trace is the
                // mirror image's
                const double *nk;
                long step = ncell;
                bool mirror = false;
                if (!at_face) {
                    nk = g.us + lbase + cell2 + side * stride;
                } else if constexpr (GM == GUARD_BUFFER) {
                    step = layer_faces;
                    nk = g.guard + ((long(leaf) * 2 * D + 2 * a + (side > 0)) * NV * NB) * step + t;
                } else {
                    mirror = L.type == dgamr::LINK_BOUNDARY;
                    nk = mirror ? g.us + lbase + cell2
                                : g.us + long(L.nbr[0]) * NV * sv + same_cell(a, side, t, N, D);
                }
                double kf[NV][NB];
#pragma unroll
                for (int v = 0; v < NV; ++v)
#pragma unroll
                    for (int m = 0; m < NB; ++m) kf[v][m] = nk[(v * NB + m) * step];
#pragma unroll
                for (int v = 0; v < NV; ++v) emit(kf[v], v, double(mirror ? side : -side));
            }
        }
    }
    if constexpr (P > 0) {
        volume_rows<D, P, EQ>(K, R, scale, gm1, gv);
    }

    // ---- surface integrals, one axis at a time.  The trace of a cell on a
    // face is a polynomial in the NBF face modes.  Its T+ goes into the
    // cell's LDS slot, the traces from outside the slab into extra slots;
    // the + neighbour (for the slab's last cells, one of the first nE
    // threads) evaluates both traces at the face points, takes the flux,
    // projects it onto the face modes and leaves those where it found T+, so
    // an axis needs two barriers and every face of the slab is done once.
    static_for<0, D>([&](auto Ai) __attribute__((always_inline)) {
        constexpr int A = Ai;
        const int stride = A == 0 ? 1 : (A == 1 ? N : N * N);
        const int ia = ijk[A];
        // neighbours inside this slab
        const bool in_m = A == D - 1 ? ia > k0 : ia > 0;
        const double sc = scale[A];
        const SlabFaces<D> sf{N, rows, layer, g.inv_n};
        double *const ext = lds + PITCH * (nslab + sf.first(A)); // 2 nE slots
        const int nE = sf.count(A);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            double tp[NBF];
            face_trace<D, P, A>(K[v], 1.0, tp);
#pragma unroll
            for (int f = 0; f < NBF; ++f) lds[lc * PITCH + v * NBF + f] = tp[f];
        }
        bool mort_m = false, mort_p = false;
        if (g.conservative) { // uniform: mortar on faces to finer leaves
            const FaceLink Lm = g.links[leaf * 2 * D + 2 * A], Lp = g.links[leaf * 2 * D + 2 * A + 1];
            mort_m = ia == 0 && Lm.type == dgamr::LINK_FINE;
            mort_p = ia == N - 1 && Lp.type == dgamr::LINK_FINE;
            if (mort_m) mortar_lift<D, P, A, EQ, double, false>(g, K, R, -1, Lm, face_t(ijk, A, N, D), sc);
            if (mort_p) mortar_lift<D, P, A, EQ, double, false>(g, K, R, +1, Lp, face_t(ijk, A, N, D), sc);
        }
        __syncthreads();
        // the - faces of all cells, then the + faces of the slab's last
        // cells; alternate axes start from the other end of the workgroup so
        // that the same waves do not take them all
        const int e = A % 2 == 0 ? lc : nslab - 1 - lc;
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
            int side = 2 * pass - 1;
            asm volatile("" : "+s"(side)); // one body for both passes
            if (side > 0 && e >= nE) break;
            const int own = side < 0 ? lc : sf.cell(A, 1, e); // whose + / - trace
            // the neighbour's trace, and where the flux modes go
            double *const nb = side < 0 && in_m ? lds + (lc - stride) * PITCH
                                           : ext + (side < 0 ? sf.slot(A, lc) : nE + e) * PITCH;
            double *const dst = side < 0 ? nb : lds + own * PITCH;
            double Phi[NV][NBF];
            face_flux<D, P, A, EQ>(
                double(side), gamma, gv,
                [&](int v, double *tr) __attribute__((always_inline)) {
                    if (side < 0) {
                        face_trace<D, P, A>(K[v], -1.0, tr);
                    } else {
#pragma unroll
                        for (int f = 0; f < NBF; ++f) tr[f] = lds[own * PITCH + v * NBF + f];
                    }
                },
                [&](int v, int f) __attribute__((always_inline)) { return nb[v * NBF + f]; }, Phi);
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int f = 0; f < NBF; ++f) dst[v * NBF + f] = Phi[v][f];
            if (side < 0 && !mort_m) lift<D, P, A, EQ>(Phi, -1, sc, R);
        }
        __syncthreads();
        if (!mort_p) {
            double Phi[NV][NBF];
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int f = 0; f < NBF; ++f) Phi[v][f] = lds[lc * PITCH + v * NBF + f];
            lift<D, P, A, EQ>(Phi, +1, sc, R);
        }
    });

    // ---- output
    if constexpr (OM == OUT_RES64) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int m = 0; m < NB; ++m) plane(g.out64, v, m)[uc] = R[v][m] * kTab<D, P>.inv_mass[m];
    } else {
        double dt;
        if (g.rate_in) {
            const double rate = __longlong_as_double((long long)*g.rate_in);
            dt = g.cfl / rate;
            if (item == 0 && threadIdx.x == 0) *g.dt_out = dt;
        } else {
            dt = g.dt[g.leaf_member ? g.leaf_member[leaf] : 0];
        }
        if (g.rate_clear && item == 0 && threadIdx.x == 0) *g.rate_clear = 0ULL;
        const double a = g.rk_a, b = g.rk_b;
        double Kn[NV][NB];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int m = 0; m < NB; ++m) Kn[v][m] = b * fma(dt * kTab<D, P>.inv_mass[m], R[v][m], K[v][m]);
        // stages 2 and 3 add the RK base state; a uniform branch keeps its
        // loads here, after the residual, instead of live through it
        if (a != 0.0) {
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int m = 0; m < NB; ++m) Kn[v][m] = fma(a, plane(g.un, v, m)[uc], Kn[v][m]);
        }
        if constexpr (LIM && EQ == EQ_EULER) limit_cell<D, P>(Kn, g.gamma);
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int m = 0; m < NB; ++m) plane(g.out64, v, m)[uc] = Kn[v][m];
        if (g.rate_out) {
            // CFL rate of the new state from its cell mean, folded over the block
            double rate = 0.0;
            if constexpr (EQ == EQ_ADVECTION) {
#pragma unroll
                for (int a2 = 0; a2 < D; ++a2) rate += fabs(g.vel[a2]) / g.geo[leaf].h[a2];
            } else {
                double U[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) U[v] = Kn[v][0];
                const double rinv = 1.0 / U[0];
                const double cs = sqrt(g.gamma * pressure_r<D>(U, g.gamma - 1.0, rinv) * rinv);
#pragma unroll
                for (int a2 = 0; a2 < D; ++a2) rate += (fabs(U[1 + a2] * rinv) + cs) / g.geo[leaf].h[a2];
            }
            block_max_to(rate, lds, g.rate_out);
        }
    }
}

// Whether the stage item contracts axis by axis: FP64, 2-D and 3-D to degree
// 1.  From degree 2 in 3-D one thread cannot hold the state, the residual
// and a face's traces and fluxes (16^3 roots, degree 2: 15.2 ms per two steps
// point by point, 16.2 axis by axis with 440 bytes of spills).  Scalar
// convection at degree 0 has nothing to contract (3-D, 150 000 cells in 2^3 /
// 8^3 blocks 65 / 22 us a step point by point, 82 / 24 axis by axis).
template <int D, int P, typename T, int EQ = EQ_EULER>
constexpr bool by_axis() { return sizeof(T) == 8 && (D == 2 || P <= 1) && (EQ == EQ_EULER || P > 0); }

// the item with the contractions point by point (kernels_points.hpp)
template <int D, int P, int GM, int OM, bool LIM, typename T, int EQ, bool MF>
__device__ __forceinline__ void stage_item_points(const StageArgs &g, int rows, int item, int total);

// T: the arithmetic of the residual, double or float (the state, the stage
// update, the limiter and the CFL rate are FP64).
// The stage kernel: one workgroup per (leaf, slab) work item, or (PERSIST,
// a grid smaller than the item count) each workgroup walks the items with
// a stride of the grid size.  With a grid that is a
// multiple of the XCD count every item a workgroup takes maps to the same
// XCD's leaf range.
template <int D, int P, int GM, int OM, bool LIM, typename T = double, int EQ = EQ_EULER, bool PERSIST = false,
          bool MF = false, bool AXIS = by_axis<D, P, T, EQ>()>
__global__ __launch_bounds__((stage_threads<D, P, T>()), (stage_min_waves<D, P, T>())) void k_stage(StageArgs g,
                                                                                                     int rows)
{
    const int total = g.nleaves * (g.N / rows);
    auto run = [&](int item) __attribute__((always_inline)) {
        if constexpr (AXIS) stage_item<D, P, GM, OM, LIM, EQ>(g, rows, item, total);
        else stage_item_points<D, P, GM, OM, LIM, T, EQ, MF>(g, rows, item, total);
    };
    if constexpr (PERSIST) {
        for (int item = blockIdx.x; item < total; item += gridDim.x) {
            run(item);
            if constexpr (AXIS) __syncthreads(); // the next item reuses the LDS
        }
    } else { // one item per workgroup: no loop to hold values across items
        run(blockIdx.x);
    }
}

// ------------------------------------------------------------------ guard fill
// One thread per guard cell (leaf, face, t): Eq. 15 copy, Eq. 16 split of the
// coarser neighbour cell, Eq. 17 combine of the 2^d finer cells, outflow
// mirror K_m (-1)^{m_axis}.
template <int D, int P, int NV = D + 2>
__global__ __launch_bounds__(256) void k_fill(FillArgs g)
{
    constexpr int NB = Tab<D, P>::NB;
    const int N = g.N, ncell = D == 2 ? N * N : N * N * N, nfc = D == 2 ? N : N * N;
    const long gid = long(blockIdx.x) * blockDim.x + threadIdx.x;
    if (gid >= long(g.nfaces) * nfc) return;
    const int fi = int(gid / nfc), t = int(gid % nfc);
    const int lf = g.work ? g.work[fi / (2 * D)] * 2 * D + fi % (2 * D) : fi;
    const int leaf = lf / (2 * D), face = lf % (2 * D);
    const int a = face / 2, side = (face & 1) ? 1 : -1;
    const FaceLink L = g.links[lf];
    const long sv = long(NB) * ncell;
    // one variable of the guard cell
    auto emit = [&](int v, const double *gk) __attribute__((always_inline)) {
        double *out = g.guard + (long(lf) * NV * NB) * nfc + t;
#pragma unroll
        for (int m = 0; m < NB; ++m) out[(v * NB + m) * nfc] = gk[m];
    };
    if (L.rot > 0) {
        // a neighbour root of another frame (Sec. 3.5): copy, split or combine
        // in the source frame, then the rotation R^n into this leaf's frame
        const RotPlan Rp = g.plans[L.rot - 1 + t];
        double ks[NV][NB];
        for (int v = 0; v < NV; ++v) {
            double kv[NB];
            if (Rp.type == dgamr::PLAN_COMBINE) {
#pragma unroll
                for (int m = 0; m < NB; ++m) kv[m] = 0.0;
                for (int ch = 0; ch < (1 << D); ++ch) {
                    const double *src = g.u + long(Rp.leaf[ch]) * NV * sv + long(v) * sv + Rp.cell[ch];
                    double kf[NB];
#pragma unroll
                    for (int n = 0; n < NB; ++n) kf[n] = src[long(n) * ncell];
                    comb_any<D, P>(ch, kf, kv);
                }
            } else {
                const double *src = g.u + long(Rp.leaf[0]) * NV * sv + long(v) * sv + Rp.cell[0];
                double kc[NB];
#pragma unroll
                for (int n = 0; n < NB; ++n) kc[n] = src[long(n) * ncell];
                if (Rp.type == dgamr::PLAN_SPLIT) split_any<D, P, double>(Rp.child, kc, kv);
                else
#pragma unroll
                    for (int n = 0; n < NB; ++n) kv[n] = kc[n];
            }
            // modes: phi_n(m xi) = sign * phi_n'(xi), exponent l of n' = exponent
            // l' of n where m[l'][l] != 0
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                int e2[3] = {0, 0, 0};
                double sg = 1.0;
                for (int lp = 0; lp < D; ++lp)
                    for (int l = 0; l < D; ++l) {
                        const int mm = Rp.m[3 * lp + l];
                        if (mm != 0) {
                            e2[l] = kTab<D, P>.e[n][lp];
                            if (mm < 0 && (kTab<D, P>.e[n][lp] & 1)) sg = -sg;
                        }
                    }
                int idx = 0;
                for (int q = 0; q < NB; ++q)
                    if (kTab<D, P>.e[q][0] == e2[0] && kTab<D, P>.e[q][1] == e2[1] && kTab<D, P>.e[q][2] == e2[2])
                        idx = q;
                ks[v][idx] = sg * kv[n];
            }
        }
        if (NV == D + 2 && !g.global_vectors) { // momentum into this leaf's frame: m_dst[l] = sum_l' m[l'][l] m_src[l']
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                double mv[3] = {0.0, 0.0, 0.0};
                for (int l = 0; l < D; ++l)
                    for (int lp = 0; lp < D; ++lp) mv[l] += double(Rp.m[3 * lp + l]) * ks[1 + lp][n];
                for (int l = 0; l < D; ++l) ks[1 + l][n] = mv[l];
            }
        }
        for (int v = 0; v < NV; ++v) emit(v, ks[v]);
        return;
    }
    if (L.type == dgamr::LINK_SAME) {
        const int c = same_cell(a, side, t, N, D);
        const double *src = g.u + long(L.nbr[0]) * NV * sv + c;
        for (int v = 0; v < NV; ++v) {
            double gk[NB];
#pragma unroll
            for (int m = 0; m < NB; ++m) gk[m] = src[v * sv + m * ncell];
            emit(v, gk);
        }
    } else if (L.type == dgamr::LINK_BOUNDARY) {
        const int c = face_cell(a, side > 0 ? N - 1 : 0, t, N, D);
        const double *src = g.u + long(leaf) * NV * sv + c;
        for (int v = 0; v < NV; ++v) {
            double gk[NB];
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const double k = src[v * sv + m * ncell];
                const int ex = kTab<D, P>.e[m][0] * (a == 0) + kTab<D, P>.e[m][1] * (a == 1) +
                               kTab<D, P>.e[m][2] * (a == 2);
                gk[m] = (ex % 2) ? -k : k;
            }
            emit(v, gk);
        }
    } else if (L.type == dgamr::LINK_COARSE) {
        // the guard cell (fine size) lies in one coarse cell; along a it is
        // the half nearest to this leaf
        const int c = coarse_cell(a, side, t, L.off, N, D);
        const int child = coarse_child(a, side, t, N, D);
        const double *src = g.u + long(L.nbr[0]) * NV * sv + c;
        for (int v = 0; v < NV; ++v) {
            double ks[NB], gk[NB];
#pragma unroll
            for (int n = 0; n < NB; ++n) ks[n] = src[v * sv + n * ncell];
            split_any<D, P, double>(child, ks, gk);
            emit(v, gk);
        }
    } else { // LINK_FINE: 2^d fine cells, 2 along a and 2^(d-1) tangential
        const double *base = g.u + long(link_nbr(L, fine_block(t, N, D))) * NV * sv;
        for (int v = 0; v < NV; ++v) {
            double acc[NB];
#pragma unroll
            for (int m = 0; m < NB; ++m) acc[m] = 0.0;
#pragma unroll
            for (int ch = 0; ch < (1 << D); ++ch) {
                const int c = fine_cell(a, side, t, ch, N, D);
                double ks[NB];
#pragma unroll
                for (int n = 0; n < NB; ++n) ks[n] = base[v * sv + n * ncell + c];
#pragma unroll
                for (int m = 0; m < NB; ++m)
#pragma unroll
                    for (int n = 0; n < NB; ++n) {
                        const double cc = kTab<D, P>.comb[ch][m][n];
                        if (cc != 0.0) acc[m] = fma(cc, ks[n], acc[m]);
                    }
            }
            emit(v, acc);
        }
    }
}

} // namespace dgk
