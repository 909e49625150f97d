// 3-D DG stage kernel with one lane per (cell, variable).
//
// Twelve cells of five conserved variables fill lanes 0..59 of a wave
// (lanes 60..63 repeat the last cell's lanes and store nothing).  Each lane
// keeps only its variable's coefficients and residual, so a cell's state
// and residual take 4 N_b registers per lane instead of 20 N_b in one
// thread.  The Euler and Rusanov fluxes need all five variables of a point:
// the lanes of a cell write five points' values to LDS records, each lane
// then computes the flux of one of the five points, and the lanes read their
// variable back, so no flux is computed twice.
//
// A workgroup covers a slab of layers of one leaf, one layer at a time along
// z.  A face between two layers needs no exchange (the same lanes hold both
// cells: the next layer is loaded while the current one is computed); x and
// y faces go through LDS as face modes as in the thread-per-cell kernel, the
// + faces of a layer's last cells computed by the cell slots that the
// layer's N^2 cells leave free (N = 8: 72 slots in 6 waves, 64 cells and 8
// faces).  Runs the fused RK stage in FP64 for the Euler equations without
// the limiter and without mortar faces; everything else takes the
// thread-per-cell kernel.
#pragma once

#include "kernels_2d.hpp"
#include "launch.hpp"

namespace dgk {

// An empty asm that takes and returns x: what x depends on is computed before
// it.  Without it the compiler sinks the residual's contractions to the
// stage update and keeps every flux of the volume integral until then.
#define DG_PIN(x) asm volatile("" : "+v"(x))

// doubles of one point's LDS record: five variables of the own and of the
// neighbour's state in, the flux out; odd, to spread the records over the banks
constexpr int kRec3v = 11;

// waves per SIMD the register budget is cut for
template <int P>
constexpr int waves_3v() { return P <= 1 ? 4 : 3; }

// Euler flux of a point's five variables: the lanes of a cell exchange the
// values of up to five points through the wave's LDS records (rec: the
// record of the cell's point 0; own: this lane's own record).
struct Lanes3 {
    double *rec, *own;
    int v;
    __device__ __forceinline__ void put(int o, int slot, double x) const { rec[o * kRec3v + slot * 5 + v] = x; }
    __device__ __forceinline__ double get(int o) const { return rec[o * kRec3v + v]; }
};

// Volume integral of this lane's variable: R_m += int F_a dphi_m/dx_a.  sc:
// 2/h_a; isE, isM: 1 on the lane of the energy / the momentum along a.
template <int P>
__device__ __forceinline__ void volume_3v(const double *K, double *R, const Lanes3 &ln, const double *sc, double gm1,
                                          double isE, const double *isM)
{
    constexpr int NB = Tab<3, P>::NB, NQ = Tab<3, P>::NQ, Q = P + 1, NB2 = Q * (Q + 1) / 2;
    double C[NB2], row[Q], rx[P], ry[P], rz[P];
    const double cm[3] = {isM[0] * sc[0], isM[1] * sc[1], isM[2] * sc[2]};
    static_for<0, (NQ + 4) / 5>([&](auto gv) __attribute__((always_inline)) {
        double val[5];
        static_for<0, 5>([&](auto ov) __attribute__((always_inline)) {
            constexpr int o = ov, q = 5 * decltype(gv)::value + o;
            if constexpr (q < NQ) {
                constexpr int qx = q % Q, qy = (q / Q) % Q, qz = q / (Q * Q);
                if constexpr (qx == 0 && qy == 0) // the polynomial on this plane
#pragma unroll
                    for (int m = 0; m < NB; ++m) {
                        const int f = mode2(kTab<3, P>.e[m][0], kTab<3, P>.e[m][1]), k = kTab<3, P>.e[m][2];
                        const double c = kRule<P>.val[qz][k];
                        if (k == 0) C[f] = K[m];
                        else if (c != 0.0) C[f] = fma(c, K[m], C[f]);
                    }
                if constexpr (qx == 0) // on this row
#pragma unroll
                    for (int i = 0; i < Q; ++i) {
                        row[i] = C[mode2(i, 0)];
#pragma unroll
                        for (int j = 1; i + j < Q; ++j) {
                            const double c = kRule<P>.val[qy][j];
                            if (c != 0.0) row[i] = fma(c, C[mode2(i, j)], row[i]);
                        }
                    }
                double s = row[0];
#pragma unroll
                for (int i = 1; i < Q; ++i) {
                    const double c = kRule<P>.val[qx][i];
                    if (c != 0.0) s = fma(c, row[i], s);
                }
                val[o] = s;
                ln.put(o, 0, s);
            }
        });
        wave_lds_sync();
        { // this lane's point: velocities times 2/h_a, and the pressure
            double U[5];
#pragma unroll
            for (int b = 0; b < 5; ++b) U[b] = ln.own[b];
            const double rinv = recip(U[0]);
            const double p = pressure_r<3>(U, gm1, rinv);
#pragma unroll
            for (int a = 0; a < 3; ++a) ln.own[a] = U[1 + a] * (rinv * sc[a]);
            ln.own[3] = p;
        }
        wave_lds_sync();
        static_for<0, 5>([&](auto ov) __attribute__((always_inline)) {
            constexpr int o = ov, q = 5 * decltype(gv)::value + o;
            if constexpr (q < NQ) {
                constexpr int qx = q % Q, qy = (q / Q) % Q, qz = q / (Q * Q);
                const double p = ln.rec[o * kRec3v + 3];
                static_for<0, 3>([&](auto Ai) __attribute__((always_inline)) {
                    constexpr int A = Ai;
                    const double us = ln.rec[o * kRec3v + A];
                    const double F = fma(val[o], us, p * fma(isE, us, cm[A]));
                    double(&r)[P] = A == 0 ? rx : (A == 1 ? ry : rz);
#pragma unroll
                    for (int i = 0; i < P; ++i) {
                        // x: modes i + 1 through their derivative; y, z: modes i < P
                        const double c = kRule<P>.w[qx] * (A == 0 ? kRule<P>.der[qx][i + 1] : kRule<P>.val[qx][i]);
                        if (c != 0.0) r[i] = qx == 0 ? c * F : fma(c, F, r[i]);
                        else if (qx == 0) r[i] = 0.0;
                    }
                });
                if constexpr (qx == Q - 1) // the row's fluxes onto the modes
#pragma unroll
                    for (int m = 0; m < NB; ++m) {
                        const int i = kTab<3, P>.e[m][0], j = kTab<3, P>.e[m][1], k = kTab<3, P>.e[m][2];
                        const double vz = kRule<P>.w[qz] * kRule<P>.val[qz][k], dz = kRule<P>.w[qz] * kRule<P>.der[qz][k];
                        const double vy = kRule<P>.w[qy] * kRule<P>.val[qy][j], dy = kRule<P>.w[qy] * kRule<P>.der[qy][j];
                        if (i > 0 && vy * vz != 0.0) R[m] = fma(vy * vz, rx[i - 1], R[m]);
                        if (j > 0 && dy * vz != 0.0) R[m] = fma(dy * vz, ry[i], R[m]);
                        if (k > 0 && vy * dz != 0.0) R[m] = fma(vy * dz, rz[i], R[m]);
                        DG_PIN(R[m]);
                    }
            }
        });
        wave_lds_sync();
        __builtin_amdgcn_sched_barrier(0);
    });
}

// Flux of one face in its face modes, this lane's variable: to the own trace,
// nbr(f) mode f of the neighbour's, side +1 / -1 the side of the own cell the
// face is on.
template <int P, int A, class Nbr>
__device__ __forceinline__ void face_flux_3v(const double *to, Nbr &&nbr, double side, double gamma, const Lanes3 &ln,
                                             double *Phi)
{
    constexpr int NF = Tab<3, P>::NF, Q = P + 1, NBF = face_modes<3, P>();
    struct {
    } none;
    double ro[Q], rn[Q], acc[Q];
#pragma unroll
    for (int f = 0; f < NBF; ++f) Phi[f] = 0.0;
    static_for<0, (NF + 4) / 5>([&](auto gv) __attribute__((always_inline)) {
        static_for<0, 5>([&](auto ov) __attribute__((always_inline)) {
            constexpr int o = ov, f = 5 * decltype(gv)::value + o;
            if constexpr (f < NF) {
                constexpr int t0 = f % Q, t1 = f / Q;
                if constexpr (t0 == 0)
#pragma unroll
                    for (int j = 0; j < Q; ++j) {
                        ro[j] = to[mode2(j, 0)];
                        rn[j] = nbr(mode2(j, 0));
#pragma unroll
                        for (int k = 1; j + k < Q; ++k) {
                            const double c = kRule<P>.val[t1][k];
                            if (c != 0.0) {
                                ro[j] = fma(c, to[mode2(j, k)], ro[j]);
                                rn[j] = fma(c, nbr(mode2(j, k)), rn[j]);
                            }
                        }
                    }
                double uo = ro[0], un = rn[0];
#pragma unroll
                for (int j = 1; j < Q; ++j) {
                    const double c = kRule<P>.val[t0][j];
                    if (c != 0.0) {
                        uo = fma(c, ro[j], uo);
                        un = fma(c, rn[j], un);
                    }
                }
                ln.put(o, 0, uo);
                ln.put(o, 1, un);
            }
        });
        wave_lds_sync();
        {
            double Uo[5], Un[5], F[5];
#pragma unroll
            for (int b = 0; b < 5; ++b) {
                Uo[b] = ln.own[b];
                Un[b] = ln.own[5 + b];
            }
            side_flux<3, A, EQ_EULER>(none, Uo, Un, side, gamma, F);
#pragma unroll
            for (int b = 0; b < 5; ++b) ln.own[b] = F[b];
        }
        wave_lds_sync();
        static_for<0, 5>([&](auto ov) __attribute__((always_inline)) {
            constexpr int o = ov, f = 5 * decltype(gv)::value + o;
            if constexpr (f < NF) {
                constexpr int t0 = f % Q, t1 = f / Q;
                const double F = ln.get(o);
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    const double c = kRule<P>.w[t0] * kRule<P>.val[t0][j];
                    if (c != 0.0) acc[j] = t0 == 0 ? c * F : fma(c, F, acc[j]);
                    else if (t0 == 0) acc[j] = 0.0;
                }
                if constexpr (t0 == Q - 1)
#pragma unroll
                    for (int j = 0; j < Q; ++j)
#pragma unroll
                        for (int k = 0; j + k < Q; ++k) {
                            const double c = kRule<P>.w[t1] * kRule<P>.val[t1][k];
                            if (c != 0.0) Phi[mode2(j, k)] = fma(c, acc[j], Phi[mode2(j, k)]);
                        }
            }
        });
        wave_lds_sync();
        __builtin_amdgcn_sched_barrier(0);
    });
}

// R_m -= side^(m_A + 1) (2/h_A) Phi_f(m), this lane's variable (before M^-1)
template <int P, int A>
__device__ __forceinline__ void lift_3v(const double *Phi, double side, double sc, double *R)
{
    const double even = -side * sc;
#pragma unroll
    for (int m = 0; m < Tab<3, P>::NB; ++m)
        R[m] = fma(kTab<3, P>.e[m][A] % 2 == 0 ? even : -sc, Phi[face_mode<3, P>(m, A)], R[m]);
#pragma unroll
    for (int m = 0; m < Tab<3, P>::NB; ++m) DG_PIN(R[m]);
}

// This lane's variable of the polynomial across block face (a, side) at
// tangential index t: the guard cell, the neighbour's cell, its split or
// combine, or at an outflow boundary the mirror image of the own cell (index
// own in the leaf).
template <int P, int GM>
__device__ __forceinline__ void far_3v(const StageArgs &g, int leaf, int v, int a, int side, int t, int own, double *kf)
{
    constexpr int NV = 5, NB = Tab<3, P>::NB;
    const int N = g.N, layer = N * N, ncell = layer * N;
    const long sv = long(NB) * ncell;
    if constexpr (GM == GUARD_BUFFER) {
        const double *gk = g.guard + ((long(leaf) * 6 + 2 * a + (side > 0)) * NV + v) * NB * layer + t;
#pragma unroll
        for (int m = 0; m < NB; ++m) kf[m] = gk[long(m) * layer];
    } else {
        const FaceLink L = g.links[leaf * 6 + 2 * a + (side > 0)];
        if (L.type == dgamr::LINK_COARSE || L.type == dgamr::LINK_FINE) {
            hanging_var<3, P, NV>(g, v, a, side, t, L, kf);
        } else {
            const bool mirror = L.type == dgamr::LINK_BOUNDARY;
            const double *nk = g.us + (mirror ? long(leaf) : long(L.nbr[0])) * NV * sv + v * sv +
                               (mirror ? own : same_cell(a, side, t, N, 3));
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const int e = kTab<3, P>.e[m][0] * (a == 0) + kTab<3, P>.e[m][1] * (a == 1) + kTab<3, P>.e[m][2] * (a == 2);
                kf[m] = nk[long(m) * ncell];
                if (mirror && (e & 1)) kf[m] = -kf[m];
            }
        }
    }
}

// What bounds it: the latencies of one layer's chain (two LDS round trips per
// group of five points, the far traces and the RK base state) with three
// waves per SIMD that the barriers keep in the same phase; at degree 3 also
// registers (spills at 168).  8^3-cell blocks, average stage with everything
// that goes before it: degree 2, 16^3 roots 2.52 ms (one thread per cell, one
// wave per SIMD) -> 1.84 ms; degree 3, 8^3 roots 1.43 ms (every lane computing
// every point's flux, faces in chunks with 12 barriers per axis, guard traces
// written by a fill before) -> 1.02 ms.  One item of six waves per workgroup
// took 2.60 ms at degree 2: 1.5 waves per SIMD.
//
// One (leaf, slab of `rows` layers) takes waves_item waves, 64 lanes per 12 of
// the layer's N^2 cells and N + faces; a workgroup holds `group` of them, so
// that its waves spread evenly over a compute unit's four SIMDs (a second
// workgroup of six waves was not placed beside the first).  lds_item: doubles
// of LDS per item.
template <int P, int GM, int OM>
__global__ __launch_bounds__(kThreads3v, waves_3v<P>()) void k_stage3v(StageArgs g, int rows, int waves_item, int group,
                                                                          int lds_item)
{
    constexpr int NV = 5, NB = Tab<3, P>::NB, NBF = face_modes<3, P>(), PITCH = (NV * NBF) | 1;
    // the RK base state loaded ahead of its use, where the registers allow (the
    // next layer is to degree 2)
    constexpr bool PREFETCH = P <= 1;
    extern __shared__ double lds_all[];
    const int N = g.N, layer = N * N, ncell = layer * N;
    const int slabs = N / rows, items = g.nleaves * slabs;
    const int wgwave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), sub = wgwave / waves_item;
    const int item = xcd_leaf(blockIdx.x, gridDim.x) * group + sub;
    const bool real = item < items; // the last workgroup may be partly empty: it repeats the last item
    const int it0 = real ? item : items - 1;
    const int li = it0 / slabs, k0 = (it0 % slabs) * rows;
    const int leaf = g.work ? g.work[li] : li; // listed leaves of a pool, or all
    const int lane = threadIdx.x & 63, wave = wgwave - sub * waves_item;
    double *const lds = lds_all + sub * lds_item;
    const int lv = lane < 5 * kCells3v ? lane : lane - 5; // lanes 60..63 repeat lanes 55..58
    const int cw = lv / 5, v = lv - 5 * cw;
    const int slot = wave * kCells3v + cw, nslots = waves_item * kCells3v;
    // slots: the layer's cells, then the + faces of the last cells of its
    // rows (x) or columns (y); the rest store nothing
    const bool is_cell = slot < layer, live = real && lane < 5 * kCells3v && is_cell;
    const bool active = lane < 5 * kCells3v && slot < layer + N;
    const int c = is_cell ? slot : layer - 1; // spare slots repeat the last cell
    const int j = div_n(c, g.inv_n), i = c - j * N;
    const int pf = is_cell ? 0 : (slot - layer < N ? slot - layer : N - 1);
    const double side = is_cell ? -1.0 : 1.0;
    double *const recs = lds + wave * 5 * kCells3v * kRec3v;
    const Lanes3 ln{recs + 5 * cw * kRec3v, recs + lv * kRec3v, v};
    double *const T = lds + waves_item * 5 * kCells3v * kRec3v; // layer + 4 N slots of PITCH
    double *const Tv = T + v * NBF;
    const double isE = v == 4 ? 1.0 : 0.0;
    const double isM[3] = {v == 1 ? 1.0 : 0.0, v == 2 ? 1.0 : 0.0, v == 3 ? 1.0 : 0.0};
    const double sc[3] = {g.geo[leaf].scale[0], g.geo[leaf].scale[1], g.geo[leaf].scale[2]};
    const double gm1 = g.gamma - 1.0;
    const long sv = long(NB) * ncell;
    // mode m's planes of this leaf in array X at a workgroup-uniform address;
    // the lanes add one 32-bit offset
    const long lbase = long(leaf) * NV * sv;
    const unsigned uc = unsigned(v) * unsigned(sv) + unsigned(c);
    auto plane = [&](auto *X, int m) __attribute__((always_inline)) { return X + (lbase + long(m) * ncell); };

    double dt = 0.0;
    if constexpr (OM == OUT_RK) {
        if (g.rate_in) {
            dt = g.cfl / __longlong_as_double((long long)*g.rate_in);
            if (blockIdx.x == 0 && threadIdx.x == 0) *g.dt_out = dt;
        } else {
            dt = g.dt[g.leaf_member ? g.leaf_member[leaf] : 0];
        }
        if (g.rate_clear && blockIdx.x == 0 && threadIdx.x == 0) *g.rate_clear = 0ULL;
    }
    // layer k of this lane's column; outside the leaf the polynomial across
    // the z face
    auto load_layer = [&](int k, double *X) __attribute__((always_inline)) {
        if (k >= 0 && k < N) { // uniform
#pragma unroll
            for (int m = 0; m < NB; ++m) X[m] = plane(g.us, m)[uc + unsigned(k * layer)];
        } else {
            far_3v<P, GM>(g, leaf, v, 2, k < 0 ? -1 : 1, c, c + (k < 0 ? 0 : N - 1) * layer, X);
        }
    };
    double K[NB], Kn[NB], R[NB]; // current and next layer; R starts with the face below
#pragma unroll
    for (int m = 0; m < NB; ++m) R[m] = 0.0;
    double rate = 0.0;
    // per iteration: load the next layer, finish the current one (from
    // it = 0), take the flux between them (from it = -1)
#pragma unroll 1
    for (int it = -2; it < rows; ++it) {
        const int k = k0 + it;
        if (P <= 2 || it < 0) load_layer(k + 1, Kn);
        double Un[NB];
        if (it >= 0) {
            // traces across the leaf's x and y faces, spread over the waves (the
            // first one is hidden from the compiler, which would otherwise hoist
            // every address out of the layer loop into registers)
            int s0 = cw * waves_item + wave;
            asm volatile("" : "+v"(s0));
            for (int s = s0; s < 4 * N; s += nslots) {
                const int a = s < 2 * N ? 0 : 1, b0 = s - 2 * N * a, sd = b0 < N ? -1 : 1, b = b0 < N ? b0 : b0 - N;
                const int n = sd < 0 ? 0 : N - 1;
                double kf[NB], tr[NBF];
                far_3v<P, GM>(g, leaf, v, a, sd, b + N * k, (a == 0 ? n + N * b : b + N * n) + k * layer, kf);
                if (a == 0) face_trace<3, P, 0>(kf, double(-sd), tr);
                else face_trace<3, P, 1>(kf, double(-sd), tr);
                if (lane < 5 * kCells3v)
#pragma unroll
                    for (int f = 0; f < NBF; ++f) Tv[(layer + s) * PITCH + f] = tr[f];
            }
            if constexpr (P > 0) volume_3v<P>(K, R, ln, sc, gm1, isE, isM);
            static_for<0, 2>([&](auto Ai) __attribute__((always_inline)) {
                constexpr int A = Ai;
                const int ia = A == 0 ? i : j, stride = A == 0 ? 1 : N, jb = A == 0 ? j : i;
                double to[NBF], Phi[NBF];
                face_trace<3, P, A>(K, 1.0, to);
                if (is_cell && lane < 5 * kCells3v)
#pragma unroll
                    for (int f = 0; f < NBF; ++f) Tv[c * PITCH + f] = to[f];
                __syncthreads();
                // the - faces of the cells, and in the spare slots the + faces
                // of the last cells; the flux modes replace T+
                const int own = A == 0 ? (N - 1) + N * pf : pf + N * (N - 1);
                const int ext = layer + 2 * N * A + (is_cell ? jb : N + pf);
                const double *const nb = Tv + (is_cell && ia > 0 ? c - stride : ext) * PITCH;
                if (is_cell) face_trace<3, P, A>(K, -1.0, to);
                else
#pragma unroll
                    for (int f = 0; f < NBF; ++f) to[f] = Tv[own * PITCH + f];
                face_flux_3v<P, A>(to, [&](int f) __attribute__((always_inline)) { return nb[f]; }, side, g.gamma, ln, Phi);
                double *const dst = Tv + (is_cell ? c - stride : own) * PITCH;
                if (active && (!is_cell || ia > 0))
#pragma unroll
                    for (int f = 0; f < NBF; ++f) dst[f] = Phi[f];
                lift_3v<P, A>(Phi, -1.0, sc[A], R); // (a spare slot's R is not used)
                __syncthreads();
#pragma unroll
                for (int f = 0; f < NBF; ++f) Phi[f] = Tv[c * PITCH + f];
                lift_3v<P, A>(Phi, 1.0, sc[A], R);
            });
            if constexpr (P > 2) load_layer(k + 1, Kn);
            if constexpr (OM == OUT_RK)
                if (PREFETCH && g.rk_a != 0.0) // uniform: stages 2 and 3 add the RK base state
#pragma unroll
                    for (int m = 0; m < NB; ++m) Un[m] = plane(g.un, m)[uc + unsigned(k * layer)];
        }
        // the face above
        double Pt[NBF];
        if (it >= -1) {
            double to[NBF], tn[NBF];
            face_trace<3, P, 2>(K, 1.0, to);
            face_trace<3, P, 2>(Kn, -1.0, tn);
            face_flux_3v<P, 2>(to, [&](int f) __attribute__((always_inline)) { return tn[f]; }, 1.0, g.gamma, ln, Pt);
        }
        if (it >= 0) {
            lift_3v<P, 2>(Pt, 1.0, sc[2], R);
            const unsigned idx = uc + unsigned(k * layer);
            if constexpr (OM == OUT_RES64) {
                if (live)
#pragma unroll
                    for (int m = 0; m < NB; ++m) plane(g.out64, m)[idx] = R[m] * kTab<3, P>.inv_mass[m];
            } else {
                const double a = g.rk_a, b = g.rk_b;
#pragma unroll
                for (int m = 0; m < NB; ++m) K[m] = b * fma(dt * kTab<3, P>.inv_mass[m], R[m], K[m]);
                if (a != 0.0) {
#pragma unroll
                    for (int m = 0; m < NB; ++m) K[m] = fma(a, PREFETCH ? Un[m] : plane(g.un, m)[idx], K[m]);
                }
                if (live)
#pragma unroll
                    for (int m = 0; m < NB; ++m) plane(g.out64, m)[idx] = K[m];
                if (g.rate_out) {
                    // CFL rate of the new state from its cell mean
                    ln.put(0, 0, K[0]);
                    wave_lds_sync();
                    double U[5];
#pragma unroll
                    for (int b2 = 0; b2 < 5; ++b2) U[b2] = ln.rec[b2];
                    wave_lds_sync();
                    const double rinv = 1.0 / U[0];
                    const double cs = sqrt(g.gamma * pressure_r<3>(U, gm1, rinv) * rinv);
                    double r = 0.0;
#pragma unroll
                    for (int a2 = 0; a2 < 3; ++a2) r += (fabs(U[1 + a2] * rinv) + cs) / g.geo[leaf].h[a2];
                    rate = nan_max(rate, r);
                }
            }
        }
#pragma unroll
        for (int m = 0; m < NB; ++m) {
            K[m] = Kn[m];
            R[m] = 0.0;
        }
        if (it >= -1) lift_3v<P, 2>(Pt, -1.0, sc[2], R);
    }
    // No rate of a spare slot, whose state took a + face's flux for a - face's,
    // nor of a repeated item, which in the last stage (un and out64 are one
    // array) may have read what the item it repeats had stored already: what
    // either computes from there is dropped
    if constexpr (OM == OUT_RK)
        if (g.rate_out) block_max_to(real && is_cell ? rate : 0.0, lds_all, g.rate_out);
}

} // namespace dgk
