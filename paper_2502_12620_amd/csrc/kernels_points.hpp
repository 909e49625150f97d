// The stage item with the contractions point by point, one thread per cell,
// for the cases the axis-by-axis item (kernels.hpp) does not take:
//  - FP32 arithmetic (the FP32 residual, and the fused stage on an FP64 state
//    read as FP64 and rounded once): contracting in another order would round
//    differently at 1e-8 of the state, which is held in FP64;
//  - FP64 in 3-D from degree 2, where one thread's state and residual alone
//    take 100 (degree 2) or 200 of its 256 doubles.  At degree 3 the
//    axis-by-axis form spills 2.7 KB per lane and 13 000 scalars, and one of
//    its builds returned wrong momenta in the residual of a conservative
//    hanging forest.  Its source is right: compiled for the host it agrees with
//    this item to 2e-15 there, whatever the order of the threads between
//    barriers and the contents of LDS (tests/native/stage_kernels_check.cpp),
//    as do the instances in use, none of whose residuals spills to memory.
//    What that build did wrong on the GPU is not known.  Steps run one lane per
//    (cell, variable) there (kernels_3d.hpp) unless they have the limiter or
//    mortar faces.
#pragma once

#include "kernels.hpp"

namespace dgk {

// Number of face points exchanged through LDS at once: all of them in 2-D,
// one at a time in 3-D (keeps the register budget to one cell's state and
// residual).
template <int D, int P>
constexpr int face_chunk() { return D == 2 ? (P == 3 ? 2 : Tab<D, P>::NF) : 1; }

// Far-side traces of block face (A, side) at the FCH face points starting
// at f0, for the cell with tangential index t (the far polynomial touches
// the face with its -side side):
//  - guard-buffer mode: the stored guard cell;
//  - inline mode: the same-level neighbour cell (Eq. 15), the split of the
//    coarser neighbour cell (Eq. 16), the combine of the 2^d finer cells
//    (Eq. 17), or at an outflow boundary the mirror image, whose trace is
//    the own trace.
template <int D, int P, int A, int GM, int FCH, int NV, typename T>
__device__ __forceinline__ void far_traces(const StageArgs &g, const T (&K)[NV][Tab<D, P>::NB], int leaf, int side,
                                           int t, const FaceLink &L, int f0, T (&Tr)[FCH][NV])
{
    constexpr int NB = Tab<D, P>::NB;
    const int N = g.N, ncell = D == 2 ? N * N : N * N * N, nfc = D == 2 ? N : N * N;
    const long sv = long(NB) * ncell;
    const int face = 2 * A + (side > 0);
    auto traces_of = [&](const T *kv, int v, int poly_side) {
#pragma unroll
        for (int fi = 0; fi < FCH; ++fi) {
            T e, o;
            trace_eo<D, P, T>(kv, A, f0 + fi, e, o);
            Tr[fi][v] = poly_side > 0 ? e + o : e - o;
        }
    };
    if (GM == GUARD_BUFFER) {
        const double *gk = g.guard + ((long(leaf) * 2 * D + face) * NV * NB) * nfc + t;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            T kv[NB];
#pragma unroll
            for (int m = 0; m < NB; ++m) kv[m] = T(gk[(long(v) * NB + m) * nfc]);
            traces_of(kv, v, -side);
        }
        return;
    }
    if (L.type == dgamr::LINK_BOUNDARY) {
#pragma unroll
        for (int v = 0; v < NV; ++v) traces_of(K[v], v, side);
    } else if (L.type == dgamr::LINK_SAME) {
        const int c = same_cell(A, side, t, N, D);
        const double *nk = g.us + long(L.nbr[0]) * NV * sv + c;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            T kv[NB];
#pragma unroll
            for (int m = 0; m < NB; ++m) kv[m] = T(nk[v * sv + m * ncell]);
            traces_of(kv, v, -side);
        }
    } else if (L.type == dgamr::LINK_COARSE) {
        const int c = coarse_cell(A, side, t, L.off, N, D);
        const int child = coarse_child(A, side, t, N, D);
        const double *ck = g.us + long(L.nbr[0]) * NV * sv + c;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            T kv[NB], gv[NB];
#pragma unroll
            for (int m = 0; m < NB; ++m) kv[m] = T(ck[v * sv + m * ncell]);
            split_any<D, P, T>(child, kv, gv);
            traces_of(gv, v, -side);
        }
    } else { // LINK_FINE
        const double *fk = g.us + long(link_nbr(L, fine_block(t, N, D))) * NV * sv;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            T gv[NB];
#pragma unroll
            for (int m = 0; m < NB; ++m) gv[m] = T(0);
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
                        if (cc != 0.0) gv[m] = fma(T(cc), kv[n], gv[m]);
                    }
            }
            traces_of(gv, v, -side);
        }
    }
}

// the volume integral on the matrix cores (kernels_mfma.hpp)
template <int D, int P>
__device__ __forceinline__ void volume_mfma(const float (&K)[D + 2][Tab<D, P>::NB], float (&R)[D + 2][Tab<D, P>::NB],
                                            float *lds, const float *scale, float gm1);
template <int D, int P>
constexpr int mfma_lds_floats();

// MF: the volume integral on the matrix cores (FP32 Euler, whole waves of
// cells; kernels_mfma.hpp)
template <int D, int P, int GM, int OM, bool LIM, typename T, int EQ, bool MF>
__device__ __forceinline__ void stage_item_points(const StageArgs &g, int rows, int item, int total)
{
    constexpr int NV = nvar<D, EQ>(), NB = Tab<D, P>::NB, NQ = Tab<D, P>::NQ, NF = Tab<D, P>::NF;
    constexpr int FCH = face_chunk<D, P>();
    extern __shared__ double lds_d[];
    T *lds = reinterpret_cast<T *>(lds_d);

    const int N = g.N, ncell = D == 2 ? N * N : N * N * N;
    const int layer = D == 2 ? N : N * N; // cells per layer of the last axis
    const int slabs = N / rows;
    const int wg = xcd_leaf(item, total);
    const int li = wg / slabs, k0 = (wg % slabs) * rows;
    const int leaf = g.work ? g.work[li] : li;
    const int lc = threadIdx.x, nslab = rows * layer;
    const int cell = lc + k0 * layer;
    int ijk[3];
    cell_ijk(cell, N, D, ijk);
    const T scale[3] = {T(g.geo[leaf].scale[0]), T(g.geo[leaf].scale[1]), T(g.geo[leaf].scale[2])};
    const long sv = long(NB) * ncell;
    const long base = long(leaf) * NV * sv + cell;
    // (v, m) plane of this leaf in array X: a workgroup-uniform address, so
    // the per-lane part of every state access is the one 32-bit cell offset
    const long lbase = long(leaf) * NV * sv;
    const unsigned uc = unsigned(cell);
    auto plane = [&](auto *X, int v, int m) __attribute__((always_inline)) { return X + (lbase + v * sv + long(m) * ncell); };

    T K[NV][NB], R[NV][NB];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int m = 0; m < NB; ++m) {
            K[v][m] = T(plane(g.us, v, m)[uc]);
            R[v][m] = T(0);
        }

    // ---- volume integral: sum_q w_q F_a(U_q) (2/h_a) dphi_m/dxi_a / M_m
    const T gamma = T(g.gamma), gm1 = T(g.gamma - 1.0);
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
    auto vol_point = [&](auto qv) __attribute__((always_inline)) {
        const int q = qv;
        T U[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            T s = T(0);
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const double c = kTake32<D, P, T> ? kPointTab32<D, P>.phi_v[q][m] : kTab<D, P>.phi_v[q][m];
                if (use_entry<D, P>(c)) s = fma(T(c), K[v][m], s);
            }
            U[v] = s;
        }
        T rinv = T(0), p = T(0);
        if constexpr (EQ == EQ_EULER) {
            rinv = recip(U[0]);
            p = pressure_r<D, T>(U, gm1, rinv);
        }
        static_for<0, D>([&](auto Ai) __attribute__((always_inline)) {
            constexpr int A = Ai;
            T F[NV];
            if constexpr (EQ == EQ_ADVECTION) F[0] = T(gv.vel[A]) * U[0];
            else euler_flux<D, A, T>(U, U[1 + A] * rinv, p, F);
#pragma unroll
            for (int v = 0; v < NV; ++v) F[v] *= scale[A];
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const double c = kTake32<D, P, T> ? kPointTab32<D, P>.dproj[A][q][m] : kTab<D, P>.dproj[A][q][m];
                // a mode of degree 0 along A has no derivative along A
                if (kTab<D, P>.e[m][A] != 0 && use_entry<D, P>(c)) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) R[v][m] = fma(T(c), F[v], R[v][m]);
                }
            }
        });
    };
    if constexpr (MF) {
        static_assert(std::is_same<T, float>::value && EQ == EQ_EULER, "matrix-core volume: FP32 Euler");
        float *wave_lds = reinterpret_cast<float *>(lds_d) + (threadIdx.x >> 6) * mfma_lds_floats<D, P>();
        // the per-wave regions alias the face exchange and the CFL fold of
        // the previous work item of a persistent workgroup: every wave
        // leaves them before any wave writes here
        __syncthreads();
        volume_mfma<D, P>(K, R, wave_lds, scale, gm1);
    } else if constexpr (unroll_points<D, P>()) {
        static_for<0, NQ>(vol_point);
    } else {
#pragma unroll 1
        for (int q = 0; q < NQ; ++q) vol_point(q);
    }

    // ---- surface integrals, one axis at a time
    static_for<0, D>([&](auto Ai) __attribute__((always_inline)) {
        constexpr int A = Ai;
        const int stride = A == 0 ? 1 : (A == 1 ? N : N * N);
        const int ia = ijk[A];
        // neighbours reachable through LDS (inside this slab)
        const bool in_m = A == D - 1 ? ia > k0 : ia > 0;
        const bool in_p = A == D - 1 ? ia < k0 + rows - 1 : ia < N - 1;
        const int t = face_t(ijk, A, N, D);
        const T sc = scale[A];
        const FaceLink Lm = g.links[leaf * 2 * D + 2 * A];
        const FaceLink Lp = g.links[leaf * 2 * D + 2 * A + 1];
        const bool mort_m = g.conservative && ia == 0 && Lm.type == dgamr::LINK_FINE;
        const bool mort_p = g.conservative && ia == N - 1 && Lp.type == dgamr::LINK_FINE;
        if (mort_m) mortar_lift<D, P, A, EQ, T, true>(g, K, R, -1, Lm, t, sc);
        if (mort_p) mortar_lift<D, P, A, EQ, T, true>(g, K, R, +1, Lp, t, sc);
        // In 3-D a cell has at most one side along A whose neighbour is not
        // in the slab (slabs hold at least two layers or the whole leaf); the
        // polynomial across it (the neighbour cell at a slab edge, or the
        // far side of a block face: guard coefficients, or inline copy /
        // split / combine / mirror) is built once here and its traces taken
        // per face point.  Read per face point, the compiler hoists both
        // sides' loads out of the point loop and holds them (3-D degree 1 with
        // slab edges: 255 registers and a spill -> 213).  Mortar faces and
        // block faces read as traces keep their own paths.  In 2-D
        // (unrolled points) the per-point reads spill less.
        constexpr bool FAR_REGS = D == 3;
        const bool edge_m = FAR_REGS ? (!in_m && !mort_m)
                                     : (A == D - 1 && !in_m && ia > 0);
        const bool edge_p = FAR_REGS ? (!in_p && !mort_p)
                                     : (A == D - 1 && !in_p && ia < N - 1);
        constexpr int NBE = FAR_REGS ? NB : 1;
        T nb[NV][NBE];
        if constexpr (FAR_REGS) {
            if (edge_m || edge_p) {
                const int side = edge_m ? -1 : 1;
                if (edge_m ? ia > 0 : ia < N - 1) { // slab edge: the neighbour cell
                    const double *nk = g.us + base + side * stride;
#pragma unroll
                    for (int v = 0; v < NV; ++v)
#pragma unroll
                        for (int m = 0; m < NB; ++m) nb[v][m] = T(nk[v * sv + m * ncell]);
                } else if (edge_m) { // (a link chosen at run time would go to scratch)
                    far_poly<D, P, A, GM, NV, T>(g, K, leaf, -1, t, Lm, nb);
                } else {
                    far_poly<D, P, A, GM, NV, T>(g, K, leaf, +1, t, Lp, nb);
                }
            } else {
#pragma unroll
                for (int v = 0; v < NV; ++v)
#pragma unroll
                    for (int m = 0; m < NB; ++m) nb[v][m] = T(0);
            }
        }
        auto face_chunk_body = [&](auto cv) __attribute__((always_inline)) {
            const int f0 = int(cv) * FCH;
            // own traces of this chunk: + side to LDS, - side kept
            T Tm[FCH][NV];
            __syncthreads();
#pragma unroll
            for (int fi = 0; fi < FCH; ++fi)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    T e, o;
                    trace_eo<D, P, T>(K[v], A, f0 + fi, e, o);
                    lds[(v * FCH + fi) * nslab + lc] = e + o;
                    Tm[fi][v] = e - o;
                }
            __syncthreads();
            // flux on the - face: left state = the left neighbour's + trace
            T Fm[FCH][NV];
            if (in_m) {
#pragma unroll
                for (int fi = 0; fi < FCH; ++fi) {
                    T TL[NV];
#pragma unroll
                    for (int v = 0; v < NV; ++v) TL[v] = lds[(v * FCH + fi) * nslab + lc - stride];
                    num_flux<D, A, EQ, T>(gv, TL, Tm[fi], gamma, Fm[fi]);
                }
            } else if (edge_m) { // slab edge inside the leaf: the layer below
#pragma unroll
                for (int fi = 0; fi < FCH; ++fi) {
                    T TL[NV];
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        T e, o;
                        if constexpr (FAR_REGS) trace_eo<D, P, T>(nb[v], A, f0 + fi, e, o);
                        else trace_eo_mem<D, P, T>(g.us + base - stride + v * sv, ncell, A, f0 + fi, e, o);
                        TL[v] = e + o;
                    }
                    num_flux<D, A, EQ, T>(gv, TL, Tm[fi], gamma, Fm[fi]);
                }
            } else if (!mort_m) {
                T TL[FCH][NV];
                far_traces<D, P, A, GM, FCH, NV, T>(g, K, leaf, -1, t, Lm, f0, TL);
#pragma unroll
                for (int fi = 0; fi < FCH; ++fi) num_flux<D, A, EQ, T>(gv, TL[fi], Tm[fi], gamma, Fm[fi]);
            } else {
#pragma unroll
                for (int fi = 0; fi < FCH; ++fi)
#pragma unroll
                    for (int v = 0; v < NV; ++v) Fm[fi][v] = T(0);
            }
            __syncthreads();
#pragma unroll
            for (int fi = 0; fi < FCH; ++fi)
#pragma unroll
                for (int v = 0; v < NV; ++v) lds[(v * FCH + fi) * nslab + lc] = Fm[fi][v];
            __syncthreads();
            T Fp[FCH][NV];
            if (in_p) {
#pragma unroll
                for (int fi = 0; fi < FCH; ++fi)
#pragma unroll
                    for (int v = 0; v < NV; ++v) Fp[fi][v] = lds[(v * FCH + fi) * nslab + lc + stride];
            } else if (edge_p) { // slab edge inside the leaf: the layer above
#pragma unroll
                for (int fi = 0; fi < FCH; ++fi) {
                    T TL[NV], TR[NV];
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        T e, o;
                        trace_eo<D, P, T>(K[v], A, f0 + fi, e, o);
                        TL[v] = e + o;
                        if constexpr (FAR_REGS) trace_eo<D, P, T>(nb[v], A, f0 + fi, e, o);
                        else trace_eo_mem<D, P, T>(g.us + base + stride + v * sv, ncell, A, f0 + fi, e, o);
                        TR[v] = e - o;
                    }
                    num_flux<D, A, EQ, T>(gv, TL, TR, gamma, Fp[fi]);
                }
            } else if (!mort_p) {
                T TR[FCH][NV];
                far_traces<D, P, A, GM, FCH, NV, T>(g, K, leaf, +1, t, Lp, f0, TR);
#pragma unroll
                for (int fi = 0; fi < FCH; ++fi) {
                    T TL[NV];
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        T e, o;
                        trace_eo<D, P, T>(K[v], A, f0 + fi, e, o);
                        TL[v] = e + o;
                    }
                    num_flux<D, A, EQ, T>(gv, TL, TR[fi], gamma, Fp[fi]);
                }
            } else {
#pragma unroll
                for (int fi = 0; fi < FCH; ++fi)
#pragma unroll
                    for (int v = 0; v < NV; ++v) Fp[fi][v] = T(0);
            }
            // lift: R_m += s_a w phi_m(+1)/M_m ((-1)^{m_A} Phi_- - Phi_+)
#pragma unroll
            for (int fi = 0; fi < FCH; ++fi) {
                const int F = f0 + fi;
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const T dm = sc * Fm[fi][v], dp = sc * Fp[fi][v];
                    const T even = dm - dp, odd = -(dm + dp);
#pragma unroll
                    for (int m = 0; m < NB; ++m) {
                        const double c = kTake32<D, P, T> ? kPointTab32<D, P>.lift_f[A][F][m] : kTab<D, P>.lift_f[A][F][m];
                        if (use_entry<D, P>(c)) R[v][m] = fma(T(c), (kTab<D, P>.e[m][A] % 2 == 0) ? even : odd, R[v][m]);
                    }
                }
            }
        };
        if constexpr (unroll_points<D, P>()) {
            static_for<0, NF / FCH>(face_chunk_body);
        } else {
#pragma unroll 1
            for (int ci = 0; ci < NF / FCH; ++ci) face_chunk_body(ci);
        }
    });

    // ---- output
    if constexpr (OM == OUT_RES64) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int m = 0; m < NB; ++m) plane(g.out64, v, m)[uc] = double(R[v][m]);
    } else if constexpr (OM == OUT_RES32) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int m = 0; m < NB; ++m) plane(g.out32, v, m)[uc] = float(R[v][m]);
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
        // FP64 update; the FP32 path re-reads U_s at full precision
        double Kn[NV][NB];
        if constexpr (std::is_same<T, double>::value) {
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int m = 0; m < NB; ++m) Kn[v][m] = b * (K[v][m] + dt * R[v][m]);
        } else if (b != 0.0) {
            // FP32 path: U_s again at full precision; inside a (uniform)
            // branch so that its loads are issued here, not held in
            // registers through the residual
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int m = 0; m < NB; ++m) Kn[v][m] = b * (plane(g.us, v, m)[uc] + dt * double(R[v][m]));
        } else {
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int m = 0; m < NB; ++m) Kn[v][m] = 0.0;
        }
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
            block_max_to(rate, lds_d, g.rate_out);
        }
    }
}

} // namespace dgk
