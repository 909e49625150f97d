// One (dim, degree) instantiation of the degree-templated kernels and their
// launchers; compiled once per pair with -DDG_D=<dim> -DDG_P=<degree> and
// -DDG_PART=<part>, the heavy kernels split over parts so that the units
// compile in parallel:
//   part 0  the dispatcher launch_stage, the 2-D lane-per-(cell, variable)
//           kernels, scalar convection, fill, limiter, projection, inheritance
//   part 1  the thread-per-cell Euler stage kernels in FP64
//   part 2  the thread-per-cell Euler stage kernels with FP32 arithmetic
//   part 3  the diffusion stage
//   part 4  the thread-per-cell Euler stage kernels with FP32 arithmetic and
//           the volume integral on the matrix cores (degree >= 2)
//   part 5  the 3-D lane-per-(cell, variable) stage kernels
#include "kernels.hpp"
#include "kernels_2d.hpp"
#include "kernels_3d.hpp"
#include "kernels_aux.hpp"
#include "kernels_ipdg.hpp"
#include "kernels_mapped.hpp"
#include "kernels_mfma.hpp"
#include "kernels_points.hpp"
#include "launch.hpp"

#ifndef DG_D
#error "DG_D must be defined"
#endif
#ifndef DG_P
#error "DG_P must be defined"
#endif
#ifndef DG_PART
#error "DG_PART must be defined"
#endif

namespace dgk {

// 2-D without the limiter: one lane per (cell, variable), a slab of rows
// per workgroup, with enough slabs to give every compute unit work.
template <int P>
hipError_t launch_stage_2v(const StageArgs &a, int gm, int om, hipStream_t s, int rows_req)
{
    int rows = a.N;
    if (rows_req > 0) {
        if (a.N % rows_req != 0 || rows_req * a.N * 4 > 512) return hipErrorInvalidValue;
        rows = rows_req;
    } else {
        while (rows * a.N * 4 > 512) rows /= 2;
        // thinner slabs until every compute unit has one, of at least a whole
        // wave (16 leaves of 8^2 cells, degree 1: 2 rows 6.7 us, 1 row 7.6)
        while (rows % 2 == 0 && rows * a.N * 4 >= 128 && long(a.nleaves) * (a.N / rows) < 256) rows /= 2;
    }
    const int slabs = a.N / rows;
    const size_t lds = sizeof(double) * (P + 1) * rows * a.N * 4;
    const dim3 grid(unsigned(a.nleaves * slabs)), block(rows * a.N * 4);
    if (gm == GUARD_BUFFER && om == OUT_RES64)
        hipLaunchKernelGGL((k_stage2v<P, GUARD_BUFFER, OUT_RES64>), grid, block, lds, s, a, rows);
    else if (gm == GUARD_INLINE && om == OUT_RK)
        hipLaunchKernelGGL((k_stage2v<P, GUARD_INLINE, OUT_RK>), grid, block, lds, s, a, rows);
    else if (gm == GUARD_BUFFER && om == OUT_RK) // far side from the (rotated) guard fill
        hipLaunchKernelGGL((k_stage2v<P, GUARD_BUFFER, OUT_RK>), grid, block, lds, s, a, rows);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// 3-D FP64 residual or fused stage with one lane per (cell, variable)
template <int P>
hipError_t launch_stage_3v(const StageArgs &args, int gm, int om, hipStream_t s, int rows_req)
{
    StageArgs a = args;
    a.inv_n = unsigned((65536 + a.N - 1) / a.N);
    const int N = a.N;
    int rows = rows_req;
    if (rows > 0) {
        if (!rows_ok_3v(N, rows)) return hipErrorInvalidValue;
    } else {
        // whole leaves, in thinner slabs (which take a z face more each) until
        // there are 1024 items, four a compute unit: 8^3 cells, degree 3, a step on
        // 720 leaves in half blocks 4.46 ms, whole 5.21; 512 leaves in half blocks
        // 3.07, whole 2.86, in quarters 3.39; 4^3 cells, 512 leaves 0.51 in half
        // blocks, 0.66 whole; 1024 or more leaves whole (1452: 1.29, half blocks 1.47)
        rows = N;
        while (rows % 2 == 0 && long(a.nleaves) * (N / rows) < 1024) rows /= 2;
    }
    const int waves = (N * N + N + kCells3v - 1) / kCells3v;
    int group = 1; // items per workgroup: whole fours of waves
    while (waves * group % 4 != 0) ++group;
    const int lds_item = waves * 5 * kCells3v * kRec3v + (N * N + 4 * N) * ((5 * face_modes<3, P>()) | 1);
    const size_t lds = sizeof(double) * size_t(lds_item) * group;
    const long items = long(a.nleaves) * (N / rows);
    const dim3 grid(unsigned((items + group - 1) / group)), block(64 * waves * group);
    if (gm == GUARD_INLINE && om == OUT_RK)
        hipLaunchKernelGGL((k_stage3v<P, GUARD_INLINE, OUT_RK>), grid, block, lds, s, a, rows, waves, group, lds_item);
    else if (gm == GUARD_BUFFER && om == OUT_RK)
        hipLaunchKernelGGL((k_stage3v<P, GUARD_BUFFER, OUT_RK>), grid, block, lds, s, a, rows, waves, group, lds_item);
    else if (gm == GUARD_BUFFER && om == OUT_RES64)
        hipLaunchKernelGGL((k_stage3v<P, GUARD_BUFFER, OUT_RES64>), grid, block, lds, s, a, rows, waves, group, lds_item);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int D, int P, typename T>
bool rows_ok(int N, int rows)
{
    const int layer = D == 2 ? N : N * N;
    // 3-D: at least two layers unless the whole leaf (a cell has at most one
    // slab edge)
    return rows >= 1 && N % rows == 0 && (D == 2 || rows >= 2 || rows == N) && rows * layer <= stage_threads<D, P, T>();
}

template <int D, int P>
int stage_rows_options(int N, int *rows, int max_options, bool fp32)
{
    int n = 0;
    for (int r = N; r >= 1 && n < max_options; --r)
        if (fp32 ? rows_ok<D, P, float>(N, r) : rows_ok<D, P, double>(N, r)) rows[n++] = r;
    return n;
}

template <int D, int P, typename T, int EQ = EQ_EULER, bool MF = false, bool AXIS = by_axis<D, P, T, EQ>()>
hipError_t launch_stage_cell(const StageArgs &args, int gm, int om, bool lim, const StageShape &sh, hipStream_t s)
{
    StageArgs a = args;
    a.inv_n = unsigned((65536 + a.N - 1) / a.N);
    // slab of `rows` layers along the last axis within the thread budget
    const int layer = D == 2 ? a.N : a.N * a.N;
    int rows = sh.rows;
    if (rows == 0) {
        rows = a.N;
        if constexpr (AXIS) {
            // the slab that fills its waves best; among equals the tallest of
            // at most stage_default_cells cells (12^2-cell blocks, 100^2 roots,
            // degree 2: 4 rows, 48 of 64 lanes, 213 us; 6 rows, 72 of 128, 271;
            // 12 rows, 144 of 192, 261)
            double best = 0.0;
            for (int r = a.N; r >= 1; --r) {
                if (!rows_ok<D, P, T>(a.N, r)) continue;
                const int cells = r * layer;
                double fill = cells / (64.0 * ((cells + 63) / 64));
                if (cells > stage_default_cells<D, P, T>()) fill -= 1e-3;
                if (fill > best) {
                    best = fill;
                    rows = r;
                }
            }
        } else {
            while (rows % 2 == 0 && rows * layer > stage_default_cells<D, P, T>()) rows /= 2;
        }
    }
    if (!rows_ok<D, P, T>(a.N, rows)) return hipErrorInvalidValue;
    const int nslab = rows * layer;
    const long items = long(a.nleaves) * (a.N / rows);
    // the face exchange (point by point: face points in chunks; axis by axis:
    // the face modes of every slab cell and of the cells outside), and the
    // workgroup maximum of the CFL rate
    size_t lds = sizeof(double) * (D + 2) * face_chunk<D, P>() * nslab;
    if constexpr (AXIS) {
        lds = sizeof(double) * stage_lds_values<D, P, nvar<D, EQ>()>(a.N, rows);
        if (lds < sizeof(double) * size_t(nslab)) lds = sizeof(double) * size_t(nslab);
    }
    if constexpr (MF) {
        // whole waves only; the volume phase's per-wave LDS regions alias the
        // face exchange's buffer
        if (nslab % 64 != 0) return hipErrorNotSupported;
        const size_t mf = sizeof(float) * size_t(mfma_lds_floats<D, P>()) * (nslab / 64);
        lds = mf > lds ? mf : lds;
    }
    const bool persist = sh.grid > 0 && sh.grid < items;
    // the persistent shape applies to the fused Euler stage (pools); every
    // other launch takes one workgroup per item
    const dim3 grid(unsigned(persist ? sh.grid : items)), block(nslab);
    const dim3 grid_all = dim3(unsigned(items));
    // the fused stage takes the far side of block faces inline (copy,
    // split, combine, mirror of the neighbour cells), or on forests with
    // rotated root frames from the guard fill; the residual entry point
    // reads guard coefficients
    if constexpr (EQ == EQ_ADVECTION) {
        // one variable: the far side is always taken inline
        if (gm == GUARD_INLINE && om == OUT_RK) {
            hipLaunchKernelGGL((k_stage<D, P, GUARD_INLINE, OUT_RK, false, T, EQ, false, false, AXIS>), grid_all, block, lds, s, a, rows);
            return hipGetLastError();
        }
        if (gm == GUARD_BUFFER && om == OUT_RES64) {
            hipLaunchKernelGGL((k_stage<D, P, GUARD_BUFFER, OUT_RES64, false, T, EQ, false, false, AXIS>), grid_all, block, lds, s, a, rows);
            return hipGetLastError();
        }
        if (gm == GUARD_BUFFER && om == OUT_RK) { // rotated root frames
            hipLaunchKernelGGL((k_stage<D, P, GUARD_BUFFER, OUT_RK, false, T, EQ, false, false, AXIS>), grid_all, block, lds, s, a, rows);
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    constexpr int GMRK = GUARD_INLINE; // the fused stage takes the far side inline
    if (gm == GMRK && om == OUT_RK) {
        if (persist && lim)
            hipLaunchKernelGGL((k_stage<D, P, GMRK, OUT_RK, true, T, EQ_EULER, true, MF, AXIS>), grid, block, lds, s, a, rows);
        else if (persist)
            hipLaunchKernelGGL((k_stage<D, P, GMRK, OUT_RK, false, T, EQ_EULER, true, MF, AXIS>), grid, block, lds, s, a, rows);
        else if (lim)
            hipLaunchKernelGGL((k_stage<D, P, GMRK, OUT_RK, true, T, EQ_EULER, false, MF, AXIS>), grid, block, lds, s, a, rows);
        else
            hipLaunchKernelGGL((k_stage<D, P, GMRK, OUT_RK, false, T, EQ_EULER, false, MF, AXIS>), grid, block, lds, s, a, rows);
        return hipGetLastError();
    }
    if (gm == GUARD_BUFFER && om == OUT_RK) {
        // the fused stage reading the far side from the guard fill (forests
        // with rotated root frames), one workgroup per item, on the vector
        // unit
        if constexpr (MF) {
            return hipErrorNotSupported;
        } else {
            if (lim)
                hipLaunchKernelGGL((k_stage<D, P, GUARD_BUFFER, OUT_RK, true, T, EQ_EULER, false, false, AXIS>), grid_all, block, lds, s, a, rows);
            else
                hipLaunchKernelGGL((k_stage<D, P, GUARD_BUFFER, OUT_RK, false, T, EQ_EULER, false, false, AXIS>), grid_all, block, lds, s, a, rows);
            return hipGetLastError();
        }
    }
    if constexpr (std::is_same<T, float>::value) {
        if (gm == GUARD_BUFFER && om == OUT_RES32) {
            hipLaunchKernelGGL((k_stage<D, P, GUARD_BUFFER, OUT_RES32, false, T, EQ_EULER, false, MF, AXIS>), grid_all, block,
                               lds, s, a, rows);
            return hipGetLastError();
        }
    } else {
        if (gm == GUARD_BUFFER && om == OUT_RES64) {
            hipLaunchKernelGGL((k_stage<D, P, GUARD_BUFFER, OUT_RES64, false, T, EQ_EULER, false, false, AXIS>), grid_all, block, lds, s, a, rows);
            return hipGetLastError();
        }
    }
    return hipErrorInvalidValue;
}

#if DG_PART == 0
// defined here, instantiated in parts 1, 2 and 5
#if DG_D == 3
extern template hipError_t launch_stage_3v<DG_P>(const StageArgs &, int, int, hipStream_t, int);
#if DG_P == 0
extern template hipError_t launch_stage_cell<DG_D, DG_P, double, EQ_EULER, false, false>(const StageArgs &, int, int, bool,
                                                                                        const StageShape &, hipStream_t);
#endif
#endif
extern template hipError_t launch_stage_cell<DG_D, DG_P, double, EQ_EULER>(const StageArgs &, int, int, bool,
                                                                          const StageShape &, hipStream_t);
extern template hipError_t launch_stage_cell<DG_D, DG_P, float, EQ_EULER>(const StageArgs &, int, int, bool,
                                                                         const StageShape &, hipStream_t);
#if DG_P >= 2 && !(DG_D == 3 && DG_P == 3)
extern template hipError_t launch_stage_cell<DG_D, DG_P, float, EQ_EULER, true>(const StageArgs &, int, int, bool,
                                                                               const StageShape &, hipStream_t);
#endif

template <int D, int P>
hipError_t launch_stage(const StageArgs &a, int gm, int om, bool lim, bool fp32, const StageShape &sh, hipStream_t s,
                        int eq)
{
    if (a.nleaves == 0) return hipSuccess;
    if (eq == EQ_ADVECTION) {
        if (fp32) return hipErrorInvalidValue;
        // four-cell blocks of one variable: the dense gather of the far traces
        // costs more than the contraction saves (degree 1, 8 000 / 500 000 cells:
        // point by point 23.6 / 350 us a step, axis by axis 27.9 / 381; degree 2:
        // 33.8 / 633 against 36.3 / 588, 60 000: 88 against 92)
        if constexpr (D == 2 && (P == 1 || P == 2))
            if (a.N == 2 && (P == 1 || a.nleaves <= 32768))
                return launch_stage_cell<D, P, double, EQ_ADVECTION, false, false>(a, gm, om, lim, sh, s);
        return launch_stage_cell<D, P, double, EQ_ADVECTION>(a, gm, om, lim, sh, s);
    }
    if (fp32) {
        if constexpr (mfma_volume<D, P>()) {
            // the volume integral on the matrix cores where the slab is whole
            // waves; otherwise (small blocks) on the vector unit
            if (sh.mfma) {
                const hipError_t e = launch_stage_cell<D, P, float, EQ_EULER, true>(a, gm, om, lim, sh, s);
                if (e != hipErrorNotSupported) return e;
            }
        }
        return launch_stage_cell<D, P, float>(a, gm, om, lim, sh, s);
    }
    if constexpr (D == 2) {
        // one lane per (cell, variable) where asked for (variant 0: small
        // forests), without the limiter.  The residual of large forests runs
        // one thread per cell too (52 x 47 roots of 12^2 cells, 12 refined
        // leaf rows, degree 3: 536 -> 202 us)
        if (!lim && sh.variant == 0) return launch_stage_2v<P>(a, gm, om, s, sh.rows);
        // (slab heights of the residual stay those of the lane kernel)
        if (om != OUT_RK && sh.rows > 0 && (a.N % sh.rows != 0 || sh.rows * a.N * 4 > 512)) return hipErrorInvalidValue;
    } else {
        if (lanes_3d(sh, lim, false, a.conservative != 0, false, a.N)) return launch_stage_3v<P>(a, gm, om, s, sh.rows);
        // degree 0 with mortar faces, whose traces the gather leaves out: point
        // by point (40 000 cells in 2^3 / 8^3 blocks, one root in ten refined,
        // 109 / 37 us a step against 115 / 42)
        if constexpr (P == 0)
            if (a.conservative) return launch_stage_cell<D, P, double, EQ_EULER, false, false>(a, gm, om, lim, sh, s);
    }
    return launch_stage_cell<D, P, double>(a, gm, om, lim, sh, s);
}

template <int D, int P>
hipError_t launch_fill(const FillArgs &a, int nfc, hipStream_t s, int nv)
{
    const long threads = long(a.nfaces) * nfc;
    const dim3 grid(unsigned((threads + 255) / 256)), block(256);
    if (nv == 1) hipLaunchKernelGGL((k_fill<D, P, 1>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_fill<D, P>), grid, block, 0, s, a);
    return hipGetLastError();
}

template <int D, int P>
hipError_t launch_limit(double *u, int N, long total, double gamma, hipStream_t s)
{
    hipLaunchKernelGGL((k_limit<D, P>), dim3(unsigned((total + 255) / 256)), dim3(256), 0, s, u, N, total, gamma);
    return hipGetLastError();
}

template <int D, int P>
hipError_t launch_project_ic(double *u, const LeafGeo *geo, int N, long total, int kind, const IcParams &prm,
                             double t, double gamma, const double *hmin, hipStream_t s, int nv)
{
    const dim3 grid(unsigned((total + 255) / 256)), block(256);
    if (nv == 1)
        hipLaunchKernelGGL((k_project_ic<D, P, 1>), grid, block, 0, s, u, geo, N, total, kind, prm, t, gamma, hmin[0],
                           hmin[1], hmin[2]);
    else
        hipLaunchKernelGGL((k_project_ic<D, P>), grid, block, 0, s, u, geo, N, total, kind, prm, t, gamma, hmin[0],
                           hmin[1], hmin[2]);
    return hipGetLastError();
}

template <int D, int P>
hipError_t launch_inherit(const double *uold, double *unew, const Inherit *inh, int N, long total, hipStream_t s,
                          int nv)
{
    const dim3 grid(unsigned((total + 255) / 256)), block(256);
    if (nv == 1) hipLaunchKernelGGL((k_inherit<D, P, 1>), grid, block, 0, s, uold, unew, inh, N, total);
    else hipLaunchKernelGGL((k_inherit<D, P>), grid, block, 0, s, uold, unew, inh, N, total);
    return hipGetLastError();
}

template hipError_t launch_stage<DG_D, DG_P>(const StageArgs &, int, int, bool, bool, const StageShape &, hipStream_t,
                                             int);
template int stage_rows_options<DG_D, DG_P>(int, int *, int, bool);
template hipError_t launch_fill<DG_D, DG_P>(const FillArgs &, int, hipStream_t, int);
template hipError_t launch_limit<DG_D, DG_P>(double *, int, long, double, hipStream_t);
template hipError_t launch_project_ic<DG_D, DG_P>(double *, const LeafGeo *, int, long, int, const IcParams &, double,
                                                   double, const double *, hipStream_t, int);
template hipError_t launch_inherit<DG_D, DG_P>(const double *, double *, const Inherit *, int, long, hipStream_t, int);
#elif DG_PART == 3
template <int D, int P>
hipError_t launch_ipdg(const IpdgArgs &a, int om, hipStream_t s)
{
    if (a.ncell_total == 0) return hipSuccess;
    const dim3 grid(unsigned((a.ncell_total + 255) / 256)), block(256);
    if (om == OUT_RES64) hipLaunchKernelGGL((k_ipdg<D, P, OUT_RES64>), grid, block, 0, s, a);
    else if (om == OUT_RK) hipLaunchKernelGGL((k_ipdg<D, P, OUT_RK>), grid, block, 0, s, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}
template hipError_t launch_ipdg<DG_D, DG_P>(const IpdgArgs &, int, hipStream_t);
#if DG_D == 2 || DG_P <= 2
template <int D, int P>
hipError_t launch_mapped(const MappedArgs &a, int eq, int om, bool lim, hipStream_t s)
{
    if (a.ncell_total == 0) return hipSuccess;
    const dim3 grid(unsigned((a.ncell_total + 127) / 128)), block(128);
    if (lim) {
        if (eq != EQ_EULER || om != OUT_RK) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_mapped<D, P, EQ_EULER, OUT_RK, true>), grid, block, 0, s, a);
    } else if (eq == EQ_ADVECTION) {
        if (om == OUT_RES64) hipLaunchKernelGGL((k_mapped<D, P, EQ_ADVECTION, OUT_RES64>), grid, block, 0, s, a);
        else if (om == OUT_RK) hipLaunchKernelGGL((k_mapped<D, P, EQ_ADVECTION, OUT_RK>), grid, block, 0, s, a);
        else return hipErrorInvalidValue;
    } else {
        if (om == OUT_RES64) hipLaunchKernelGGL((k_mapped<D, P, EQ_EULER, OUT_RES64>), grid, block, 0, s, a);
        else if (om == OUT_RK) hipLaunchKernelGGL((k_mapped<D, P, EQ_EULER, OUT_RK>), grid, block, 0, s, a);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <int D, int P>
hipError_t launch_mapped_limit(double *u, const LeafGeo *geo, int N, long total, double gamma, hipStream_t s)
{
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL((k_mapped_limit<D, P>), dim3(unsigned((total + 127) / 128)), dim3(128), 0, s, u, geo, N, total,
                       gamma);
    return hipGetLastError();
}
template <int D, int P>
hipError_t launch_mapped_rate(const MappedArgs &a, int eq, int nleaves, int block, double *leaf_max, hipStream_t s)
{
    if (eq == EQ_ADVECTION)
        hipLaunchKernelGGL((k_mapped_rate<D, P, EQ_ADVECTION>), dim3(nleaves), dim3(block), 0, s, a, leaf_max);
    else
        hipLaunchKernelGGL((k_mapped_rate<D, P, EQ_EULER>), dim3(nleaves), dim3(block), 0, s, a, leaf_max);
    return hipGetLastError();
}
template <int D, int P>
hipError_t launch_mapped_totals(const MappedArgs &a, int eq, int nleaves, int block, double *part, hipStream_t s)
{
    if (eq == EQ_ADVECTION)
        hipLaunchKernelGGL((k_mapped_totals_leaf<D, P, EQ_ADVECTION>), dim3(nleaves), dim3(block), 0, s, a, part);
    else
        hipLaunchKernelGGL((k_mapped_totals_leaf<D, P, EQ_EULER>), dim3(nleaves), dim3(block), 0, s, a, part);
    return hipGetLastError();
}
template <int D, int P>
hipError_t launch_mapped_ic(double *u, const LeafGeo *geo, int N, long total, int kind, const IcParams &prm,
                            double t, double gamma, int nv, hipStream_t s)
{
    const dim3 grid(unsigned((total + 127) / 128)), block(128);
    if (nv == 1)
        hipLaunchKernelGGL((k_mapped_project_ic<D, P, 1>), grid, block, 0, s, u, geo, N, total, kind, prm, t, gamma);
    else
        hipLaunchKernelGGL((k_mapped_project_ic<D, P, D + 2>), grid, block, 0, s, u, geo, N, total, kind, prm, t,
                           gamma);
    return hipGetLastError();
}
template hipError_t launch_mapped<DG_D, DG_P>(const MappedArgs &, int, int, bool, hipStream_t);
template hipError_t launch_mapped_limit<DG_D, DG_P>(double *, const LeafGeo *, int, long, double, hipStream_t);
template hipError_t launch_mapped_rate<DG_D, DG_P>(const MappedArgs &, int, int, int, double *, hipStream_t);
template hipError_t launch_mapped_totals<DG_D, DG_P>(const MappedArgs &, int, int, int, double *, hipStream_t);
template hipError_t launch_mapped_ic<DG_D, DG_P>(double *, const LeafGeo *, int, long, int, const IcParams &, double,
                                                 double, int, hipStream_t);
#endif
#elif DG_PART == 5
#if DG_D == 3
template hipError_t launch_stage_3v<DG_P>(const StageArgs &, int, int, hipStream_t, int);
#endif
#elif DG_PART == 1
template hipError_t launch_stage_cell<DG_D, DG_P, double, EQ_EULER>(const StageArgs &, int, int, bool,
                                                                   const StageShape &, hipStream_t);
#if DG_D == 3 && DG_P == 0
template hipError_t launch_stage_cell<DG_D, DG_P, double, EQ_EULER, false, false>(const StageArgs &, int, int, bool,
                                                                                 const StageShape &, hipStream_t);
#endif
#elif DG_PART == 2
template hipError_t launch_stage_cell<DG_D, DG_P, float, EQ_EULER>(const StageArgs &, int, int, bool,
                                                                  const StageShape &, hipStream_t);
#else
#if DG_P >= 2 && !(DG_D == 3 && DG_P == 3)
template hipError_t launch_stage_cell<DG_D, DG_P, float, EQ_EULER, true>(const StageArgs &, int, int, bool,
                                                                        const StageShape &, hipStream_t);
#endif
#endif

} // namespace dgk
