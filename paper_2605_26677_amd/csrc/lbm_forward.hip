// Forward kernels of the D2Q4 x 6 vectorial LBM on gfx950: the fused collide-stream step
// (Sec. 3.7), the traction-wall F^b solve (Sec. 3.6), the second-order initialisation
// (Sec. 3.4) and the recoveries from stored post-collision populations (Sec. 3.5).  The
// per-node update is in lbm_collide.hpp, the two-level kernels in lbm_pair.hip.
//
// Layout: populations, u* and records in 64-node row tiles holding all their planes
// contiguously (tile_base in lbm_device.hpp).  One thread per node, one wavefront per
// tile, kTilesPerBlock tiles per workgroup; the tile order is remapped so that each of the
// eight XCDs sweeps a contiguous band of rows (its L2 then serves the one-element overlap
// of the x -/+ 1 pulls between adjacent tiles).  Each stored value is written once per
// pass, with non-temporal stores.
#include <algorithm>

#include "lbm_collide.hpp"
#include "lbm_device.hpp"
#include "lbm_internal.hpp"
#include "lbm_kernel_util.hpp"

namespace lbm {

// F^b of every link of the traction edges at step n -> n+1 (Sec. 3.6; boundary_F), from the
// wall nodes' stored populations of level n.
//
// One launch covers every traction edge (each edge reads level n only and writes its own
// slice of the staging buffer), one wavefront per workgroup and one lane per link: the
// solve is latency-bound, so the links are spread over as many compute units as there are
// wavefronts.  The edge's normal axis AX is a template parameter (fixed per edge, so per
// wavefront): with the axis known, F, the tangent and the per-node vectors index with
// constants and stay in registers.
template <int ST, int LAW, bool FIELDS, bool LINES, int AX>
__device__ __forceinline__ void traction_solve(const TractionArgs& a, int e) {
    using Tr = Storage<ST>;
    using R = typename Tr::real;
    using T = typename Tr::pop_t;
    constexpr bool SH = Tr::shifted;
    const Common& cm = a.cm;
    const EdgeGeom G = edge_geom(e);
    const int L = (AX == 0) ? cm.ny : cm.nx;
    const int s = (int(blockIdx.x) - a.eblk[e]) * kTracWin + int(threadIdx.x);
    if (s >= L) return;
    const int64_t n = int64_t(cm.nx) * cm.ny;
    const R hdt = R(0.5 * cm.dt);

    // U of level n at the wall node
    const XY n0 = edge_node(G, cm.nx, cm.ny, 0, s);
    double b0, b1;
    body_at<FIELDS>(cm, n0.y * cm.nx + n0.x, n, a.r_n, b0, b1);
    R Uw[6];
    if constexpr (LINES) {
        // level n+1 of the two-level step, from the wall line of the staging buffer
        const T* lv = (const T*)wall_lines(a.aux, cm.nx, cm.ny).lines + line_slot(cm.nx, cm.ny, e, 0, s) * 24;
        recover_vals<T, R>(lv, 1, hdt * R(b0), hdt * R(b1), Uw);
    } else {
        recover_node<T, R>((const T*)a.pop, cm.ntile, n0.x, n0.y, hdt * R(b0), hdt * R(b1), Uw);
    }
    const R Tv[2] = {edge_value<R>(a.ed, e, 0, s, L), edge_value<R>(a.ed, e, 1, s, L)};
    R mu, lam, Fb[4];
    params_at<FIELDS, R>(cm, n0.y * cm.nx + n0.x, mu, lam);
    if (!boundary_F<R, LAW, SH, AX>(cm, R(G.NA), Uw, Tv, mu, lam, Fb)) atomicOr(cm.fault, (uint32_t)LBM_FAULT_NEWTON);
    R* aux = (R*)a.aux + 4 * (int64_t)(edge_off(cm.nx, cm.ny, e) + s);
#pragma unroll
    for (int k = 0; k < 4; ++k) aux[k] = Fb[k];
}

template <int ST, int LAW, bool FIELDS, bool LINES>
__global__ void __launch_bounds__(kTracWin) traction_kernel(TractionArgs a) {
    int e = 0;
    while (e < 3 && int(blockIdx.x) >= a.eblk[e + 1]) ++e;
    if (e == LBM_XMIN || e == LBM_XMAX) traction_solve<ST, LAW, FIELDS, LINES, 0>(a, e);
    else traction_solve<ST, LAW, FIELDS, LINES, 1>(a, e);
}

// ---------------------------------------------------------------- the fused step
// (the wall links and the collision of a node: lbm_collide.hpp)

template <int ST, int LAW, bool WALLS, bool FIELDS>
__global__ void __launch_bounds__(kBlock) step_kernel(StepArgs a) {
    using Tr = Storage<ST>;
    using R = typename Tr::real;
    using T = typename Tr::pop_t;
    constexpr bool SH = Tr::shifted;
    const Common& cm = a.cm;
    const int nx = cm.nx, ny = cm.ny, ntile = cm.ntile;
    int x, y;
    if (!tile_thread(nx, ny, ntile, x, y)) return;
    const int64_t n = int64_t(nx) * ny;
    const T* __restrict__ src = (const T*)a.src;
    T* __restrict__ dst = (T*)a.dst;
    const int idx = y * nx + x;
    const int64_t own = tile_base(ntile, 24, x, y);

    // pull sources: q0 (1,0) from (x-1, y), q1 (0,1) from (x, y-1), q2 (-1,0) from (x+1, y),
    // q3 (0,-1) from (x, y+1) (eq:streaming); a source beyond a wall is a missing link.
    int xm = x - 1, xp = x + 1, ym = y - 1, yp = y + 1;
    bool miss0 = false, miss1 = false, miss2 = false, miss3 = false;
    if (xm < 0) { if (WALLS && !cm.periodic_x) { miss0 = true; xm = x; } else xm = nx - 1; }
    if (xp >= nx) { if (WALLS && !cm.periodic_x) { miss2 = true; xp = x; } else xp = 0; }
    if (ym < 0) { if (WALLS && !cm.periodic_y) { miss1 = true; ym = y; } else ym = ny - 1; }
    if (yp >= ny) { if (WALLS && !cm.periodic_y) { miss3 = true; yp = y; } else yp = 0; }
    const int64_t sb[4] = {tile_base(ntile, 24, xm, y), tile_base(ntile, 24, x, ym),
                           tile_base(ntile, 24, xp, y), tile_base(ntile, 24, x, yp)};

    // x-neighbour pulls come from the own tile (but for one lane), so issue them first
    R g[4][6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        g[0][k] = R(src[sb[0] + k * kTile]);
        g[2][k] = R(src[sb[2] + (12 + k) * kTile]);
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        g[1][k] = R(src[sb[1] + (6 + k) * kTile]);
        g[3][k] = R(src[sb[3] + (18 + k) * kTile]);
    }

    if constexpr (WALLS) {
        if (miss0) wall_link<T, R>(cm, a.ed, a.aux, LBM_XMIN, y, src + own, kTile, g[0]);
        if (miss2) wall_link<T, R>(cm, a.ed, a.aux, LBM_XMAX, y, src + own, kTile, g[2]);
        if (miss1) wall_link<T, R>(cm, a.ed, a.aux, LBM_YMIN, x, src + own, kTile, g[1]);
        if (miss3) wall_link<T, R>(cm, a.ed, a.aux, LBM_YMAX, x, src + own, kTile, g[3]);
    }

    double bd0, bd1;
    body_at<FIELDS>(cm, idx, n, a.r_np1, bd0, bd1);
    R mu, lam;
    params_at<FIELDS, R>(cm, idx, mu, lam);
    const R dt = kval<R>(cm.dt, cm.f_dt);
    R out[4][6], U[6], J;
    collide_node<R, LAW, SH>(cm, g, R(bd0), R(bd1), mu, lam, out, U, J);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int k = 0; k < 6; ++k) store_stream(dst + own + (6 * q + k) * kTile, to_storage<T>(out[q][k]));

    // displacement quadrature u*^{n+2} = u*^{n+1} + dt v^{n+1} (eq:trapezoid-u)
    if (!a.ustar) {
        // replay for the adjoint: the accumulator is not needed
    } else if constexpr (ST == LBM_F64_PLAIN) {
        double* us = (double*)a.ustar + tile_base(ntile, 2, x, y);
        store_stream(us, us[0] + dt * U[0]);
        store_stream(us + kTile, us[kTile] + dt * U[1]);
    } else {
        // u* = U + S: S += dt v; at a block boundary S moves into U (ustar_refs)
        const UstarRefs r = ustar_refs(a.ustar, ntile, ny, x, y);
#pragma unroll
        for (int cpt = 0; cpt < 2; ++cpt) {
            const float sn = r.S[cpt * kTile] + float(dt * U[cpt]);
            if (a.fold) {
                store_stream(r.U + cpt * kTile, r.U[cpt * kTile] + double(sn));
                store_stream(r.S + cpt * kTile, 0.0f);
            } else {
                store_stream(r.S + cpt * kTile, sn);
            }
        }
    }

    if (a.record) write_record<R, SH>(a.record, ntile, x, y, U);

    bool nonfinite = false;
#pragma unroll
    for (int k = 0; k < 6; ++k) nonfinite |= !finite_r(U[k]);
    const bool jbad = J <= R(0);
    if (nonfinite || jbad)
        atomicOr(cm.fault, (jbad ? (uint32_t)LBM_FAULT_J : 0u) | (nonfinite ? (uint32_t)LBM_FAULT_NONFINITE : 0u));
}

// ---------------------------------------------------------------- recoveries

template <int ST, bool FIELDS, int MODE>   // MODE 0 moments (double), 1 record (R), 2 displacement
__global__ void __launch_bounds__(kBlock) recover_kernel(RecoverArgs a) {
    using Tr = Storage<ST>;
    using R = typename Tr::real;
    using T = typename Tr::pop_t;
    constexpr bool SH = Tr::shifted;
    const Common& cm = a.cm;
    const int64_t n = int64_t(cm.nx) * cm.ny;
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    const int y = int(idx / cm.nx), x = int(idx - int64_t(y) * cm.nx);
    double b0, b1;
    body_at<FIELDS>(cm, (int)idx, n, a.r_n, b0, b1);
    const double hdt = 0.5 * cm.dt;
    R U[6];
    recover_node<T, R>((const T*)a.pop, cm.ntile, x, y, R(hdt * b0), R(hdt * b1), U);
    if constexpr (MODE == 0) {
        double* out = (double*)a.out;
        for (int k = 0; k < 6; ++k) {
            double v = double(U[k]);
            if (!SH && (k == 2 || k == 5)) v -= 1.0;
            out[k * n + idx] = v;
        }
    } else if constexpr (MODE == 1) {
        R* out = (R*)a.out + tile_base(cm.ntile, 6, x, y);
        for (int k = 0; k < 6; ++k) {
            R v = U[k];
            if (!SH && (k == 2 || k == 5)) v -= R(1);
            out[k * kTile] = v;
        }
    } else {
        double* out = (double*)a.out;
        for (int cpt = 0; cpt < 2; ++cpt) {
            double ustar;
            if constexpr (ST == LBM_F64_PLAIN) {
                ustar = ((const double*)a.ustar)[tile_base(cm.ntile, 2, x, y) + cpt * kTile];
            } else {
                const UstarRefs r = ustar_refs(const_cast<void*>(a.ustar), cm.ntile, cm.ny, x, y);
                ustar = r.U[cpt * kTile] + double(r.S[cpt * kTile]);
            }
            out[cpt * n + idx] = ustar - hdt * double(U[cpt]);
        }
    }
}

// ---------------------------------------------------------------- stresses

// P(F) and sigma = J^{-1} P F^T (Sec. 3.5) of the recovered state, in FP64 from the
// stored populations (shifted evaluation for every storage: F - I is formed first).
template <int ST, int LAW, bool FIELDS>
__global__ void __launch_bounds__(kBlock) stress_kernel(RecoverArgs a) {
    using Tr = Storage<ST>;
    using R = typename Tr::real;
    using T = typename Tr::pop_t;
    constexpr bool SH = Tr::shifted;
    const Common& cm = a.cm;
    const int64_t n = int64_t(cm.nx) * cm.ny;
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    const int y = int(idx / cm.nx), x = int(idx - int64_t(y) * cm.nx);
    double b0, b1;
    body_at<FIELDS>(cm, (int)idx, n, a.r_n, b0, b1);
    const double hdt = 0.5 * cm.dt;
    R U[6];
    recover_node<T, R>((const T*)a.pop, cm.ntile, x, y, R(hdt * b0), R(hdt * b1), U);
    double ft[4] = {double(U[2]), double(U[3]), double(U[4]), double(U[5])};
    if (!SH) { ft[0] -= 1.0; ft[3] -= 1.0; }
    double mu, lam;
    params_at<FIELDS, double>(cm, (int)idx, mu, lam);
    double P[4], J;
    piola<double, LAW, true>(ft, mu, lam, law_consts<double>(cm), P, J);
    double* Po = (double*)a.out;
    for (int k = 0; k < 4; ++k) Po[k * n + idx] = P[k];
    if (a.out2) {
        const double F[4] = {1.0 + ft[0], ft[1], ft[2], 1.0 + ft[3]};
        const double iJ = 1.0 / J;
        double* So = (double*)a.out2;
        So[idx] = iJ * (P[0] * F[0] + P[1] * F[1]);
        So[n + idx] = iJ * (P[0] * F[2] + P[1] * F[3]);
        So[2 * n + idx] = iJ * (P[2] * F[2] + P[3] * F[3]);
    }
}

// ---------------------------------------------------------------- diagnostics

// Sums (k < 7), minimum (k = 7) and maxima (k > 7) of the diagnostics.
__device__ __forceinline__ double diag_join(int k, double m, double o) {
    return k == 7 ? fmin(m, o) : k >= 8 ? fmax(m, o) : m + o;
}

// The tree reduction of a workgroup's values of every diagnostic, in column 0 at the end.
__device__ __forceinline__ void diag_reduce(double (*red)[kBlock]) {
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int k = 0; k < LBM_DIAG_COUNT; ++k)
                red[k][threadIdx.x] = diag_join(k, red[k][threadIdx.x], red[k][threadIdx.x + w]);
        __syncthreads();
    }
}

// Directions of the acoustic-tensor scan (one degree apart).
constexpr int kScanDirs = 180;

// The larger eigenvalue of Q_ik = n_A C_iAkB n_B (symmetrised) for the direction n.
template <typename R>
__device__ __forceinline__ R acoustic_max(const R C[16], R n0, R n1) {
    const R nn[2] = {n0, n1};
    R Q[4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            R v = R(0);
#pragma unroll
            for (int A = 0; A < 2; ++A)
#pragma unroll
                for (int B = 0; B < 2; ++B) v += nn[A] * C[8 * i + 4 * A + 2 * k + B] * nn[B];
            Q[2 * i + k] = v;
        }
    const R tr = R(0.5) * (Q[0] + Q[3]);
    const R dd = R(0.5) * (Q[0] - Q[3]);
    const R off = R(0.5) * (Q[1] + Q[2]);
    return tr + sqrt_r(dd * dd + off * off);
}

// Bounds of a node's scan, in FP32: lo <= the largest of its kScanDirs values <= hi.  With
// phi = 2 theta the entries of Q are first-order trigonometric polynomials, the larger eigenvalue
// is T(phi) + sqrt(S(phi)), T of first and S of second order.  The samples are kBoundDirs of the
// scan's own directions, so that the largest one is no larger than the scan (between them a
// compressed St. Venant-Kirchhoff node exceeded its own scan by up to 38 %, and a node with a
// larger scan was skipped).  They bound the eigenvalue from above too: between two samples T and S
// exceed their chords by at most |T''| h^2/8 and |S''| h^2/8 (h the step of phi), and the square
// root of a linear S its own chord by (dS)^2 / (32 Smin^(3/2)).  Both bounds keep 4e-5 of the
// largest |C_iAkB| apart from the samples: the FP32 scan's rotated directions drift by 5e-6 in
// |n|^2 and 6e-7 in angle, and |Q| <= |C| (Frobenius, at most 4 times that entry); with the
// rounding of either side that makes 8e-6 |C|.  All is formed for C divided by that entry: the
// fourth powers of the moduli would leave FP32's range (of moduli of 1e-12 the bound was 0.3 %
// below the scan).  hi is not finite where S may vanish or the state is not
// finite: no bound.
constexpr int kBoundDirs = 15;                       // every twelfth direction of the scan (18: 3 % slower)
static_assert(kScanDirs % kBoundDirs == 0, "the samples are directions of the scan");

template <typename R>
__device__ __forceinline__ void scan_bounds(const R C[16], float& lo, float& hi) {
    float top = 0.0f;
#pragma unroll
    for (int k = 0; k < 16; ++k) top = fmaxf(top, fabsf(float(C[k])));
    const float scale = __builtin_amdgcn_rcpf(top);
    float z[3][3];                                  // T, (Q00 - Q11)/2, (Q01 + Q10)/2
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        // coefficients of 1, cos phi, sin phi of Q_ik = (C_i0k0 + C_i1k1)/2 + ...
        auto coef = [&](int i, int k, int j) {
            const float a = float(C[8 * i + 2 * k]), b = float(C[8 * i + 4 + 2 * k + 1]);
            const float c = float(C[8 * i + 2 * k + 1]), d = float(C[8 * i + 4 + 2 * k]);
            return j == 0 ? 0.5f * (a + b) : j == 1 ? 0.5f * (a - b) : 0.5f * (c + d);
        };
#pragma unroll
        for (int j = 0; j < 3; ++j)
            z[m][j] = scale * (m == 0 ? 0.5f * (coef(0, 0, j) + coef(1, 1, j))
                             : m == 1 ? 0.5f * (coef(0, 0, j) - coef(1, 1, j)) : 0.5f * (coef(0, 1, j) + coef(1, 0, j)));
    }
    float p[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};     // S = p0 + p1 cos + p2 sin + p3 cos 2phi + p4 sin 2phi
#pragma unroll
    for (int m = 1; m < 3; ++m) {
        p[0] += z[m][0] * z[m][0] + 0.5f * (z[m][1] * z[m][1] + z[m][2] * z[m][2]);
        p[1] += 2.0f * z[m][0] * z[m][1];
        p[2] += 2.0f * z[m][0] * z[m][2];
        p[3] += 0.5f * (z[m][1] * z[m][1] - z[m][2] * z[m][2]);
        p[4] += z[m][1] * z[m][2];
    }
    constexpr float h = 6.2831853f / kBoundDirs;
    const float t12 = __builtin_amdgcn_sqrtf(z[0][1] * z[0][1] + z[0][2] * z[0][2]);
    const float p12 = __builtin_amdgcn_sqrtf(p[1] * p[1] + p[2] * p[2]);
    const float p34 = __builtin_amdgcn_sqrtf(p[3] * p[3] + p[4] * p[4]);
    const float smin = p[0] - p12 - p34;
    const float eS = (p12 + 4.0f * p34) * (h * h / 8.0f), dS = (p12 + 2.0f * p34) * h;
    constexpr float cs[kBoundDirs] = {1.0f, 0.91354546f, 0.66913061f, 0.30901699f, -0.10452846f, -0.50000000f,
                                      -0.80901699f, -0.97814760f, -0.97814760f, -0.80901699f, -0.50000000f,
                                      -0.10452846f, 0.30901699f, 0.66913061f, 0.91354546f};
    constexpr float sn[kBoundDirs] = {0.0f, 0.40673664f, 0.74314483f, 0.95105652f, 0.99452190f, 0.86602540f,
                                      0.58778525f, 0.20791169f, -0.20791169f, -0.58778525f, -0.86602540f,
                                      -0.99452190f, -0.95105652f, -0.74314483f, -0.40673664f};
    lo = hi = -1e30f;
#pragma unroll
    for (int k = 0; k < kBoundDirs; ++k) {
        const float T = z[0][0] + z[0][1] * cs[k] + z[0][2] * sn[k];
        const float B = z[1][0] + z[1][1] * cs[k] + z[1][2] * sn[k];
        const float D = z[2][0] + z[2][1] * cs[k] + z[2][2] * sn[k];
        const float S = B * B + D * D;
        lo = fmaxf(lo, T + __builtin_amdgcn_sqrtf(S));
        hi = fmaxf(hi, T + __builtin_amdgcn_sqrtf(S + eS));
    }
    lo = top * (lo - 4e-5f);
    // 1.01: the rounding of smin, at most 0.6 % where it is accepted
    hi += t12 * (h * h / 8.0f) + 1.01f * dS * dS * __builtin_amdgcn_rcpf(32.0f * smin * __builtin_amdgcn_sqrtf(smin)) + 4e-5f;
    hi *= top;
    const bool in_range = top > 1e-30f && top < 1e30f;
    if (!in_range || !(smin > 1e-4f * p[0])) hi = __builtin_inff();
    if (!in_range) lo = 0.0f;
}

// One partial row of LBM_DIAG_COUNT values per workgroup.  The direction scan of the acoustic
// tensor (180 directions, some 10 000 instructions per node) was the whole cost: 4.06 ms of
// 4096^2 in FP32.  Only nodes that can hold the workgroup's largest value take it now: those
// whose upper bound reaches the largest lower bound seen so far (scan_bounds), so that the result
// is that of the full scan, whatever the order in which that floor is raised.  A wavefront with
// few such nodes takes them one by one, its lanes sharing the directions.  Four wavefronts per
// SIMD in the shifted storages: at most 128 registers, which costs no spills.  The laws of the
// invariants took up to 138, and with them three: FP32 at 739 x 396 with per-node moduli, us per
// call, MR 37 -> 31, Yeoh 36 -> 32, Gent 37 -> 32; 1500 x 1100 78 -> 73, 76 -> 70, 78 -> 71.
template <int ST, int LAW, bool FIELDS>
__global__ void __launch_bounds__(kBlock, ST == LBM_F64_PLAIN ? 1 : 4) diag_kernel(RecoverArgs a) {
    using Tr = Storage<ST>;
    using R = typename Tr::real;
    using T = typename Tr::pop_t;
    constexpr bool SH = Tr::shifted;
    const Common& cm = a.cm;
    const int64_t n = int64_t(cm.nx) * cm.ny;
    __shared__ R dirs[2][kScanDirs];
    __shared__ int floor_bits;                      // the largest lower bound, as the bits of a float >= 0
    __shared__ double red[LBM_DIAG_COUNT][kBlock];
    if (threadIdx.x == 0) {
        floor_bits = 0;
        // 1-degree rotation for the direction scan of the acoustic tensor
        const R cd = R(0.99984769515639123916), sd = R(0.017452406437283512820);
        R cs = R(1), sn = R(0);
        for (int t = 0; t < kScanDirs; ++t) {
            dirs[0][t] = cs;
            dirs[1][t] = sn;
            const R c2 = cs * cd - sn * sd;
            sn = sn * cd + cs * sd;
            cs = c2;
        }
    }
    __syncthreads();
    double acc[LBM_DIAG_COUNT];
#pragma unroll
    for (int k = 0; k < LBM_DIAG_COUNT; ++k) acc[k] = 0.0;
    acc[7] = 1e300;
    const double hdt = 0.5 * cm.dt;
    const int lane = threadIdx.x & (kTile - 1);
    for (int64_t base = int64_t(blockIdx.x) * blockDim.x; base < n; base += int64_t(gridDim.x) * blockDim.x) {
        const int64_t idx = base + threadIdx.x;
        const bool valid = idx < n;
        R C[16];
        float lo = 0.0f, hi = -1.0f;
        if (valid) {
            const int y = int(idx) / cm.nx, x = int(idx) - y * cm.nx;
            double b0, b1;
            body_at<FIELDS>(cm, (int)idx, n, a.r_n, b0, b1);
            R U[6];
            recover_node<T, R>((const T*)a.pop, cm.ntile, x, y, R(hdt * b0), R(hdt * b1), U);
            R mu, lam;
            params_at<FIELDS, R>(cm, (int)idx, mu, lam);
            R ft[4] = {U[2], U[3], U[4], U[5]};
            if (!SH) { ft[0] -= R(1); ft[3] -= R(1); }
            acc[0] += double(U[0]);
            acc[1] += double(U[1]);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[2 + k] += double(ft[k]);
            const R W = energy<R, LAW, true>(ft, mu, lam, law_consts<R>(cm));
            acc[6] += double(R(0.5) * (U[0] * U[0] + U[1] * U[1]) + W);
            const R J = R(1) + ft[0] + ft[3] + (ft[0] * ft[3] - ft[1] * ft[2]);
            acc[7] = fmin(acc[7], double(J));
            acc[8] = fmax(acc[8], double(sqrt_r(ft[0] * ft[0] + ft[1] * ft[1] + ft[2] * ft[2] + ft[3] * ft[3])));
            tangent<R, LAW, true>(ft, mu, lam, law_consts<R>(cm), C);
            scan_bounds<R>(C, lo, hi);
            // one update per wavefront where a lane raises the floor
            if (isfinite(lo) && lo > 0.0f && __float_as_int(lo) > *(volatile int*)&floor_bits)
                atomicMax(&floor_bits, __float_as_int(lo));
        }
        if (base == int64_t(blockIdx.x) * blockDim.x) __syncthreads();
        const float thr = __int_as_float(*(volatile int*)&floor_bits);
        const bool odd = valid && !isfinite(hi);
        const uint64_t want = __ballot(valid && !(hi < thr));
        if (__ballot(odd) != 0 || __popcll(want) > 40) {
            if (valid && !(hi < thr)) {
                R best = R(0);
                for (int t = 0; t < kScanDirs; ++t) {
                    const R lmax = acoustic_max<R>(C, dirs[0][t], dirs[1][t]);
                    best = best > lmax ? best : lmax;
                }
                acc[9] = fmax(acc[9], double(sqrt_r(best)) / cm.c);
            }
        } else {
            for (uint64_t m = want; m != 0; m &= m - 1) {
                const int src = __ffsll((unsigned long long)m) - 1;
                R D[16];
                for (int k = 0; k < 16; ++k) D[k] = __shfl(C[k], src);
                R best = R(0);
                for (int t = lane; t < kScanDirs; t += kTile) {
                    const R lmax = acoustic_max<R>(D, dirs[0][t], dirs[1][t]);
                    best = best > lmax ? best : lmax;
                }
                // each lane keeps the largest of its own directions (the square root is monotone)
                acc[9] = fmax(acc[9], double(sqrt_r(best)) / cm.c);
            }
        }
    }
    acc[6] *= cm.dx * cm.dx;
    // block reduction in FP64
    double* part = (double*)a.scratch + int64_t(blockIdx.x) * LBM_DIAG_COUNT;
    for (int k = 0; k < LBM_DIAG_COUNT; ++k) red[k][threadIdx.x] = acc[k];
    diag_reduce(red);
    if (threadIdx.x < LBM_DIAG_COUNT) part[threadIdx.x] = red[threadIdx.x][0];
}

__global__ void __launch_bounds__(kBlock) diag_final_kernel(const double* part, int nblocks, double* out) {
    __shared__ double red[LBM_DIAG_COUNT][kBlock];
    for (int k = 0; k < LBM_DIAG_COUNT; ++k) {
        double m = (k == 7) ? 1e300 : 0.0;
        for (int b = threadIdx.x; b < nblocks; b += blockDim.x) m = diag_join(k, m, part[b * LBM_DIAG_COUNT + k]);
        red[k][threadIdx.x] = m;
    }
    diag_reduce(red);
    if (threadIdx.x < LBM_DIAG_COUNT) out[threadIdx.x] = red[threadIdx.x][0];
}

// ---------------------------------------------------------------- initialisation

// U0 = (v0, F - I) as 6 double planes, F - I = (Fbar - I) + grad u0 by second-order
// differences.
__global__ void __launch_bounds__(kBlock) init_state_kernel(InitArgs a) {
    const Common& cm = a.cm;
    const int nx = cm.nx, ny = cm.ny;
    const int64_t n = int64_t(nx) * ny;
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    const int y = int(idx / nx), x = int(idx - int64_t(y) * nx);
    double* U0 = (double*)a.scratch;
    U0[idx] = a.v0[idx];
    U0[n + idx] = a.v0[n + idx];
    const double inv2h = 1.0 / (2.0 * cm.dx);
    for (int cpt = 0; cpt < 2; ++cpt) {
        double gx = 0.0, gy = 0.0;
        if (a.u0) {
            const double* u = a.u0 + cpt * n;
            gx = fd_along<double>([&](int s) { return u[int64_t(y) * nx + s]; }, x, nx, cm.periodic_x, inv2h);
            gy = fd_along<double>([&](int s) { return u[int64_t(s) * nx + x]; }, y, ny, cm.periodic_y, inv2h);
        }
        U0[(2 + 2 * cpt) * n + idx] = (a.Fbar[2 * cpt] - (cpt == 0 ? 1.0 : 0.0)) + gx;
        U0[(3 + 2 * cpt) * n + idx] = (a.Fbar[2 * cpt + 1] - (cpt == 1 ? 1.0 : 0.0)) + gy;
    }
}

// Second-order populations (eq:init-compact with eq:init-Zq-components, eq:init-deltaPq,
// eq:init-expanded) in FP64 shifted form, then the first collision (level 0) and u*^1.
//
// REST (no initial displacement and F = I): U0 = (v0, 0), so the kernel reads v0 itself and
// needs no pass that forms U0.  The general form keeps 30 loads of U0 and its neighbours and
// the tangent in flight at two wavefronts per SIMD and was bound by their latency: 8192^2 FP32
// 6.6 ms and 0.75 ms for U0.
template <int ST, int LAW, bool FIELDS, bool REST>
__global__ void __launch_bounds__(kBlock) init_pop_kernel(InitArgs a) {
    using Tr = Storage<ST>;
    using T = typename Tr::pop_t;
    constexpr bool SH = Tr::shifted;
    const Common& cm = a.cm;
    const int nx = cm.nx, ny = cm.ny;
    const int64_t n = int64_t(nx) * ny;
    int x, y;
    if (!tile_thread(nx, ny, cm.ntile, x, y)) return;
    const int64_t idx = int64_t(y) * nx + x;
    const double* U0p = REST ? a.v0 : (const double*)a.scratch;
    const double c = cm.c, dt = cm.dt, hdt = 0.5 * cm.dt;
    const double inv2h = 1.0 / (2.0 * cm.dx);
    double U0[6], dX[6], dY[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        if (REST && k >= 2) {
            U0[k] = dX[k] = dY[k] = 0.0;
            continue;
        }
        const double* pl = U0p + k * n;
        U0[k] = pl[idx];
        if (!REST && a.dUdX) {
            dX[k] = a.dUdX[k * n + idx];
            dY[k] = a.dUdY[k * n + idx];
        } else {
            dX[k] = fd_along<double>([&](int s) { return pl[int64_t(y) * nx + s]; }, x, nx, cm.periodic_x, inv2h);
            dY[k] = fd_along<double>([&](int s) { return pl[int64_t(s) * nx + x]; }, y, ny, cm.periodic_y, inv2h);
        }
    }
    double mu, lam, b0, b1;
    params_at<FIELDS, double>(cm, (int)idx, mu, lam);
    body_at<FIELDS>(cm, (int)idx, n, a.r0, b0, b1);
    double C[16], P0[4], J;
    tangent<double, LAW, true>(&U0[2], mu, lam, law_consts<double>(cm), C);
    piola<double, LAW, true>(&U0[2], mu, lam, law_consts<double>(cm), P0, J);
    // d_alpha P = C : d_alpha F
    double dPX[4], dPY[4];
    for (int iA = 0; iA < 4; ++iA) {
        double sx = 0.0, sy = 0.0;
        for (int kB = 0; kB < 4; ++kB) {
            sx += C[4 * iA + kB] * dX[2 + kB];
            sy += C[4 * iA + kB] * dY[2 + kB];
        }
        dPX[iA] = sx;
        dPY[iA] = sy;
    }
    const double PhiX[6] = {-P0[0], -P0[2], -U0[0], 0.0, -U0[1], 0.0};
    const double PhiY[6] = {-P0[1], -P0[3], 0.0, -U0[0], 0.0, -U0[1]};
    double g0[4][6];
    for (int q = 0; q < 4; ++q) {
        const double i = dir_i(q), j = dir_j(q);
        double Z[6];
        Z[0] = b0 + dPX[0] + dPY[1] + c * (i * dX[0] + j * dY[0]);
        Z[1] = b1 + dPX[2] + dPY[3] + c * (i * dX[1] + j * dY[1]);
        Z[2] = dX[0] + c * (i * dX[2] + j * dY[2]);
        Z[3] = dY[0] + c * (i * dX[3] + j * dY[3]);
        Z[4] = dX[1] + c * (i * dX[4] + j * dY[4]);
        Z[5] = dY[1] + c * (i * dX[5] + j * dY[5]);
        double dP[4];
        for (int iA = 0; iA < 4; ++iA) {
            double sacc = 0.0;
            for (int kB = 0; kB < 4; ++kB) sacc += C[4 * iA + kB] * Z[2 + kB];
            dP[iA] = sacc;
        }
        const double D[6] = {
            0.25 * (Z[0] - (2.0 / c) * (i * dP[0] + j * dP[1])),
            0.25 * (Z[1] - (2.0 / c) * (i * dP[2] + j * dP[3])),
            0.25 * (Z[2] - (2.0 * i / c) * Z[0]),
            0.25 * (Z[3] - (2.0 * j / c) * Z[0]),
            0.25 * (Z[4] - (2.0 * i / c) * Z[1]),
            0.25 * (Z[5] - (2.0 * j / c) * Z[1]),
        };
        for (int k = 0; k < 6; ++k) {
            const double feq = 0.25 * (U0[k] + (2.0 / c) * (i * PhiX[k] + j * PhiY[k]));
            g0[q][k] = feq - hdt * D[k];
        }
    }
    // first collision at level 0 (eq:moment-U, eq:collision)
    double U[6];
    for (int k = 0; k < 6; ++k) U[k] = g0[0][k] + g0[1][k] + g0[2][k] + g0[3][k];
    U[0] += hdt * b0;
    U[1] += hdt * b1;
    double P[4];
    piola<double, LAW, true>(&U[2], mu, lam, law_consts<double>(cm), P, J);
    const double QX[6] = {-P[0], -P[2], -U[0], 0.0, -U[1], 0.0};
    const double QY[6] = {-P[1], -P[3], 0.0, -U[0], 0.0, -U[1]};
    const double srcw = dt * (2.0 - cm.omega) * 0.125;
    T* dst = (T*)a.dst + tile_base(cm.ntile, 24, x, y);
    for (int q = 0; q < 4; ++q) {
        const double i = dir_i(q), j = dir_j(q);
        for (int k = 0; k < 6; ++k) {
            const double feq = 0.25 * (U[k] + (2.0 / c) * (i * QX[k] + j * QY[k]));
            double v = g0[q][k] + cm.omega * (feq - g0[q][k]);
            if (k == 0) v += srcw * b0;
            if (k == 1) v += srcw * b1;
            if (!SH && (k == 2 || k == 5)) v += 0.25;
            dst[(6 * q + k) * kTile] = T(v);
        }
    }
    // u*^1 = u0 - (dt/2) v0 + dt v^0 (eq:trapezoid-u)
    for (int cpt = 0; cpt < 2; ++cpt) {
        const double u0 = a.u0 ? a.u0[cpt * n + idx] : 0.0;
        const double us1 = u0 - hdt * a.v0[cpt * n + idx] + dt * U[cpt];
        if constexpr (ST == LBM_F64_PLAIN) {
            ((double*)a.ustar)[tile_base(cm.ntile, 2, x, y) + cpt * kTile] = us1;
        } else {
            const UstarRefs r = ustar_refs(a.ustar, cm.ntile, cm.ny, x, y);
            r.U[cpt * kTile] = us1;
            r.S[cpt * kTile] = 0.0f;
        }
    }
    bool bad = !(J > 0.0);
    if (bad) atomicOr(cm.fault, (uint32_t)LBM_FAULT_J);
}

// ---------------------------------------------------------------- dispatch

static inline unsigned nblocks(int64_t n) { return unsigned((n + kBlock - 1) / kBlock); }

template <int ST, int LAW>
static hipError_t step_st_law(const StepArgs& a, hipStream_t s) {
    const bool walls = !(a.cm.periodic_x && a.cm.periodic_y);
    const bool fields = a.cm.mu || a.cm.lam || a.cm.body;
    const dim3 grid(unsigned((int64_t(a.cm.ntile) * a.cm.ny + kTilesPerBlock - 1) / kTilesPerBlock));
    const dim3 block(kTile * kTilesPerBlock);
    if (walls) {
        if (fields) hipLaunchKernelGGL((step_kernel<ST, LAW, true, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((step_kernel<ST, LAW, true, false>), grid, block, 0, s, a);
    } else {
        if (fields) hipLaunchKernelGGL((step_kernel<ST, LAW, false, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((step_kernel<ST, LAW, false, false>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

template <int ST>
static hipError_t step_st(const StepArgs& a, hipStream_t s) {
    switch (a.cm.material) {
        case LBM_LOGNH: return step_st_law<ST, LBM_LOGNH>(a, s);
        case LBM_NH: return step_st_law<ST, LBM_NH>(a, s);
        case LBM_MR: return step_st_law<ST, LBM_MR>(a, s);
        case LBM_YEOH: return step_st_law<ST, LBM_YEOH>(a, s);
        case LBM_GENT: return step_st_law<ST, LBM_GENT>(a, s);
        default: return step_st_law<ST, LBM_SVK>(a, s);
    }
}

// The two-level bulk launch.  On a grid with walls, the blocks whose level-(n+1) region
// keeps two nodes away from every wall line run the periodic instantiation (no wall code:
// compiled in, the wall branches cost every node about a sixth of its speed), and only the
// blocks along the walls run the wall instantiation.
hipError_t launch_step(const StepArgs& a, hipStream_t s) {
    switch (a.cm.storage) {
        case LBM_F32_SHIFTED: return step_st<LBM_F32_SHIFTED>(a, s);
        case LBM_F16_SHIFTED: return step_st<LBM_F16_SHIFTED>(a, s);
        default: return step_st<LBM_F64_PLAIN>(a, s);
    }
}

template <int ST, int LAW>
static hipError_t traction_st_law(const TractionArgs& a, hipStream_t s) {
    const bool fields = a.cm.mu || a.cm.lam || a.cm.body;
    const dim3 grid(unsigned(a.eblk[4])), block(kTracWin);
    if (a.lines) {
        if (fields) hipLaunchKernelGGL((traction_kernel<ST, LAW, true, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((traction_kernel<ST, LAW, false, true>), grid, block, 0, s, a);
    } else {
        if (fields) hipLaunchKernelGGL((traction_kernel<ST, LAW, true, false>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((traction_kernel<ST, LAW, false, false>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

template <int ST>
static hipError_t traction_st(const TractionArgs& a, hipStream_t s) {
    switch (a.cm.material) {
        case LBM_LOGNH: return traction_st_law<ST, LBM_LOGNH>(a, s);
        case LBM_NH: return traction_st_law<ST, LBM_NH>(a, s);
        case LBM_MR: return traction_st_law<ST, LBM_MR>(a, s);
        case LBM_YEOH: return traction_st_law<ST, LBM_YEOH>(a, s);
        case LBM_GENT: return traction_st_law<ST, LBM_GENT>(a, s);
        default: return traction_st_law<ST, LBM_SVK>(a, s);
    }
}

hipError_t launch_traction(TractionArgs a, hipStream_t s) {
    // workgroup ranges of the traction edges; nothing to launch without one
    a.eblk[0] = 0;
    for (int e = 0; e < 4; ++e) {
        const int L = (e == LBM_XMIN || e == LBM_XMAX) ? a.cm.ny : a.cm.nx;
        a.eblk[e + 1] = a.eblk[e] + (a.cm.bc[e] == LBM_TRACTION ? (L + kTracWin - 1) / kTracWin : 0);
    }
    if (a.eblk[4] == 0) return hipSuccess;
    switch (a.cm.storage) {
        case LBM_F32_SHIFTED: return traction_st<LBM_F32_SHIFTED>(a, s);
        case LBM_F16_SHIFTED: return traction_st<LBM_F16_SHIFTED>(a, s);
        default: return traction_st<LBM_F64_PLAIN>(a, s);
    }
}

template <int MODE>
static hipError_t recover_dispatch(const RecoverArgs& a, hipStream_t s) {
    const bool fields = a.cm.body != nullptr;
    const dim3 grid(nblocks(int64_t(a.cm.nx) * a.cm.ny));
#define LBM_RECOVER(ST_)                                                                         \
    if (fields) hipLaunchKernelGGL((recover_kernel<ST_, true, MODE>), grid, dim3(kBlock), 0, s, a); \
    else hipLaunchKernelGGL((recover_kernel<ST_, false, MODE>), grid, dim3(kBlock), 0, s, a);
    switch (a.cm.storage) {
        case LBM_F32_SHIFTED: { LBM_RECOVER(LBM_F32_SHIFTED) break; }
        case LBM_F16_SHIFTED: { LBM_RECOVER(LBM_F16_SHIFTED) break; }
        default: { LBM_RECOVER(LBM_F64_PLAIN) break; }
    }
#undef LBM_RECOVER
    return hipGetLastError();
}

hipError_t launch_moments(const RecoverArgs& a, hipStream_t s) { return recover_dispatch<0>(a, s); }
hipError_t launch_record(const RecoverArgs& a, hipStream_t s) { return recover_dispatch<1>(a, s); }
hipError_t launch_displacement(const RecoverArgs& a, hipStream_t s) { return recover_dispatch<2>(a, s); }

template <int ST, int LAW>
static void stress_st_law(const RecoverArgs& a, hipStream_t s) {
    const bool fields = a.cm.mu || a.cm.lam || a.cm.body;
    const dim3 grid(nblocks(int64_t(a.cm.nx) * a.cm.ny));
    if (fields) hipLaunchKernelGGL((stress_kernel<ST, LAW, true>), grid, dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((stress_kernel<ST, LAW, false>), grid, dim3(kBlock), 0, s, a);
}

template <int ST>
static void stress_st(const RecoverArgs& a, hipStream_t s) {
    switch (a.cm.material) {
        case LBM_LOGNH: stress_st_law<ST, LBM_LOGNH>(a, s); break;
        case LBM_NH: stress_st_law<ST, LBM_NH>(a, s); break;
        case LBM_MR: stress_st_law<ST, LBM_MR>(a, s); break;
        case LBM_YEOH: stress_st_law<ST, LBM_YEOH>(a, s); break;
        case LBM_GENT: stress_st_law<ST, LBM_GENT>(a, s); break;
        default: stress_st_law<ST, LBM_SVK>(a, s); break;
    }
}

hipError_t launch_stress(const RecoverArgs& a, hipStream_t s) {
    switch (a.cm.storage) {
        case LBM_F32_SHIFTED: stress_st<LBM_F32_SHIFTED>(a, s); break;
        case LBM_F16_SHIFTED: stress_st<LBM_F16_SHIFTED>(a, s); break;
        default: stress_st<LBM_F64_PLAIN>(a, s); break;
    }
    return hipGetLastError();
}

template <int ST, int LAW>
static void diag_st_law(const RecoverArgs& a, hipStream_t s) {
    const bool fields = a.cm.mu || a.cm.lam || a.cm.body;
    const int64_t n = int64_t(a.cm.nx) * a.cm.ny;
    const unsigned nb = unsigned(std::min<int64_t>(kDiagBlocks, (n + kBlock - 1) / kBlock));
    if (fields) hipLaunchKernelGGL((diag_kernel<ST, LAW, true>), dim3(nb), dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((diag_kernel<ST, LAW, false>), dim3(nb), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(diag_final_kernel, dim3(1), dim3(kBlock), 0, s, (const double*)a.scratch, (int)nb,
                       (double*)a.out);
}

template <int ST>
static void diag_st(const RecoverArgs& a, hipStream_t s) {
    switch (a.cm.material) {
        case LBM_LOGNH: diag_st_law<ST, LBM_LOGNH>(a, s); break;
        case LBM_NH: diag_st_law<ST, LBM_NH>(a, s); break;
        case LBM_MR: diag_st_law<ST, LBM_MR>(a, s); break;
        case LBM_YEOH: diag_st_law<ST, LBM_YEOH>(a, s); break;
        case LBM_GENT: diag_st_law<ST, LBM_GENT>(a, s); break;
        default: diag_st_law<ST, LBM_SVK>(a, s); break;
    }
}

hipError_t launch_diagnostics(const RecoverArgs& a, hipStream_t s) {
    switch (a.cm.storage) {
        case LBM_F32_SHIFTED: diag_st<LBM_F32_SHIFTED>(a, s); break;
        case LBM_F16_SHIFTED: diag_st<LBM_F16_SHIFTED>(a, s); break;
        default: diag_st<LBM_F64_PLAIN>(a, s); break;
    }
    return hipGetLastError();
}

template <int ST, int LAW>
static void init_st_law(const InitArgs& a, hipStream_t s) {
    const bool fields = a.cm.mu || a.cm.lam || a.cm.body;
    const dim3 grid(unsigned((int64_t(a.cm.ntile) * a.cm.ny + kBlock / kTile - 1) / (kBlock / kTile)));
    if (a.rest) {
        if (fields) hipLaunchKernelGGL((init_pop_kernel<ST, LAW, true, true>), grid, dim3(kBlock), 0, s, a);
        else hipLaunchKernelGGL((init_pop_kernel<ST, LAW, false, true>), grid, dim3(kBlock), 0, s, a);
    } else {
        if (fields) hipLaunchKernelGGL((init_pop_kernel<ST, LAW, true, false>), grid, dim3(kBlock), 0, s, a);
        else hipLaunchKernelGGL((init_pop_kernel<ST, LAW, false, false>), grid, dim3(kBlock), 0, s, a);
    }
}

template <int ST>
static void init_st(const InitArgs& a, hipStream_t s) {
    switch (a.cm.material) {
        case LBM_LOGNH: init_st_law<ST, LBM_LOGNH>(a, s); break;
        case LBM_NH: init_st_law<ST, LBM_NH>(a, s); break;
        case LBM_MR: init_st_law<ST, LBM_MR>(a, s); break;
        case LBM_YEOH: init_st_law<ST, LBM_YEOH>(a, s); break;
        case LBM_GENT: init_st_law<ST, LBM_GENT>(a, s); break;
        default: init_st_law<ST, LBM_SVK>(a, s); break;
    }
}

hipError_t launch_init_state(const InitArgs& a, hipStream_t s) {
    const dim3 grid(nblocks(int64_t(a.cm.nx) * a.cm.ny));
    hipLaunchKernelGGL(init_state_kernel, grid, dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_init(const InitArgs& a, hipStream_t s) {
    InitArgs b = a;
    b.rest = !a.u0 && a.Fbar[0] == 1.0 && a.Fbar[1] == 0.0 && a.Fbar[2] == 0.0 && a.Fbar[3] == 1.0;
    if (!b.rest) {
        const dim3 grid(nblocks(int64_t(a.cm.nx) * a.cm.ny));
        hipLaunchKernelGGL(init_state_kernel, grid, dim3(kBlock), 0, s, b);
    }
    return launch_init_given(b, s);
}

// The populations from U0 already in a.scratch (and its derivatives, if given).
hipError_t launch_init_given(const InitArgs& a, hipStream_t s) {
    switch (a.cm.storage) {
        case LBM_F32_SHIFTED: init_st<LBM_F32_SHIFTED>(a, s); break;
        case LBM_F16_SHIFTED: init_st<LBM_F16_SHIFTED>(a, s); break;
        default: init_st<LBM_F64_PLAIN>(a, s); break;
    }
    return hipGetLastError();
}

}  // namespace lbm
