// Several adjoint levels per launch with the levels in between in LDS, the transpose of
// patch_kernel on the same patches (lbm_adjoint_advance).  Every node's arithmetic is adj_node
// and adj_link, as in the single adjoint step, and the gradients are updated in its order, so
// the result is bit for bit that of as many single steps.
//
// What bounds it is what bounds patch_kernel: the latency of a node's chain per level and of
// the launch on small grids, the vector instructions with the halo's repeated work on larger
// ones.  On grids with walls it replaces six launches per pair of levels (two bulk kernels, the
// wall pass, two traction stages and the scatter).
#include "lbm_adjoint.hpp"
#include "lbm_device.hpp"
#include "lbm_internal.hpp"
#include "lbm_kernel_util.hpp"
#include "lbm_patch.hpp"

namespace lbm {

// The terms of one traction link (adj_link) at level t of the launch: normal along axis AX (lo:
// the edge at coordinate 0), position s of the edge, l: lambda_d of the wall node.
template <typename R, int LAW, int AX>
__device__ __forceinline__ void patch_adj_link(const PatchAdjArgs& a, int t, bool lo, int s, const R ft[4],
                                               const R l[4], R mu, R lam, R out[4]) {
    const Common& cm = a.cm;
    constexpr int E0 = AX == 0 ? LBM_XMIN : LBM_YMIN, E1 = E0 + 1;
    const int L = AX == 0 ? cm.ny : cm.nx;
    const double* fl = lo ? a.field[t - 1][E0] : a.field[t - 1][E1];
    R w[2], Fbar[4];
#pragma unroll
    for (int c = 0; c < 2; ++c)
        w[c] = fl ? R(fl[c * L + s]) : lo ? R(a.value[t - 1][E0][c]) : R(a.value[t - 1][E1][c]);
#pragma unroll
    for (int k = 0; k < 4; ++k) Fbar[k] = R(0.5) * l[k];
    adj_link<R, LAW, AX>(cm, lo ? R(-1) : R(1), ft, w, Fbar, mu, lam, a.g_mu || a.g_lam, out);
}

// Exchange through LDS as in patch_kernel, mirrored: the adjoint pulls lambda_q from X + c_q.
// After an odd level a node writes lambda_q to its own slot opp(q), after an even level to the
// slot q of the neighbour X - c_q that pulls it; the next level reads slot opp(q) of the
// neighbour X + c_q (t even) or the own slot q (t odd).  At a wall the slot of the outgoing
// direction takes D lambda_d of the node itself, which lies where the other parity would read.
template <int ST, int LAW, bool WALLS, bool FIELDS>
__global__ void __launch_bounds__(kPatchAdjThreads) patch_adj_kernel(PatchAdjArgs a) {
    using R = typename Storage<ST>::real;
    constexpr bool F64 = ST == LBM_F64_PLAIN;
    constexpr int NS = 25;
    extern __shared__ __attribute__((aligned(16))) char patch_smem[];
    R* sh = (R*)patch_smem;
    const Common& cm = a.cm;
    const int nx = cm.nx, ny = cm.ny, ntile = cm.ntile, levels = a.levels, halo = levels - 1;
    const int64_t n = int64_t(nx) * ny;
    int pw, ph, px0, py0, px1, py1;
    patch_at(a.map, pw, ph, px0, py0, px1, py1);
    const PatchPos pos = patch_pos(threadIdx.x, pw, ph);
    const int X = px0 + pos.x, Y = py0 + pos.y;
    const int rw = pw + 2 * halo, rh = ph + 2 * halo;
    const bool valid = pos.ring < levels && (!WALLS || ((cm.periodic_x || (X >= 0 && X < nx)) &&
                                                        (cm.periodic_y || (Y >= 0 && Y < ny))));
    const bool core = valid && pos.ring == 0 && X < px1 && Y < py1;
    const int xr = wrap_index(X, nx), yr = wrap_index(Y, ny);
    R* own = sh + ((pos.y + halo) * rw + (pos.x + halo)) * NS;
    R* const xm = own - NS;
    R* const xp = own + NS;
    R* const ym = own - rw * NS;
    R* const yp = own + rw * NS;
    R* const lnk = sh + rw * rh * NS;             // the traction terms of the links, 4 each

    const R* __restrict__ src = (const R*)a.src;
    const bool gpar = a.g_mu || a.g_lam, gbody = a.g_body != nullptr;
    R mu = kval<R>(cm.mu0, cm.f_mu0), lam = kval<R>(cm.lam0, cm.f_lam0);
    bool xlo = false, xhi = false, ylo = false, yhi = false, probe = false;
    if (valid) {
        const int idx = yr * nx + xr;
        params_at<FIELDS, R>(cm, idx, mu, lam);
        double ps[2];
        probe = probe_at<R>(a, xr, yr, ps);
        if (WALLS) {
            xlo = !cm.periodic_x && xr == 0;
            xhi = !cm.periodic_x && xr == nx - 1;
            ylo = !cm.periodic_y && yr == 0;
            yhi = !cm.periodic_y && yr == ny - 1;
        }
    }
    // the traction edges of a wall node, x edge first
    const bool tx = WALLS && ((xlo && cm.bc[LBM_XMIN] == LBM_TRACTION) || (xhi && cm.bc[LBM_XMAX] == LBM_TRACTION));
    const bool ty = WALLS && ((ylo && cm.bc[LBM_YMIN] == LBM_TRACTION) || (yhi && cm.bc[LBM_YMAX] == LBM_TRACTION));
    // FP32 block sums of the gradients (FP64 storage: the gradients themselves) of a patch node;
    // a traction wall node also holds its FP64 mu and lam gradients, which its links' terms
    // enter at every level
    R gs[4] = {R(0), R(0), R(0), R(0)};
    double wg[2] = {0.0, 0.0};
    if (core) {
        const int64_t id = int64_t(yr) * nx + xr;
        if constexpr (F64) {
            if (a.g_mu) gs[0] = a.g_mu[id];
            if (a.g_lam) gs[1] = a.g_lam[id];
            if (a.g_body) {
                gs[2] = a.g_body[id];
                gs[3] = a.g_body[n + id];
            }
        } else {
            if (gpar || gbody) {
                const float* g = (const float*)a.gsum + tile_base(ntile, 4, xr, yr);
#pragma unroll
                for (int j = 0; j < 4; ++j) gs[j] = g[j * kTile];
            }
            if (tx || ty) {
                if (a.g_mu) wg[0] = a.g_mu[id];
                if (a.g_lam) wg[1] = a.g_lam[id];
            }
        }
    }
    R ft[4] = {R(0), R(0), R(0), R(0)};
    auto load_record = [&](int t, int x, int y) {
        const R* rec = (const R*)a.rec[t - 1] + tile_base(ntile, 6, x, y);
#pragma unroll
        for (int k = 0; k < 4; ++k) ft[k] = rec[(2 + k) * kTile];
    };
    if (valid) load_record(1, xr, yr);

    const bool rim = WALLS && ((!cm.periodic_x && (px0 - halo <= 0 || px0 + pw + halo >= nx)) ||
                               (!cm.periodic_y && (py0 - halo <= 0 || py0 + ph + halo >= ny)));
    // The terms of every traction link of the region at level t, one lane per link, the links
    // of x-edges and of y-edges on wavefronts of their own.
    auto solve_links = [&](int t, int px0, int py0) {
        asm volatile("" : "+s"(px0), "+s"(py0));     // formed here, not kept through the loop
        const bool nbr = (t & 1) == 0;
        const bool elo = !cm.periodic_x && px0 - halo <= 0 && cm.bc[LBM_XMIN] == LBM_TRACTION;
        const bool ehi = !cm.periodic_x && px0 + pw + halo >= nx && cm.bc[LBM_XMAX] == LBM_TRACTION;
        const bool flo = !cm.periodic_y && py0 - halo <= 0 && cm.bc[LBM_YMIN] == LBM_TRACTION;
        const bool fhi = !cm.periodic_y && py0 + ph + halo >= ny && cm.bc[LBM_YMAX] == LBM_TRACTION;
        const int xlinks = (int(elo) + int(ehi)) * rh, xpad = (xlinks + kTile - 1) & ~(kTile - 1);
        const int links = xpad + (int(flo) + int(fhi)) * rw;
        for (int j = threadIdx.x; j < links; j += blockDim.x) {
            const bool ax = j >= xpad;
            int i = ax ? j - xpad : j;
            if (!ax && i >= xlinks) continue;
            const bool lo = ax ? (flo && i < rw) : (elo && i < rh);
            if (i >= (ax ? rw : rh)) i -= ax ? rw : rh;
            const int LX = ax ? px0 - halo + i : (lo ? 0 : nx - 1), LY = ax ? (lo ? 0 : ny - 1) : py0 - halo + i;
            const int cx = LX - px0, cy = LY - py0;
            const int ring = max(max(max(-cx, cx - pw + 1), max(-cy, cy - ph + 1)), 0);
            const bool inside = (cm.periodic_x || (LX >= 0 && LX < nx)) && (cm.periodic_y || (LY >= 0 && LY < ny));
            if (!inside || ring > levels - t) continue;
            const int wx = wrap_index(LX, nx), wy = wrap_index(LY, ny);
            const R* rec = (const R*)a.rec[t - 1] + tile_base(ntile, 6, wx, wy);
            R fr[4], l[4], pm, pl, out[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) fr[k] = rec[(2 + k) * kTile];
            params_at<FIELDS, R>(cm, wy * nx + wx, pm, pl);
            // lambda_d of the node, d = 0, 2, 1, 3 at XMIN, XMAX, YMIN, YMAX
            if (t == 1) {
                const R* s = src + tile_base(ntile, 24, wx, wy) + (ax ? (lo ? 6 : 18) : (lo ? 0 : 12)) * kTile;
#pragma unroll
                for (int k = 0; k < 4; ++k) l[k] = s[(2 + k) * kTile];
            } else {
                const R* o = sh + ((cy + halo) * rw + (cx + halo)) * NS;
                const R* s = ax ? (lo ? (nbr ? o + 18 : o - rw * NS + 6) : (nbr ? o + 6 : o + rw * NS + 18))
                                : (lo ? (nbr ? o + 12 : o - NS) : (nbr ? o : o + NS + 12));
#pragma unroll
                for (int k = 0; k < 4; ++k) l[k] = s[2 + k];
            }
            R* to;
            if (ax) {
                patch_adj_link<R, LAW, 1>(a, t, lo, wx, fr, l, pm, pl, out);
                to = lnk + 4 * (2 * rh + (lo ? 0 : rw) + cx + halo);
            } else {
                patch_adj_link<R, LAW, 0>(a, t, lo, wy, fr, l, pm, pl, out);
                to = lnk + 4 * ((lo ? 0 : rh) + cy + halo);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) to[k] = out[k];
        }
    };

    const double hdt64 = 0.5 * cm.dt;
    for (int t = 1; t <= levels; ++t) {
        const bool act = valid && pos.ring <= levels - t;
        // opaque per level: addresses in memory are formed where they are used
        int x = xr, y = yr;
        asm volatile("" : "+v"(x), "+v"(y));
        if (rim) {
            if (t > 1) __syncthreads();
            solve_links(t, px0, py0);
            __syncthreads();
        } else if (t > 1) {
            __syncthreads();
        }
        R l[4][6], out[4][6];
        if (act) {
            if (t == 1) {
                int x0 = wrap_dec(x, nx), x1 = wrap_inc(x, nx), y0 = wrap_dec(y, ny), y1 = wrap_inc(y, ny);
                if (WALLS) {                       // a source beyond a wall: the own lambda_d
                    if (xlo) x0 = x;
                    if (xhi) x1 = x;
                    if (ylo) y0 = y;
                    if (yhi) y1 = y;
                }
                const R* s0 = src + tile_base(ntile, 24, x1, y) + (WALLS && xhi ? 12 : 0) * kTile;
                const R* s1 = src + tile_base(ntile, 24, x, y1) + (WALLS && yhi ? 18 : 6) * kTile;
                const R* s2 = src + tile_base(ntile, 24, x0, y) + (WALLS && xlo ? 0 : 12) * kTile;
                const R* s3 = src + tile_base(ntile, 24, x, y0) + (WALLS && ylo ? 6 : 18) * kTile;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    l[0][k] = s0[k * kTile];
                    l[1][k] = s1[k * kTile];
                    l[2][k] = s2[k * kTile];
                    l[3][k] = s3[k * kTile];
                }
            } else {
                const bool nbr = (t & 1) == 0;
                const R* r0 = nbr ? (WALLS && xhi ? own : xp + 12) : (WALLS && xhi ? xp + 12 : own);
                const R* r1 = nbr ? (WALLS && yhi ? own + 6 : yp + 18) : (WALLS && yhi ? yp + 18 : own + 6);
                const R* r2 = nbr ? (WALLS && xlo ? own + 12 : xm) : (WALLS && xlo ? xm : own + 12);
                const R* r3 = nbr ? (WALLS && ylo ? own + 18 : ym + 6) : (WALLS && ylo ? ym + 6 : own + 18);
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    l[0][k] = r0[k];
                    l[1][k] = r1[k];
                    l[2][k] = r2[k];
                    l[3][k] = r3[k];
                }
            }
            if (WALLS && (xlo || xhi || ylo || yhi)) {
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    if (xhi) l[0][k] = D_sign<R>(cm.bc[LBM_XMAX], k) * l[0][k];
                    if (yhi) l[1][k] = D_sign<R>(cm.bc[LBM_YMAX], k) * l[1][k];
                    if (xlo) l[2][k] = D_sign<R>(cm.bc[LBM_XMIN], k) * l[2][k];
                    if (ylo) l[3][k] = D_sign<R>(cm.bc[LBM_YMIN], k) * l[3][k];
                }
            }
            R inc[4];
            const R fm[4] = {ft[0], ft[1], ft[2], ft[3]};
            if (t < levels && pos.ring < levels - t) load_record(t + 1, x, y);
            adj_node<R, LAW>(cm, l, fm, mu, lam, R(a.r[t - 1]), gpar, gbody, out, inc);
            double ps[2];
            if (probe) {
                probe_at<R>(a, x, y, ps);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    out[q][0] += R(ps[0]);
                    out[q][1] += R(ps[1]);
                }
            }
            const R* lx = lnk + 4 * ((xlo ? 0 : rh) + pos.y + halo);
            const R* ly = lnk + 4 * (2 * rh + (ylo ? 0 : rw) + pos.x + halo);
            if (tx) {
                const R t0 = lx[0], t1 = lx[1];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    out[q][3] += t0;
                    out[q][5] += t1;
                }
            }
            if (ty) {
                const R t0 = ly[0], t1 = ly[1];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    out[q][2] += t0;
                    out[q][4] += t1;
                }
            }
            if (t < levels) {
                const bool mine = (t & 1) != 0;
                R* w0 = mine ? own + 12 : xm;
                R* w1 = mine ? own + 18 : ym + 6;
                R* w2 = mine ? own : xp + 12;
                R* w3 = mine ? own + 6 : yp + 18;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    w0[k] = out[0][k];
                    w1[k] = out[1][k];
                    w2[k] = out[2][k];
                    w3[k] = out[3][k];
                }
            } else if (core) {
                R* d = (R*)a.dst + tile_base(ntile, 24, x, y);
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int k = 0; k < 6; ++k) d[(6 * q + k) * kTile] = out[q][k];
            }
            if (core) {
                // the gradients in the order of a single step: this level's increments (block
                // sum, fold), its probe body term, its links' mu and lam terms
                const int64_t id = int64_t(y) * nx + x;
                if constexpr (F64) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) gs[j] += double(inc[j]);
                    if (probe) {
                        gs[2] += a.r[t - 1] * hdt64 * ps[0];
                        gs[3] += a.r[t - 1] * hdt64 * ps[1];
                    }
                    if (tx) { gs[0] += double(lx[2]); gs[1] += double(lx[3]); }
                    if (ty) { gs[0] += double(ly[2]); gs[1] += double(ly[3]); }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) gs[j] = gs[j] + float(inc[j]);
                    if (t == a.fold) {
                        if (tx || ty) {
                            wg[0] += double(gs[0]);
                            wg[1] += double(gs[1]);
                        } else {
                            if (a.g_mu) a.g_mu[id] += double(gs[0]);
                            if (a.g_lam) a.g_lam[id] += double(gs[1]);
                        }
                        if (a.g_body) {
                            a.g_body[id] += double(gs[2]);
                            a.g_body[n + id] += double(gs[3]);
                        }
                        gs[0] = gs[1] = gs[2] = gs[3] = 0.0f;
                    }
                    if (probe && a.g_body) {
                        a.g_body[id] += a.r[t - 1] * hdt64 * ps[0];
                        a.g_body[n + id] += a.r[t - 1] * hdt64 * ps[1];
                    }
                    if (tx) { wg[0] += double(lx[2]); wg[1] += double(lx[3]); }
                    if (ty) { wg[0] += double(ly[2]); wg[1] += double(ly[3]); }
                }
            }
        }
    }
    if (core) {
        int x = xr, y = yr;
        asm volatile("" : "+v"(x), "+v"(y));
        const int64_t id = int64_t(y) * nx + x;
        if constexpr (F64) {
            if (a.g_mu) a.g_mu[id] = gs[0];
            if (a.g_lam) a.g_lam[id] = gs[1];
            if (a.g_body) {
                a.g_body[id] = gs[2];
                a.g_body[n + id] = gs[3];
            }
        } else {
            float* g = (float*)a.gsum + tile_base(ntile, 4, x, y);
            double* const g64[4] = {a.g_mu, a.g_lam, a.g_body, a.g_body};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (g64[j]) g[j * kTile] = gs[j];
            if (tx || ty) {
                if (a.g_mu) a.g_mu[id] = wg[0];
                if (a.g_lam) a.g_lam[id] = wg[1];
            }
        }
    }
}

// ---------------------------------------------------------------- dispatch

template <int ST, int LAW>
static hipError_t patch_adj_st_law(const PatchAdjArgs& a, hipStream_t s) {
    using R = typename Storage<ST>::real;
    const bool fields = a.cm.mu || a.cm.lam || a.cm.body;
    const bool walls = !(a.cm.periodic_x && a.cm.periodic_y);
    const int rw = a.map.pw + 2 * (a.levels - 1), rh = a.map.ph + 2 * (a.levels - 1);
    const size_t lds = (size_t(rw) * rh * 25 + (walls ? size_t(8) * (rw + rh) : 0)) * sizeof(R);
    const dim3 grid(unsigned(a.map.nwg)), block(unsigned((rw * rh + kTile - 1) / kTile * kTile));
    if (block.x > unsigned(kPatchAdjThreads) || lds > size_t(kPatchLds)) return hipErrorInvalidValue;
    if (walls) {
        if (fields) hipLaunchKernelGGL((patch_adj_kernel<ST, LAW, true, true>), grid, block, lds, s, a);
        else hipLaunchKernelGGL((patch_adj_kernel<ST, LAW, true, false>), grid, block, lds, s, a);
    } else {
        if (fields) hipLaunchKernelGGL((patch_adj_kernel<ST, LAW, false, true>), grid, block, lds, s, a);
        else hipLaunchKernelGGL((patch_adj_kernel<ST, LAW, false, false>), grid, block, lds, s, a);
    }
    return hipGetLastError();
}

template <int ST>
static hipError_t patch_adj_st(const PatchAdjArgs& a, hipStream_t s) {
    switch (a.cm.material) {
        case LBM_LOGNH: return patch_adj_st_law<ST, LBM_LOGNH>(a, s);
        case LBM_NH: return patch_adj_st_law<ST, LBM_NH>(a, s);
        case LBM_MR: return patch_adj_st_law<ST, LBM_MR>(a, s);
        case LBM_YEOH: return patch_adj_st_law<ST, LBM_YEOH>(a, s);
        case LBM_GENT: return patch_adj_st_law<ST, LBM_GENT>(a, s);
        default: return patch_adj_st_law<ST, LBM_SVK>(a, s);
    }
}

hipError_t launch_patch_adjoint(const PatchAdjArgs& a, hipStream_t s) {
    // the adjoint populations are in the compute type: one kernel serves both shifted storages
    if (a.cm.storage == LBM_F64_PLAIN) return patch_adj_st<LBM_F64_PLAIN>(a, s);
    return patch_adj_st<LBM_F32_SHIFTED>(a, s);
}

}  // namespace lbm
