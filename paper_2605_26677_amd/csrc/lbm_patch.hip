// Several levels of the fused collide-stream per launch with the levels in between in LDS:
// a workgroup owns a rectangular patch of nodes, one node per thread, and takes the patch and
// the halo it needs from f*^n to f*^{n+T}, walls included.  Every node's arithmetic is
// collide_node, wall_rule and boundary_F, as in the single-step kernels, and each
// intermediate level is rounded to the storage type, so the result is bit for bit that of as
// many single steps.
//
// What bounds it: on grids up to about 300^2 the latency of one node's chain per level (some
// 250 dependent instructions, 1.1 us with the barrier; a traction solve adds 700, 3.3 us) and
// about 4 us per launch (dispatch, first loads, last stores), which the levels of a launch
// share; on larger ones the vector instructions, the halo's repeated work included (1.4 times
// the patch at 4 levels of 16 x 16).  The sizes of patch and launch follow from that trade-off
// (patch_plan).  Measured: 64^2 FP64 5.9 -> 1.8 us per level, 256^2 FP32 3.1 -> 2.2, 1024^2
// FP32 with traction walls 33 -> 21 (the single steps and pairs it replaces, with their traction
// and wall passes).
#include "lbm_collide.hpp"
#include "lbm_device.hpp"
#include "lbm_internal.hpp"
#include "lbm_kernel_util.hpp"
#include "lbm_patch.hpp"

namespace lbm {

// The boundary data of step t of the launch at position s of the edge whose normal lies along
// axis AX (lo: the edge at coordinate 0, else the one at the far end).
template <typename R, int AX>
__device__ __forceinline__ void patch_edge_data(const PatchArgs& a, int t, bool lo, int s, R w[2]) {
    constexpr int E0 = AX == 0 ? LBM_XMIN : LBM_YMIN, E1 = E0 + 1;
    const int L = AX == 0 ? a.cm.ny : a.cm.nx;
    const double* fl = lo ? a.field[t][E0] : a.field[t][E1];
#pragma unroll
    for (int c = 0; c < 2; ++c) w[c] = fl ? R(fl[c * L + s]) : lo ? R(a.value[t][E0][c]) : R(a.value[t][E1][c]);
}

// The missing link of a wall node from its own outgoing populations o and its F of the same
// level (U[2 .. 5]; traction edges).  Returns false when the traction solve failed.
template <typename R, int LAW, bool SH, int AX>
__device__ __forceinline__ bool patch_link(const PatchArgs& a, int t, bool lo, int s, const R o[6], const R U[6],
                                           R mu, R lam, R out[6]) {
    const Common& cm = a.cm;
    const R NA = lo ? R(-1) : R(1);
    const bool velocity = (AX == 0 ? (lo ? cm.bc[LBM_XMIN] : cm.bc[LBM_XMAX])
                                   : (lo ? cm.bc[LBM_YMIN] : cm.bc[LBM_YMAX])) == LBM_VELOCITY;
    R w[2], Fb[4] = {R(0), R(0), R(0), R(0)};
    patch_edge_data<R, AX>(a, t, lo, s, w);
    const bool ok = velocity || boundary_F<R, LAW, SH, AX>(cm, NA, U, w, mu, lam, Fb);
    wall_rule<R>(velocity, AX == 0 ? NA : R(0), AX == 1 ? NA : R(0), w[0], w[1], R(cm.c), o, Fb, out);
    return ok;
}

// The missing link of a velocity wall node, into the slot it is read from.  o: the node's
// outgoing populations, `stride` apart.
template <typename R, int AX, typename T>
__device__ __forceinline__ void patch_velocity_link(const PatchArgs& a, int t, bool lo, int s, const T* o, int stride,
                                                    R* slot) {
    const R NA = lo ? R(-1) : R(1), none[4] = {R(0), R(0), R(0), R(0)};
    R w[2], in[6], out[6];
    patch_edge_data<R, AX>(a, t, lo, s, w);
#pragma unroll
    for (int k = 0; k < 6; ++k) in[k] = R(o[k * stride]);
    wall_rule<R>(true, AX == 0 ? NA : R(0), AX == 1 ? NA : R(0), w[0], w[1], R(a.cm.c), in, none, out);
#pragma unroll
    for (int k = 0; k < 6; ++k) slot[k] = out[k];
}

// Exchange through LDS.  A node's 24 populations, rounded to the storage type, take 25
// words of the compute type (odd: lanes at consecutive nodes hit different banks, and every
// plane is an immediate offset), in one buffer, used in the pull-swap order: after an odd level t a node
// writes f*_q to its own slot of the opposite direction, after an even level to the slot q of
// the neighbour it streams to; the next level then reads f_q from slot opp(q) of the
// neighbour it pulls from (t even) or from its own slot q (t odd).  A node writes exactly the
// slots it has just read, so one barrier per level separates the levels.
// (27 with per-node parameters on a grid with traction edges: mu and lam for the link solves)
constexpr int patch_stride(bool params) { return params ? 27 : 25; }

// Grids without walls, with velocity walls only, and with traction edges.
enum { kNoWalls, kVelocityWalls, kTractionWalls };

template <int ST, int LAW, int WALLS, bool FIELDS>
__global__ void __launch_bounds__(patch_threads(ST == LBM_F64_PLAIN, WALLS == kTractionWalls)) patch_kernel(PatchArgs a) {
    using Tr = Storage<ST>;
    using R = typename Tr::real;
    using T = typename Tr::pop_t;
    constexpr bool SH = Tr::shifted;
    constexpr bool LINKS = WALLS == kTractionWalls;
    constexpr int NS = patch_stride(LINKS && FIELDS);
    extern __shared__ __attribute__((aligned(16))) char patch_smem[];
    R* sh = (R*)patch_smem;
    const Common& cm = a.cm;
    const int nx = cm.nx, ny = cm.ny, ntile = cm.ntile, levels = a.levels;
    const int64_t n = int64_t(nx) * ny;
    int pw, ph, px0, py0, px1, py1;
    patch_at(a.map, pw, ph, px0, py0, px1, py1);
    const PatchPos pos = patch_pos(threadIdx.x, pw, ph);
    const int X = px0 + pos.x, Y = py0 + pos.y;
    const int rw = pw + 2 * (levels - 1);
    const bool valid = pos.ring < levels && (!WALLS || ((cm.periodic_x || (X >= 0 && X < nx)) &&
                                                        (cm.periodic_y || (Y >= 0 && Y < ny))));
    const bool core = valid && pos.ring == 0 && X < px1 && Y < py1;
    const int xr = wrap_index(X, nx), yr = wrap_index(Y, ny);
    R* own = sh + ((pos.y + levels - 1) * rw + (pos.x + levels - 1)) * NS;
    // the neighbours a node pulls q0 .. q3 from, and streams q2, q3, q0, q1 to
    R* const nb0 = own - NS;
    R* const nb1 = own - rw * NS;
    R* const nb2 = own + NS;
    R* const nb3 = own + rw * NS;

    const T* __restrict__ src = (const T*)a.src;
    R mu = kval<R>(cm.mu0, cm.f_mu0), lam = kval<R>(cm.lam0, cm.f_lam0);
    float bf[2] = {0.0f, 0.0f};
    bool xw = false, yw = false;                 // the node has a missing link along x / y
    if (WALLS && valid) {
        xw = !cm.periodic_x && (xr == 0 || xr == nx - 1);
        yw = !cm.periodic_y && (yr == 0 || yr == ny - 1);
    }
    if (valid) {
        const int idx = yr * nx + xr;
        params_at<FIELDS, R>(cm, idx, mu, lam);
        if (FIELDS && cm.body) {
            bf[0] = cm.body[idx];
            bf[1] = cm.body[n + idx];
        }
        if (LINKS && FIELDS) {
            own[NS - 2] = mu;
            own[NS - 1] = lam;
        }
    }
    // the displacement accumulator of the patch's nodes
    R u0 = R(0), u1 = R(0);
    float sf0 = 0.0f, sf1 = 0.0f;                // the block sums moved into U at a fold
    if (core && a.ustar) {
        if constexpr (ST == LBM_F64_PLAIN) {
            const double* up = (const double*)a.ustar + tile_base(ntile, 2, xr, yr);
            u0 = up[0];
            u1 = up[kTile];
        } else {
            const float* sp = ustar_refs(a.ustar, ntile, ny, xr, yr).S;
            u0 = sp[0];
            u1 = sp[kTile];
        }
    }
    const R dt = kval<R>(cm.dt, cm.f_dt);
    auto body_level = [&](int t, R& B0, R& B1) {  // B of level n + t
        if (FIELDS && cm.body) {
            B0 = R(a.r[t] * double(bf[0]));
            B1 = R(a.r[t] * double(bf[1]));
        } else {
            B0 = kval<R>(a.r[t] * cm.b0[0], a.fb[t][0]);
            B1 = kval<R>(a.r[t] * cm.b0[1], a.fb[t][1]);
        }
    };
    uint32_t fault = 0;
    // Grids with traction edges: a patch whose region touches a wall solves the missing links of a level first: one lane
    // per link, the links of x-edges and of y-edges on wavefronts of their own, so that no
    // wavefront takes one solve after the other.  A link reads its node's populations of level
    // n + t - 1 (in memory, or where the node wrote them in LDS) and writes its value into the
    // slot the node is about to read (a slot whose neighbour lies beyond the wall: no other
    // thread touches it).
    const int halo = levels - 1;
    const bool rim = LINKS && ((!cm.periodic_x && (px0 - halo <= 0 || px0 + pw + halo >= nx)) ||
                               (!cm.periodic_y && (py0 - halo <= 0 || py0 + ph + halo >= ny)));
    auto solve_links = [&](int t, int px0, int py0) {
        asm volatile("" : "+s"(px0), "+s"(py0));     // formed here, not kept through the loop
        const int rh = ph + 2 * halo;
        const bool xlo = !cm.periodic_x && px0 - halo <= 0, xhi = !cm.periodic_x && px0 + pw + halo >= nx;
        const bool ylo = !cm.periodic_y && py0 - halo <= 0, yhi = !cm.periodic_y && py0 + ph + halo >= ny;
        const int xlinks = (int(xlo) + int(xhi)) * rh, xpad = (xlinks + kTile - 1) & ~(kTile - 1);
        const int links = xpad + (int(ylo) + int(yhi)) * rw;
        const bool nbr = (t & 1) == 0;
        for (int j = threadIdx.x; j < links; j += blockDim.x) {
            const bool ax = j >= xpad;              // the axis of the normal (per wavefront)
            int i = ax ? j - xpad : j;
            if (!ax && i >= xlinks) continue;
            const bool lo = ax ? (ylo && i < rw) : (xlo && i < rh);
            if (i >= (ax ? rw : rh)) i -= ax ? rw : rh;
            const int LX = ax ? px0 - halo + i : (lo ? 0 : nx - 1), LY = ax ? (lo ? 0 : ny - 1) : py0 - halo + i;
            const int cx = LX - px0, cy = LY - py0;
            const int ring = max(max(max(-cx, cx - pw + 1), max(-cy, cy - ph + 1)), 0);
            const bool inside = (cm.periodic_x || (LX >= 0 && LX < nx)) && (cm.periodic_y || (LY >= 0 && LY < ny));
            if (!inside || ring > levels - t) continue;
            R* o = sh + ((cy + halo) * rw + (cx + halo)) * NS;
            R* const m0 = o - NS;
            R* const m1 = o - rw * NS;
            R* const m2 = o + NS;
            R* const m3 = o + rw * NS;
            R out[6], U[6], lk[6];
            const int wx = wrap_index(LX, nx), wy = wrap_index(LY, ny);
            auto gather = [&](auto get) {
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const R v0 = get(0, k), v1 = get(1, k), v2 = get(2, k), v3 = get(3, k);
                    U[k] = R(0) + v0 + v1 + v2 + v3;         // as recover_vals sums
                    out[k] = ax ? (lo ? v3 : v1) : (lo ? v2 : v0);
                }
            };
            if (t == 1) {
                const T* s = src + tile_base(ntile, 24, wx, wy);
                gather([&](int q, int k) { return R(s[(6 * q + k) * kTile]); });
            } else {
                const R* const w[4] = {nbr ? o + 12 : m2, nbr ? o + 18 : m3 + 6, nbr ? o : m0 + 12, nbr ? o + 6 : m1 + 18};
                gather([&](int q, int k) { return w[q][k]; });
            }
            const R pm = FIELDS ? o[NS - 2] : mu, pl = FIELDS ? o[NS - 1] : lam;
            bool ok;
            R* slot;
            if (ax) {
                ok = patch_link<R, LAW, SH, 1>(a, t - 1, lo, wx, out, U, pm, pl, lk);
                slot = lo ? (nbr ? m1 + 18 : o + 6) : (nbr ? m3 + 6 : o + 18);
            } else {
                ok = patch_link<R, LAW, SH, 0>(a, t - 1, lo, wy, out, U, pm, pl, lk);
                slot = lo ? (nbr ? m0 + 12 : o) : (nbr ? m2 : o + 12);
            }
#pragma unroll
            for (int k = 0; k < 6; ++k) slot[k] = lk[k];
            if (!ok) fault |= LBM_FAULT_NEWTON;
        }
    };
    for (int t = 1; t <= levels; ++t) {
        const bool act = valid && pos.ring <= levels - t;
        // opaque per level: addresses in memory, used at one level each, are formed where they
        // are used instead of being kept in registers through the loop
        int x = xr, y = yr;
        asm volatile("" : "+v"(x), "+v"(y));
        R gq[4][6], f[4][6];
        // Velocity walls alone: a link takes no solve, and the node's own thread forms it from the
        // populations that it wrote itself, so that the patches at a wall have one barrier per
        // level as all others (128^2 FP32 4.2 -> 3.4 us per level, 512^2 FP64 16.7 -> 12.6, against the
        // lanes and barriers of solve_links; where only some of the edges are velocity walls
        // the solves' lanes take these links along).
        if (WALLS == kVelocityWalls && act && (xw || yw)) {
            const bool nbr = (t & 1) == 0;
            const T* s = src + tile_base(ntile, 24, x, y);
            if (xw) {
                const bool lo = x == 0;
                // the outgoing q2 at XMIN (q0 at XMAX) lies where level t - 1 wrote it
                R* slot = lo ? (nbr ? nb0 + 12 : own) : (nbr ? nb2 : own + 12);
                const R* o = lo ? (nbr ? own : nb0 + 12) : (nbr ? own + 12 : nb2);
                if (t == 1) patch_velocity_link<R, 0>(a, t - 1, lo, y, s + (lo ? 12 : 0) * kTile, kTile, slot);
                else patch_velocity_link<R, 0>(a, t - 1, lo, y, o, 1, slot);
            }
            if (yw) {
                const bool lo = y == 0;
                R* slot = lo ? (nbr ? nb1 + 18 : own + 6) : (nbr ? nb3 + 6 : own + 18);
                const R* o = lo ? (nbr ? own + 6 : nb1 + 18) : (nbr ? own + 18 : nb3 + 6);
                if (t == 1) patch_velocity_link<R, 1>(a, t - 1, lo, x, s + (lo ? 18 : 6) * kTile, kTile, slot);
                else patch_velocity_link<R, 1>(a, t - 1, lo, x, o, 1, slot);
            }
        }
        if (rim) {
            if (FIELDS || t > 1) __syncthreads();
            solve_links(t, px0, py0);
            __syncthreads();
        } else if (t > 1) {
            __syncthreads();
        }
        if (t == 1) {
            if (act) {
                int xm = wrap_dec(x, nx), xp = wrap_inc(x, nx), ym = wrap_dec(y, ny), yp = wrap_inc(y, ny);
                if (WALLS) {                             // a source beyond a wall: any readable node
                    if (xw) { if (x == 0) xm = x; else xp = x; }
                    if (yw) { if (y == 0) ym = y; else yp = y; }
                }
                const T* s0 = src + tile_base(ntile, 24, xm, y);
                const T* s1 = src + tile_base(ntile, 24, x, ym);
                const T* s2 = src + tile_base(ntile, 24, xp, y);
                const T* s3 = src + tile_base(ntile, 24, x, yp);
        #pragma unroll
                for (int k = 0; k < 6; ++k) {
                    gq[0][k] = R(s0[k * kTile]);
                    gq[1][k] = R(s1[(6 + k) * kTile]);
                    gq[2][k] = R(s2[(12 + k) * kTile]);
                    gq[3][k] = R(s3[(18 + k) * kTile]);
                }
            }
        } else {
            if (act) {
                const bool nbr = (t & 1) == 0;
                const R* r0 = nbr ? nb0 + 12 : own;
                const R* r1 = nbr ? nb1 + 18 : own + 6;
                const R* r2 = nbr ? nb2 : own + 12;
                const R* r3 = nbr ? nb3 + 6 : own + 18;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    gq[0][k] = r0[k];
                    gq[1][k] = r1[k];
                    gq[2][k] = r2[k];
                    gq[3][k] = r3[k];
                }
            }
        }
        if (act) {
            if (WALLS && t == 1 && (xw || yw)) {   // the other pulls came from memory
                const int dx = x == 0 ? 0 : 2, dy = y == 0 ? 1 : 3;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const R vx = own[6 * dx + k], vy = own[6 * dy + k];
                    if (xw) { gq[0][k] = x == 0 ? vx : gq[0][k]; gq[2][k] = x == 0 ? gq[2][k] : vx; }
                    if (yw) { gq[1][k] = y == 0 ? vy : gq[1][k]; gq[3][k] = y == 0 ? gq[3][k] : vy; }
                }
            }
            R B0, B1, U[6], J;
            body_level(t, B0, B1);
            collide_node<R, LAW, SH>(cm, gq, B0, B1, mu, lam, f, U, J);
            bool nonfinite = false;
#pragma unroll
            for (int k = 0; k < 6; ++k) nonfinite |= !finite_r(U[k]);
            if (nonfinite) fault |= LBM_FAULT_NONFINITE;
            if (J <= R(0)) fault |= LBM_FAULT_J;
            if (core) {
                if (a.rec[t - 1]) {
                    R* rec = (R*)a.rec[t - 1] + tile_base(ntile, 6, x, y);
                    if (a.rec_planes == 6) {
                        rec[0] = U[0];
                        rec[kTile] = U[1];
                    }
                    rec[2 * kTile] = SH ? U[2] : U[2] - R(1);
                    rec[3 * kTile] = U[3];
                    rec[4 * kTile] = U[4];
                    rec[5 * kTile] = SH ? U[5] : U[5] - R(1);
                }
                // displacement quadrature (eq:trapezoid-u), with the folds of single steps
                if constexpr (ST == LBM_F64_PLAIN) {
                    u0 = u0 + dt * U[0];
                    u1 = u1 + dt * U[1];
                } else {
                    u0 = u0 + float(dt * U[0]);
                    u1 = u1 + float(dt * U[1]);
                    if (t == a.fold) {
                        sf0 = u0;
                        sf1 = u1;
                        u0 = u1 = 0.0f;
                    }
                }
            }
            if (t < levels) {
                const bool mine = (t & 1) != 0;
                R* w0 = mine ? own + 12 : nb2;
                R* w1 = mine ? own + 18 : nb3 + 6;
                R* w2 = mine ? own : nb0 + 12;
                R* w3 = mine ? own + 6 : nb1 + 18;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    w0[k] = R(to_storage<T>(f[0][k]));
                    w1[k] = R(to_storage<T>(f[1][k]));
                    w2[k] = R(to_storage<T>(f[2][k]));
                    w3[k] = R(to_storage<T>(f[3][k]));
                }
            } else if (core) {
                T* d = (T*)a.dst + tile_base(ntile, 24, x, y);
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int k = 0; k < 6; ++k) d[(6 * q + k) * kTile] = to_storage<T>(f[q][k]);
            }
        }
    }
    if (core && a.ustar) {
        int x = xr, y = yr;
        asm volatile("" : "+v"(x), "+v"(y));
        if constexpr (ST == LBM_F64_PLAIN) {
            double* up = (double*)a.ustar + tile_base(ntile, 2, x, y);
            up[0] = u0;
            up[kTile] = u1;
        } else {
            const UstarRefs r = ustar_refs(a.ustar, ntile, ny, x, y);
            r.S[0] = u0;
            r.S[kTile] = u1;
            if (a.fold) {
                r.U[0] = r.U[0] + double(sf0);
                r.U[kTile] = r.U[kTile] + double(sf1);
            }
        }
    }
    if (fault) atomicOr(cm.fault, fault);
}

// ---------------------------------------------------------------- dispatch

template <int ST, int LAW, int WALLS>
static hipError_t patch_st_law_walls(const PatchArgs& a, hipStream_t s) {
    const bool fields = a.cm.mu || a.cm.lam || a.cm.body;
    const int nodes = (a.map.pw + 2 * (a.levels - 1)) * (a.map.ph + 2 * (a.levels - 1));
    const size_t lds =
        size_t(nodes) * patch_stride(WALLS == kTractionWalls && fields) * sizeof(typename Storage<ST>::real);
    const dim3 grid(unsigned(a.map.nwg)), block(unsigned((nodes + kTile - 1) / kTile * kTile));
    if (block.x > unsigned(patch_threads(ST == LBM_F64_PLAIN, WALLS == kTractionWalls)) || lds > size_t(kPatchLds))
        return hipErrorInvalidValue;
    if (fields) hipLaunchKernelGGL((patch_kernel<ST, LAW, WALLS, true>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((patch_kernel<ST, LAW, WALLS, false>), grid, block, lds, s, a);
    return hipGetLastError();
}

template <int ST, int LAW>
static hipError_t patch_st_law(const PatchArgs& a, hipStream_t s) {
    if (a.cm.periodic_x && a.cm.periodic_y) return patch_st_law_walls<ST, LAW, kNoWalls>(a, s);
    bool traction = false;
    for (int e = 0; e < 4; ++e) traction |= a.cm.bc[e] == LBM_TRACTION;
    if (traction) return patch_st_law_walls<ST, LAW, kTractionWalls>(a, s);
    return patch_st_law_walls<ST, LAW, kVelocityWalls>(a, s);
}

template <int ST>
static hipError_t patch_st(const PatchArgs& a, hipStream_t s) {
    switch (a.cm.material) {
        case LBM_LOGNH: return patch_st_law<ST, LBM_LOGNH>(a, s);
        case LBM_NH: return patch_st_law<ST, LBM_NH>(a, s);
        case LBM_MR: return patch_st_law<ST, LBM_MR>(a, s);
        case LBM_YEOH: return patch_st_law<ST, LBM_YEOH>(a, s);
        case LBM_GENT: return patch_st_law<ST, LBM_GENT>(a, s);
        default: return patch_st_law<ST, LBM_SVK>(a, s);
    }
}

hipError_t launch_patch(const PatchArgs& a, hipStream_t s) {
    switch (a.cm.storage) {
        case LBM_F32_SHIFTED: return patch_st<LBM_F32_SHIFTED>(a, s);
        case LBM_F16_SHIFTED: return patch_st<LBM_F16_SHIFTED>(a, s);
        default: return patch_st<LBM_F64_PLAIN>(a, s);
    }
}

}  // namespace lbm
