// C ABI of the library (declared in include/lbm.h): argument validation, buffer sizes and
// the launch sequence of each entry point.  No allocation, no synchronisation.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>

#include "lbm_device.hpp"
#include "lbm_internal.hpp"

using namespace lbm;

namespace {

// Device scratch of lbm_diagnostics_noalloc: the per-workgroup partial sums of the
// diagnostics reduction, kDiagBlocks x LBM_DIAG_COUNT doubles (80 KiB), enough for every
// grid because the reduction kernel strides over the nodes with at most kDiagBlocks
// workgroups.  Every GPU the library runs on holds its own copy until the process ends.
// On the host this name is only a stand-in for the symbol: host code uses the device
// address that scratch_address obtains for the current device.
__device__ __align__(256) double scratch[kDiagBlocks * LBM_DIAG_COUNT];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device.
lbm_status scratch_address(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LBM_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LBM_ERR_LAUNCH;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return LBM_OK;
}

bool any_wall(const lbm_params* p) {
    for (int e = 0; e < 4; ++e)
        if (p->bc[e] != LBM_PERIODIC) return true;
    return false;
}

bool has_traction(const lbm_params* p) {
    for (int e = 0; e < 4; ++e)
        if (p->bc[e] == LBM_TRACTION) return true;
    return false;
}

size_t real_size(const lbm_params* p) { return p->storage == LBM_F64_PLAIN ? 8 : 4; }

size_t pop_elem_size(const lbm_params* p) {
    return p->storage == LBM_F64_PLAIN ? 8 : (p->storage == LBM_F16_SHIFTED ? 2 : 4);
}

Common make_common(const lbm_params* p, const lbm_state* s) {
    Common cm{};
    cm.nx = p->nx;
    cm.ny = p->ny;
    cm.ntile = (p->nx + kTile - 1) / kTile;
    for (int e = 0; e < 4; ++e) cm.bc[e] = p->bc[e];
    cm.periodic_x = p->bc[LBM_XMIN] == LBM_PERIODIC;
    cm.periodic_y = p->bc[LBM_YMIN] == LBM_PERIODIC;
    cm.material = p->material;
    cm.storage = p->storage;
    cm.dx = p->dx;
    cm.c = p->c;
    cm.omega = p->omega;
    cm.dt = p->dx / p->c;
    cm.newton_max_iter = p->newton_max_iter > 0 ? p->newton_max_iter : 8;
    cm.newton_tol = p->newton_tol > 0 ? p->newton_tol : (p->storage == LBM_F64_PLAIN ? 1e-14 : 1e-6);
    for (int k = 0; k < 3; ++k) cm.law_k[k] = p->law_k[k];
    cm.k_omq = 0.25 * cm.omega;
    cm.k_cq = 0.5 * cm.omega / cm.c;
    cm.k_srcw = cm.dt * (2.0 - cm.omega) * 0.125;
    cm.k_hdt = 0.5 * cm.dt;
    cm.k_c2 = 2.0 / cm.c;
    cm.k_hc = 0.5 / cm.c;
    if (s) {
        cm.mu0 = s->mu0;
        cm.lam0 = s->lam0;
        cm.b0[0] = s->b0[0];
        cm.b0[1] = s->b0[1];
        cm.mu = s->mu;
        cm.lam = s->lam;
        cm.body = s->body;
        cm.body_prev = s->body_prev;
        cm.fault = s->fault;
    }
    cm.f_omq = float(cm.k_omq);
    cm.f_cq = float(cm.k_cq);
    cm.f_srcw = float(cm.k_srcw);
    cm.f_hdt = float(cm.k_hdt);
    cm.f_c2 = float(cm.k_c2);
    cm.f_hc = float(cm.k_hc);
    cm.f_dt = float(cm.dt);
    cm.f_mu0 = float(cm.mu0);
    cm.f_lam0 = float(cm.lam0);
    for (int k = 0; k < 3; ++k) cm.f_law_k[k] = float(cm.law_k[k]);
    cm.f_omega = float(cm.omega);
    return cm;
}

EdgeData make_edges(const lbm_edge_data* ed) {
    EdgeData out{};
    if (ed) {
        for (int e = 0; e < 4; ++e) {
            out.value[e][0] = ed->value[e][0];
            out.value[e][1] = ed->value[e][1];
            out.field[e] = ed->field[e];
        }
    }
    return out;
}

lbm_status check_state(const lbm_params* p, const lbm_state* s, bool need_ustar = true) {
    if (!s || !s->pop[0] || !s->pop[1] || !s->fault) return LBM_ERR_ARG;
    if (need_ustar && !s->ustar) return LBM_ERR_ARG;
    if (s->cur != 0 && s->cur != 1) return LBM_ERR_ARG;
    if (has_traction(p) && !s->aux) return LBM_ERR_ARG;
    return LBM_OK;
}

// Compute units of the current device, queried once per device (256 on an MI355X).
int compute_units() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int v = cached[dev].load(std::memory_order_relaxed);
    if (v > 0) return v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    cached[dev].store(v, std::memory_order_relaxed);
    return v;
}

lbm_status launched(hipError_t e) { return e == hipSuccess ? LBM_OK : LBM_ERR_LAUNCH; }

// Uniform predeformation: I when none is given; rejected unless finite with det > 0.
bool predeformation(const double* Fbar, double out[4]) {
    const double I[4] = {1.0, 0.0, 0.0, 1.0};
    const double* f = Fbar ? Fbar : I;
    for (int k = 0; k < 4; ++k) {
        if (!isfinite(f[k])) return false;
        out[k] = f[k];
    }
    return out[0] * out[3] - out[1] * out[2] > 0.0;
}

// The P-wave speed at F = I bounding the material's waves: sqrt(lam + 2 mu) for the
// Lame-parametrised laws, sqrt(lam + 4 G / 3) for the invariant laws (small-strain shear
// modulus G, plane Lame constant lam - 2 G / 3).
double p_wave_speed(const lbm_params* p, double mu_max, double lam_max) {
    double cp2 = lam_max + 2.0 * mu_max;
    if (p->material == LBM_MR || p->material == LBM_YEOH || p->material == LBM_GENT) {
        const double G = p->material == LBM_MR ? 2.0 * (p->law_k[0] + p->law_k[1]) * mu_max
                       : p->material == LBM_YEOH ? 2.0 * p->law_k[0] * mu_max : mu_max;
        cp2 = lam_max + 4.0 / 3.0 * G;
    }
    return sqrt(fmax(cp2, 0.0));
}

// Growth per step of the modes a traction wall carries at omega = 2, measured (FP64, 512^2,
// from noise; walls on all four sides, with a velocity corner, and on two sides only) at
// P-wave ratios c_p / c of 0.0505 ... 0.283, and the rate at which 2 - omega damps them.
constexpr int kWallTable = 6;
constexpr double kWallRatio[kWallTable] = {0.0505, 0.0707, 0.101, 0.141, 0.202, 0.283};
constexpr double kWallGrowth0[kWallTable] = {3.3e-4, 2.7e-4, 2.5e-4, 3.7e-4, 1.76e-3, 4.35e-3};
constexpr double kWallDamping = 0.45;
constexpr double kWallGrowthMax = 2e-4;   // e-folding in 5000 steps

}  // namespace

extern "C" {

size_t lbm_tile_width(void) { return (size_t)kTile; }

size_t lbm_padded_nodes(const lbm_params* p) {
    const size_t ntile = ((size_t)p->nx + kTile - 1) / kTile;
    return ntile * kTile * (size_t)p->ny;
}

size_t lbm_pop_bytes(const lbm_params* p) { return 24 * lbm_padded_nodes(p) * pop_elem_size(p); }

size_t lbm_ustar_bytes(const lbm_params* p) {
    // FP64: 2 double planes; shifted storages: 2 float planes S and 2 double planes U
    return p->storage == LBM_F64_PLAIN ? 2 * lbm_padded_nodes(p) * 8 : lbm_padded_nodes(p) * (2 * 4 + 2 * 8);
}

// F^b of every link (4 values), and for the two-level step the wall lines of level n+1
// (2 lines of 24 values per link) and U^{n+1} of the wall nodes (6 values), 8 bytes each
// (WallLines in lbm_kernel_util.hpp).
size_t lbm_aux_bytes(const lbm_params* p) { return (size_t)(2 * p->nx + 2 * p->ny) * (4 + 2 * 24 + 6) * 8; }

size_t lbm_record_bytes(const lbm_params* p) { return 6 * lbm_padded_nodes(p) * real_size(p); }

size_t lbm_adj_bytes(const lbm_params* p) { return 24 * lbm_padded_nodes(p) * real_size(p); }

size_t lbm_adj_sum_bytes(const lbm_params* p) { return 4 * lbm_padded_nodes(p) * sizeof(float); }

size_t lbm_diag_scratch_bytes(const lbm_params* p) {
    (void)p;
    return (size_t)kDiagBlocks * LBM_DIAG_COUNT * sizeof(double);
}

lbm_status lbm_check_params(const lbm_params* p) {
    if (!p) return LBM_ERR_ARG;
    if (p->nx < 3 || p->ny < 3) return LBM_ERR_ARG;
    if ((int64_t)p->nx * (int64_t)p->ny >= ((int64_t)1 << 31)) return LBM_ERR_ARG;
    if (p->material < LBM_LOGNH || p->material > LBM_GENT) return LBM_ERR_ARG;
    if (p->material == LBM_MR &&
        !(p->law_k[0] >= 0 && p->law_k[1] >= 0 && p->law_k[0] + p->law_k[1] > 0)) return LBM_ERR_ARG;
    if (p->material == LBM_YEOH &&
        !(p->law_k[0] > 0 && isfinite(p->law_k[1]) && isfinite(p->law_k[2]))) return LBM_ERR_ARG;
    if (p->material == LBM_GENT && !(p->law_k[0] > 0 && isfinite(p->law_k[0]))) return LBM_ERR_ARG;
    if (p->storage < LBM_F32_SHIFTED || p->storage > LBM_F64_PLAIN) return LBM_ERR_ARG;
    for (int e = 0; e < 4; ++e)
        if (p->bc[e] < LBM_PERIODIC || p->bc[e] > LBM_TRACTION) return LBM_ERR_ARG;
    if ((p->bc[LBM_XMIN] == LBM_PERIODIC) != (p->bc[LBM_XMAX] == LBM_PERIODIC)) return LBM_ERR_ARG;
    if ((p->bc[LBM_YMIN] == LBM_PERIODIC) != (p->bc[LBM_YMAX] == LBM_PERIODIC)) return LBM_ERR_ARG;
    if (any_wall(p) && (p->nx < 4 || p->ny < 4)) return LBM_ERR_ARG;
    if (!(p->dx > 0) || !(p->c > 0) || !(p->omega > 0) || !(p->omega <= 2.0)) return LBM_ERR_ARG;
    return LBM_OK;
}

double lbm_wall_mode_growth(const lbm_params* p, double mu_max, double lam_max) {
    if (!p || !(p->c > 0)) return 0.0;
    bool traction = false;
    for (int e = 0; e < 4; ++e) traction |= p->bc[e] == LBM_TRACTION;
    if (!traction) return 0.0;
    const double r = p_wave_speed(p, mu_max, lam_max) / p->c;
    double g0;
    if (r <= kWallRatio[0]) {
        g0 = kWallGrowth0[0];
    } else {
        int i = 1;
        while (i < kWallTable - 1 && r > kWallRatio[i]) ++i;
        // linear between the measured points, and along the last segment beyond them
        const double t = (r - kWallRatio[i - 1]) / (kWallRatio[i] - kWallRatio[i - 1]);
        g0 = kWallGrowth0[i - 1] + t * (kWallGrowth0[i] - kWallGrowth0[i - 1]);
    }
    return g0 - kWallDamping * (2.0 - p->omega);
}

lbm_status lbm_check_cfl(const lbm_params* p, double mu_max, double lam_max) {
    if (!p || !(p->c > 0)) return LBM_ERR_ARG;
    if (p_wave_speed(p, mu_max, lam_max) / p->c > 0.5) return LBM_ERR_CFL;
    if (lbm_wall_mode_growth(p, mu_max, lam_max) > kWallGrowthMax) return LBM_ERR_CFL;
    return LBM_OK;
}

lbm_status lbm_init(const lbm_params* p, lbm_state* s, const double* v0, const double* u0,
                    const double* Fbar, double r0, void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if ((st = check_state(p, s)) != LBM_OK) return st;
    if (!v0) return LBM_ERR_ARG;
    double F0[4];
    if (!predeformation(Fbar, F0)) return LBM_ERR_ARG;
    if (!p->force_unstable) {
        const double mu = s->mu ? s->mu_max : s->mu0;
        const double lam = s->lam ? s->lam_max : s->lam0;
        if ((st = lbm_check_cfl(p, mu, lam)) != LBM_OK) return st;
    }
    InitArgs a{};
    a.cm = make_common(p, s);
    a.v0 = v0;
    a.u0 = u0;
    for (int k = 0; k < 4; ++k) a.Fbar[k] = F0[k];
    a.r0 = r0;
    a.scratch = s->pop[1 - s->cur];
    a.dst = s->pop[s->cur];
    a.ustar = s->ustar;
    return launched(launch_init(a, (hipStream_t)stream));
}

lbm_status lbm_init_state(const lbm_params* p, lbm_state* s, const double* U0, const double* dUdX,
                          const double* dUdY, const double* u0, double r0, void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if ((st = check_state(p, s)) != LBM_OK) return st;
    if (!U0 || !dUdX || !dUdY) return LBM_ERR_ARG;
    if (!p->force_unstable) {
        const double mu = s->mu ? s->mu_max : s->mu0;
        const double lam = s->lam ? s->lam_max : s->lam0;
        if ((st = lbm_check_cfl(p, mu, lam)) != LBM_OK) return st;
    }
    InitArgs a{};
    a.cm = make_common(p, s);
    a.v0 = U0;                       // planes 0, 1 of U0 are v0
    a.u0 = u0;
    a.r0 = r0;
    a.scratch = const_cast<double*>(U0);
    a.dst = s->pop[s->cur];
    a.ustar = s->ustar;
    a.dUdX = dUdX;
    a.dUdY = dUdY;
    return launched(launch_init_given(a, (hipStream_t)stream));
}

lbm_status lbm_step(const lbm_params* p, lbm_state* s, int64_t n, double r_n, double r_np1,
                    const lbm_edge_data* at_half, void* record, void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if ((st = check_state(p, s, false)) != LBM_OK) return st;
    if (any_wall(p) && !at_half) return LBM_ERR_ARG;
    const hipStream_t hs = (hipStream_t)stream;
    const Common cm = make_common(p, s);
    const EdgeData ed = make_edges(at_half);
    {
        TractionArgs t{};
        t.cm = cm;
        if (cm.body_prev) t.cm.body = cm.body_prev;
        t.pop = s->pop[s->cur];
        t.aux = s->aux;
        t.r_n = r_n;
        t.ed = ed;
        if (launch_traction(t, hs) != hipSuccess) return LBM_ERR_LAUNCH;
    }
    StepArgs a{};
    a.cm = cm;
    a.src = s->pop[s->cur];
    a.dst = s->pop[1 - s->cur];
    a.ustar = s->ustar;
    a.aux = s->aux;
    a.record = record;
    a.fold = (n + 1) % kUstarBlock == 0;
    a.r_np1 = r_np1;
    a.ed = ed;
    if (launch_step(a, hs) != hipSuccess) return LBM_ERR_LAUNCH;
    s->cur = 1 - s->cur;
    return LBM_OK;
}

lbm_status lbm_step2(const lbm_params* p, lbm_state* s, int64_t n, double r_n, double r_np1, double r_np2,
                     const lbm_edge_data* at_half, const lbm_edge_data* at_half_next, void* record1, void* record2,
                     void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if ((st = check_state(p, s, false)) != LBM_OK) return st;
    const bool walls = any_wall(p);
    if (walls && (!at_half || !at_half_next || !s->aux)) return LBM_ERR_ARG;
    const hipStream_t hs = (hipStream_t)stream;
    Step2Args a{};
    a.cm = make_common(p, s);
    a.cm.body_prev = nullptr;                    // the body field is that of every level
    a.src = s->pop[s->cur];
    a.dst = s->pop[1 - s->cur];
    a.ustar = s->ustar;
    a.aux = s->aux;
    a.ed = make_edges(at_half);
    a.ed2 = make_edges(at_half_next);
    a.record1 = record1;
    a.record2 = record2;
    a.fold1 = (n + 1) % kUstarBlock == 0;
    a.fold2 = (n + 2) % kUstarBlock == 0;
    a.nstrip = (p->nx + kPairCols - 1) / kPairCols;
    a.r_np1 = r_np1;
    a.r_np2 = r_np2;
    for (int k = 0; k < 2; ++k) {
        a.fb1[k] = float(r_np1 * a.cm.b0[k]);
        a.fb2[k] = float(r_np2 * a.cm.b0[k]);
    }
    // F^b of level n from f*^n, as lbm_step takes it
    {
        TractionArgs t{};
        t.cm = a.cm;
        t.pop = a.src;
        t.aux = s->aux;
        t.r_n = r_n;
        t.ed = a.ed;
        if (launch_traction(t, hs) != hipSuccess) return LBM_ERR_LAUNCH;
    }
    if (launch_step2(a, hs) != hipSuccess) return LBM_ERR_LAUNCH;
    if (walls) {
        // F^b of level n+1 from the wall lines the bulk kernel wrote, then the wall nodes
        {
            TractionArgs t{};
            t.cm = a.cm;
            t.pop = nullptr;
            t.aux = s->aux;
            t.r_n = r_np1;
            t.ed = a.ed2;
            t.lines = 1;
            if (launch_traction(t, hs) != hipSuccess) return LBM_ERR_LAUNCH;
        }
        Step2Args w = a;
        w.wall_pass = 1;
        if (launch_step2(w, hs) != hipSuccess) return LBM_ERR_LAUNCH;
    }
    s->cur = 1 - s->cur;
    return LBM_OK;
}

// Workgroups of the multi-level kernels: spans of kMarchTiles tiles per row, segments of
// `seg` rows.  A segment repeats 2 (levels - 1) rows of the first level and fewer of the
// later ones, and the launch runs in rounds of one workgroup per compute unit: the length
// between 8 and 1024 rows that minimises rounds x iterations per workgroup (8192^2: 205
// rows in three full rounds; with at most 64 rows, 62 rows in ten rounds ran 4 % slower).
static bool march_geometry(int tiles, int per_span, int rows, int levels, int& nspan, int& seg, int& nwg, FastDiv& d_nspan) {
    nspan = (tiles + per_span - 1) / per_span;
    const int cus = compute_units();
    int best = 8;
    int64_t best_cost = -1;
    for (int sg = 8; sg <= 1024; ++sg) {
        const int64_t ns = (rows + sg - 1) / sg;
        const int64_t rounds = (ns * nspan + cus - 1) / cus;
        const int64_t cost = rounds * (sg + 2 * (levels - 1));
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = sg; }
    }
    seg = best < rows ? best : rows;
    const int64_t nseg = (rows + seg - 1) / seg;
    if (nseg * nspan > 0x7fffffff) return false;
    nwg = int(nseg * nspan);
    d_nspan = fast_div(nspan);
    return true;
}

// The march over tiles [tile0, tile1) of the rows [row0, row1), level n -> n + levels, into the
// other population buffer (s->cur is not flipped).
static lbm_status march_launch(const lbm_params* p, const lbm_state* s, int64_t n, int levels, const double* r_next,
                               void* const* records, int record_planes, int tile0, int tile1, int row0, int row1,
                               hipStream_t hs) {
    MarchArgs a{};
    a.cm = make_common(p, s);
    a.cm.body_prev = nullptr;
    a.src = s->pop[s->cur];
    a.dst = s->pop[1 - s->cur];
    a.ustar = s->ustar;
    a.levels = levels;
    a.rec_planes = records ? record_planes : 6;
    for (int t = 0; t < levels; ++t) {
        a.fold[t] = (n + 1 + t) % kUstarBlock == 0;
        a.rec[t] = records ? records[t] : nullptr;
        a.r[t] = r_next[t];
        for (int k = 0; k < 2; ++k) a.fb[t][k] = float(r_next[t] * a.cm.b0[k]);
    }
    a.tile0 = tile0;
    a.tile1 = tile1;
    a.row0 = row0;
    a.row1 = row1;
    if (!march_geometry(tile1 - tile0, march_tiles(p->storage == LBM_F64_PLAIN), row1 - row0, levels, a.nspan, a.seg,
                        a.nwg, a.d_nspan))
        return LBM_ERR_UNSUPPORTED;
    return launched(launch_march(a, hs));
}

lbm_status lbm_step_multi(const lbm_params* p, lbm_state* s, int64_t n, int levels, const double* r_next,
                          void* const* records, int record_planes, void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if ((st = check_state(p, s, false)) != LBM_OK) return st;
    if (levels < 2 || levels > kMarchMaxLevels || !r_next) return LBM_ERR_ARG;
    if (records) {
        for (int t = 0; t < levels; ++t)
            if (!records[t]) return LBM_ERR_ARG;
        if (record_planes != 6 && record_planes != 4) return LBM_ERR_ARG;
    } else if (!s->ustar) {
        return LBM_ERR_ARG;
    }
    if (any_wall(p)) return LBM_ERR_UNSUPPORTED;
    // the replay form: records, no accumulator, shifted storages
    if (records && (s->ustar || p->storage == LBM_F64_PLAIN)) return LBM_ERR_UNSUPPORTED;
    st = march_launch(p, s, n, levels, r_next, records, record_planes, 0, (p->nx + kTile - 1) / kTile, 0, p->ny,
                      (hipStream_t)stream);
    if (st != LBM_OK) return st;
    s->cur = 1 - s->cur;
    return LBM_OK;
}

}  // extern "C"

// ---------------------------------------------------------------- several steps per call

namespace {

// Geometry of a patch launch: levels per launch and the nodes of a patch.
struct PatchPlan {
    int levels, pw, ph;
};

bool invariant_material(const lbm_params* p) {
    return p->material == LBM_MR || p->material == LBM_YEOH || p->material == LBM_GENT;
}

// What a patch launch costs, in arbitrary units (only the choice between plans uses it):
// `launch` once; every further round of patches on a compute unit, `round`; and per level and
// round the larger of `level` (one node's chain of dependent instructions and the barrier, with
// walls the traction solves before it) and `wave` for every wavefront of the level, of which
// patches of one compute unit beyond the first add the share `share` (they fill each other's
// waits).  Patches of 32 columns cost `row` times that (FP32 rows of 32 nodes are whole cache
// lines: 256^2, 6 levels 2.39 us per level at 32 x 8, 2.66 at 16 x 16).  `waves` wavefronts fit
// a compute unit.  Fitted to sweeps over 2 .. 8 levels and patches of 4 x 4 to 32 x 16 nodes on
// 18 grids of 64 x 64 to 1024 x 1024 nodes (log-NH and Gent): the chosen plan is 1 to 5 % slower
// than the best of the sweep on average, 25 % at worst.  Patches are used up to `side`^2 nodes.
struct PatchCost {
    double launch, level, wave, round, share, row;
    int side, threads, waves;
};

// Levels per launch and patch with the least cost per level, or levels = 0 beyond c.side^2.
PatchPlan patch_choice(const lbm_params* p, const PatchCost& c, int words, bool links) {
    static const int kLevels[] = {2, 3, 4, 6, 8};
    static const int kShapes[][2] = {{4, 4},   {8, 4},   {8, 8},   {12, 8}, {12, 12}, {16, 8},
                                     {16, 12}, {16, 16}, {20, 16}, {32, 8}, {32, 12}, {32, 16}};
    PatchPlan best{0, 0, 0};
    if (int64_t(p->nx) * p->ny > int64_t(c.side) * c.side) return best;
    double least = 0.0;
    const int cus = compute_units(), size = int(real_size(p));
    for (const auto& sh : kShapes) {
        const int pw = std::min(sh[0], p->nx), ph = std::min(sh[1], p->ny);
        const int64_t nwg = int64_t((p->nx + pw - 1) / pw) * ((p->ny + ph - 1) / ph);
        const int per_cu = int((nwg + cus - 1) / cus);
        for (const int T : kLevels) {
            const int nodes = (pw + 2 * (T - 1)) * (ph + 2 * (T - 1));
            const int lds = (nodes * words + (links ? 8 * (pw + ph + 4 * (T - 1)) : 0)) * size;
            if (nodes > c.threads || lds > kPatchLds) break;
            const int at_once = std::max(1, std::min(kPatchLds / lds, c.waves / ((nodes + kTile - 1) / kTile)));
            const int rounds = (per_cu + at_once - 1) / at_once;
            double t = c.launch + (rounds - 1) * c.round;
            for (int k = 0; k < T; ++k)
                t += std::max(c.level * rounds, c.wave * ((per_cu - 1) * c.share + 1.0) *
                                                    (((pw + 2 * k) * (ph + 2 * k) + kTile - 1) / kTile));
            if (pw >= 32) t *= c.row;
            if (best.levels == 0 || t / T < least) {
                least = t / T;
                best = PatchPlan{T, pw, ph};
            }
        }
    }
    return best;
}

// Periodic grids of about 280^2 nodes and more, where one launch takes two or more patches per
// compute unit: the model above misses how the patches of a unit share it, and there the plan was
// read off sweeps instead.  The first entry that holds the storage, the law and the grid's side
// sqrt(nx ny) decides; levels = 0: pairs of levels.  Measured on all plans and the pairs over grids
// of 1:1, 4:1 and 1:4, uniform and per-node parameters, log-NH, svk, MR, Yeoh and Gent (times over
// the best of all, averaged over the grids of a size): the model's plans reach 1.48 and, where the
// pairs are better, were up to 1.54 times as slow as these.
struct PlanRange {
    int storage, laws;               // laws: bits of the materials
    int lo, hi;                      // sides [lo, hi)
    PatchPlan plan;
};
constexpr int kLameLaws = 1 << LBM_LOGNH | 1 << LBM_NH | 1 << LBM_SVK;
constexpr int kInvariantLaws = 1 << LBM_MR | 1 << LBM_YEOH | 1 << LBM_GENT;
constexpr int kAllLaws = kLameLaws | kInvariantLaws;

const PlanRange kForwardRanges[] = {
    // this 1.00 to 1.03 (at 352^2 1.09), model 1.00 to 1.10, pairs 1.00 to 1.47
    {LBM_F32_SHIFTED, kLameLaws, 354, 440, {4, 32, 12}},
    // pairs 1.00 to 1.07, model 1.04 to 1.31, {4, 32, 12} 1.00 to 1.18; from 400^2 on pairs 1.01 to 1.35
    {LBM_F32_SHIFTED, kInvariantLaws, 354, 388, {0, 0, 0}},
    {LBM_F32_SHIFTED, kInvariantLaws, 395, 430, {4, 32, 12}},
    // 1.00 to 1.02, model 1.03 to 1.19, pairs 1.41 to 1.51 (610^2 to 690^2 1.00 / 1.02 to 1.09; 700^2
    // the other way, 1.05 / 1.00)
    {LBM_F32_SHIFTED, kAllLaws, 720, 1 << 15, {3, 32, 8}},
    // 1.00 to 1.02, model 1.01 to 1.13, pairs 1.02 to 1.15 (at 350^2 1.10 / 1.00); Yeoh: pairs 1.00 to
    // 1.03, model 1.08 to 1.27
    {LBM_F16_SHIFTED, kAllLaws & ~(1 << LBM_YEOH), 354, 435, {4, 32, 12}},
    {LBM_F16_SHIFTED, 1 << LBM_YEOH, 354, 435, {0, 0, 0}},
    // pairs 1.00 to 1.03, model 1.00 to 1.31, {3, 32, 8} 1.05 to 1.16: up to here the two buffers of
    // the pairs fit the L2s of the eight dies (32 MB); at 430^2 pairs 1.10, model 1.00; at 580^2
    // 1.07 / 1.01
    {LBM_F16_SHIFTED, kAllLaws, 435, 577, {0, 0, 0}},
    // 1.02 to 1.07, model 1.00 to 1.14, pairs 1.16 to 1.24 (per-node Gent and Yeoh: pairs 3 to 8 %
    // faster without records, 5 to 10 % slower with them)
    {LBM_F16_SHIFTED, kAllLaws, 720, 1 << 15, {3, 32, 8}},
    // per-node Yeoh: pairs 1.00, {3, 16, 8} 1.07 to 1.09, model 1.11 to 1.16
    {LBM_F64_PLAIN, 1 << LBM_YEOH, 365, 390, {0, 0, 0}},
    // 1.00 to 1.10, model 1.01 to 1.24, pairs 1.00 to 1.55 (272^2: 1.03 to 1.09 / 1.00 to 1.05)
    {LBM_F64_PLAIN, kAllLaws, 285, 1 << 15, {3, 16, 8}},
};
const PlanRange kAdjointRanges[] = {
    // pairs 1.00 to 1.04 (383^2 log-NH 1.08), model 1.05 to 1.28, {3, 16, 8} 1.04 to 1.11
    {LBM_F32_SHIFTED, kLameLaws, 310, 390, {0, 0, 0}},
    // pairs 1.00, model 1.00 to 1.12 (Gent 1.01 to 1.09 / 0.98 to 1.06)
    {LBM_F32_SHIFTED, 1 << LBM_MR | 1 << LBM_YEOH, 335, 388, {0, 0, 0}},
    // 1.00 to 1.03, model 0.99 to 1.17, pairs 1.02 to 1.55
    {LBM_F64_PLAIN, kLameLaws, 285, 1 << 15, {3, 16, 8}},
    // Gent: pairs 1.00 to 1.06, model 1.07 to 1.13
    {LBM_F64_PLAIN, 1 << LBM_GENT, 312, 388, {0, 0, 0}},
    // Yeoh: pairs 1.00 to 1.09, model 1.08 to 1.20 (at 200^2 1.04 / 1.01, at 279^2 1.23 / 1.00, at
    // 392^2 1.09 / 1.00)
    {LBM_F64_PLAIN, 1 << LBM_YEOH, 210, 268, {0, 0, 0}},
    {LBM_F64_PLAIN, 1 << LBM_YEOH, 302, 388, {0, 0, 0}},
};

// The entry for a periodic grid (nullptr: the model decides), on grids no narrower than those of
// the sweeps.
template <int N>
const PatchPlan* ranged_plan(const lbm_params* p, int storage, const PlanRange (&ranges)[N]) {
    if (p->nx < 2 * kTile || p->ny < kTile) return nullptr;
    const int64_t nodes = int64_t(p->nx) * p->ny;
    for (const PlanRange& r : ranges)
        if (r.storage == storage && (r.laws >> p->material & 1) && nodes >= int64_t(r.lo) * r.lo &&
            nodes < int64_t(r.hi) * r.hi)
            return &r.plan;
    return nullptr;
}

// The plan of patch_kernel.  Where it stops (side) the other kernels are faster.  Measured us
// per level, patches against the pairs, single steps and multi-level launches they replace
// (log-NH, uniform parameters):
//   FP32 periodic  64^2 1.7 / 2.8, 256^2 2.2 / 2.9, 512^2 5.2 / 8.3, 1000^2 15.2 / 23.1, and
//                  1130^2 27.7 / 19.6 (march_kernel from 1024^2 on; FP16 16.7 / 19.0, svk with
//                  per-node mu and lam 18.2 / 19.1)
//   FP32 traction  64^2 5.6 / 11.7, 256^2 6.2 / 11.6, 512^2 8.5 / 18.7, 1024^2 20.9 / 33.8
//                  (from 1100^2 on the march of the inner rectangle, see kRimNodes)
//   FP32 velocity  64^2 2.7 / 5.3, 256^2 3.6 / 6.0, 512^2 6.5 / 12.1, 1024^2 16.1 / 25.7; FP16
//                  512^2 7.0 / 9.5, 1024^2 17.0 / 21.7
//   FP64 periodic  64^2 2.0 / 3.8, 256^2 3.5 / 4.1, 700^2 15.4 / 22.8, 1024^2 48 / 43; with
//                  records 600^2 13.8 / 18.5, 850^2 41 / 38
//   FP64 traction  64^2 8.9 / 15.1, 256^2 9.1 / 16.3, 640^2 19.7 / 36.9, 850^2 39.8 / 38.1
//   FP64 velocity  64^2 3.2 / 5.6, 256^2 4.8 / 7.2, 640^2 14.3 / 27.2, 850^2 33.6 / 29.6
// (the traction solves of a wall node, some 700 dependent instructions per level, bound the
// small walled grids).  FP16 has no fit of its own: it takes kShifted's constants and, with traction
// edges, kTraction's (those plans are 1.06 to 1.22 times the best on 256^2 to 1090^2, the pairs 1.38
// to 2.08).
PatchPlan patch_plan(const lbm_params* p) {
    static const PatchCost kShifted{12.7, 0.84, 0.457, 3.43, 1.0, 0.92, 1024, patch_threads(false, false), 24};
    static const PatchCost kVelocity{2.80, 0.306, 0.032, 0.600, 1.0, 0.92, 1100, patch_threads(false, false), 24};
    static const PatchCost kTraction{18.4, 1.37, 0.090, 3.58, 0.57, 1.0, 1100, patch_threads(false, true), 24};
    static const PatchCost kHalf{12.7, 0.84, 0.457, 3.43, 1.0, 1.0, 1150, patch_threads(false, false), 24};
    static const PatchCost kHalfVelocity{12.7, 0.84, 0.457, 3.43, 1.0, 1.0, 1100, patch_threads(false, false), 24};
    static const PatchCost kPlain{7.71, 8.22, 1.31, 3.42, 0.96, 1.0, 750, patch_threads(true, false), 12};
    static const PatchCost kPlainTraction{22.0, 2.19, 0.872, 0.921, 0.129, 1.0, 750, patch_threads(true, true), 12};
    const bool walls = any_wall(p), traction = has_traction(p);
    const bool plain = p->storage == LBM_F64_PLAIN, half = p->storage == LBM_F16_SHIFTED;
    const int64_t nodes = int64_t(p->nx) * p->ny;
    const PatchCost& c = plain ? (traction ? kPlainTraction : kPlain)
                               : traction ? kTraction
                                          : half ? (walls ? kHalfVelocity : kHalf) : (walls ? kVelocity : kShifted);
    if (nodes > int64_t(c.side) * c.side) return PatchPlan{0, 0, 0};
    if (!walls)
        if (const PatchPlan* r = ranged_plan(p, p->storage, kForwardRanges)) return *r;
    // FP16 between velocity walls, all laws: this 1.00 to 1.01, model 1.10 to 1.17, pairs 1.14 to 1.24
    if (half && walls && !traction && nodes >= 365 * 365 && nodes < 400 * 400)
        return PatchPlan{3, std::min(16, p->nx), std::min(8, p->ny)};
    return patch_choice(p, c, traction ? 27 : 25, false);
}

// The rectangle of a walled grid that the multi-level kernels take (march_kernel; the patches
// take the rest): whole tiles and rows at least `levels` nodes away from every wall line.
struct Inner {
    int tile0, tile1, row0, row1;
};

Inner inner_rect(const lbm_params* p, int levels, int ph) {
    const bool perx = p->bc[LBM_XMIN] == LBM_PERIODIC, pery = p->bc[LBM_YMIN] == LBM_PERIODIC;
    Inner in{0, (p->nx + kTile - 1) / kTile, 0, p->ny};
    if (!perx) {
        in.tile0 = 1;
        in.tile1 = (p->nx - levels) / kTile;
    }
    if (!pery) {
        in.row0 = ph;
        in.row1 = p->ny - ph;
    }
    return in;
}

// Side of the patches around the rectangle.
constexpr int kRimPatch = 16;

// us per level of four levels by march_kernel (with patches around its rectangle on a grid with
// walls) and of two levels by the pairs, from what the launches do: the march wins where the
// rectangle fills its spans, and loses on narrow grids and where the patches beside it cost more
// than it saves.
//   march: launch (with patches) + iteration * (iterations of a workgroup) + node * (nodes of the
//          rectangle, repeated rows included) + rim * (nodes of the patches; between velocity walls,
//          with traction) + link * (traction links)
//   pairs: pair + tile * (nodes of whole tiles) + node2 * nodes + link2 * (links of velocity walls,
//          of traction walls)
// Nodes in millions, links in 10 000.  Fitted to 2 886 grids without records and 1 008 with a record
// of every level (seven wall layouts, widths of 64 to 4500, log-NH and Gent, uniform and per-node
// parameters).  On those and 2 886 more (svk, MR, Yeoh) the pick, which favours the march by 3 %, is
// 0.1 to 1.1 % slower than the better one on average; the march everywhere was 0.1 to 8 % slower, up to
// 1.98 times (FP64 MR, periodic, 64 columns; 257 columns between traction walls 1.79; FP16 Yeoh
// 1.47).  FP32 with the Lame-type laws has no entry: the march was 1.00 to 1.82 times as fast.
struct MarchCost {
    int storage, laws, records;
    double launch, iteration, node, rim[2], link;
    double pair, tile, node2, link2[2];
};
const MarchCost kMarchCosts[] = {
    {LBM_F64_PLAIN, kLameLaws, 0, 4.42, 0.94, 5.17, {52.56, 81.77}, 18.15, 6.49, 19.40, 20.72, {13.84, 28.44}},
    {LBM_F64_PLAIN, kInvariantLaws, 0, 4.54, 1.36, 3.45, {59.03, 96.04}, 35.17, 9.81, 21.69, 19.02, {12.15, 25.25}},
    {LBM_F16_SHIFTED, kLameLaws, 0, 2.41, 0.83, 3.46, {22.32, 25.04}, 5.56, 5.33, 15.88, 0.0, {5.62, 12.88}},
    {LBM_F16_SHIFTED, kLameLaws, 1, 2.49, 0.90, 3.32, {28.84, 33.98}, 3.30, 5.56, 19.47, 0.0, {6.67, 14.84}},
    {LBM_F16_SHIFTED, kInvariantLaws, 0, 2.45, 1.02, 4.20, {20.78, 28.06}, 8.70, 6.20, 16.63, 0.0, {5.27, 13.71}},
    {LBM_F16_SHIFTED, kInvariantLaws, 1, 2.14, 1.13, 3.30, {27.37, 36.27}, 6.30, 6.17, 20.33, 0.0, {5.80, 15.44}},
    {LBM_F32_SHIFTED, kInvariantLaws, 0, 1.97, 0.89, 5.23, {23.91, 28.44}, 8.85, 4.96, 13.38, 7.86, {7.19, 15.73}},
    {LBM_F32_SHIFTED, kInvariantLaws, 1, 2.17, 1.02, 5.23, {26.79, 32.92}, 6.99, 5.45, 17.50, 7.79, {8.11, 16.79}},
};

// Whether the march is expected to be faster than the pairs (march_kernel's grids with walls, and
// FP64 on periodic ones).
bool march_pays(const lbm_params* p, bool records) {
    const MarchCost* c = nullptr;
    for (const MarchCost& m : kMarchCosts)
        if (m.storage == p->storage && (m.laws >> p->material & 1) && m.records == int(records)) c = &m;
    if (!c) return true;
    const Inner in = inner_rect(p, kMarchMaxLevels, kRimPatch);
    const int rows = in.row1 - in.row0;
    int nspan, seg, nwg;
    FastDiv d;
    if (in.tile1 <= in.tile0 || rows < 1 ||
        !march_geometry(in.tile1 - in.tile0, march_tiles(p->storage == LBM_F64_PLAIN), rows, kMarchMaxLevels, nspan,
                        seg, nwg, d))
        return false;
    const int cus = compute_units(), halo = 2 * (kMarchMaxLevels - 1);
    const double nodes = double(p->nx) * p->ny;
    const double inner = double(rows) * (std::min(in.tile1 * kTile, p->nx) - in.tile0 * kTile);
    double links[2] = {0.0, 0.0};                // of velocity and of traction walls
    for (int e = 0; e < 4; ++e)
        if (p->bc[e] != LBM_PERIODIC) links[p->bc[e] == LBM_TRACTION] += edge_len(p->nx, p->ny, e);
    double march = c->iteration * ((nwg + cus - 1) / cus) * (seg + halo) + c->node * 1e-6 * inner * (seg + halo) / seg;
    if (any_wall(p)) march += c->launch + c->rim[links[1] > 0.0] * 1e-6 * (nodes - inner) + c->link * 1e-4 * links[1];
    const double tiles = double((p->nx + kTile - 1) / kTile) * kTile * p->ny;
    const double pairs = c->pair + c->tile * 1e-6 * tiles + c->node2 * 1e-6 * nodes +
                         1e-4 * (c->link2[0] * links[0] + c->link2[1] * links[1]);
    return march < 1.03 * pairs;
}

enum Route { kRouteStep, kRoutePair, kRouteMulti, kRouteRim, kRoutePatch };

// Nodes from which a grid with walls may take the march of its inner rectangle (FP32 log-NH, two
// traction-free pairs of edges, us per level, march and patches around it against patches alone
// and pairs: 1050^2 25 / 23 / 34, 1250^2 33 / 49 / 44; 2200^2 73 / - / 120; 4096^2 with per-node mu
// and lam 0.23 ms / - / 0.43).
constexpr int64_t kRimNodes = 1100 * 1100;

// What a call of lbm_advance forms once: the patch plan (levels = 0: none), and whether march_kernel
// takes the grid, without records and with a record of every level.
struct AdvancePlan {
    PatchPlan patch;
    bool march, replay;
};

AdvancePlan advance_plan(const lbm_params* p) {
    AdvancePlan a{patch_plan(p), false, false};
    if (a.patch.levels) return a;
    const bool walls = any_wall(p), f64 = p->storage == LBM_F64_PLAIN;
    const int64_t nodes = int64_t(p->nx) * p->ny;
    if (walls && (p->nx < 4 * kTile || p->ny < 4 * kTile)) return a;
    if (f64) {
        const int side = invariant_material(p) ? (walls ? 1250 : 1100) : (walls ? 850 : 750);
        a.march = nodes >= int64_t(side) * side && march_pays(p, false);
    } else if (walls) {
        a.march = nodes >= kRimNodes && march_pays(p, false);
        a.replay = nodes >= kRimNodes && march_pays(p, true);
    } else {
        a.march = nodes >= 1024 * 1024;
        a.replay = nodes >= 2048 * 2048;
    }
    return a;
}

// The launch that takes the next of `left` steps, and its levels (records: as lbm_advance's,
// from the next step on, or NULL).
Route advance_route(const lbm_params* p, const lbm_state* s, const AdvancePlan& plan, int64_t left,
                    void* const* records, PatchPlan& pl) {
    pl = PatchPlan{1, 0, 0};
    if (s->body_prev) return kRouteStep;
    if (plan.patch.levels) {
        pl = plan.patch;
        pl.levels = int(std::min<int64_t>(plan.patch.levels, left));
        return kRoutePatch;
    }
    const int64_t nodes = int64_t(p->nx) * p->ny;
    const bool walls = any_wall(p);
    if (left >= 2) {
        // march_kernel: without records (4 levels, or what is left without leaving a single step
        // over) and, in the shifted storages, with a record of every level; on a grid with walls
        // its inner rectangle, and the patches the rest
        const int levels = int(std::min<int64_t>(kMarchMaxLevels, left));
        int recs = 0;
        for (int t = 0; records && t < levels; ++t) recs += records[t] != nullptr;
        const bool go = recs == 0 ? plan.march && s->ustar && (levels > 2 || p->storage != LBM_F64_PLAIN)
                                  : plan.replay && recs == kMarchMaxLevels && !s->ustar;
        if (go) {
            pl.levels = recs == 0 && left - levels == 1 && levels > 2 ? levels - 1 : levels;
            pl.pw = pl.ph = kRimPatch;
            return walls ? kRouteRim : kRouteMulti;
        }
    }
    if (left >= 2 && (!walls || nodes >= 416 * 416)) {
        pl.levels = 2;
        return kRoutePair;
    }
    return kRouteStep;
}

// The patches of the whole grid, those whose region reaches a wall first (their traction solves
// take longer, and the first workgroups are dealt over the XCDs one by one; with only the ragged
// last row and column among the first, the far walls of a grid of whole patches came last and on
// one XCD: 384^2 FP64 Gent 23.3 -> 14.3 us per level, 512^2 FP32 log-NH 10.4 -> 8.5), or of the
// grid outside the rectangle `in`.
PatchMap patch_map(const lbm_params* p, const PatchPlan& pl, const Inner* in = nullptr) {
    PatchMap m{};
    m.pw = pl.pw;
    m.ph = pl.ph;
    auto add = [&](int x0, int y0, int x1, int y1) {
        if (x0 >= x1 || y0 >= y1) return;
        PatchRect& pr = m.rect[m.nrect++];
        pr.x0 = x0;
        pr.y0 = y0;
        pr.x1 = x1;
        pr.y1 = y1;
        pr.first = m.nwg;
        pr.npx = (x1 - x0 + pl.pw - 1) / pl.pw;
        pr.d_npx = fast_div(pr.npx);
        m.nwg += pr.npx * ((y1 - y0 + pl.ph - 1) / pl.ph);
    };
    const bool perx = p->bc[LBM_XMIN] == LBM_PERIODIC, pery = p->bc[LBM_YMIN] == LBM_PERIODIC;
    const int pw = pl.pw, ph = pl.ph;
    const int halo = pl.levels - 1;
    auto low = [halo](int w, int n) { return std::min((halo / w + 1) * w, n); };
    auto high = [halo](int w, int n, int lo) { return std::max(lo, (std::max(n - halo - w, 0) + w - 1) / w * w); };
    int x1 = perx ? 0 : low(pw, p->nx), y1 = pery ? 0 : low(ph, p->ny);
    int x2 = perx ? p->nx : std::min(high(pw, p->nx, x1), p->nx);
    int y2 = pery ? p->ny : std::min(high(ph, p->ny, y1), p->ny);
    if (in) {
        x1 = in->tile0 * kTile;
        x2 = std::min(in->tile1 * kTile, p->nx);
        y1 = in->row0;
        y2 = in->row1;
    }
    add(0, 0, p->nx, y1);
    add(0, y2, p->nx, p->ny);
    add(0, y1, x1, y2);
    add(x2, y1, p->nx, y2);
    if (!in) add(x1, y1, x2, y2);
    return m;
}

lbm_status patch_launch(const lbm_params* p, lbm_state* s, int64_t n, const PatchPlan& pl, const double* r,
                        const lbm_edge_data* edges, void* const* records, int record_planes, hipStream_t hs,
                        const Inner* in = nullptr) {
    PatchArgs a{};
    a.cm = make_common(p, s);
    a.cm.body_prev = nullptr;
    a.src = s->pop[s->cur];
    a.dst = s->pop[1 - s->cur];
    a.ustar = s->ustar;
    a.levels = pl.levels;
    a.rec_planes = record_planes;
    for (int t = 0; t <= pl.levels; ++t) {
        a.r[t] = r[t];
        for (int k = 0; k < 2; ++k) a.fb[t][k] = float(r[t] * a.cm.b0[k]);
    }
    for (int t = 0; t < pl.levels; ++t) {
        if ((n + 1 + t) % kUstarBlock == 0) a.fold = t + 1;
        a.rec[t] = records ? records[t] : nullptr;
        if (!edges) continue;
        for (int e = 0; e < 4; ++e) {
            for (int k = 0; k < 2; ++k) a.value[t][e][k] = edges[t].value[e][k];
            a.field[t][e] = edges[t].field[e];
        }
    }
    a.map = patch_map(p, pl, in);
    if (launch_patch(a, hs) != hipSuccess) return LBM_ERR_LAUNCH;
    if (!in) s->cur = 1 - s->cur;
    return LBM_OK;
}

// The plan of patch_adj_kernel (us per level, patches against the pairs and single steps,
// per-node mu and lam, gradients of mu, lam and b):
//   FP32 periodic  128^2 2.6 / 3.6, 256^2 3.4 / 3.7, 512^2 7.6 / 9.9, 850^2 18.4 / 23.0,
//                  1024^2 32 / 29
//   FP32 walls     128^2 5.0 / 18.1, 256^2 5.9 / 22.4, 512^2 10.2 / 26.6, 1024^2 37 / 48,
//                  1448^2 74 / 82 (between two velocity walls 1050^2 37.5 / 39.9, 1448^2 72 / 70)
//   FP64 periodic  64^2 2.6 / 4.9, 256^2 4.5 / 6.0, 512^2 11.9 / 17.5, 1024^2 62 / 60
//   FP64 walls     64^2 6.8 / 22.1, 256^2 9.0 / 28.4, 700^2 38 / 51, 1024^2 86 / 82 (between two
//                  velocity walls 512^2 18 / 27, 850^2 61 / 55)
// The invariant-based laws differentiate their stress in forward mode, whose registers leave
// fewer wavefronts; their halo work costs more (Gent, FP32 periodic: 512^2 13.0 / 14.8,
// 1024^2 47 / 43; walls 512^2 16.4 / 35.7, 1024^2 57 / 65; FP64 256^2 8.2 / 8.4, 512^2 29 / 30,
// walls 512^2 39 / 53, 1024^2 154 / 134).
PatchPlan patch_adj_plan(const lbm_params* p) {
    static const PatchCost kShifted{24.6, 2.20, 0.585, 67.3, 0.83, 1.0, 900, kPatchAdjThreads, 24};
    static const PatchCost kShiftedWalls{25.9, 1.19, 0.123, 15.5, 0.436, 1.0, 1300, kPatchAdjThreads, 24};
    static const PatchCost kPlain{6.58, 0.230, 0.0297, 2.43, 0.626, 1.0, 800, kPatchAdjThreads, 12};
    static const PatchCost kPlainWalls{2.01, 5.73, 0.732, 1.65, 1.0, 1.0, 780, kPatchAdjThreads, 12};
    static const PatchCost kInvShifted{3.18, 4.20, 0.808, 0.66, 0.54, 1.0, 920, kPatchAdjThreads, 24};
    static const PatchCost kInvShiftedWalls{3.09, 37.5, 4.19, 6.26, 0.55, 1.0, 1030, kPatchAdjThreads, 24};
    static const PatchCost kInvPlain{10.8, 20.7, 2.81, 1.91, 0.90, 1.0, 420, kPatchAdjThreads, 12};
    static const PatchCost kInvPlainWalls{3.77, 13.0, 1.50, 2.38, 1.0, 1.0, 700, kPatchAdjThreads, 12};
    const bool walls = any_wall(p), plain = p->storage == LBM_F64_PLAIN, traction = has_traction(p);
    const PatchCost& c = invariant_material(p)
                             ? (plain ? (walls ? kInvPlainWalls : kInvPlain) : (walls ? kInvShiftedWalls : kInvShifted))
                             : (plain ? (walls ? kPlainWalls : kPlain) : (walls ? kShiftedWalls : kShifted));
    // Smaller limits (patches / pairs, over the better one).  The FP64 kernels of MR and Yeoh keep up
    // to 99 of their registers in scratch memory: periodic MR 128^2 1.00 / 1.03, 180^2 1.09 / 1.00,
    // 340^2 1.44 / 1.00.  FP64 between velocity walls (a channel and four walls): MR 580^2 1.00 /
    // 1.02, 640^2 1.05 / 1.00; Yeoh 580^2 1.00 / 1.08, 700^2 1.12 / 1.00; Gent 640^2 1.00 / 1.01,
    // 700^2 1.07 / 1.00.  FP32 between velocity walls: MR and Yeoh 750^2 1.00 / 1.04, 820^2 1.05 /
    // 1.00, 1000^2 1.17 / 1.00; the Lame-type laws 1099^2 1.00 / 1.10, 1200^2 1.08 / 1.00.
    const bool mr = p->material == LBM_MR, yeoh = p->material == LBM_YEOH;
    int side = c.side;
    if (plain && !walls && mr) side = 150;
    if (plain && walls && !traction && invariant_material(p)) side = mr ? 590 : yeoh ? 630 : 690;
    if (!plain && walls && !traction) side = mr || yeoh ? 800 : invariant_material(p) ? side : 1130;
    const int64_t nodes = int64_t(p->nx) * p->ny;
    if (nodes > int64_t(side) * side) return PatchPlan{0, 0, 0};
    if (!walls)
        if (const PatchPlan* r = ranged_plan(p, plain ? LBM_F64_PLAIN : LBM_F32_SHIFTED, kAdjointRanges)) return *r;
    return patch_choice(p, c, 25, walls);
}

lbm_status patch_adj_launch(const lbm_params* p, const lbm_state* fwd, lbm_adj_state* adj, int64_t m,
                            const PatchPlan& pl, const double* r, const lbm_edge_data* edges,
                            const void* const* records, hipStream_t hs) {
    PatchAdjArgs a{};
    a.cm = make_common(p, fwd);
    a.src = adj->adj[adj->cur];
    a.dst = adj->adj[1 - adj->cur];
    a.levels = pl.levels;
    a.map = patch_map(p, pl);
    for (int t = 0; t < pl.levels; ++t) {
        if ((m - t) % kGradBlock == 0) a.fold = t + 1;
        a.rec[t] = records[t];
        a.r[t] = r[t];
        if (!edges) continue;
        for (int e = 0; e < 4; ++e) {
            for (int k = 0; k < 2; ++k) a.value[t][e][k] = edges[t].value[e][k];
            a.field[t][e] = edges[t].field[e];
        }
    }
    a.g_mu = adj->g_mu;
    a.g_lam = adj->g_lam;
    a.g_body = adj->g_body;
    a.gsum = adj->gsum;
    a.pmask = adj->nprobe > 0 ? adj->probe_mask : nullptr;
    a.pfield = adj->nprobe > 0 ? adj->probe_field : nullptr;
    a.probe_weight = a.cm.dt;                    // every level of the launch is below N
    if (launch_patch_adjoint(a, hs) != hipSuccess) return LBM_ERR_LAUNCH;
    adj->cur = 1 - adj->cur;
    return LBM_OK;
}

}  // namespace

extern "C" {

int lbm_advance_levels(const lbm_params* p, const lbm_state* s, int64_t left, void* const* records) {
    if (lbm_check_params(p) != LBM_OK || !s || left < 1) return 0;
    PatchPlan pl;
    advance_route(p, s, advance_plan(p), left, records, pl);
    return pl.levels;
}

lbm_status lbm_advance(const lbm_params* p, lbm_state* s, int64_t n, int64_t count, const double* r,
                       const lbm_edge_data* edges, void* const* records, int record_planes, void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if ((st = check_state(p, s, false)) != LBM_OK) return st;
    if (count < 0 || !r) return LBM_ERR_ARG;
    if (any_wall(p) && (!edges || !s->aux)) return LBM_ERR_ARG;
    if (records && record_planes != 6 && record_planes != 4) return LBM_ERR_ARG;
    const AdvancePlan plan = advance_plan(p);
    for (int64_t i = 0; i < count;) {
        const int64_t left = count - i;
        void* const* rec = records ? records + i : nullptr;
        const lbm_edge_data* ed = edges ? edges + i : nullptr;
        PatchPlan pl;
        switch (advance_route(p, s, plan, left, rec, pl)) {
            case kRoutePatch: st = patch_launch(p, s, n + i, pl, r + i, ed, rec, record_planes, (hipStream_t)stream); break;
            case kRouteRim: {
                const Inner in = inner_rect(p, pl.levels, pl.ph);
                void* const* all = rec && rec[0] ? rec : nullptr;
                st = patch_launch(p, s, n + i, pl, r + i, ed, all, record_planes, (hipStream_t)stream, &in);
                if (st == LBM_OK)
                    st = march_launch(p, s, n + i, pl.levels, r + i + 1, all, record_planes, in.tile0, in.tile1, in.row0,
                                      in.row1, (hipStream_t)stream);
                if (st == LBM_OK) s->cur = 1 - s->cur;
                break;
            }
            case kRouteMulti:
                st = lbm_step_multi(p, s, n + i, pl.levels, r + i + 1, rec && rec[0] ? rec : nullptr, record_planes,
                                    stream);
                break;
            case kRoutePair:
                st = lbm_step2(p, s, n + i, r[i], r[i + 1], r[i + 2], ed, ed ? ed + 1 : nullptr, rec ? rec[0] : nullptr,
                               rec ? rec[1] : nullptr, stream);
                break;
            default: st = lbm_step(p, s, n + i, r[i], r[i + 1], ed, rec ? rec[0] : nullptr, stream); break;
        }
        if (st != LBM_OK) return st;
        i += pl.levels;
    }
    return LBM_OK;
}

static lbm_status recover_common(const lbm_params* p, const lbm_state* s, double r_n, void* out,
                                 RecoverArgs& a, bool need_ustar = false) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if ((st = check_state(p, s, need_ustar)) != LBM_OK) return st;
    if (!out) return LBM_ERR_ARG;
    a = RecoverArgs{};
    a.cm = make_common(p, s);
    a.pop = s->pop[s->cur];
    a.ustar = s->ustar;
    a.r_n = r_n;
    a.out = out;
    return LBM_OK;
}

lbm_status lbm_displacement(const lbm_params* p, const lbm_state* s, double r_n, double* u_out, void* stream) {
    RecoverArgs a;
    lbm_status st = recover_common(p, s, r_n, u_out, a, true);
    if (st != LBM_OK) return st;
    return launched(launch_displacement(a, (hipStream_t)stream));
}

lbm_status lbm_moments(const lbm_params* p, const lbm_state* s, double r_n, double* U_out, void* stream) {
    RecoverArgs a;
    lbm_status st = recover_common(p, s, r_n, U_out, a);
    if (st != LBM_OK) return st;
    return launched(launch_moments(a, (hipStream_t)stream));
}

lbm_status lbm_record_state(const lbm_params* p, const lbm_state* s, double r_n, void* record, void* stream) {
    RecoverArgs a;
    lbm_status st = recover_common(p, s, r_n, record, a);
    if (st != LBM_OK) return st;
    return launched(launch_record(a, (hipStream_t)stream));
}

lbm_status lbm_stress(const lbm_params* p, const lbm_state* s, double r_n, double* P_out, double* sigma_out,
                      void* stream) {
    RecoverArgs a;
    lbm_status st = recover_common(p, s, r_n, P_out, a);
    if (st != LBM_OK) return st;
    a.out2 = sigma_out;
    return launched(launch_stress(a, (hipStream_t)stream));
}

lbm_status lbm_diagnostics(const lbm_params* p, const lbm_state* s, double r_n, double* out, void* scratch,
                           void* stream) {
    RecoverArgs a;
    lbm_status st = recover_common(p, s, r_n, out, a);
    if (st != LBM_OK) return st;
    if (!scratch) return LBM_ERR_ARG;
    a.scratch = scratch;
    return launched(launch_diagnostics(a, (hipStream_t)stream));
}

lbm_status lbm_diagnostics_noalloc(const lbm_params* p, const lbm_state* s, double r_n, double* out,
                                   void* stream) {
    if (p && lbm_diag_scratch_bytes(p) > sizeof(scratch)) return LBM_ERR_UNSUPPORTED;
    void* ptr = nullptr;
    const lbm_status st = scratch_address(&ptr);
    if (st != LBM_OK) return st;
    return lbm_diagnostics(p, s, r_n, out, ptr, stream);
}

lbm_status lbm_adjoint_step(const lbm_params* p, const lbm_state* fwd, lbm_adj_state* adj, int64_t m,
                            double r_m, const lbm_edge_data* at_half, const void* record_m, void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if (!fwd || !adj || !adj->adj[0] || !adj->adj[1] || !record_m) return LBM_ERR_ARG;
    if (adj->cur != 0 && adj->cur != 1) return LBM_ERR_ARG;
    if (has_traction(p) && !adj->aux) return LBM_ERR_ARG;
    if (adj->nprobe < 0 || (adj->nprobe > 0 && (!adj->probe || !adj->ubar))) return LBM_ERR_ARG;
    if (m < 0 || m > adj->nsteps) return LBM_ERR_ARG;
    if (any_wall(p) && !at_half) return LBM_ERR_ARG;
    if (p->storage != LBM_F64_PLAIN && (adj->g_mu || adj->g_lam || adj->g_body) && !adj->gsum)
        return LBM_ERR_ARG;
    AdjArgs a{};
    a.cm = make_common(p, fwd);
    a.src = adj->adj[adj->cur];
    a.dst = adj->adj[1 - adj->cur];
    a.record = record_m;
    a.g_mu = adj->g_mu;
    a.g_lam = adj->g_lam;
    a.g_body = adj->g_body;
    a.gsum = adj->gsum;
    a.fold = m % kGradBlock == 0;
    a.aux = adj->aux;
    a.r_m = r_m;
    a.ed = make_edges(at_half);
    a.probe = adj->probe;
    a.ubar = adj->ubar;
    a.nprobe = adj->nprobe;
    a.probe_weight = (m == adj->nsteps ? 0.5 : 1.0) * a.cm.dt;
    if (adj->nprobe > 0 && adj->probe_mask && adj->probe_field) {
        a.pmask = adj->probe_mask;
        a.pfield = adj->probe_field;
    }
    if (launch_adjoint(a, (hipStream_t)stream) != hipSuccess) return LBM_ERR_LAUNCH;
    adj->cur = 1 - adj->cur;
    return LBM_OK;
}

size_t lbm_probe_mask_bytes(const lbm_params* p) {
    if (lbm_check_params(p) != LBM_OK) return 0;
    return size_t((p->nx + kTile - 1) / kTile) * size_t(p->ny) * sizeof(uint64_t);
}

lbm_status lbm_adjoint_probe_table(const lbm_params* p, const lbm_adj_state* adj, uint64_t* mask, double* field,
                                   void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if (!adj || !mask || !field) return LBM_ERR_ARG;
    if (adj->nprobe < 0 || (adj->nprobe > 0 && (!adj->probe || !adj->ubar))) return LBM_ERR_ARG;
    const Common cm = make_common(p, nullptr);
    return launched(launch_probe_table(cm, adj->probe, adj->ubar, adj->nprobe, mask, field, (hipStream_t)stream));
}

lbm_status lbm_adjoint_step2(const lbm_params* p, const lbm_state* fwd, lbm_adj_state* adj, int64_t m, double r_m,
                             double r_mm1, const lbm_edge_data* at_half, const lbm_edge_data* at_half_prev,
                             const void* record_m, const void* record_mm1, const uint64_t* mask,
                             const double* field, void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if (!fwd || !adj || !adj->adj[0] || !adj->adj[1] || !record_m || !record_mm1) return LBM_ERR_ARG;
    if (any_wall(p) && (!at_half || !at_half_prev || !adj->aux)) return LBM_ERR_ARG;
    if (adj->cur != 0 && adj->cur != 1) return LBM_ERR_ARG;
    if (adj->nprobe < 0 || (adj->nprobe > 0 && (!adj->probe || !adj->ubar || !mask || !field))) return LBM_ERR_ARG;
    if (m < 1 || m >= adj->nsteps) return LBM_ERR_ARG;
    if (p->storage != LBM_F64_PLAIN && (adj->g_mu || adj->g_lam || adj->g_body) && !adj->gsum)
        return LBM_ERR_ARG;
    Adj2Args a{};
    a.cm = make_common(p, fwd);
    a.src = adj->adj[adj->cur];
    a.dst = adj->adj[1 - adj->cur];
    a.rec1 = record_m;
    a.rec2 = record_mm1;
    a.g_mu = adj->g_mu;
    a.g_lam = adj->g_lam;
    a.g_body = adj->g_body;
    a.gsum = adj->gsum;
    a.fold1 = m % kGradBlock == 0;
    a.fold2 = (m - 1) % kGradBlock == 0;
    a.nstrip = (p->nx + kTile - 1) / kTile;
    {
        const int nblk = (p->ny + kPairRows - 1) / kPairRows;
        a.map = pair_map(a.nstrip, nblk, 0, a.nstrip, 0, nblk);
    }
    a.r1 = r_m;
    a.r2 = r_mm1;
    a.pmask = adj->nprobe > 0 ? mask : nullptr;
    a.pfield = adj->nprobe > 0 ? field : nullptr;
    a.probe_weight = a.cm.dt;                    // levels m and m - 1 are below N
    a.aux = adj->aux;
    if (any_wall(p)) {
        a.ed1 = make_edges(at_half);
        a.ed2 = make_edges(at_half_prev);
    }
    if (launch_adjoint2(a, (hipStream_t)stream) != hipSuccess) return LBM_ERR_LAUNCH;
    adj->cur = 1 - adj->cur;
    return LBM_OK;
}

lbm_status lbm_adjoint_step_multi(const lbm_params* p, const lbm_state* fwd, lbm_adj_state* adj, int64_t m,
                                  int levels, const double* r, const void* const* records, const uint64_t* mask,
                                  const double* field, void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if (!fwd || !adj || !adj->adj[0] || !adj->adj[1] || !r || !records) return LBM_ERR_ARG;
    if (levels < 2 || levels > kMarchMaxLevels) return LBM_ERR_ARG;
    if (adj->cur != 0 && adj->cur != 1) return LBM_ERR_ARG;
    if (adj->nprobe < 0 || (adj->nprobe > 0 && (!adj->probe || !adj->ubar || !mask || !field))) return LBM_ERR_ARG;
    if (m - (levels - 1) < 0 || m >= adj->nsteps) return LBM_ERR_ARG;
    for (int t = 0; t < levels; ++t)
        if (!records[t]) return LBM_ERR_ARG;
    if (any_wall(p) || p->storage == LBM_F64_PLAIN) return LBM_ERR_UNSUPPORTED;
    if ((adj->g_mu || adj->g_lam || adj->g_body) && !adj->gsum) return LBM_ERR_ARG;
    MarchAdjArgs a{};
    a.cm = make_common(p, fwd);
    a.src = adj->adj[adj->cur];
    a.dst = adj->adj[1 - adj->cur];
    for (int t = 0; t < levels; ++t) {
        a.rec[t] = records[t];
        a.r[t] = r[t];
        a.fold[t] = (m - t) % kGradBlock == 0;
    }
    a.g_mu = adj->g_mu;
    a.g_lam = adj->g_lam;
    a.g_body = adj->g_body;
    a.gsum = adj->gsum;
    a.pmask = adj->nprobe > 0 ? mask : nullptr;
    a.pfield = adj->nprobe > 0 ? field : nullptr;
    a.probe_weight = a.cm.dt;                    // every level of the pass is below N
    a.levels = levels;
    if (!march_geometry((p->nx + kTile - 1) / kTile, kMarchTiles, p->ny, levels, a.nspan, a.seg, a.nwg, a.d_nspan))
        return LBM_ERR_UNSUPPORTED;
    if (launch_march_adjoint(a, (hipStream_t)stream) != hipSuccess) return LBM_ERR_LAUNCH;
    adj->cur = 1 - adj->cur;
    return LBM_OK;
}

lbm_status lbm_adjoint_advance(const lbm_params* p, const lbm_state* fwd, lbm_adj_state* adj, int64_t m, int64_t count,
                               const double* r, const lbm_edge_data* edges, const void* const* records,
                               void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if (!fwd || !adj || !adj->adj[0] || !adj->adj[1] || !r || !records) return LBM_ERR_ARG;
    if (adj->cur != 0 && adj->cur != 1) return LBM_ERR_ARG;
    if (adj->nprobe < 0 || (adj->nprobe > 0 && (!adj->probe || !adj->ubar))) return LBM_ERR_ARG;
    if (count < 0 || m - (count - 1) < 0 || m > adj->nsteps) return LBM_ERR_ARG;
    for (int64_t i = 0; i < count; ++i)
        if (!records[i]) return LBM_ERR_ARG;
    const bool walls = any_wall(p), plain = p->storage == LBM_F64_PLAIN;
    if (walls && (!edges || !adj->aux)) return LBM_ERR_ARG;
    if (!plain && (adj->g_mu || adj->g_lam || adj->g_body) && !adj->gsum) return LBM_ERR_ARG;
    // the kernels of several levels take the probe sources from the probe table
    const bool table = adj->nprobe == 0 || (adj->probe_mask && adj->probe_field);
    const PatchPlan plan = patch_adj_plan(p);
    for (int64_t i = 0; i < count;) {
        const int64_t left = count - i, lm = m - i;
        const lbm_edge_data* ed = edges ? edges + i : nullptr;
        PatchPlan pl = plan;
        pl.levels = int(std::min<int64_t>(pl.levels, left));
        const int multi = invariant_material(p) ? 3 : 4;
        int done = 1;
        if (!table || lm == adj->nsteps) {
            st = lbm_adjoint_step(p, fwd, adj, lm, r[i], ed, records[i], stream);
        } else if (pl.levels) {
            done = pl.levels;
            st = patch_adj_launch(p, fwd, adj, lm, pl, r + i, ed, records + i, (hipStream_t)stream);
        } else if (!walls && !plain && left >= multi && int64_t(p->nx) * p->ny >= 2048 * 2048) {
            done = multi;
            st = lbm_adjoint_step_multi(p, fwd, adj, lm, multi, r + i, records + i, adj->probe_mask, adj->probe_field,
                                        stream);
        } else if (left >= 2) {
            done = 2;
            st = lbm_adjoint_step2(p, fwd, adj, lm, r[i], r[i + 1], ed, ed ? ed + 1 : nullptr, records[i],
                                   records[i + 1], adj->probe_mask, adj->probe_field, stream);
        } else {
            st = lbm_adjoint_step(p, fwd, adj, lm, r[i], ed, records[i], stream);
        }
        if (st != LBM_OK) return st;
        i += done;
    }
    return LBM_OK;
}

lbm_status lbm_adjoint_init(const lbm_params* p, const lbm_state* fwd, lbm_adj_state* adj, const double* v0,
                            const double* u0, const double* Fbar, double r0, double* g_v0, void* stream) {
    lbm_status st = lbm_check_params(p);
    if (st != LBM_OK) return st;
    if (!fwd || !adj || !adj->adj[0] || !adj->adj[1] || !v0 || !g_v0) return LBM_ERR_ARG;
    double F0[4];
    if (!predeformation(Fbar, F0)) return LBM_ERR_ARG;
    if (adj->cur != 0 && adj->cur != 1) return LBM_ERR_ARG;
    if (adj->nprobe < 0 || (adj->nprobe > 0 && (!adj->probe || !adj->ubar))) return LBM_ERR_ARG;
    AdjInitArgs a{};
    a.cm = make_common(p, fwd);
    a.lam0 = adj->adj[adj->cur];
    a.scratch = adj->adj[1 - adj->cur];
    a.v0 = v0;
    a.u0 = u0;
    for (int k = 0; k < 4; ++k) a.Fbar[k] = F0[k];
    a.r0 = r0;
    a.g_mu = adj->g_mu;
    a.g_lam = adj->g_lam;
    a.g_body = adj->g_body;
    a.g_v0 = g_v0;
    a.probe = adj->probe;
    a.ubar = adj->ubar;
    a.nprobe = adj->nprobe;
    return launched(launch_adjoint_init(a, (hipStream_t)stream));
}

const char* lbm_status_string(lbm_status st) {
    switch (st) {
        case LBM_OK: return "ok";
        case LBM_ERR_ARG: return "invalid argument";
        case LBM_ERR_UNSUPPORTED: return "unsupported combination";
        case LBM_ERR_CFL: return "lattice speed too low for the material (bulk: P-wave speed above c/2; traction walls: wall modes grow, see lbm_wall_mode_growth)";
        case LBM_ERR_LAUNCH: return "kernel launch failed";
        default: return "unknown status";
    }
}

const char* lbm_version(void) { return "tlvlbm 0.1 (gfx950)"; }

}  // extern "C"
