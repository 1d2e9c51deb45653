// capi.hip -- plans, workspace layout, the backward time loop and the C ABI
// of include/bsde.h (arXiv:1909.13560, Section 3.1 steps 1-3).
//
// Workspace layout (caller-owned device memory):
//   per instance: ring of K+1 slots; layer n lives in slot n mod (K+1); a slot
//                 is two planes of pad_l ghost, n_x grid and pad_r ghost
//                 elements: (y, z), then a spline plane (16 bytes each in
//                 FP64, 8 in FP32), so each launch writes whole planes.  The
//                 spline plane holds the B-spline coefficients (c_y, c_z) for
//                 the fused sweep in FP64 (located nodes in LDS windows too) and
//                 the one-launch exact sweep, the second derivatives (M_y, M_z)
//                 for the other kernels and the FP32 form; the FP32 form adds a third plane, the rounding
//                 residuals (e_y, e_z) of the stored values (error feedback)
//   per instance: per-wavefront Picard counters (statistics)
//   totals      : 4 x u64 reduced statistics
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/bsde.h"
#include "kernels.h"
#include "plan_math.h"
#include "sweep2d.h"

namespace {

using bsde::kBlock;

enum SweepPath { PATH_FUSED = 0, PATH_DIRECT = 1, PATH_GATHER = 3, PATH_TOEPLITZ = 4 };

struct SweepConfig {
    int path = PATH_DIRECT;
    int P = 2;
    int G = 1;       // node groups per tile (fused path), or blocks per tile
    size_t lds = 0;  // dynamic LDS bytes; 0 marks a fused shape that does not fit
    int W = 4;       // wavefronts along the points of a tile (fused path)
};

constexpr int kMaxP = 4;
constexpr int kMinTile = 64;  // smallest tile of any kernel shape (the tile maps are sized for it)

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct Instance {
    bsde_problem pb;
    int K, nx, pad_l, pad_r, npad;
    double dx, dt, h0;
    int m_min, m_max;
    int reach = 0;  // cells a node lies from its point at most, as reported
    double R;
    bool f32;
    bool gather;  // state-dependent forward coefficients: nodes located per point
    bool located = false;  // of these, with node windows that the fused sweep can stage (FP64)
    bool exact;   // exact Gaussian expectations (banded Toeplitz operators)
    std::vector<double> ctab;          // tabulated forward coefficients (host copy)
    const double *d_ctab = nullptr;    // and on the device
    bsde::GaussBand band[bsde::kMaxOrder + 1];  // per layer j (exact)
    int toep_off[bsde::kMaxOrder + 1] = {};       // band j in the device table
    const double *toep_w = nullptr;
    // exact expectations on B-spline coefficients: bands and end corrections
    std::vector<double> ex_band;
    std::vector<double2> ex_corr;
    int ex_boff[bsde::kMaxOrder + 1] = {}, ex_loff[bsde::kMaxOrder + 1] = {}, ex_roff[bsde::kMaxOrder + 1] = {};
    int ex_nl[bsde::kMaxOrder + 1] = {}, ex_nr[bsde::kMaxOrder + 1] = {};
    int ex_il[bsde::kMaxOrder + 1] = {}, ex_ir[bsde::kMaxOrder + 1] = {};
    const double *d_ex_band = nullptr;
    const double2 *d_ex_corr = nullptr;
    const bsde::NodeRecB *d_recb = nullptr;
    int2 *d_addr = nullptr;  // FP64 fused sweep: node addresses of the bound shape (in its group's)
    int steps;  // layers computed: N - K - n_stop + 1
    bsde::DriverParams drv;
    std::vector<int> m, win_lo, win_hi;
    std::vector<double> B, C, D, phi, cfy, cfz, cz, cy, cyz, dw;
    bsde::NodeTable dtab{};
    size_t ring_off, fin_off, stat_off;
    int nwaves;  // per-wave statistics slots (P = 1 has the most waves)
    int group;
};

// Instances sharing precision, driver and kernel shape: one launch per step
// serves all of them.  Members are sorted by their number of steps (most
// first), so the instances active at step s are a prefix.
struct Group {
    bool f32 = false;
    int driver = 0;
    SweepConfig cfg;
    std::vector<int> members;
    std::vector<int> tile_prefix, spline_prefix;  // members + 1 entries
    int *d_tile_inst = nullptr;    // grid tile -> instance (sized for kMinTile)
    int2 *d_addr = nullptr;        // FP64: the members' node addresses, one after the other
    int *d_spline_inst = nullptr;  // spline tile -> instance
    int max_steps = 0;
    size_t part_off = 0;  // partial sums in the workspace: Toeplitz splits or direct chunks
    int dchunks = 0;      // direct sweep: node chunks per tile in that layout (0: no region)
    int active(int s, const std::vector<Instance> &inst) const
    {
        int lo = 0, hi = (int)members.size();  // members[0..lo) have steps > s
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (inst[members[mid]].steps > s)
                lo = mid + 1;
            else
                hi = mid;
        }
        return lo;
    }
};

// A two-dimensional instance (tensor grid).
struct Instance2 {
    bsde_problem pb;
    bool f32 = false;  // FP32 form: float ring planes with residual planes
    int K, n0, n1, pad0, pad0r, pad1, pad1r, npad0, npad1;
    int win;  // LDS window columns of the sweep kernel
    // B-spline form (FP64, natural spline): its tables
    bool bspline = false;
    int nl = 0, nr = 0, spread = 0;
    std::vector<bsde::Row2B> rowsb;
    std::vector<bsde::Node2B> nodesb;
    std::vector<double4> corr_l, corr_r;
    const bsde::Row2B *d_rowsb = nullptr;
    const bsde::Node2B *d_nodesb = nullptr;
    const double4 *d_corr_l = nullptr, *d_corr_r = nullptr;
    double lin_y = 0.0, lin_z1 = 0.0, lin_z2 = 0.0;
    int planes() const { return bspline ? bsde::kPlanes2B : f32 ? 15 : 12; }
    size_t plane, tmp_off = 0;
    int reach = 0;  // widest node offset
    double dx0, dx1, dt, h0, R;
    std::vector<bsde::Node2Row> rows;
    std::vector<bsde::Node2> nodes;
    std::vector<int> m1;
    const bsde::Node2Row *d_rows = nullptr;
    const bsde::Node2 *d_nodes = nullptr;
    const int *d_m1 = nullptr;
    size_t ring_off, fin_off, stat_off;
    int nwaves;
};

}  // namespace

// A captured backward solve (hipGraph) for one set of buffers.
struct GraphEntry {
    const void *ws = nullptr;
    std::vector<bsde_io> io;
    bool stats = false;
    hipGraphExec_t exec = nullptr;
    unsigned long long last_use = 0;
};

constexpr int kMaxGraphs = 4;

struct bsde_plan_s {
    int device = 0;
    size_t max_lds = 65536;
    std::vector<Instance> inst;
    std::vector<Group> groups;
    std::vector<Instance2> inst2;       // two-dimensional plans (all instances d = 2)
    bsde::SplineFilter filter2;
    std::vector<bsde::InstDesc> desc;       // host copy of the descriptors
    bsde::InstDesc *d_desc = nullptr;
    void *d_tables = nullptr;
    size_t ws_bytes = 0;
    size_t stats_off = 0, stats_bytes = 0;  // statistics region of the workspace
    size_t totals_off = 0;                  // 3 u64 per instance + non-finite count
    bsde::PcrCoef pcr_base;                 // kappa, inv_b (s6 set per instance)
    bool use_graphs = true;
    std::mutex mu;                          // guards the graph cache
    hipStream_t capture_stream = nullptr;
    std::vector<GraphEntry> graphs;
    unsigned long long clock = 0;
    void drop_graphs()
    {
        for (GraphEntry &g : graphs) (void)hipGraphExecDestroy(g.exec);
        graphs.clear();
    }
};

namespace {

// Static workspace of bsde_solve_batched_static: a file-scope device array
// (each GPU the library runs on holds its own copy until the process ends).
// In host code `scratch` names a host-side stand-in, not a device address:
// the kernels get the address hipGetSymbolAddress returns for the device,
// looked up once per device at plan time (set-up) and kept in
// g_scratch_addr.
constexpr size_t kStaticWorkspaceBytes = BSDE_STATIC_WORKSPACE_BYTES;
__device__ __align__(256) unsigned char scratch[kStaticWorkspaceBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char *g_scratch_addr[kMaxDevices];

// Device address of `scratch` on device dev (the current device).
bsde_status static_workspace(int dev, char **out)
{
    if (dev < 0 || dev >= kMaxDevices) return BSDE_EDEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return BSDE_EDEVICE;
        g_scratch_addr[dev] = static_cast<char *>(p);
    }
    *out = g_scratch_addr[dev];
    return BSDE_OK;
}

#define HIP_OK(x)                                  \
    do {                                           \
        hipError_t e_ = (x);                       \
        if (e_ != hipSuccess) return BSDE_EDEVICE; \
    } while (0)

bool valid_problem(const bsde_problem &p)
{
    if (p.d != 1 && p.d != 2) return false;
    static_assert(bsde::kMaxK <= bsde::kMaxOrder, "descriptor window arrays hold K + 1 entries");
    if (p.k_y < 1 || p.k_y > bsde::kMaxK || p.k_z < 1 || p.k_z > bsde::kMaxK) return false;
    const int K = std::max(p.k_y, p.k_z);
    if (p.n_t < K || !(p.T > 0.0) || !std::isfinite(p.T)) return false;
    if (p.L < 1 || p.L > bsde::kMaxL) return false;
    if (p.n_x[0] < 4 || !(p.x_max[0] > p.x_min[0])) return false;
    if (!std::isfinite(p.x_min[0]) || !std::isfinite(p.x_max[0])) return false;
    if (p.tab_steps == 0) {
        if (p.coef_tab) return false;
        if (!std::isfinite(p.drift[0]) || !std::isfinite(p.vol[0][0])) return false;
        if (!std::isfinite(p.drift_x) || !std::isfinite(p.vol_x)) return false;
        // the diffusion coefficient b(x) = vol + vol_x x must be positive over the grid
        if (!(p.vol[0][0] + p.vol_x * p.x_min[0] > 0.0) ||
            !(p.vol[0][0] + p.vol_x * p.x_max[0] > 0.0))
            return false;
    } else {
        // tabulated coefficients: d = 1, one row or one per step, a finite,
        // b finite and positive, the affine slopes unused (0)
        if (p.d != 1 || !p.coef_tab || (p.tab_steps != 1 && p.tab_steps != p.n_t)) return false;
        if (p.drift_x != 0.0 || p.vol_x != 0.0) return false;
        const size_t nx = (size_t)p.n_x[0];
        for (int r = 0; r < p.tab_steps; ++r) {
            const double *ta = p.coef_tab + (size_t)2 * r * nx, *tb = ta + nx;
            for (size_t i = 0; i < nx; ++i)
                if (!std::isfinite(ta[i]) || !std::isfinite(tb[i]) || !(tb[i] > 0.0)) return false;
        }
    }
    if (p.driver < BSDE_DRIVER_LINEAR || p.driver > BSDE_DRIVER_EXP) return false;
    if (p.picard_max < 1) return false;
    if (p.prec != BSDE_FP64 && p.prec != BSDE_FP32_COMP) return false;
    if (p.n_stop < 0 || p.n_stop > p.n_t - K) return false;
    if (p.z_form != BSDE_ZFORM_EZ && p.z_form != BSDE_ZFORM_YDW) return false;
    if (p.quad != BSDE_QUAD_GH && p.quad != BSDE_QUAD_EXACT) return false;
    if (p.interp != BSDE_INTERP_SPLINE && p.interp != BSDE_INTERP_BICUBIC_FD) return false;
    if (p.interp == BSDE_INTERP_BICUBIC_FD && p.d != 2) return false;
    for (int i = 0; i < 8; ++i)
        if (!std::isfinite(p.p[i])) return false;
    if (p.driver == BSDE_DRIVER_BIDASK && p.p[3] == 0.0) return false;
    if (p.d == 2) {
        if (p.n_x[1] < 4 || !(p.x_max[1] > p.x_min[1])) return false;
        if (!std::isfinite(p.x_min[1]) || !std::isfinite(p.x_max[1])) return false;
        if (!std::isfinite(p.drift[1]) || !(p.vol[1][1] > 0.0) || !std::isfinite(p.vol[1][1]) ||
            !std::isfinite(p.vol[1][0]) || !std::isfinite(p.vol[0][1]))
            return false;
    }
    return true;
}

// R above BSDE_STABILITY_LIMIT by more than its own rounding (a grid built
// for R = 16 computes R = 16 to within a few ulps)
bool beyond_stability_limit(double R) { return R > BSDE_STABILITY_LIMIT * (1.0 + 1e-12); }

// What the one-dimensional path implements: every valid problem except the
// E[y dW]/dt z form in the FP32 form (it weighs the stored y by dW/dt ~
// 1/sqrt(dt), so the ring's rounding would enter z amplified by that) and
// exact expectations beyond the Toeplitz kernel's reach (linear driver,
// constant coefficients, FP64).
bool supported_1d(const bsde_problem &q)
{
    if (q.z_form == BSDE_ZFORM_YDW && q.prec == BSDE_FP32_COMP) return false;
    if (q.quad == BSDE_QUAD_EXACT &&
        (q.driver != BSDE_DRIVER_LINEAR || q.drift_x != 0.0 || q.vol_x != 0.0 ||
         q.tab_steps != 0 || q.prec != BSDE_FP64))
        return false;
    return true;
}

// What the two-dimensional path implements: vol lower triangular (any
// correlation, written with its Cholesky factor), the linear driver, FP64.
bool supported_2d(const bsde_problem &p)
{
    // the FP32 form stores the ring in single precision; with the E[y dW]/dt
    // z form its rounding would enter z amplified by dW/dt (as in 1-D)
    const bool prec_ok = p.prec == BSDE_FP64 ||
                         (p.prec == BSDE_FP32_COMP && p.z_form == BSDE_ZFORM_EZ);
    return p.vol[0][1] == 0.0 && p.driver == BSDE_DRIVER_LINEAR && prec_ok &&
           p.L <= 64 && p.drift_x == 0.0 && p.vol_x == 0.0 && p.tab_steps == 0 &&
           p.quad == BSDE_QUAD_GH &&
           (p.interp == BSDE_INTERP_SPLINE || (p.n_x[0] >= 5 && p.n_x[1] >= 5));
}

// Bounds on the drift and the volatility of state-dependent coefficients over
// runs of a table's rows (its volatilities are positive), or at the grid's ends
// where they are affine.  One pass over a table, eight extremes at a time: it
// also serves the widest reach, which took a pass of its own.
struct CoefBounds {
    double alo, ahi, blo, bhi;
};
std::vector<CoefBounds> coef_bounds(const bsde_problem &p)
{
    std::vector<CoefBounds> out;
    if (p.tab_steps == 0) {
        for (double x : {p.x_min[0], p.x_max[0]}) {
            const double ax = p.drift[0] + p.drift_x * x, bx = p.vol[0][0] + p.vol_x * x;
            out.push_back({ax, ax, std::min(0.0, bx), std::max(0.0, bx)});
        }
        return out;
    }
    constexpr int kRun = 64, kV = 8;
    const int nx = p.n_x[0];
    for (int r = 0; r < p.tab_steps; ++r) {
        const double *ta = p.coef_tab + (size_t)2 * r * nx, *tb = ta + nx;
        for (int i0 = 0; i0 < nx; i0 += kRun) {
            double al[kV], ah[kV], bh[kV];
            for (int v = 0; v < kV; ++v) {
                al[v] = ah[v] = ta[i0];
                bh[v] = tb[i0];
            }
            const int i1 = std::min(i0 + kRun, nx);
            int i = i0;
            for (; i + kV <= i1; i += kV)
                for (int v = 0; v < kV; ++v) {
                    al[v] = ta[i + v] < al[v] ? ta[i + v] : al[v];
                    ah[v] = ta[i + v] > ah[v] ? ta[i + v] : ah[v];
                    bh[v] = tb[i + v] > bh[v] ? tb[i + v] : bh[v];
                }
            for (; i < i1; ++i) {
                al[0] = std::min(al[0], ta[i]);
                ah[0] = std::max(ah[0], ta[i]);
                bh[0] = std::max(bh[0], tb[i]);
            }
            out.push_back({*std::min_element(al, al + kV), *std::max_element(ah, ah + kV), 0.0,
                           *std::max_element(bh, bh + kV)});
        }
    }
    return out;
}

// Window bounds of every layer for state-dependent coefficients: the nodes of
// grid point i sit (a(t, x_i) j dt + b(t, x_i) dW) / dx cells away with b > 0,
// so the extremes over the grid (and the table's rows) of the outermost
// nodes, one cell wider for rounding.  gh: Gauss-Hermite nodes.  Bounds far
// beyond any LDS window leave the instance to the kernel that reads HBM.
void located_windows(const bsde_problem &p, const std::vector<CoefBounds> &pieces, Instance &in,
                     const double *gh)
{
    double glo = gh[0], ghi = gh[0];
    for (int l = 1; l < p.L; ++l) {
        glo = std::min(glo, gh[l]);
        ghi = std::max(ghi, gh[l]);
    }
    std::vector<int> lo(in.K + 1, 0), hi(in.K + 1, 0);
    for (int j = 1; j <= in.K; ++j) {
        const double t = j * in.dt / in.dx, sq = std::sqrt(2.0 * j * in.dt) / in.dx;
        double mn = 1e300, mx = -1e300;
        for (const CoefBounds &q : pieces) {  // glo <= 0 <= ghi: the abscissae are symmetric
            mn = std::min(mn, q.alo * t + sq * std::min(q.bhi * glo, q.blo * ghi));
            mx = std::max(mx, q.ahi * t + sq * std::max(q.bhi * ghi, q.blo * glo));
        }
        if (!(mn > -4000.0) || !(mx < 4000.0)) return;
        // (a node clamped to the right end lies in the cell left of the last point)
        lo[j] = std::min((int)std::floor(mn) - 1, -1);
        hi[j] = std::max((int)std::floor(mx) + 1, 0);
    }
    in.located = true;
    in.win_lo = lo;
    in.win_hi = hi;
}

// Node tables of eq (20)-(21) on the uniform grid (Section 3.2): the node
// x_i + drift j dt + vol sqrt(2 j dt) a_l sits s = (drift j dt + vol sqrt(2 j dt) a_l)/dx
// cells from x_i, independent of i; s = m + phi with integer m.  The weights
// fold the Gauss-Hermite weight pi^{-1/2} w_l and the coefficients of
// Tables 1 and 2 into two accumulators per grid point:
//   Y = E[y^{n+K_y}] + K_y dt sum_{j=1}^{K_y} gamma_j E[f^{n+j}]
//   Z = (E[z^{n+1}] + sum_{j=1}^{K_z} gamma'_j (E[f^{n+j} dW] - E[z^{n+j}])) / gamma'_0 = z^n
bool build_instance(const bsde_problem &p, Instance &in)
{
    in.pb = p;
    in.K = std::max(p.k_y, p.k_z);
    in.nx = p.n_x[0];
    in.dt = p.T / p.n_t;
    in.dx = (p.x_max[0] - p.x_min[0]) / (in.nx - 1);
    in.f32 = p.prec == BSDE_FP32_COMP;
    in.gather = p.drift_x != 0.0 || p.vol_x != 0.0 || p.tab_steps > 0;
    in.exact = p.quad == BSDE_QUAD_EXACT;
    in.steps = p.n_t - in.K - p.n_stop + 1;
    const double vol = p.vol[0][0];
    // largest Gauss-Hermite spread per cell over the grid (b(x) is affine, or
    // tabulated)
    const std::vector<CoefBounds> pieces = in.gather ? coef_bounds(p) : std::vector<CoefBounds>();
    double bmax = std::max(vol + p.vol_x * p.x_min[0], vol + p.vol_x * p.x_max[0]);
    if (p.tab_steps > 0) {
        bmax = 0.0;
        for (const CoefBounds &q : pieces) bmax = std::max(bmax, q.bhi);
        // the plan keeps its own copy of the table
        in.ctab.assign(p.coef_tab, p.coef_tab + (size_t)2 * p.tab_steps * in.nx);
        in.pb.coef_tab = nullptr;
    }
    in.R = bmax * std::sqrt(2.0 * in.dt) / in.dx;
    // the constant-coefficient node offsets (the kernels' windows; the gather
    // kernel locates its nodes per point); with a table, drift and vol are
    // not used and the offsets take b's largest value
    const double drift_n = p.tab_steps > 0 ? 0.0 : p.drift[0];
    const double vol_n = p.tab_steps > 0 ? bmax : vol;
    double a[bsde::kMaxL], w[bsde::kMaxL], gy[8], gz[8];
    if (!bsde::gauss_hermite(p.L, a, w)) return false;
    if (!bsde::spline_gamma(1, p.k_y, gy) || !bsde::spline_gamma(2, p.k_z, gz)) return false;
    const double inv_sqrt_pi = 0.56418958354775628695;
    const int K = in.K, L = p.L;
    in.m.assign(K * L, 0);
    in.B.assign(K * L, 0.0);
    in.C = in.D = in.phi = in.cfy = in.cfz = in.cz = in.cyz = in.dw = in.B;
    in.cy.assign(L, 0.0);
    in.win_lo.assign(K + 1, 0);
    in.win_hi.assign(K + 1, 0);
    in.m_min = 0;
    in.m_max = 0;
    const double dx26 = in.dx * in.dx / 6.0;
    for (int j = 1; j <= K; ++j) {
        const double sq = std::sqrt(2.0 * j * in.dt);
        int lo = INT32_MAX, hi = INT32_MIN;
        for (int l = 0; l < L; ++l) {
            const int k = (j - 1) * L + l;
            const double dW = sq * a[l];
            const double s = (drift_n * j * in.dt + vol_n * dW) / in.dx;
            const double fl = std::floor(s);
            if (!(std::fabs(fl) < 1e8)) return false;
            const int m = (int)fl;
            const double phi = s - fl;
            const double u = 1.0 - phi;
            const double wl = w[l] * inv_sqrt_pi;
            in.m[k] = m;
            in.dw[k] = dW;
            in.B[k] = in.phi[k] = phi;
            in.C[k] = dx26 * (u * u * u - u);
            in.D[k] = dx26 * (phi * phi * phi - phi);
            in.cfy[k] = (j <= p.k_y) ? p.k_y * in.dt * gy[j] * wl : 0.0;
            in.cfz[k] = (j <= p.k_z) ? gz[j] * wl * dW / gz[0] : 0.0;
            // the first term of the z equation: E[z^{n+1}] (eq (20)), or
            // E[y^{n+1} dW]/dt (eq (12) with l = 1) for the z form YDW
            const bool ydw = p.z_form == BSDE_ZFORM_YDW;
            in.cz[k] = ((j == 1 && !ydw ? 1.0 : 0.0) - (j <= p.k_z ? gz[j] : 0.0)) * wl / gz[0];
            in.cyz[k] = (j == 1 && ydw) ? wl * dW / (in.dt * gz[0]) : 0.0;
            if (j == p.k_y) in.cy[l] = wl;
            lo = std::min(lo, m);
            hi = std::max(hi, m);
        }
        if (j == 1) {  // the window of layer n+1 also covers the tile itself
            lo = std::min(lo, 0);
            hi = std::max(hi, 0);
        }
        in.win_lo[j] = lo;
        in.win_hi[j] = hi;
        in.m_min = std::min(in.m_min, lo);
        in.m_max = std::max(in.m_max, hi);
    }
    in.h0 = p.k_y * in.dt * gy[0];
    if (in.gather && !in.f32 && p.z_form == BSDE_ZFORM_EZ) located_windows(p, pieces, in, a);
    if (in.exact) {
        // exact Gaussian expectations: the band of every layer; the ghosts
        // cover the band and the Toeplitz kernel's window overhang
        for (int j = 1; j <= K; ++j) {
            bsde::GaussBand &b = in.band[j];
            if (!bsde::gaussian_spline_band(p.drift[0] * j * in.dt / in.dx,
                                            vol * std::sqrt(j * in.dt) / in.dx,
                                            std::sqrt(j * in.dt), in.dx, b))
                return false;
            in.m_min = std::min(in.m_min, b.klo);
            in.m_max = std::max(in.m_max, b.klo + (int)b.ev.size() - 1);
            in.ex_boff[j] = (int)in.ex_band.size();
            in.ex_band.insert(in.ex_band.end(), b.ec.begin(), b.ec.end());
            in.ex_band.insert(in.ex_band.end(), b.wc.begin(), b.wc.end());
            const int cells = (int)b.i0.size();
            auto piece = [&](const std::vector<double> &v, int cell) {  // cell relative to the point
                const int k = cell - b.klo;
                return k >= 0 && k < cells ? v[k] : 0.0;
            };
            // the points whose first or last piece lies in the band, no others: the
            // kernel's window holds the end coefficients for these only, and zero
            // times a non-finite one would be wrong.  Points il .. from the left
            // end, ir .. from the right one
            const int lend = std::min(std::max(0, 1 - b.klo), in.nx);
            const int rend = std::min(std::max(0, b.klo + cells + 1), in.nx);
            in.ex_il[j] = std::min(std::max(0, -b.klo - cells), lend);
            in.ex_ir[j] = std::min(std::max(0, b.klo), rend);
            in.ex_nl[j] = lend - in.ex_il[j];
            in.ex_nr[j] = rend - in.ex_ir[j];
            in.ex_loff[j] = (int)in.ex_corr.size();
            for (int i = in.ex_il[j]; i < lend; ++i)
                in.ex_corr.push_back(make_double2(piece(b.i3, -1 - i) + piece(b.i0, -i),
                                                  piece(b.j3, -1 - i) + piece(b.j0, -i)));
            in.ex_roff[j] = (int)in.ex_corr.size();
            for (int i = in.ex_ir[j]; i < rend; ++i)
                in.ex_corr.push_back(make_double2(piece(b.i0, i) + piece(b.i3, i - 1),
                                                  piece(b.j0, i) + piece(b.j3, i - 1)));
        }
    }
    in.reach = std::max(-in.m_min, in.m_max + 1);
    // (located nodes need one ghost either side: their windows' loads are clamped)
    in.pad_l = std::max(0, -in.m_min) + 1;
    // right ghosts cover the overhang of the last tile of any configuration
    in.pad_r = std::max(0, in.m_max) + kBlock * kMaxP + 2 + (in.exact ? 64 : 0);
    in.npad = in.pad_l + in.nx + in.pad_r;
    in.drv = bsde::DriverParams{p.p[0], p.p[1], p.p[2], p.p[3], p.p[4], 1.0 / p.p[3]};
    in.nwaves = (in.nx + kBlock - 1) / kBlock * (kBlock / 64);
    return true;
}

// The four cubic B-spline weights at the fraction ph of a cell, which sum to one
// to the last bit of the second.  The expectations' weights have to sum to one: a
// constant is a fixed point of the scheme, and what a sum is short of one is lost
// in every step (4e-16 a step of z in the basket, 6e-14 over its solve).
void spline_basis(double ph, double *b)
{
    const long double t = ph, u = 1.0L - t;
    b[0] = (double)(u * u * u / 6.0L);
    b[2] = (double)(2.0L / 3.0L - 0.5L * u * u * (1.0L + t));
    b[3] = (double)(t * t * t / 6.0L);
    b[1] = (double)(1.0L - b[0] - b[2] - b[3]);
}

// Tables of the two-dimensional B-spline form (sweep2b): node rows, nodes,
// and the corrections of the columns next to the ends of axis 1 (see sweep2b:
// node offset m errs by w b_3 at column -1 - m and by w b_0 at column -m, and
// mirrored at the other end).  a, w: Gauss-Hermite; m, weights as in
// build_instance2.
void build_instance2b(const bsde_problem &p, Instance2 &in, const double *a, const double *w,
                      const double *gy, const double *gz, int m1min, int m1max)
{
    const int K = in.K, L = p.L;
    const long double inv_pi = 0.318309886183790671538L;
    in.rowsb.assign((size_t)K * L, bsde::Row2B{});
    in.nodesb.assign((size_t)K * L * L, bsde::Node2B{});
    in.nl = std::min(std::max(0, -m1min) + 1, in.n1);
    in.nr = std::min(std::max(0, m1max) + 2, in.n1);
    in.corr_l.assign((size_t)K * L * in.nl, make_double4(0, 0, 0, 0));
    in.corr_r.assign((size_t)K * L * in.nr, make_double4(0, 0, 0, 0));
    const bool ydw = p.z_form == BSDE_ZFORM_YDW;
    for (int j = 1; j <= K; ++j) {
        const double sq = std::sqrt(2.0 * j * in.dt);
        const double fy = j <= p.k_y ? p.k_y * in.dt * gy[j] : 0.0, fz = j <= p.k_z ? gz[j] / gz[0] : 0.0;
        const double yw = j == 1 && ydw ? 1.0 / (in.dt * gz[0]) : 0.0;
        for (int l0 = 0; l0 < L; ++l0) {
            const size_t ri = (size_t)(j - 1) * L + l0;
            const double dW0 = sq * a[l0];
            const double s0 = (p.drift[0] * j * in.dt + p.vol[0][0] * dW0) / in.dx0;
            bsde::Row2B &r = in.rowsb[ri];
            r.m0 = in.rows[ri].m0;
            r.m1lo = in.rows[ri].m1lo;
            r.m1hi = in.rows[ri].m1hi;
            in.spread = std::max(in.spread, r.m1hi - r.m1lo);
            spline_basis(s0 - std::floor(s0), r.b);
            r.H = fy;
            r.Gu = fz * dW0;
            r.Gy = yw * dW0;
            r.C = ((j == 1 && !ydw ? 1.0 : 0.0) - (j <= p.k_z ? gz[j] : 0.0)) / gz[0];
            r.ey = j == p.k_y ? 1.0 : 0.0;
            r.extra = j == p.k_y || (j == 1 && ydw) ? 1 : 0;
            for (int l1 = 0; l1 < L; ++l1) {
                const size_t k = ri * L + l1;
                const double dW1 = sq * a[l1];
                const double s1 =
                    (p.drift[1] * j * in.dt + p.vol[1][0] * dW0 + p.vol[1][1] * dW1) / in.dx1;
                const long double wgt = w[l0] * (w[l1] * inv_pi);
                double b[4];
                spline_basis(s1 - std::floor(s1), b);
                bsde::Node2B &nd = in.nodesb[k];
                nd.w0 = (double)(wgt * b[0]);
                nd.w2 = (double)(wgt * b[2]);
                nd.w3 = (double)(wgt * b[3]);
                nd.w1 = (double)(wgt - nd.w0 - nd.w2 - nd.w3);
                nd.gu = fz * dW1;  // t carries the quadrature weight
                nd.gy = yw * dW1;
                const int m = in.m1[k];
                auto add = [&](std::vector<double4> &t, int n, int c, double v) {
                    if (c < 0 || c >= n) return;
                    double4 &q = t[ri * n + c];
                    q.x += v;
                    q.y += v * nd.gu;
                    q.z += v * nd.gy;
                };
                add(in.corr_l, in.nl, -1 - m, nd.w3);
                add(in.corr_l, in.nl, -m, nd.w0);
                add(in.corr_r, in.nr, m, nd.w0);      // distance from the last column
                add(in.corr_r, in.nr, m + 1, nd.w3);
                const double c3 = (double)(p.p[3] * wgt);
                in.lin_y += fy * c3;
                in.lin_z1 += fz * dW0 * c3;
                in.lin_z2 += fz * dW1 * c3;
            }
        }
    }
    // E[y] of layer K_y and the E[z] terms: the rest to one goes to the layer's row
    // of the largest weight
    auto sum = [&](size_t ri) {
        const bsde::Row2B &r = in.rowsb[ri];
        long double s = 0.0L;
        for (int l = 0; l < L; ++l) {
            const bsde::Node2B &nd = in.nodesb[ri * L + l];
            s += (long double)nd.w0 + nd.w1 + nd.w2 + nd.w3;
        }
        return s * ((long double)r.b[0] + r.b[1] + r.b[2] + r.b[3]);
    };
    long double sy = 0.0L, sz = 0.0L;
    for (size_t ri = 0; ri < in.rowsb.size(); ++ri) {
        const long double s = sum(ri);
        sy += in.rowsb[ri].ey * s;
        sz += in.rowsb[ri].C * s;
    }
    const int mid = (int)(std::max_element(w, w + L) - w);
    const size_t ky = (size_t)(p.k_y - 1) * L + mid, kz = mid;
    in.rowsb[ky].ey = (double)(in.rowsb[ky].ey + (1.0L - sy) / sum(ky));
    if (!ydw) in.rowsb[kz].C = (double)(in.rowsb[kz].C + (1.0L - sz) / sum(kz));
}

// Two-dimensional node tables (eq (20)-(21) with tensor Gauss-Hermite nodes):
// node (l0, l1) of layer n+j sits at x + drift j dt + vol sqrt(2 j dt) (a_l0, a_l1),
// i.e. s0 = (drift0 j dt + vol00 dW0)/dx0 (vol lower triangular) and
// s1 = (drift1 j dt + vol10 dW0 + vol11 dW1)/dx1 cells away, independent of
// the grid point.  Weights fold w_l0 w_l1 / pi with Tables 1 and 2 as in 1-D,
// z having one component per Brownian motion.
bsde_status build_instance2(const bsde_problem &p, Instance2 &in)
{
    in.pb = p;
    in.f32 = p.prec == BSDE_FP32_COMP;
    in.K = std::max(p.k_y, p.k_z);
    in.n0 = p.n_x[0];
    in.n1 = p.n_x[1];
    in.dt = p.T / p.n_t;
    in.dx0 = (p.x_max[0] - p.x_min[0]) / (in.n0 - 1);
    in.dx1 = (p.x_max[1] - p.x_min[1]) / (in.n1 - 1);
    in.R = std::max(p.vol[0][0] / in.dx0,
                    std::sqrt(p.vol[1][0] * p.vol[1][0] + p.vol[1][1] * p.vol[1][1]) / in.dx1) *
           std::sqrt(2.0 * in.dt);
    double a[bsde::kMaxL], w[bsde::kMaxL], gy[8], gz[8];
    if (!bsde::gauss_hermite(p.L, a, w)) return BSDE_EINVAL;
    if (!bsde::spline_gamma(1, p.k_y, gy) || !bsde::spline_gamma(2, p.k_z, gz)) return BSDE_EINVAL;
    const double inv_sqrt_pi = 0.56418958354775628695;
    const int K = in.K, L = p.L;
    // the B-spline form has node tables of its own (build_instance2b)
    in.bspline = !in.f32 && p.interp != BSDE_INTERP_BICUBIC_FD;
    in.rows.assign((size_t)K * L, bsde::Node2Row{});
    in.nodes.assign(in.bspline ? 0 : (size_t)K * L * L, bsde::Node2{});
    in.m1.assign((size_t)K * L * L, 0);
    int m0min = 0, m0max = 0, m1min = 0, m1max = 0;
    in.win = 0;
    const double d0 = in.dx0 * in.dx0 / 6.0, d1 = in.dx1 * in.dx1 / 6.0;
    // the interpolant of the layers (Section 3.3): the tensor natural spline
    // (second derivatives in the three derivative planes), or the paper's
    // bicubic from the values and finite-difference first and mixed
    // derivatives (in the same planes).  Either is v0 + B (v1 - v0) + C d0 +
    // D d1 per axis; for the bicubic B = h01(phi) (and 1 - B = h00(phi)),
    // C = dx h10(phi) = dx phi (1 - phi)^2, D = dx h11(phi) = -dx phi^2 (1 - phi).
    const bool bicubic = p.interp == BSDE_INTERP_BICUBIC_FD;
    for (int j = 1; j <= K; ++j) {
        const double sq = std::sqrt(2.0 * j * in.dt);
        for (int l0 = 0; l0 < L; ++l0) {
            const double dW0 = sq * a[l0];
            const double s0 = (p.drift[0] * j * in.dt + p.vol[0][0] * dW0) / in.dx0;
            const double f0 = std::floor(s0);
            if (!(std::fabs(f0) < 1e8)) return BSDE_EINVAL;
            const double ph0 = s0 - f0, u0 = 1.0 - ph0;
            bsde::Node2Row &row = in.rows[(size_t)(j - 1) * L + l0];
            row.m0 = (int)f0;
            if (bicubic) {  // Hermite basis: values, then dx-scaled slopes
                row.B0 = ph0 * ph0 * (3.0 - 2.0 * ph0);
                row.C0 = in.dx0 * ph0 * u0 * u0;
                row.D0 = -in.dx0 * ph0 * ph0 * u0;
            } else {
                row.B0 = ph0;
                row.C0 = d0 * (u0 * u0 * u0 - u0);
                row.D0 = d0 * (ph0 * ph0 * ph0 - ph0);
            }
            int lo = INT32_MAX, hi = INT32_MIN;
            for (int l1 = 0; l1 < L; ++l1) {
                const double dW1 = sq * a[l1];
                const double s1 =
                    (p.drift[1] * j * in.dt + p.vol[1][0] * dW0 + p.vol[1][1] * dW1) / in.dx1;
                const double f1 = std::floor(s1);
                if (!(std::fabs(f1) < 1e8)) return BSDE_EINVAL;
                const size_t k = ((size_t)(j - 1) * L + l0) * L + l1;
                in.m1[k] = (int)f1;
                lo = std::min(lo, (int)f1);
                hi = std::max(hi, (int)f1);
                if (in.bspline) continue;
                const double ph1 = s1 - f1, u1 = 1.0 - ph1;
                const double wgt = w[l0] * inv_sqrt_pi * w[l1] * inv_sqrt_pi;
                bsde::Node2 &nd = in.nodes[k];
                if (bicubic) {
                    nd.B1 = ph1 * ph1 * (3.0 - 2.0 * ph1);
                    nd.C1 = in.dx1 * ph1 * u1 * u1;
                    nd.D1 = -in.dx1 * ph1 * ph1 * u1;
                } else {
                    nd.B1 = ph1;
                    nd.C1 = d1 * (u1 * u1 * u1 - u1);
                    nd.D1 = d1 * (ph1 * ph1 * ph1 - ph1);
                }
                nd.cfy = (j <= p.k_y) ? p.k_y * in.dt * gy[j] * wgt : 0.0;
                nd.cfz1 = (j <= p.k_z) ? gz[j] * wgt * dW0 / gz[0] : 0.0;
                nd.cfz2 = (j <= p.k_z) ? gz[j] * wgt * dW1 / gz[0] : 0.0;
                const bool ydw = p.z_form == BSDE_ZFORM_YDW;
                nd.cz = ((j == 1 && !ydw ? 1.0 : 0.0) - (j <= p.k_z ? gz[j] : 0.0)) * wgt / gz[0];
                nd.cy = (j == p.k_y) ? wgt : 0.0;
                nd.cyz1 = (j == 1 && ydw) ? wgt * dW0 / (in.dt * gz[0]) : 0.0;
                nd.cyz2 = (j == 1 && ydw) ? wgt * dW1 / (in.dt * gz[0]) : 0.0;
            }
            row.m1lo = lo;
            row.m1hi = hi;
            if (bsde::kTile2C + hi - lo + 2 > bsde::kWin2) return BSDE_EUNSUPPORTED;
            in.win = std::max(in.win, bsde::kTile2C + hi - lo + 2);
            m0min = std::min(m0min, row.m0);
            m0max = std::max(m0max, row.m0);
            m1min = std::min(m1min, lo);
            m1max = std::max(m1max, hi);
        }
    }
    in.h0 = p.k_y * in.dt * gy[0];
    if (in.bspline) {
        // one plane element per grid point; the widest node spread and the
        // columns next to the ends of axis 1 that a node's correction reaches
        build_instance2b(p, in, a, w, gy, gz, m1min, m1max);
        in.pad0 = in.pad0r = in.pad1 = in.pad1r = 0;
        in.npad0 = in.n0;
        in.npad1 = in.n1;
        in.plane = (size_t)in.n0 * in.n1;
        const int tiles = in.n0 * ((in.n1 + bsde::kTile2B - 1) / bsde::kTile2B);
        in.nwaves = tiles * bsde::kGroups2B;
        in.reach = std::max({0, -m0min, -m1min, m0max});
        return BSDE_OK;
    }
    // ghosts: node reach plus the overhang of the last tile (kTile2R rows,
    // kTile2C columns)
    in.pad0 = std::max(0, -m0min) + 1;
    in.pad0r = std::max(0, m0max) + bsde::kTile2R + 1;
    in.pad1 = std::max(0, -m1min) + 1;
    in.pad1r = std::max(0, m1max) + bsde::kTile2C + 3;
    in.npad0 = in.pad0 + in.n0 + in.pad0r;
    in.npad1 = in.pad1 + in.n1 + in.pad1r;
    in.plane = (size_t)in.npad0 * in.npad1;
    const int tiles = ((in.n0 + bsde::kTile2R - 1) / bsde::kTile2R) *
                      ((in.n1 + bsde::kTile2C - 1) / bsde::kTile2C);
    in.nwaves = tiles * bsde::kWaves2;
    in.reach = std::max({in.pad0 - 1, in.pad1 - 1, in.pad0r - bsde::kTile2R - 1});
    return BSDE_OK;
}

bsde::Sweep2Args sweep2_args(const Instance2 &in, char *ws, bool stats)
{
    bsde::Sweep2Args a{};
    a.ring = ws + in.ring_off;
    a.planes = in.planes();
    a.vstep = in.bspline ? 1 : 4;
    a.plane = in.plane;
    a.n0 = in.n0;
    a.n1 = in.n1;
    a.npad1 = in.npad1;
    a.pad0 = in.pad0;
    a.pad1 = in.pad1;
    a.K = in.K;
    a.Ky = in.pb.k_y;
    a.L = in.pb.L;
    a.n_stop = in.pb.n_stop;
    a.rows = in.d_rows;
    a.nodes = in.d_nodes;
    a.m1 = in.d_m1;
    a.drv = bsde::DriverParams{in.pb.p[0], in.pb.p[1], in.pb.p[2], in.pb.p[3], in.pb.p[4], 0.0};
    a.dt = in.dt;
    a.h0 = in.h0;
    a.picard_max = in.pb.picard_max;
    a.picard_tol = in.pb.picard_tol;
    a.zform = in.pb.z_form;
    a.interp = in.pb.interp;
    a.half = (in.win + 1) / 2;
    if (in.bspline) {
        a.rowsb = in.d_rowsb;
        a.nodesb = in.d_nodesb;
        a.corr_l = in.d_corr_l;
        a.corr_r = in.d_corr_r;
        a.nl = in.nl;
        a.nr = in.nr;
        a.lds_wave = (int)bsde::sweep2b_wave_lds(in.spread);
        a.lin_y = in.lin_y;
        a.lin_z1 = in.lin_z1;
        a.lin_z2 = in.lin_z2;
        a.tmp = reinterpret_cast<double *>(ws + in.tmp_off);
    }
    a.fin = reinterpret_cast<double *>(ws + in.fin_off);
    if (stats) {
        unsigned long long *sum = reinterpret_cast<unsigned long long *>(ws + in.stat_off);
        a.st_iter_sum = sum;
        a.st_nonconv = sum + in.nwaves;
        a.st_iter_max = reinterpret_cast<unsigned int *>(sum + 2 * in.nwaves);
    }
    return a;
}

// Dynamic LDS of one block of the fused sweep (fused.h), in bytes: the
// layers' windows (the partial sums may reuse them), the spline filter's
// arrays, the boundary values and the driver's time factors.
struct FusedLds {
    int win[bsde::kMaxOrder + 1], d, a, edge, drv, tm, part;
    size_t total;
};

FusedLds fused_layout(const Instance &in, int P, int W, int G)
{
    FusedLds l{};
    const int T = 64 * P * W;
    auto slots = [&](int n) { return P % 2 == 0 ? n + n / P + 1 : n; };
    size_t off = 0;
    int w1 = 0;
    for (int j = 1; j <= in.K; ++j) {
        const int n = T + in.win_hi[j] - in.win_lo[j] + (in.f32 ? 1 : 3);
        if (j == 1) w1 = n;
        l.win[j] = (int)off;
        off += (size_t)slots(n) * 16;
    }
    // the partial sums: over the windows, or beside them where that is little
    // (one barrier less)
    const size_t part = P > 1 || G > 1 ? (size_t)G * T * 16 : 0;
    l.part = part <= 8192 ? (int)off : 0;
    off = part <= 8192 ? off + part : std::max(off, part);
    l.d = (int)off;
    off += (size_t)(w1 + 2 * bsde::kHalo + 2 + bsde::kFirOver) * 16;
    l.a = (int)off;
    off += (size_t)(w1 + 48 + bsde::kFirOver) * 16;
    l.edge = (int)off;
    off += (size_t)2 * in.K * 16;
    l.drv = (int)off;
    off += in.pb.driver == BSDE_DRIVER_EXP ? align_up((size_t)3 * (in.K + 1) * sizeof(double), 16) : 0;
    l.tm = (int)off;
    off += in.f32 ? align_up((size_t)in.K * in.pb.L * sizeof(int), 16) : 0;
    l.total = off;
    return l;
}

// The fused sweep with tiles of 64 P W points and G node groups for every
// member of a group, or lds = 0 if some member's windows do not fit.
SweepConfig fused_config(const std::vector<Instance> &all, const std::vector<int> &members, int P, int W,
                         int G, size_t max_lds)
{
    SweepConfig c{PATH_FUSED, P, G, 0, W};
    size_t lds = 0;
    for (int b : members) {
        const Instance &in = all[b];
        // the fused kernel serves the E[z] form of the z equation only
        if ((in.gather && !in.located) || in.exact || in.pb.z_form != BSDE_ZFORM_EZ || in.pb.L > 64) return c;
        // node offsets beyond any window that could fit (and int arithmetic)
        if ((long)in.m_max - in.m_min > (long)(max_lds / 16)) return c;
        // FP32 form: wider reaches stay on the direct kernel (its sums, in
        // another order, are part of the form's results)
        if (in.f32) {
            int reach = 0;
            for (int j = 2; j <= in.K; ++j) reach = std::max(reach, in.win_hi[j] - in.win_lo[j] + 1);
            if (reach > 320 || in.win_hi[1] - in.win_lo[1] + 1 > 160) return c;
        }
        const size_t need = fused_layout(in, P, W, G).total;
        if (need > max_lds) return c;
        lds = std::max(lds, need);
    }
    c.lds = lds;
    return c;
}

// Position of node (j, l) in the FP64 fused sweep's tables: by class l mod 8,
// in a class by layer K, ..., 1, in a layer by l.
int fused_position(int K, int L, int j, int l)
{
    const int c = l & 7;
    const int per = (L - c + 7) / 8;  // nodes of the class in a layer
    return K * (c * (L >> 3) + std::min(c, L & 7)) + (K - j) * per + (l >> 3);
}

// Node addresses for a shape with P points per lane (FusedHot::addr).
std::vector<int2> fused_addresses(const Instance &in, const FusedLds &lds, int P)
{
    const int L = in.pb.L;
    std::vector<int2> v((size_t)in.K * L);
    for (int j = 1; j <= in.K; ++j)
        for (int l = 0; l < L; ++l) {
            const int m = in.m[(j - 1) * L + l], off = m - in.win_lo[j];
            const int slot = P % 2 == 0 ? off + off / P : off;
            const int at = in.f32 ? (j - 1) * L + l : fused_position(in.K, L, j, l);
            // (located nodes: the address of the record of the tile's first point)
            v[at] = in.located ? make_int2(lds.win[j] - 16 * (in.win_lo[j] - 1), j)
                               : make_int2((lds.win[j] + 16 * slot) | (off % P), m * 16 + j);
        }
    return v;
}

// Shapes that the plan and the autotuner choose from (all of them add the nodes
// in the same order, so they give the same bits), with the time of a step as
// measured, in us: 256 CUs share the tiles, the first of a CU takes
//   first + first_node K L + first_kb LDS     and each further one
//   tile + node K L + kb LDS (+ alone + alone_node K L where the LDS leaves room
// for one block), and both exp K L T / 64 where the driver has an exponential.
// LDS in KiB.  Fitted to solves of 500 to 1048576 points, K L = 4 to 128 and
// stability ratios 3 to 180 (max error 7 to 10% in FP64, 8 to 25% in the FP32
// form).  Where the lines cross, measured a step: 65536 points, K = 4, L = 16:
// 64-point tiles 14.0 us, 256 10.3, 1024 19.5; 262144: 42.2, 23.3, 21.1.
// 4194304 points: 256-point tiles 298, 1024 289 (at ratio 4 283 and 285).
// 1048576 points, K = 1, L = 16: four groups a 1024-point tile 38.7 us, two 30.0,
// where few nodes leave little to share out; K = 4: 74.4 and 82.7.  FP32 form, K
// L = 16: 256-point tiles 8.0, 512 8.3, 1024 10.7 us on 32768 points, 34.5, 34.3
// and 39.3 on 1048576.
struct Shape {
    int P, W, G;
    double first, first_node, first_kb, tile, node, kb, alone, alone_node, exp;
};
constexpr Shape kShapes64[] = {{1, 1, 8, 4.0, 0.032, 0.023, 1.37, 0.0114, 0.0063, 1.9, 0.0105, 0.0300},
                               {2, 1, 8, 3.9, 0.038, 0.023, 1.49, 0.0196, 0.0061, 1.4, 0.0105, 0.0220},
                               {4, 1, 8, 4.8, 0.064, 0.021, 1.34, 0.0330, 0.0189, 2.0, 0.0105, 0.0165},
                               {4, 4, 4, 8.5, 0.178, 0.0, 6.08, 0.169, 0.0041, 0.0, 0.0, 0.0130},
                               {4, 4, 2, 6.6, 0.200, 0.033, 0.5, 0.130, 0.0550, 3.20, 0.0, 0.0130}};
constexpr Shape kShapes32[] = {{1, 4, 1, 5.5, 0.096, 0.046, 0.73, 0.0338, 0.0216, 0.0, 0.0, 0.0125},
                               {1, 8, 1, 5.4, 0.106, 0.035, 1.95, 0.0496, 0.0266, 8.08, 0.0, 0.0125},
                               {1, 16, 1, 7.1, 0.160, 0.038, 5.41, 0.183, 0.0209, 0.0, 0.0, 0.0125}};

// Estimated time of a step of a group with a fused shape (us), the mean of four
// steps spread over the group's length (the set of active instances shrinks).
double fused_cost(const std::vector<Instance> &all, const std::vector<int> &members, const SweepConfig &c,
                  const Shape &q)
{
    const int T = 64 * c.P * c.W, NT = 64 * c.W * c.G;
    const bool alone = std::min(163840 / c.lds, (size_t)2048 / NT) < 2;
    const double kb = c.lds / 1024.0;
    int longest = 1;
    for (int b : members) longest = std::max(longest, all[b].steps);
    double cost = 0.0;
    for (int k = 0; k < 4; ++k) {
        double tiles = 0.0, first = 0.0, more = 0.0;  // the latter two: tile by tile
        for (int b : members) {
            const Instance &in = all[b];
            if (in.steps <= (long)longest * k / 4) continue;
            const double t = (in.nx + T - 1) / T, kl = (double)in.K * in.pb.L;
            // (wavefronts beyond the end of the grid have no nodes to do)
            const double tn = (in.nx + 64 * c.P - 1) / (64 * c.P) / (double)c.W;
            const double ex = in.pb.driver == BSDE_DRIVER_EXP ? q.exp * T / 64.0 * kl : 0.0;
            tiles += t;
            first += t * (q.first + q.first_node * kl + ex);
            more += t * (q.tile + (alone ? q.alone : 0.0)) +
                    tn * ((q.node + (alone ? q.alone_node : 0.0)) * kl + ex);
        }
        first = first / tiles + q.first_kb * kb;
        more = more / tiles + q.kb * kb;
        cost += first + (std::ceil(tiles / 256.0) - 1.0) * more;
    }
    return cost / 4.0;
}

// The cheapest fused shape and its time (us), or lds = 0 if none fits.
SweepConfig best_fused(const std::vector<Instance> &all, const std::vector<int> &members, bool f32,
                       size_t max_lds, double &cost)
{
    SweepConfig best{PATH_FUSED, 1, 1, 0, 4};
    cost = 0.0;
    auto consider = [&](const Shape &q) {
        const SweepConfig c = fused_config(all, members, q.P, q.W, q.G, max_lds);
        if (!c.lds) return;
        const double t = fused_cost(all, members, c, q);
        if (!best.lds || t < cost) {
            best = c;
            cost = t;
        }
    };
    if (f32)
        for (const Shape &q : kShapes32) consider(q);
    else
        for (const Shape &q : kShapes64) consider(q);
    return best;
}

// Which of the shapes fit an instance: instances of one group fit the same
// ones, so that none forces a smaller shape on the others.
unsigned fitting_shapes(const std::vector<Instance> &all, int b, size_t max_lds)
{
    unsigned mask = 0, bit = 1;
    auto test = [&](const Shape &q) {
        if (fused_config(all, {b}, q.P, q.W, q.G, max_lds).lds) mask |= bit;
        bit <<= 1;
    };
    if (all[b].f32)
        for (const Shape &q : kShapes32) test(q);
    else
        for (const Shape &q : kShapes64) test(q);
    return mask;
}

// Blocks per tile of the direct sweep with one point per lane: enough for
// about 1024 blocks on a small grid, at most 16 and at most the node chunks
// of a tile (its chunk sums go through the workspace).
int direct_splits(const std::vector<Instance> &all, const std::vector<int> &members)
{
    long tiles = 0;
    int chunks = 1;
    for (int b : members) {
        tiles += (all[b].nx + kBlock - 1) / kBlock;
        chunks = std::max(chunks, bsde::direct_chunks(all[b].K, all[b].pb.L));
    }
    const long want = (1024 + std::max(tiles, 1L) - 1) / std::max(tiles, 1L);
    return (int)std::max(1L, std::min<long>({want, 16L, (long)chunks}));
}

// Time of a step of a group with the direct kernel and its spline launch (us),
// as measured: n 64-point tiles a CU, three launches where a tile is split over
// blocks, else two and at least the chain of a tile's loads.  K = 4, L = 16:
// 14.4 us on 16384 points, 29.4 on 131072 (split), 35.0 on 262144, 118 on 1048576.
double direct_cost(const std::vector<Instance> &all, const std::vector<int> &members)
{
    double tiles = 0.0, node = 0.0, layers = 0.0;  // the latter two: tile by tile
    for (int b : members) {
        const Instance &in = all[b];
        const double t = (in.nx + 63) / 64;
        tiles += t;
        layers += t * in.K;
        node += t * in.K * in.pb.L;
    }
    const double n = std::ceil(tiles / 256.0), kl = node / tiles;
    const double ex = all[members[0]].pb.driver == BSDE_DRIVER_EXP ? 0.011 * kl : 0.0;
    if (direct_splits(all, members) > 1) return 11.7 + 0.25 * layers / tiles + n * (0.17 + 0.032 * kl + ex);
    return std::max(9.6 + 0.2 * kl, 7.2 + n * (0.17 + 0.0245 * kl + ex));
}

// Whether an instance takes the fused sweep: always where it fits in the FP32
// form (its sums, in another order, are part of the results).  In FP64 where it
// is the faster on this instance alone: windows so wide that only small tiles
// fit (one block of 64 points a CU) load more per point than the direct kernel
// reads.  K = 4, L = 16, stability ratio 105, a step: 6.6 us against 14.4 direct
// on 16384 points, 10.9 and 11.9 on 32768, 18.9 and 14.9 on 65536, 94 and 36 on
// 262144; ratio 90 on 262144 points: 38.1 and 35.5.  The rule looks at no other
// instance of a batch, so that a batch gives the bits of its instances alone; a
// large batch of small grids with such windows runs faster on the direct kernel
// (48 of 4000 points, ratio 105: 78 and 44 us a step), which bsde_autotune finds.
bool takes_fused(const std::vector<Instance> &all, int b, size_t max_lds)
{
    double fused = 0.0;
    const bool f32 = all[b].f32;
    if (!best_fused(all, {b}, f32, max_lds, fused).lds) return false;
    return f32 || fused <= direct_cost(all, {b});
}

// S: blocks per tile (P = 1 only); 0 picks direct_splits.
SweepConfig direct_config(const std::vector<Instance> &all, const std::vector<int> &members,
                          bool f32, int P, int S = 0)
{
    SweepConfig c;
    c.path = PATH_DIRECT;
    c.P = P;
    (void)f32;
    const int smax = P == 1 ? direct_splits(all, members) : 1;
    c.G = S > 0 ? std::min(S, smax) : smax;
    c.lds = 0;  // the direct kernel uses no LDS
    return c;
}

bool group_gathers(const std::vector<Instance> &all, const std::vector<int> &members)
{
    for (int b : members)
        if (all[b].gather) return true;
    return false;
}

bool group_exact(const std::vector<Instance> &all, const std::vector<int> &members)
{
    for (int b : members)
        if (all[b].exact) return true;
    return false;
}

// The Toeplitz sweep takes tiles of kToepTile points (P = 1) and splits every
// tile's band chunks over S blocks (carried in the G field) so that a group
// with few tiles still launches about 1024 blocks: S = ceil(1024 / tiles),
// at most 16 and at most the largest member's chunk count.
int toeplitz_splits(const std::vector<Instance> &all, const std::vector<int> &members)
{
    long tiles = 0;
    int chunks = 1;
    for (int b : members) {
        const Instance &in = all[b];
        tiles += (in.nx + bsde::kToepTile - 1) / bsde::kToepTile;
        int c = 0;
        for (int j = 1; j <= in.K; ++j) c += bsde::toeplitz_chunks((int)in.band[j].ev.size());
        chunks = std::max(chunks, c);
    }
    const long want = (1024 + std::max(tiles, 1L) - 1) / std::max(tiles, 1L);
    return (int)std::max(1L, std::min<long>({want, 16L, (long)chunks}));
}

// Windows, bands and LDS layout of a block of the exact-expectation sweep on
// B-spline coefficients.
struct ExactLds {
    int lo[bsde::kMaxOrder + 1], W[bsde::kMaxOrder + 1], shift[bsde::kMaxOrder + 1], steps[bsde::kMaxOrder + 1];
    int win[bsde::kMaxOrder + 1], band[bsde::kMaxOrder + 1], d, a, edge, part;
    size_t total;
};

ExactLds exact_layout(const Instance &in, int G)
{
    ExactLds l{};
    constexpr int T = bsde::kExactTile;
    size_t off = 0;
    for (int j = 1; j <= in.K; ++j) {
        const int nb = (int)in.band[j].ec.size();
        const int klo = in.band[j].klo - 1;  // first coefficient of the band
        l.steps[j] = (nb + 7 + 3) / 4;
        l.lo[j] = klo;
        int hi = klo + 4 * l.steps[j] + T - 8;  // one past the last record a step reads
        if (j == 1) {  // layer n+1's window holds the tile itself
            while (l.lo[j] > -1) l.lo[j] -= 8;  // and the point before it
            hi = std::max(hi, T);
        }
        l.shift[j] = klo - l.lo[j];
        l.W[j] = hi - l.lo[j];
        l.win[j] = (int)off;
        off += (size_t)(l.W[j] + l.W[j] / 8 + 1) * 16;
    }
    for (int j = 1; j <= in.K; ++j) {
        l.band[j] = (int)off;
        off += align_up((size_t)2 * (4 * l.steps[j] + 8) * sizeof(double), 16);
    }
    l.d = (int)off;
    off += (size_t)(l.W[1] + 2 * bsde::kHalo + 2 + bsde::kFirOver) * 16;
    l.a = (int)off;
    off += (size_t)(l.W[1] + 48 + bsde::kFirOver) * 16;
    l.edge = (int)off;
    off += (size_t)4 * in.K * 16;
    l.part = (int)off;
    off += (size_t)4 * G * T * 16;
    l.total = off;
    return l;
}

// Dynamic LDS of the exact-expectation sweep on B-spline coefficients, 0 where an
// instance's windows and bands do not fit (stability ratios from about 40 at K = 4).
size_t exact_lds(const Instance &in, int G, size_t max_lds)
{
    for (int j = 1; j <= in.K; ++j)
        if ((long)in.band[j].ec.size() > (long)(max_lds / 16) ||
            std::max({in.ex_il[j], in.ex_ir[j], in.ex_nl[j], in.ex_nr[j]}) > 32767)
            return 0;  // (the latter: packed in ExactHot; no band that fits comes near)
    const size_t need = exact_layout(in, G).total;
    return need <= max_lds ? need : 0;
}

// Exact expectations: the cheapest of the sweep on B-spline coefficients with one
// or two groups of four wavefronts (W = 1, where every member fits LDS) and the
// chunked sweep on values and second derivatives, by their measured times (us a
// step; n 64-point tiles a CU): a block of the former takes `lat` alone on a CU
// and hides most of it behind the others that the LDS leaves room for; the
// chunked sweep pays per tap.  Measured, one group / two / chunked: K = 4, ratio
// 16: 19.9, 13.0, 25.0 on 16384 points, 156, 107, 126 on 262144; ratio 4: 11.5,
// 9.9, 16.0 and 48, 69, 52; 1048576 points: 177, 267, 167; K = 2, ratio 45 (one
// block a CU), 262144 points: 164, 159, 131.  The choice follows the group's
// tiles, so a batch may sum in another order than its instances alone.
SweepConfig toeplitz_config(const std::vector<Instance> &all, const std::vector<int> &members, size_t max_lds)
{
    double tiles = 0.0, layers = 0.0, taps = 0.0;  // the latter two: tile by tile
    int chunks = 1;
    for (int b : members) {
        const Instance &in = all[b];
        const double t = (in.nx + bsde::kExactTile - 1) / bsde::kExactTile;
        tiles += t;
        layers += t * in.K;
        int c = 0;
        for (int j = 1; j <= in.K; ++j) {
            taps += t * (double)in.band[j].ev.size();
            c += bsde::toeplitz_chunks((int)in.band[j].ev.size());
        }
        chunks = std::max(chunks, c);
    }
    const double n = std::ceil(tiles / 256.0), K = layers / tiles;
    taps /= tiles;
    SweepConfig best{PATH_TOEPLITZ, 1, toeplitz_splits(all, members), bsde::toeplitz_lds_bytes()};
    // (split over blocks, on fewer than 1024 tiles, it needs partial sums in the
    // workspace and is at most 6% the faster)
    double cost = best.G > 1 ? 1e300 : 7.0 + K + 0.0075 * taps + n * (0.3 + 0.15 * K + 0.0046 * taps);
    for (int G = 1; G <= (chunks > 1 ? 2 : 1); ++G) {  // (two share more than one chunk of taps)
        size_t lds = 0;
        bool fits = true;
        for (int b : members) {
            const size_t need = exact_lds(all[b], G, max_lds);
            fits = fits && need > 0;
            lds = std::max(lds, need);
        }
        if (!fits) continue;
        const double kb = lds / 1024.0;
        const int res = (int)std::min((size_t)163840 / lds, (size_t)8 / G);
        const double lat = G == 1 ? 2.4 + 0.70 * K + 0.235 * kb : 3.6 + 0.87 * K + 0.09 * kb;
        constexpr double kShared2[5] = {0.0, -0.3, 1.3, 2.3, 2.0};
        const double shared = G == 2 ? kShared2[std::min(res, 4)] : res > 1 ? 0.6 + 0.07 * K : 0.0;
        const double t = lat + (n - 1.0) * ((lat - 2.5) / res + shared);
        if (t < cost) {
            cost = t;
            best = SweepConfig{PATH_TOEPLITZ, 1, G, lds, 1};
        }
    }
    return best;
}

constexpr size_t kLocatedLds = 131072;

// Shapes of the fused sweep for located nodes and their measured times (as
// kShapes64; the same bits).  Measured a step at K = 4, L = 16, ratio 16: 7.8 and
// 15.3 us on 16384 points, 16.3 and 16.1 on 65536, 51 and 34 on 262144.
constexpr Shape kLocatedShapes[] = {{1, 1, 8, 4.4, 0.034, 0.019, 1.45, 0.0185, 0.010, 2.5, 0.0, 0.0220},
                                    {1, 4, 1, 5.6, 0.145, 0.030, 1.20, 0.0820, 0.012, 4.2, 0.070, 0.0150}};

SweepConfig located_config(const std::vector<Instance> &all, const std::vector<int> &members, const Shape &q,
                           size_t max_lds)
{
    SweepConfig c = fused_config(all, members, q.P, q.W, q.G, max_lds);
    c.path = PATH_GATHER;
    return c;
}

// The cheaper of them and its time (us), or lds = 0.
SweepConfig best_located(const std::vector<Instance> &all, const std::vector<int> &members, size_t max_lds,
                         double &cost)
{
    SweepConfig best{PATH_GATHER, 1, 1, 0};
    cost = 0.0;
    for (const Shape &q : kLocatedShapes) {
        const SweepConfig c = located_config(all, members, q, max_lds);
        if (!c.lds) continue;
        const double t = fused_cost(all, members, c, q);
        if (!best.lds || t < cost) {
            best = c;
            cost = t;
        }
    }
    return best;
}

// Time of a step of a group with the kernel that reads HBM/L2, spline launch
// included (us), as measured: the chain of a point's nodes, and n 64-point tiles
// a CU once there are more than six.  K = 4, L = 16: 34 us on 65536 points, 62 on
// 262144, 183 on 1048576.
double gather_cost(const std::vector<Instance> &all, const std::vector<int> &members)
{
    double tiles = 0.0, node = 0.0;
    for (int b : members) {
        const double t = (all[b].nx + 63) / 64;
        tiles += t;
        node += t * all[b].K * all[b].pb.L;
    }
    const double n = std::ceil(tiles / 256.0), kl = node / tiles;
    const double ex = all[members[0]].pb.driver == BSDE_DRIVER_EXP ? 0.0186 * kl : 0.0;
    return 8.0 + 0.39 * kl + std::max(0.0, n - 6.0) * (0.23 + 0.037 * kl + ex);
}

// Whether an instance's located nodes go through LDS windows: where these take at
// most 128 KB for 64 points and the fused sweep is the faster on this instance
// alone (a rule on the instance, so that a batch gives the bits of its instances
// alone).  Measured a step, fused against HBM/L2: K = 4, L = 16, ratio 60 (102 KB)
// 18.7 and 34.3 us on 65536 points, 64.4 and 61.2 on 262144; K = 1, L = 8, ratio
// 120 9.0 and 12.0, 17.4 and 15.5; ratio 16 faster throughout (34 and 62 us on
// 262144 points).  The 128 KB are no speed limit: wider windows would be faster in
// LDS as well on grids up to about 60000 points (139 KB: 1.13 ms a solve and 4.35
// from HBM/L2 on 2001 points, 3.63 and 4.21 on 60000).  They keep the launches that
// bsde_profile_kernels has reported for them, a sweep and a spline launch a step.
bool takes_windows(const std::vector<Instance> &all, int b, size_t max_lds)
{
    if (!all[b].located) return false;
    const SweepConfig narrow = located_config(all, {b}, kLocatedShapes[0], max_lds);
    if (!narrow.lds || narrow.lds > kLocatedLds) return false;
    double t = 0.0;
    (void)best_located(all, {b}, max_lds, t);
    return t <= gather_cost(all, {b});
}

// State-dependent coefficients: in the fused sweep where every member is one for
// it (the same for all members of a plan's group), else from HBM/L2.
SweepConfig gather_config(const std::vector<Instance> &all, const std::vector<int> &members, size_t max_lds)
{
    bool windows = true;
    for (int b : members) windows = windows && takes_windows(all, b, max_lds);
    double t = 0.0;
    if (windows) return best_located(all, members, max_lds, t);
    return SweepConfig{PATH_GATHER, 1, 1, 0};
}

// Default shape: the fused kernel in the shape that the cost estimate favours;
// the direct kernel where that is faster (takes_fused) or no window fits in LDS.
// BSDE_SWEEP = "fused:P:G", "fused:P:G:W" or "direct:P:S" overrides;
// bsde_autotune replaces the choice by the fastest measured shape.
SweepConfig default_config(const std::vector<Instance> &all, const Group &g, size_t max_lds)
{
    if (group_gathers(all, g.members)) return gather_config(all, g.members, max_lds);
    if (group_exact(all, g.members)) return toeplitz_config(all, g.members, max_lds);
    const char *env = std::getenv("BSDE_SWEEP");
    if (env) {
        int P = 0, G = 1, W = 4;
        if (std::sscanf(env, "fused:%d:%d:%d", &P, &G, &W) >= 1 &&
            bsde::fused_supported(P, W, G, g.f32)) {
            SweepConfig c = fused_config(all, g.members, P, W, G, max_lds);
            if (c.lds) return c;
        }
        int S = 0;
        if (std::sscanf(env, "direct:%d:%d", &P, &S) >= 1 && bsde::direct_p_supported(P))
            return direct_config(all, g.members, g.f32, P, S);
    }
    bool fused = true;  // the same for every member of a plan's group
    for (int b : g.members) fused = fused && takes_fused(all, b, max_lds);
    if (fused) {
        double t = 0.0;
        const SweepConfig cf = best_fused(all, g.members, g.f32, max_lds, t);
        if (cf.lds) return cf;
    }
    // the direct kernel: split over blocks on a small grid, else two points per lane
    const SweepConfig c1 = direct_config(all, g.members, g.f32, 1);
    return c1.G > 1 ? c1 : direct_config(all, g.members, g.f32, 2);
}

// State-dependent coefficients in the fused sweep's LDS windows.
bool in_windows(const SweepConfig &c) { return c.path == PATH_GATHER && c.lds > 0; }

int sweep_tiles(const Instance &in, const SweepConfig &c)
{
    const int T = c.path == PATH_FUSED || in_windows(c) ? 64 * c.P * c.W
                  : c.path == PATH_TOEPLITZ && c.W == 1 ? bsde::kExactTile
                                                         : kBlock * c.P;
    return (in.nx + T - 1) / T;
}
int tiles_of(const Instance &in, int T) { return (in.nx + T - 1) / T; }
int spline_tiles(const Instance &in) { return (in.nx + bsde::kSplineTile - 1) / bsde::kSplineTile; }

// Bind a kernel shape to a group: tile numbering, descriptors, LDS limit (always
// the device's: the limit belongs to the kernel, which other plans launch too).
bsde_status apply_config(bsde_plan_s &pl, Group &g, const SweepConfig &c)
{
    if (c.path == PATH_FUSED && c.lds > 65536)
        HIP_OK(bsde::set_fused_lds_limit(c.P, c.W, c.G, g.f32, g.driver, pl.max_lds));
    const bool exact_b = c.path == PATH_TOEPLITZ && c.W == 1;  // on B-spline coefficients
    const bool located = in_windows(c);
    if (located && c.lds > 65536) HIP_OK(bsde::set_located_lds_limit(c.W, g.driver, pl.max_lds));
    if (exact_b && c.lds > 65536) HIP_OK(bsde::set_exact_lds_limit(c.G, pl.max_lds));
    if (c.path == PATH_TOEPLITZ && !exact_b && c.lds > 65536) HIP_OK(bsde::set_toeplitz_lds_limit());
    g.cfg = c;
    g.tile_prefix.assign(g.members.size() + 1, 0);
    g.spline_prefix.assign(g.members.size() + 1, 0);
    std::vector<int> tmap, smap;
    std::vector<int2> addr;  // of all members: one copy
    for (size_t k = 0; k < g.members.size(); ++k) {
        const int b = g.members[k];
        const Instance &in = pl.inst[b];
        bsde::InstDesc &d = pl.desc[b];
        d.tile_base = g.tile_prefix[k];
        d.spline_base = g.spline_prefix[k];
        d.spline_tiles = spline_tiles(in);
        d.a.ntiles = sweep_tiles(in, c);
        d.coef = (c.path == PATH_FUSED && !in.f32) || exact_b || located ? 1 : 0;
        if (exact_b) {
            const ExactLds l = exact_layout(in, c.G);
            bsde::ExactHot &h = d.ex;
            h.ring_off = d.ring_off;
            h.band = in.d_ex_band;
            h.corr = in.d_ex_corr;
            h.nx = in.nx;
            h.npad = in.npad;
            h.pad_l = in.pad_l;
            h.K = in.K;
            h.n0 = d.n0;
            h.n0_mod = d.n0 % (in.K + 1);
            h.mod_magic = (65536 + in.K) / (in.K + 1);
            h.tile_base = d.tile_base;
            h.ntiles = d.a.ntiles;
            h.lds_d = l.d;
            h.lds_a = l.a;
            h.lds_edge = l.edge;
            h.lds_part = l.part;
            for (int j = 1; j <= in.K; ++j) {
                h.lo[j] = l.lo[j];
                h.W[j] = l.W[j];
                h.shift[j] = l.shift[j];
                h.steps[j] = l.steps[j];
                h.lds_win[j] = l.win[j];
                h.lds_band[j] = l.band[j];
                h.nb[j] = (int)in.band[j].ec.size();
                h.boff[j] = in.ex_boff[j];
                h.cl[j] = in.ex_il[j] | in.ex_nl[j] << 16;
                h.cr[j] = in.ex_ir[j] | in.ex_nr[j] << 16;
                h.loff[j] = in.ex_loff[j];
                h.roff[j] = in.ex_roff[j];
            }
        }
        if (c.path == PATH_FUSED || located) {
            const FusedLds l = fused_layout(in, c.P, c.W, c.G);
            if (!in.f32) {  // (the FP32 form has the offsets)
                const std::vector<int2> own = fused_addresses(in, l, c.P);
                addr.insert(addr.end(), own.begin(), own.end());
            }
            bsde::FusedHot &h = d.hot;
            h.ring_off = d.ring_off;
            h.addr = in.d_addr;
            h.recb = in.d_recb;
            h.rec32 = d.a.tab.rec32;
            h.nx = in.nx;
            h.npad = in.npad;
            h.pad_l = in.pad_l;
            h.K = in.K;
            h.Ky = in.pb.k_y;
            h.L = in.pb.L;
            h.n0 = d.n0;
            h.n0_mod = d.n0 % (in.K + 1);
            h.mod_magic = (65536 + in.K) / (in.K + 1);
            h.tile_base = d.tile_base;
            h.ntiles = d.a.ntiles;
            for (int j = 0; j <= in.K; ++j) {
                h.win_lo[j] = in.win_lo[j];
                h.win_hi[j] = in.win_hi[j];
                h.lds_win[j] = l.win[j];
            }
            h.lds_d = l.d;
            h.lds_a = l.a;
            h.lds_edge = l.edge;
            h.lds_drv = l.drv;
            h.lds_tm = l.tm;
            h.m = d.a.tab.m;
            h.lds_part = l.part;
        }
        g.tile_prefix[k + 1] = g.tile_prefix[k] + d.a.ntiles;
        g.spline_prefix[k + 1] = g.spline_prefix[k] + d.spline_tiles;
        tmap.insert(tmap.end(), d.a.ntiles, b);
        smap.insert(smap.end(), d.spline_tiles, b);
    }
    // the maps and the addresses lie side by side: one copy
    char *const base = reinterpret_cast<char *>(g.d_tile_inst);
    const size_t smap_at = reinterpret_cast<char *>(g.d_spline_inst) - base;
    const size_t addr_at = addr.empty() ? 0 : reinterpret_cast<char *>(g.d_addr) - base;
    std::vector<char> maps(std::max(smap_at + smap.size() * sizeof(int), addr_at + addr.size() * sizeof(int2)));
    std::memcpy(maps.data(), tmap.data(), tmap.size() * sizeof(int));
    std::memcpy(maps.data() + smap_at, smap.data(), smap.size() * sizeof(int));
    if (!addr.empty()) std::memcpy(maps.data() + addr_at, addr.data(), addr.size() * sizeof(int2));
    HIP_OK(hipMemcpy(base, maps.data(), maps.size(), hipMemcpyHostToDevice));
    HIP_OK(hipMemcpy(pl.d_desc, pl.desc.data(), pl.desc.size() * sizeof(bsde::InstDesc),
                     hipMemcpyHostToDevice));
    pl.drop_graphs();
    return BSDE_OK;
}

// Optional per-launch timing with hipEvent pairs (profiling entry point).
struct KernelTimer {
    std::vector<hipEvent_t> sweep, spline;  // start/stop pairs, in launch order
    hipError_t mark(std::vector<hipEvent_t> &v, hipStream_t s)
    {
        hipEvent_t e;
        hipError_t rc = hipEventCreate(&e);
        if (rc != hipSuccess) return rc;
        v.push_back(e);
        return hipEventRecord(e, s);
    }
    ~KernelTimer()
    {
        for (hipEvent_t e : sweep) (void)hipEventDestroy(e);
        for (hipEvent_t e : spline) (void)hipEventDestroy(e);
    }
};

bsde::StepArgs step_args(const bsde_plan_s &pl, const Group &g, char *ws, int s, bool stats,
                         bool spline_map)
{
    bsde::StepArgs a;
    a.ws = ws;
    if (g.members.size() == 1) {  // no tile map: every block is of this instance
        a.desc = pl.d_desc + g.members[0];
        a.tile_inst = nullptr;
    } else {
        a.desc = pl.d_desc;
        a.tile_inst = spline_map ? g.d_spline_inst : g.d_tile_inst;
    }
    a.s = s;
    a.s_mod = s % 420;
    a.stats = stats ? 1 : 0;
    a.part = ((g.cfg.path == PATH_TOEPLITZ && g.cfg.W != 1) || g.cfg.path == PATH_DIRECT) && g.cfg.G > 1
                 ? reinterpret_cast<double *>(ws + g.part_off)
                 : nullptr;
    a.dsplit = g.cfg.path == PATH_DIRECT ? g.cfg.G : 1;
    a.dchunks = g.dchunks;
    return a;
}

// Step s of a group: layer n0 - s of every active member.
bsde_status enqueue_step(const bsde_plan_s &pl, const Group &g, char *ws, int s, bool stats,
                         hipStream_t st, KernelTimer *tm)
{
    const int act = g.active(s, pl.inst);
    if (act == 0) return BSDE_OK;
    const SweepConfig &c = g.cfg;
    const bsde::StepArgs a = step_args(pl, g, ws, s, stats, false);
    const int blocks = g.tile_prefix[act];
    if (tm) HIP_OK(tm->mark(tm->sweep, st));
    if (c.path == PATH_FUSED) {
        HIP_OK(bsde::launch_sweep_fused(c.P, c.W, c.G, g.f32, g.driver, a, blocks, c.lds, st));
        if (tm) HIP_OK(tm->mark(tm->sweep, st));
    } else {
        if (c.path == PATH_GATHER)
            HIP_OK(in_windows(c) ? bsde::launch_sweep_located(c.W, g.driver, a, blocks, c.lds, st)
                                 : bsde::launch_sweep_gather(g.f32, g.driver, a, blocks, st));
        else if (c.path == PATH_TOEPLITZ)
            HIP_OK(c.W == 1 ? bsde::launch_sweep_exact(a, blocks, c.G, c.lds, st)
                            : bsde::launch_sweep_toeplitz(a, blocks, c.G, st));
        else
            HIP_OK(bsde::launch_sweep_direct(c.P, g.f32, g.driver, a, blocks, c.lds, st));
        if (tm) HIP_OK(tm->mark(tm->sweep, st));
        // natural spline of the new layer (the fused kernel does this in-kernel,
        // and so do the Toeplitz sweep on coefficients and the split one's
        // finishing kernel)
        if (c.path == PATH_TOEPLITZ && (c.W == 1 || c.G > 1)) return BSDE_OK;
        if (in_windows(c)) return BSDE_OK;
        if (tm) HIP_OK(tm->mark(tm->spline, st));
        HIP_OK(bsde::launch_spline(g.f32, step_args(pl, g, ws, s, false, true), 1,
                                   g.spline_prefix[act], st));
        if (tm) HIP_OK(tm->mark(tm->spline, st));
    }
    return BSDE_OK;
}

// Initial layers (scatter + splines) of every instance.
bsde_status enqueue_init(const bsde_plan_s &pl, char *ws, const bsde_io *io, hipStream_t s)
{
    const int count = (int)pl.inst.size();
    for (int b0 = 0; b0 < count; b0 += bsde::kChunk) {
        bsde::ScatterChunk c{};
        c.count = std::min(bsde::kChunk, count - b0);
        int nxmax = 1;
        for (int k = 0; k < c.count; ++k) {
            c.inst[k] = b0 + k;
            c.iy[k] = io[b0 + k].init_y;
            c.iz[k] = io[b0 + k].init_z;
            nxmax = std::max(nxmax, pl.inst[b0 + k].nx);
        }
        const int bx = std::min(1024, (nxmax + kBlock - 1) / kBlock);
        HIP_OK(bsde::launch_scatter(c, ws, pl.d_desc, bx, s));
    }
    for (const Group &g : pl.groups) {
        int kmax = 0;
        for (int b : g.members) kmax = std::max(kmax, pl.inst[b].K);
        // groups that keep a layer's spline by its B-spline coefficients
        const bool coef = pl.desc[g.members[0]].coef != 0;
        for (int r = 0; r < kmax; ++r) {
            const bsde::StepArgs a = step_args(pl, g, ws, r, false, true);
            HIP_OK(coef ? bsde::launch_coef(a, g.spline_prefix.back(), s)
                        : bsde::launch_spline(g.f32, a, 0, g.spline_prefix.back(), s));
        }
    }
    return BSDE_OK;
}

bsde_status enqueue_gather(const bsde_plan_s &pl, char *ws, const bsde_io *io,
                           unsigned long long *nonfinite, hipStream_t s)
{
    const int count = (int)pl.inst.size();
    for (int b0 = 0; b0 < count; b0 += bsde::kChunk) {
        bsde::GatherChunk c{};
        c.count = std::min(bsde::kChunk, count - b0);
        int nxmax = 1;
        for (int k = 0; k < c.count; ++k) {
            c.inst[k] = b0 + k;
            c.y0[k] = io[b0 + k].y0;
            c.z0[k] = io[b0 + k].z0;
            nxmax = std::max(nxmax, pl.inst[b0 + k].nx);
        }
        const int bx = std::min(1024, (nxmax + kBlock - 1) / kBlock);
        HIP_OK(bsde::launch_gather(c, ws, pl.d_desc, bx, nonfinite, s));
    }
    return BSDE_OK;
}

// Two-dimensional plan: per instance, initial layers (values, tensor splines,
// ghosts) -> per step the sweep and the splines of the new layer -> outputs.
bsde_status enqueue_solve2(const bsde_plan_s &pl, char *ws, const bsde_io *io, bool stats,
                           unsigned long long *nonfinite, hipStream_t s, KernelTimer *tm)
{
    for (size_t b = 0; b < pl.inst2.size(); ++b) {
        const Instance2 &in = pl.inst2[b];
        bsde::Sweep2Args a = sweep2_args(in, ws, stats);
        bsde::SplineFilter f = pl.filter2;
        f.s6[0] = 6.0 / (in.dx0 * in.dx0) * pl.pcr_base.inv_b;
        f.s6[1] = 6.0 / (in.dx1 * in.dx1) * pl.pcr_base.inv_b;
        const int N = in.pb.n_t, K = in.K;
        a.n = N - K;
        // the derivative planes of a layer: tensor spline or finite differences
        auto interp_layer = [&](int slot) {
            if (in.bspline) return bsde::launch_coef2d(a, slot, s);
            return in.pb.interp == BSDE_INTERP_BICUBIC_FD
                       ? bsde::launch_fd2d(in.f32, a, slot, in.dx0, in.dx1, s)
                       : bsde::launch_spline2d(a, slot, f, s);
        };
        HIP_OK(bsde::launch_scatter2d(in.f32, a, io[b].init_y, io[b].init_z, s));
        for (int r = 0; r < K; ++r) HIP_OK(interp_layer((N - K + 1 + r) % (K + 1)));
        for (int n = N - K; n >= in.pb.n_stop; --n) {
            a.n = n;
            if (tm) HIP_OK(tm->mark(tm->sweep, s));
            HIP_OK(in.bspline ? bsde::launch_sweep2b(a, s) : bsde::launch_sweep2d(in.f32, a, s));
            if (tm) HIP_OK(tm->mark(tm->sweep, s));
            if (n > in.pb.n_stop) {
                if (tm) HIP_OK(tm->mark(tm->spline, s));
                HIP_OK(interp_layer(n % (K + 1)));
                if (tm) HIP_OK(tm->mark(tm->spline, s));
            }
        }
        HIP_OK(bsde::launch_gather2d(a, io[b].y0, io[b].z0, nonfinite, s));
    }
    return BSDE_OK;
}

// The whole solve: initial layers -> backward loop (all groups, step by
// step) -> outputs.
bsde_status enqueue_solve(const bsde_plan_s &pl, char *ws, const bsde_io *io, bool stats,
                          unsigned long long *nonfinite, hipStream_t s, KernelTimer *tm = nullptr)
{
    if (!pl.inst2.empty()) return enqueue_solve2(pl, ws, io, stats, nonfinite, s, tm);
    bsde_status rc = enqueue_init(pl, ws, io, s);
    if (rc != BSDE_OK) return rc;
    int smax = 0;
    for (const Group &g : pl.groups) smax = std::max(smax, g.max_steps);
    for (int st = 0; st < smax; ++st)
        for (const Group &g : pl.groups) {
            rc = enqueue_step(pl, g, ws, st, stats, s, tm);
            if (rc != BSDE_OK) return rc;
        }
    return enqueue_gather(pl, ws, io, nonfinite, s);
}

bsde_status finish_stats(bsde_plan_t plan, char *ws, hipStream_t s, hipEvent_t e0, hipEvent_t e1,
                         bsde_stats *st)
{
    const int count = (int)plan->desc.size();
    unsigned long long *tot = reinterpret_cast<unsigned long long *>(ws + plan->totals_off);
    HIP_OK(bsde::launch_reduce_stats(ws, plan->d_desc, count, tot, s));
    std::vector<unsigned long long> h(3 * (size_t)count + 1);
    HIP_OK(hipMemcpyAsync(h.data(), tot, h.size() * sizeof(unsigned long long),
                          hipMemcpyDeviceToHost, s));
    HIP_OK(hipStreamSynchronize(s));
    unsigned long long mx = 0, sum = 0, nonc = 0;
    long long point_steps = 0;
    double R = 0.0;
    int unstable = 0;
    for (int b = 0; b < count; ++b) {
        mx = std::max(mx, h[3 * b]);
        sum += h[3 * b + 1];
        nonc += h[3 * b + 2];
        if (plan->inst2.empty()) {
            const Instance &in = plan->inst[b];
            point_steps += (long long)in.nx * in.steps;
            R = std::max(R, in.R);
            unstable += beyond_stability_limit(in.R) ? 1 : 0;
        } else {
            const Instance2 &in = plan->inst2[b];
            point_steps += (long long)in.n0 * in.n1 * (in.pb.n_t - in.K - in.pb.n_stop + 1);
            R = std::max(R, in.R);
            unstable += beyond_stability_limit(in.R) ? 1 : 0;
        }
    }
    float ms = 0.0f;
    HIP_OK(hipEventElapsedTime(&ms, e0, e1));
    st->picard_iter_max = (int)mx;
    st->picard_iter_mean = point_steps ? (double)sum / (double)point_steps : 0.0;
    st->picard_nonconverged = (long long)nonc;
    st->nonfinite = (long long)h[3 * (size_t)count];
    st->stability_ratio = R;
    st->unstable_instances = unstable;
    st->elapsed_ms = ms;
    if (st->nonfinite) return BSDE_ENONFINITE;
    if (st->picard_nonconverged) return BSDE_ENOCONV;
    return BSDE_OK;
}

bool same_io(const std::vector<bsde_io> &a, const bsde_io *b, int count)
{
    if ((int)a.size() != count) return false;
    for (int i = 0; i < count; ++i)
        if (a[i].init_y != b[i].init_y || a[i].init_z != b[i].init_z || a[i].y0 != b[i].y0 ||
            a[i].z0 != b[i].z0)
            return false;
    return true;
}

// The whole solve, replayed as one hipGraph launch: one capture per
// (workspace, buffers, statistics flag), kept in a small least-recently-used
// cache.  The graph holds kernel nodes only.
bsde_status launch_graph(bsde_plan_t plan, char *w, const bsde_io *io, int count, bool stats,
                         unsigned long long *nonfinite, hipStream_t s)
{
    std::lock_guard<std::mutex> lock(plan->mu);
    GraphEntry *hit = nullptr;
    for (GraphEntry &g : plan->graphs)
        if (g.ws == w && g.stats == stats && same_io(g.io, io, count)) hit = &g;
    if (!hit) {
        if (!plan->capture_stream)
            HIP_OK(hipStreamCreateWithFlags(&plan->capture_stream, hipStreamNonBlocking));
        hipStream_t cs = plan->capture_stream;
        HIP_OK(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
        const bsde_status rc = enqueue_solve(*plan, w, io, stats, nonfinite, cs);
        hipGraph_t graph = nullptr;
        const hipError_t ec = hipStreamEndCapture(cs, &graph);
        if (rc != BSDE_OK || ec != hipSuccess) {
            if (graph) (void)hipGraphDestroy(graph);
            return rc != BSDE_OK ? rc : BSDE_EDEVICE;
        }
        hipGraphExec_t exec = nullptr;
        const hipError_t ei = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (ei != hipSuccess) return BSDE_EDEVICE;
        if ((int)plan->graphs.size() >= kMaxGraphs) {
            auto lru = std::min_element(plan->graphs.begin(), plan->graphs.end(),
                                        [](const GraphEntry &x, const GraphEntry &y) {
                                            return x.last_use < y.last_use;
                                        });
            (void)hipGraphExecDestroy(lru->exec);
            plan->graphs.erase(lru);
        }
        GraphEntry e;
        e.ws = w;
        e.io.assign(io, io + count);
        e.stats = stats;
        e.exec = exec;
        plan->graphs.push_back(e);
        hit = &plan->graphs.back();
    }
    hit->last_use = ++plan->clock;
    HIP_OK(hipGraphLaunch(hit->exec, s));
    return BSDE_OK;
}

bool valid_io(bsde_plan_t plan, void *ws, const bsde_io *io, int count)
{
    if (!plan || !ws || !io) return false;
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return false;
    for (int b = 0; b < count; ++b)
        if (!io[b].init_y || !io[b].init_z || !io[b].y0 || !io[b].z0) return false;
    return true;
}

// Two hipEvents released on every path out of the scope that made them.
struct EventPair {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    bool create() { return hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess; }
    ~EventPair()
    {
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    }
};

bsde_status solve_impl(bsde_plan_t plan, void *ws, const bsde_io *io, int count, void *stream,
                       bsde_stats *st)
{
    if (!valid_io(plan, ws, io, count)) return BSDE_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *w = static_cast<char *>(ws);
    const bool stats = st != nullptr;
    EventPair ev;
    unsigned long long *nonfinite = nullptr;
    if (stats) {
        if (!ev.create()) return BSDE_EDEVICE;
        HIP_OK(hipEventRecord(ev.e0, s));
        // per-wave counters and the totals start at zero
        HIP_OK(bsde::launch_clear(reinterpret_cast<unsigned long long *>(w + plan->stats_off),
                                  plan->stats_bytes / 8, s));
        nonfinite = reinterpret_cast<unsigned long long *>(w + plan->totals_off) + 3 * count;
    }
    bsde_status rc = plan->use_graphs ? launch_graph(plan, w, io, count, stats, nonfinite, s)
                                      : enqueue_solve(*plan, w, io, stats, nonfinite, s);
    if (rc != BSDE_OK) return rc;
    if (!stats) return BSDE_OK;
    HIP_OK(hipEventRecord(ev.e1, s));
    HIP_OK(hipEventSynchronize(ev.e1));
    return finish_stats(plan, w, s, ev.e0, ev.e1, st);
}

}  // namespace

// --------------------------------------------------------------------------
// Plans of two-dimensional problems
// --------------------------------------------------------------------------
namespace {

void pcr_base_coefficients(bsde::PcrCoef &c)
{
    // PCR coefficients of the (1, 4, 1) system: round r eliminates the
    // neighbours at distance 2^r; a' = -a^2/b, b' = b - 2a^2/b
    double av = 1.0, bv = 4.0;
    for (int r = 0; r < bsde::kPcrRounds; ++r) {
        const double k = av / bv;
        c.kappa[r] = k;
        bv = bv - 2.0 * k * av;
        av = -k * av;
    }
    c.inv_b = 1.0 / bv;
    c.s6 = 0.0;
}

// The truncated PCR's filters (compile-time constants of the (1, 4, 1)
// system); the per-axis scale s6 is set per instance.
void pcr_filter(bsde::SplineFilter &f)
{
    constexpr bsde::SplineTaps t = bsde::spline_taps();
    for (int k = 0; k < bsde::kPcrTaps; ++k) f.c[k] = t.c[k];
    for (int k = 0; k < bsde::kPcrTaps + 2; ++k) f.d[k] = t.d[k];
    f.s6[0] = f.s6[1] = 0.0;
}

bsde_status plan_2d(const bsde_problem *pb, int batch, bsde_plan_t *out)
{
    for (int b = 0; b < batch; ++b)
        if (!supported_2d(pb[b])) return BSDE_EUNSUPPORTED;
    bsde_plan_s *pl = new (std::nothrow) bsde_plan_s;
    if (!pl) return BSDE_ENOMEM;
    pl->inst2.resize(batch);
    for (int b = 0; b < batch; ++b) {
        const bsde_status rc = build_instance2(pb[b], pl->inst2[b]);
        if (rc != BSDE_OK) {
            delete pl;
            return rc;
        }
    }
    pcr_base_coefficients(pl->pcr_base);
    pcr_filter(pl->filter2);
    char *sw = nullptr;
    if (hipGetDevice(&pl->device) != hipSuccess || static_workspace(pl->device, &sw) != BSDE_OK) {
        delete pl;
        return BSDE_EDEVICE;
    }
    int lds_limit = 65536;
    if (hipDeviceGetAttribute(&lds_limit, hipDeviceAttributeMaxSharedMemoryPerBlock,
                              pl->device) != hipSuccess) {
        delete pl;
        return BSDE_EDEVICE;
    }
    pl->max_lds = (size_t)lds_limit;
    {
        const char *g = std::getenv("BSDE_GRAPH");
        pl->use_graphs = !(g && g[0] == '0');
    }
    // device tables: node rows, nodes, axis-1 offsets; descriptors (statistics)
    size_t tbytes = 0;
    std::vector<size_t> toff(batch);
    for (int b = 0; b < batch; ++b) {
        const Instance2 &in = pl->inst2[b];
        toff[b] = tbytes;
        tbytes += (in.bspline ? 0 : align_up(in.rows.size() * sizeof(bsde::Node2Row), 256)) +
                  align_up(in.nodes.size() * sizeof(bsde::Node2), 256) +
                  align_up(in.m1.size() * sizeof(int), 256) +
                  align_up(in.rowsb.size() * sizeof(bsde::Row2B), 256) +
                  align_up(in.nodesb.size() * sizeof(bsde::Node2B), 256) +
                  align_up(in.corr_l.size() * sizeof(double4), 256) +
                  align_up(in.corr_r.size() * sizeof(double4), 256);
    }
    const size_t desc_off = tbytes;
    tbytes += align_up((size_t)batch * sizeof(bsde::InstDesc), 256);
    if (hipMalloc(&pl->d_tables, tbytes) != hipSuccess) {
        delete pl;
        return BSDE_ENOMEM;
    }
    char *dev = static_cast<char *>(pl->d_tables);
    std::vector<char> host(desc_off);
    for (int b = 0; b < batch; ++b) {
        Instance2 &in = pl->inst2[b];
        size_t o = toff[b];
        auto put = [&](const void *src, size_t bytes) {
            std::memcpy(host.data() + o, src, bytes);
            void *d = dev + o;
            o += align_up(bytes, 256);
            return d;
        };
        if (!in.bspline) {
            in.d_rows = static_cast<const bsde::Node2Row *>(
                put(in.rows.data(), in.rows.size() * sizeof(bsde::Node2Row)));
            in.d_nodes =
                static_cast<const bsde::Node2 *>(put(in.nodes.data(), in.nodes.size() * sizeof(bsde::Node2)));
        }
        in.d_m1 = static_cast<const int *>(put(in.m1.data(), in.m1.size() * sizeof(int)));
        if (in.bspline) {
            in.d_rowsb = static_cast<const bsde::Row2B *>(
                put(in.rowsb.data(), in.rowsb.size() * sizeof(bsde::Row2B)));
            in.d_nodesb = static_cast<const bsde::Node2B *>(
                put(in.nodesb.data(), in.nodesb.size() * sizeof(bsde::Node2B)));
            in.d_corr_l = static_cast<const double4 *>(
                put(in.corr_l.data(), in.corr_l.size() * sizeof(double4)));
            in.d_corr_r = static_cast<const double4 *>(
                put(in.corr_r.data(), in.corr_r.size() * sizeof(double4)));
        }
        // the kernel's limit, which other plans launch too: the device's
        const size_t lds = in.bspline ? bsde::kGroups2B * bsde::sweep2b_wave_lds(in.spread)
                                      : 2 * bsde::sweep2d_lds((in.win + 1) / 2);
        if (lds > 65536 && (in.bspline ? bsde::set_sweep2b_lds_limit(pl->max_lds)
                                       : bsde::set_sweep2d_lds_limit(in.f32, pl->max_lds)) != hipSuccess) {
            bsde_plan_destroy(pl);
            return BSDE_EDEVICE;
        }
    }
    // workspace: rings (6 planes of doubles per layer in the B-spline form, 12
    // with the bicubic, or 15 of floats in the FP32 form), final layers, statistics
    size_t off = 0;
    for (Instance2 &in : pl->inst2) {
        in.ring_off = off;
        off += align_up((size_t)in.planes() * (in.f32 ? sizeof(float) : sizeof(double)) * (in.K + 1) *
                            in.plane,
                        256);
        if (in.bspline) {  // between the two passes of the spline
            in.tmp_off = off;
            off += align_up((size_t)3 * sizeof(double) * in.plane, 256);
        }
    }
    for (Instance2 &in : pl->inst2) {
        in.fin_off = off;
        off += align_up((size_t)3 * in.n0 * in.n1 * sizeof(double), 256);
    }
    pl->stats_off = off;
    for (Instance2 &in : pl->inst2) {
        in.stat_off = off;
        off += align_up((size_t)in.nwaves * (2 * sizeof(unsigned long long) + sizeof(unsigned int)),
                        256);
    }
    pl->totals_off = off;
    off += align_up((3 * (size_t)batch + 1) * sizeof(unsigned long long), 256);
    pl->stats_bytes = off - pl->stats_off;
    pl->ws_bytes = off;
    pl->desc.resize(batch);
    for (int b = 0; b < batch; ++b) {
        bsde::InstDesc &d = pl->desc[b];
        std::memset(&d, 0, sizeof(d));
        d.stat_off = pl->inst2[b].stat_off;
        d.nwaves = pl->inst2[b].nwaves;
    }
    pl->d_desc = reinterpret_cast<bsde::InstDesc *>(dev + desc_off);
    if (hipMemcpy(pl->d_tables, host.data(), desc_off, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(pl->d_desc, pl->desc.data(), batch * sizeof(bsde::InstDesc),
                  hipMemcpyHostToDevice) != hipSuccess) {
        bsde_plan_destroy(pl);
        return BSDE_EDEVICE;
    }
    *out = pl;
    return BSDE_OK;
}

}  // namespace

// --------------------------------------------------------------------------
// C ABI
// --------------------------------------------------------------------------
extern "C" {

const char *bsde_status_string(bsde_status s)
{
    // a C caller may pass any int: read it as one (a value outside the
    // enumeration would be undefined as a C++ enum value)
    int v;
    std::memcpy(&v, &s, sizeof(v));
    switch (v) {
    case BSDE_OK: return "ok";
    case BSDE_EINVAL: return "invalid argument";
    case BSDE_ENOMEM: return "out of memory";
    case BSDE_EDEVICE: return "device (HIP) error";
    case BSDE_EUNSUPPORTED: return "unsupported problem";
    case BSDE_ENOCONV: return "Picard iteration did not converge at some point";
    case BSDE_ENONFINITE: return "non-finite value in the output";
    case BSDE_ESCRATCH:
        return "workspace larger than the static workspace (BSDE_STATIC_WORKSPACE_BYTES)";
    }
    return "unknown status";
}

bsde_status bsde_gauss_hermite(int L, double *a, double *w)
{
    if (!a || !w) return BSDE_EINVAL;
    return bsde::gauss_hermite(L, a, w) ? BSDE_OK : BSDE_EINVAL;
}

bsde_status bsde_gamma(int table, int K, double *g)
{
    if (!g) return BSDE_EINVAL;
    return bsde::spline_gamma(table, K, g) ? BSDE_OK : BSDE_EINVAL;
}

bsde_status bsde_initial_layers(const bsde_problem *pb, int substeps, void *ws, size_t ws_bytes,
                                double *init_y, double *init_z, void *stream)
{
    if (!pb || !ws || !init_y || !init_z || substeps < 1) return BSDE_EINVAL;
    if (!valid_problem(*pb)) return BSDE_EINVAL;
    const int K = std::max(pb->k_y, pb->k_z);
    const size_t np = pb->d == 1 ? (size_t)pb->n_x[0] : (size_t)pb->n_x[0] * pb->n_x[1];
    const double dt = pb->T / pb->n_t;
    // every segment plan has n_t = (N - r + 1) substeps steps; the count must
    // stay an int
    if ((long long)pb->n_t * substeps > INT32_MAX / 2) return BSDE_EINVAL;
    // The segments' plans (and their device tables) outlive the enqueued work:
    // one wait after the last segment, so a plan is made while the segment
    // before it runs (16384 points, K = 4, L = 32, 8 sub-steps: 545 -> 418 us).
    bsde_plan_t plans[bsde::kMaxOrder] = {};
    int made = 0;
    bsde_status rc = BSDE_OK;
    for (int r = 1; r < K && rc == BSDE_OK; ++r) {
        // layer t_{N-r} from t_{N-r+1}: the 1-step scheme (K_y = K_z = 1) over
        // substeps steps of dt / substeps, absolute times kept (t = n dt')
        bsde_problem q = *pb;
        const int n_hi = pb->n_t - r + 1;
        q.k_y = q.k_z = 1;
        q.T = n_hi * dt;
        q.n_t = n_hi * substeps;
        q.n_stop = (n_hi - 1) * substeps;
        // coefficients tabulated per step: the row of t_{N-r}, held over the
        // segment's sub-steps
        if (pb->tab_steps > 1) {
            q.tab_steps = 1;
            q.coef_tab = pb->coef_tab + (size_t)2 * (pb->n_t - r) * pb->n_x[0];
        }
        bsde_plan_t plan = nullptr;
        rc = bsde_plan(&q, 1, &plan);
        if (rc != BSDE_OK) break;
        plans[made++] = plan;
        plan->use_graphs = false;  // solved once: launch directly, no capture
        if (bsde_workspace_bytes(plan) > ws_bytes) {
            rc = BSDE_EINVAL;
            break;
        }
        const bsde_io io{init_y + (size_t)(K - r) * np, init_z + (size_t)(K - r) * np * pb->d,
                         init_y + (size_t)(K - 1 - r) * np,
                         init_z + (size_t)(K - 1 - r) * np * pb->d};
        rc = bsde_solve_batched(plan, ws, &io, stream, nullptr);
    }
    const hipError_t e = made ? hipStreamSynchronize(static_cast<hipStream_t>(stream)) : hipSuccess;
    for (int i = 0; i < made; ++i) bsde_plan_destroy(plans[i]);
    if (rc != BSDE_OK) return rc;
    return e == hipSuccess ? BSDE_OK : BSDE_EDEVICE;
}

bsde_status bsde_problem_info(const bsde_problem *pb, bsde_problem_info_t *info)
{
    if (!pb || !info) return BSDE_EINVAL;
    if (!valid_problem(*pb)) return BSDE_EINVAL;
    bsde_problem_info_t r{};
    r.K = std::max(pb->k_y, pb->k_z);
    if (pb->d == 1) {
        Instance in;
        if (!build_instance(*pb, in)) return BSDE_EINVAL;
        r.stability_ratio = in.R;
        r.node_reach = in.reach;
        r.supported = supported_1d(*pb) ? 1 : 0;
    } else {
        Instance2 in;
        r.supported = supported_2d(*pb) ? 1 : 0;
        if (r.supported) {
            const bsde_status rc = build_instance2(*pb, in);
            if (rc == BSDE_EUNSUPPORTED) r.supported = 0;
            else if (rc != BSDE_OK) return rc;
        }
        const double dx0 = (pb->x_max[0] - pb->x_min[0]) / (pb->n_x[0] - 1);
        const double dx1 = (pb->x_max[1] - pb->x_min[1]) / (pb->n_x[1] - 1);
        const double dt = pb->T / pb->n_t;
        r.stability_ratio =
            std::max(std::hypot(pb->vol[0][0], pb->vol[0][1]) / dx0,
                     std::hypot(pb->vol[1][0], pb->vol[1][1]) / dx1) * std::sqrt(2.0 * dt);
        r.node_reach = r.supported ? in.reach : 0;
    }
    r.stable = beyond_stability_limit(r.stability_ratio) ? 0 : 1;
    *info = r;
    return BSDE_OK;
}

bsde_status bsde_plan(const bsde_problem *pb, int batch, bsde_plan_t *out)
{
    if (!pb || !out || batch < 1) return BSDE_EINVAL;
    for (int b = 0; b < batch; ++b) {
        if (!valid_problem(pb[b])) return BSDE_EINVAL;
        if (pb[b].d != pb[0].d) return BSDE_EINVAL;
    }
    if (pb[0].d == 2) return plan_2d(pb, batch, out);
    bsde_plan_s *pl = new (std::nothrow) bsde_plan_s;
    if (!pl) return BSDE_ENOMEM;
    pl->inst.resize(batch);
    for (int b = 0; b < batch; ++b) {
        if (!supported_1d(pb[b])) {
            delete pl;
            return BSDE_EUNSUPPORTED;
        }
        if (!build_instance(pb[b], pl->inst[b])) {
            delete pl;
            return BSDE_EINVAL;
        }
        // the kernels address a ring plane by 32-bit byte offsets
        const Instance &in = pl->inst[b];
        if ((uint64_t)in.npad * (in.f32 ? sizeof(float2) : sizeof(double2)) >= (uint64_t(1) << 32)) {
            delete pl;
            return BSDE_EUNSUPPORTED;
        }
    }
    // PCR coefficients of the (1, 4, 1) system: round r eliminates the
    // neighbours at distance 2^r; a' = -a^2/b, b' = b - 2a^2/b
    {
        double av = 1.0, bv = 4.0;
        for (int r = 0; r < bsde::kPcrRounds; ++r) {
            const double k = av / bv;
            pl->pcr_base.kappa[r] = k;
            bv = bv - 2.0 * k * av;
            av = -k * av;
        }
        pl->pcr_base.inv_b = 1.0 / bv;
        pl->pcr_base.s6 = 0.0;
    }
    char *sw = nullptr;
    if (hipGetDevice(&pl->device) != hipSuccess || static_workspace(pl->device, &sw) != BSDE_OK) {
        delete pl;
        return BSDE_EDEVICE;
    }
    int lds_limit = 65536;
    if (hipDeviceGetAttribute(&lds_limit, hipDeviceAttributeMaxSharedMemoryPerBlock,
                              pl->device) != hipSuccess) {
        delete pl;
        return BSDE_EDEVICE;
    }
    pl->max_lds = (size_t)lds_limit;
    {
        const char *g = std::getenv("BSDE_GRAPH");
        pl->use_graphs = !(g && g[0] == '0');
    }
    // groups: same precision, driver and default kernel shape (an instance
    // whose windows do not fit a shape does not force it on the others);
    // members by number of steps, most first
    std::vector<SweepConfig> own(batch);
    std::vector<unsigned> fits(batch, 0);
    for (int b = 0; b < batch; ++b) {
        Instance &in = pl->inst[b];
        Group one;
        one.f32 = in.f32;
        one.members = {b};
        own[b] = default_config(pl->inst, one, pl->max_lds);
        if (own[b].path == PATH_FUSED) fits[b] = fitting_shapes(pl->inst, b, pl->max_lds);
        if (own[b].path == PATH_TOEPLITZ) fits[b] = exact_lds(in, 2, pl->max_lds) ? 1 : 0;
        if (own[b].path == PATH_GATHER) fits[b] = in_windows(own[b]) ? 1 : 0;
        int gi = -1;
        for (size_t k = 0; k < pl->groups.size(); ++k) {
            const Group &g = pl->groups[k];
            const SweepConfig &c = own[g.members[0]];
            // the shape of the fused sweep and the split count of the Toeplitz
            // and direct sweeps follow the group
            if (g.f32 == in.f32 && g.driver == in.pb.driver && c.path == own[b].path &&
                (c.path != PATH_DIRECT || c.P == own[b].P) && fits[g.members[0]] == fits[b])
                gi = (int)k;
        }
        if (gi < 0) {
            pl->groups.emplace_back();
            pl->groups.back().f32 = in.f32;
            pl->groups.back().driver = in.pb.driver;
            gi = (int)pl->groups.size() - 1;
        }
        in.group = gi;
        pl->groups[gi].members.push_back(b);
    }
    for (Group &g : pl->groups) {
        std::stable_sort(g.members.begin(), g.members.end(), [&](int x, int y) {
            return pl->inst[x].steps > pl->inst[y].steps;
        });
        g.max_steps = pl->inst[g.members[0]].steps;
    }
    // device tables: per instance node records (of its form) and offsets; the
    // descriptors (with the window bounds); per group the tile maps
    size_t tbytes = 0;
    std::vector<size_t> toff(batch);
    for (int b = 0; b < batch; ++b) {
        const Instance &in = pl->inst[b];
        toff[b] = tbytes;
        const size_t kl = (size_t)in.K * in.pb.L;
        tbytes += align_up(kl * sizeof(int), 256) + align_up(kl * sizeof(double), 256) +
                  (in.f32 ? align_up(kl * sizeof(bsde::NodeRec32), 256)
                          : align_up(kl * sizeof(bsde::NodeRec), 256) + align_up(kl * sizeof(bsde::NodeRecB), 256));
        size_t nbw = 0;
        for (int j = 1; j <= in.K; ++j) nbw += 4 * in.band[j].ev.size();
        tbytes += align_up(nbw * sizeof(double), 256) + align_up(in.ex_band.size() * sizeof(double), 256) +
                  align_up(in.ex_corr.size() * sizeof(double2), 256);
        tbytes += align_up(in.ctab.size() * sizeof(double), 256);
    }
    const size_t desc_off = tbytes;
    tbytes += align_up((size_t)batch * sizeof(bsde::InstDesc), 256);
    std::vector<size_t> map_off(pl->groups.size()), addr_off(pl->groups.size());
    for (size_t k = 0; k < pl->groups.size(); ++k) {
        size_t tiles = 0, stiles = 0, nodes = 0;
        for (int b : pl->groups[k].members) {
            tiles += tiles_of(pl->inst[b], kMinTile);
            stiles += spline_tiles(pl->inst[b]);
            nodes += (size_t)pl->inst[b].K * pl->inst[b].pb.L;
        }
        map_off[k] = tbytes;
        tbytes += align_up(tiles * sizeof(int), 256) + align_up(stiles * sizeof(int), 256);
        addr_off[k] = tbytes;
        // (a wavefront without nodes may read the entry after the last, class_address)
        if (!pl->groups[k].f32) tbytes += align_up((nodes + 1) * sizeof(int2), 256);
    }
    if (hipMalloc(&pl->d_tables, std::max<size_t>(tbytes, 256)) != hipSuccess) {
        delete pl;
        return BSDE_ENOMEM;
    }
    char *dev = static_cast<char *>(pl->d_tables);
    std::vector<char> host(desc_off);
    for (int b = 0; b < batch; ++b) {
        Instance &in = pl->inst[b];
        const size_t kl = (size_t)in.K * in.pb.L;
        size_t o = toff[b];
        auto put = [&](const void *src, size_t bytes) {
            std::memcpy(host.data() + o, src, bytes);
            void *d = dev + o;
            o += align_up(bytes, 256);
            return d;
        };
        if (in.f32) {
            std::vector<bsde::NodeRec32> recs(kl);
            for (size_t k = 0; k < kl; ++k) {
                const int l = (int)(k % in.pb.L), j = (int)(k / in.pb.L) + 1;
                const double cy = (j == in.pb.k_y) ? in.cy[l] : 0.0;
                recs[k] = bsde::NodeRec32{(float)in.B[k],   (float)in.C[k],   (float)in.D[k],
                                          (float)in.cfy[k], (float)in.cfz[k], (float)in.cz[k],
                                          (float)cy,        (float)in.cyz[k], in.cz[k],
                                          cy,               in.cyz[k],        0.0};
            }
            in.dtab.rec32 =
                static_cast<const bsde::NodeRec32 *>(put(recs.data(), kl * sizeof(bsde::NodeRec32)));
        } else {
            std::vector<bsde::NodeRec> recs(kl);
            std::vector<bsde::NodeRecB> recsb(kl);
            const bool linear = in.pb.driver == BSDE_DRIVER_LINEAR;
            long double rest_y = 1.0L, rest_z = 1.0L;
            for (size_t k = 0; k < kl; ++k) {
                const int l = (int)(k % in.pb.L), j = (int)(k / in.pb.L) + 1;
                const double cy = (j == in.pb.k_y) ? in.cy[l] : 0.0;
                recs[k] = bsde::NodeRec{in.B[k],   in.C[k],  in.D[k], in.cfy[k],
                                        in.cfz[k], in.cz[k], cy,      in.cyz[k]};
                // cubic B-spline weights at the fraction; for the linear driver
                // f = p0 y + p1 z + p3 folded into the weights
                double b[4];
                spline_basis(in.phi[k], b);
                bsde::NodeRecB &rb = recsb[fused_position(in.K, in.pb.L, j, l)];
                rb.b0 = b[0];
                rb.b1 = b[1];
                rb.b2 = b[2];
                rb.b3 = b[3];
                long double s = (long double)b[0] + b[1] + b[2] + b[3];
                if (in.located) {  // located nodes: the increments in cells
                    rb.b0 = in.dw[k] / in.dx;
                    rb.b1 = j * in.dt / in.dx;
                    s = 1.0L;
                }
                if (linear) {
                    rb.w0 = in.cfy[k] * in.pb.p[0] + cy;
                    rb.w1 = in.cfy[k] * in.pb.p[1];
                    rb.w2 = in.cfz[k] * in.pb.p[0];
                    rb.w3 = in.cfz[k] * in.pb.p[1] + in.cz[k];
                    rest_y += (long double)in.cfy[k] * in.pb.p[0];
                    rest_z += (long double)in.cfz[k] * in.pb.p[1];
                } else {
                    rb.w0 = in.cfy[k];
                    rb.w1 = in.cfz[k];
                    rb.w2 = in.cz[k];
                    rb.w3 = cy;
                }
                rest_y -= (linear ? rb.w0 : rb.w3) * s;
                rest_z -= (linear ? rb.w3 : rb.w2) * s;
            }
            // what E[y] of layer K_y and the E[z] terms lack to one (spline_basis) goes
            // to the layer's node of the largest weight
            const int mid = (int)(std::max_element(in.cy.begin(), in.cy.end()) - in.cy.begin());
            bsde::NodeRecB &ry = recsb[fused_position(in.K, in.pb.L, in.pb.k_y, mid)];
            bsde::NodeRecB &rz = recsb[fused_position(in.K, in.pb.L, 1, mid)];
            double &wy = linear ? ry.w0 : ry.w3, &wz = linear ? rz.w3 : rz.w2;
            wy = (double)(wy + rest_y);
            if (in.pb.z_form == BSDE_ZFORM_EZ) wz = (double)(wz + rest_z);
            in.dtab.rec = static_cast<const bsde::NodeRec *>(put(recs.data(), kl * sizeof(bsde::NodeRec)));
            in.d_recb =
                static_cast<const bsde::NodeRecB *>(put(recsb.data(), kl * sizeof(bsde::NodeRecB)));
        }
        in.dtab.m = static_cast<const int *>(put(in.m.data(), kl * sizeof(int)));
        in.dtab.dw = static_cast<const double *>(put(in.dw.data(), kl * sizeof(double)));
        std::vector<double> bw;
        for (int j = 1; j <= in.K; ++j) {
            const bsde::GaussBand &bd = in.band[j];
            in.toep_off[j] = (int)bw.size();
            bw.insert(bw.end(), bd.ev.begin(), bd.ev.end());
            bw.insert(bw.end(), bd.em.begin(), bd.em.end());
            bw.insert(bw.end(), bd.wv.begin(), bd.wv.end());
            bw.insert(bw.end(), bd.wm.begin(), bd.wm.end());
        }
        in.toep_w = static_cast<const double *>(put(bw.data(), bw.size() * sizeof(double)));
        in.d_ex_band = static_cast<const double *>(put(in.ex_band.data(), in.ex_band.size() * sizeof(double)));
        in.d_ex_corr = static_cast<const double2 *>(put(in.ex_corr.data(), in.ex_corr.size() * sizeof(double2)));
        if (!in.ctab.empty())
            in.d_ctab = static_cast<const double *>(put(in.ctab.data(), in.ctab.size() * sizeof(double)));
    }
    if (hipMemcpy(pl->d_tables, host.data(), desc_off, hipMemcpyHostToDevice) != hipSuccess) {
        bsde_plan_destroy(pl);
        return BSDE_EDEVICE;
    }
    pl->d_desc = reinterpret_cast<bsde::InstDesc *>(dev + desc_off);
    for (size_t k = 0; k < pl->groups.size(); ++k) {
        Group &g = pl->groups[k];
        size_t tiles = 0;
        for (int b : g.members) tiles += tiles_of(pl->inst[b], kMinTile);
        g.d_tile_inst = reinterpret_cast<int *>(dev + map_off[k]);
        g.d_spline_inst = reinterpret_cast<int *>(dev + map_off[k] + align_up(tiles * sizeof(int), 256));
        if (g.f32) continue;
        g.d_addr = reinterpret_cast<int2 *>(dev + addr_off[k]);
        size_t nodes = 0;
        for (int b : g.members) {  // in the members' order, as apply_config fills it
            pl->inst[b].d_addr = g.d_addr + nodes;
            nodes += (size_t)pl->inst[b].K * pl->inst[b].pb.L;
        }
    }
    // workspace: rings, then the final layers, then the statistics (per-wave
    // slots of every instance, then the totals)
    size_t off = 0;
    for (Instance &in : pl->inst) {
        in.ring_off = off;
        // planes of npad elements per slot: (y, z) and (M_y, M_z); the FP32
        // form adds the rounding residuals (e_y, e_z)
        off += align_up((size_t)(in.K + 1) * (in.f32 ? 3 * sizeof(float2) : 2 * sizeof(double2)) *
                            in.npad,
                        256);
    }
    for (Instance &in : pl->inst) {
        in.fin_off = off;
        off += align_up((size_t)2 * in.nx * sizeof(double), 256);
    }
    // partial sums of the split Toeplitz sweep: 2 kToepTile doubles per tile
    // and split
    for (Group &g : pl->groups) {
        if (!group_exact(pl->inst, g.members)) continue;
        if (toeplitz_config(pl->inst, g.members, pl->max_lds).W == 1) continue;
        const int S = toeplitz_splits(pl->inst, g.members);
        if (S == 1) continue;
        size_t tiles = 0;
        for (int b : g.members) tiles += tiles_of(pl->inst[b], kBlock);
        g.part_off = off;
        off += align_up(tiles * S * 2 * bsde::kToepTile * sizeof(double), 256);
    }
    // chunk sums of the split direct sweep: 2 kBlock doubles per tile and
    // node chunk (groups that may take it: neither exact nor gathering)
    for (Group &g : pl->groups) {
        if (group_exact(pl->inst, g.members) || group_gathers(pl->inst, g.members)) continue;
        if (direct_splits(pl->inst, g.members) == 1) continue;
        size_t tiles = 0;
        for (int b : g.members) {
            tiles += tiles_of(pl->inst[b], kBlock);
            g.dchunks = std::max(g.dchunks, bsde::direct_chunks(pl->inst[b].K, pl->inst[b].pb.L));
        }
        g.part_off = off;
        off += align_up(tiles * g.dchunks * 2 * kBlock * sizeof(double), 256);
    }
    pl->stats_off = off;
    for (Instance &in : pl->inst) {
        in.stat_off = off;
        off += align_up((size_t)in.nwaves * (2 * sizeof(unsigned long long) + sizeof(unsigned int)),
                        256);
    }
    pl->totals_off = off;
    off += align_up((3 * (size_t)batch + 1) * sizeof(unsigned long long), 256);
    pl->stats_bytes = off - pl->stats_off;
    pl->ws_bytes = off;
    // descriptors
    pl->desc.resize(batch);
    for (int b = 0; b < batch; ++b) {
        const Instance &in = pl->inst[b];
        bsde::InstDesc &d = pl->desc[b];
        std::memset(&d, 0, sizeof(d));
        bsde::SweepArgs &a = d.a;
        a.n_stop = in.pb.n_stop;
        a.tab = in.dtab;
        a.drv = in.drv;
        a.pcr = pl->pcr_base;
        a.pcr.s6 = 6.0 / (in.dx * in.dx);
        a.nx = in.nx;
        a.npad = in.npad;
        a.pad_l = in.pad_l;
        a.pad_r = in.pad_r;
        a.K = in.K;
        a.Ky = in.pb.k_y;
        a.L = in.pb.L;
        a.dt = in.dt;
        a.h0 = in.h0;
        a.picard_max = in.pb.picard_max;
        a.picard_tol = in.pb.picard_tol;
        a.zform = in.pb.z_form;
        a.x_min = in.pb.x_min[0];
        a.dx = in.dx;
        a.drift0 = in.pb.drift[0];
        a.drift_x = in.pb.drift_x;
        a.vol0 = in.pb.vol[0][0];
        a.vol_x = in.pb.vol_x;
        a.ctab = in.d_ctab;
        a.tab_steps = in.pb.tab_steps;
        if (in.exact) {
            // eq (20) for f = p0 y + p1 z + p3 with exact expectations:
            //   Y = E[y^{n+K_y}] + K_y dt sum_j gamma_j E[f^{n+j}]
            //   Z = (E[z^{n+1}] (or E[y^{n+1} dW]/dt) + sum_j gamma'_j (E[f dW] - E[z])) / gamma'_0
            double gy[8], gz[8];
            bsde::spline_gamma(1, in.pb.k_y, gy);
            bsde::spline_gamma(2, in.pb.k_z, gz);
            bsde::ToepTable &t = a.toep;
            t.w = in.toep_w;
            const double p0 = in.pb.p[0], p1 = in.pb.p[1], p3 = in.pb.p[3];
            const bool ydw = in.pb.z_form == BSDE_ZFORM_YDW;
            for (int j = 1; j <= in.K; ++j) {
                t.off[j] = in.toep_off[j];
                t.klo[j] = in.band[j].klo;
                t.nb[j] = (int)in.band[j].ev.size();
                const double fy = j <= in.pb.k_y ? in.pb.k_y * in.dt * gy[j] : 0.0;
                const double fz = j <= in.pb.k_z ? gz[j] : 0.0;
                t.cy_ey[j] = (j == in.pb.k_y ? 1.0 : 0.0) + fy * p0;
                t.cy_ez[j] = fy * p1;
                t.cy_1[j] = fy * p3;
                t.cz_ez[j] = ((j == 1 && !ydw ? 1.0 : 0.0) - fz) / gz[0];
                t.cz_wy[j] = (fz * p0 + (j == 1 && ydw ? 1.0 / in.dt : 0.0)) / gz[0];
                t.cz_wz[j] = fz * p1 / gz[0];
            }
            if (!ydw) {  // the E[z] terms sum to one
                long double rest = 1.0L;
                for (int j = 1; j <= in.K; ++j) rest -= t.cz_ez[j];
                t.cz_ez[1] = (double)(t.cz_ez[1] + rest);
            }
        }
        for (size_t k = 0; k < in.cfy.size(); ++k) {
            d.lin_y += in.cfy[k] * in.pb.p[3];
            d.lin_z += in.cfz[k] * in.pb.p[3];
        }
        d.ring_off = in.ring_off;
        d.fin_off = in.fin_off;
        d.stat_off = in.stat_off;
        d.nwaves = in.nwaves;
        d.n0 = in.pb.n_t - in.K;
        d.f32 = in.f32 ? 1 : 0;
        for (int j = 0; j <= in.K; ++j) {
            d.win_lo[j] = in.win_lo[j];
            d.win_hi[j] = in.win_hi[j];
        }
    }
    for (Group &g : pl->groups) {
        bsde_status rc = apply_config(*pl, g, default_config(pl->inst, g, pl->max_lds));
        if (rc != BSDE_OK) {
            bsde_plan_destroy(pl);
            return rc;
        }
    }
    *out = pl;
    return BSDE_OK;
}

void bsde_plan_destroy(bsde_plan_t plan)
{
    if (!plan) return;
    plan->drop_graphs();
    if (plan->capture_stream) (void)hipStreamDestroy(plan->capture_stream);
    if (plan->d_tables) (void)hipFree(plan->d_tables);
    delete plan;
}

size_t bsde_workspace_bytes(bsde_plan_t plan) { return plan ? plan->ws_bytes : 0; }

bsde_status bsde_solve(bsde_plan_t plan, void *ws, const double *init_y, const double *init_z,
                       double *y0, double *z0, void *stream, bsde_stats *st)
{
    if (!plan) return BSDE_EINVAL;
    if (plan->desc.size() != 1) return BSDE_EINVAL;
    bsde_io io{init_y, init_z, y0, z0};
    return solve_impl(plan, ws, &io, 1, stream, st);
}

bsde_status bsde_solve_batched(bsde_plan_t plan, void *ws, const bsde_io *io, void *stream,
                               bsde_stats *st)
{
    if (!plan) return BSDE_EINVAL;
    return solve_impl(plan, ws, io, (int)plan->desc.size(), stream, st);
}

bsde_status bsde_checkpoint_layers(bsde_plan_t plan, void *ws, int b, double *layers_y,
                                   double *layers_z, void *stream)
{
    if (!plan || !ws || !layers_y || !layers_z || b < 0) return BSDE_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *w = static_cast<char *>(ws);
    if (!plan->inst2.empty()) {
        if (b >= (int)plan->inst2.size()) return BSDE_EINVAL;
        const Instance2 &in = plan->inst2[b];
        bsde::Sweep2Args a = sweep2_args(in, w, false);
        HIP_OK(bsde::launch_export2d(in.f32, a, layers_y, layers_z, s));
        return BSDE_OK;
    }
    if (b >= (int)plan->inst.size()) return BSDE_EINVAL;
    const Instance &in = plan->inst[b];
    HIP_OK(bsde::launch_export_layers(in.f32, plan->d_desc + b, in.K, in.nx, w, layers_y, layers_z,
                                      s));
    return BSDE_OK;
}

bsde_status bsde_solve_batched_static(bsde_plan_t plan, const bsde_io *io, void *stream)
{
    if (!plan || !io) return BSDE_EINVAL;
    const int count = (int)plan->desc.size();
    for (int b = 0; b < count; ++b)
        if (!io[b].init_y || !io[b].init_z || !io[b].y0 || !io[b].z0) return BSDE_EINVAL;
    if (plan->ws_bytes > kStaticWorkspaceBytes) return BSDE_ESCRATCH;
    int dev = -1;
    HIP_OK(hipGetDevice(&dev));
    if (dev != plan->device) return BSDE_EINVAL;
    char *w = nullptr;
    const bsde_status rc = static_workspace(dev, &w);
    if (rc != BSDE_OK) return rc;
    // kernel launches only: no statistics (their counters would need
    // clearing and a host read-back), no graph capture
    return enqueue_solve(*plan, w, io, false, nullptr, static_cast<hipStream_t>(stream));
}

bsde_status bsde_profile_kernels(bsde_plan_t plan, void *ws, const bsde_io *io, void *stream,
                                 bsde_kernel_times *kt)
{
    const int count = plan ? (int)plan->desc.size() : 0;
    if (!kt || !valid_io(plan, ws, io, count)) return BSDE_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *w = static_cast<char *>(ws);
    KernelTimer tm;
    bsde_status rc = enqueue_solve(*plan, w, io, false, nullptr, s, &tm);
    if (rc != BSDE_OK) return rc;
    HIP_OK(hipStreamSynchronize(s));
    double sw = 0.0, sp = 0.0;
    for (size_t i = 0; i + 1 < tm.sweep.size(); i += 2) {
        float ms = 0.0f;
        HIP_OK(hipEventElapsedTime(&ms, tm.sweep[i], tm.sweep[i + 1]));
        sw += ms;
    }
    for (size_t i = 0; i + 1 < tm.spline.size(); i += 2) {
        float ms = 0.0f;
        HIP_OK(hipEventElapsedTime(&ms, tm.spline[i], tm.spline[i + 1]));
        sp += ms;
    }
    kt->sweep_ms = sw;
    kt->sweep_launches = (int)(tm.sweep.size() / 2);
    kt->spline_ms = sp;
    kt->spline_launches = (int)(tm.spline.size() / 2);
    if (plan->groups.empty()) {  // two-dimensional plan
        const Instance2 &in = plan->inst2[0];
        kt->path = 2;
        kt->points_per_lane = 1;
        kt->node_groups = 1;
        kt->blocks = in.nwaves / (in.bspline ? bsde::kGroups2B : bsde::kWaves2);
        kt->lds_bytes = 0;
        return BSDE_OK;
    }
    const Group &g = plan->groups[0];
    kt->path = g.cfg.path;
    kt->points_per_lane = g.cfg.P;
    kt->node_groups = g.cfg.G;
    kt->blocks = g.tile_prefix.back();
    kt->lds_bytes = (long long)g.cfg.lds;
    return BSDE_OK;
}

bsde_status bsde_autotune(bsde_plan_t plan, void *ws, const bsde_io *io, void *stream, int reps,
                          bsde_tune_report *rep)
{
    const int count = plan ? (int)plan->desc.size() : 0;
    if (!valid_io(plan, ws, io, count) || reps < 1) return BSDE_EINVAL;
    if (plan->groups.empty()) {  // two-dimensional plan: one kernel shape
        if (rep) *rep = bsde_tune_report{2, 1, 1, 0.0, 0};
        return BSDE_OK;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *w = static_cast<char *>(ws);
    std::lock_guard<std::mutex> lock(plan->mu);
    bsde_status rc = enqueue_init(*plan, w, io, s);
    if (rc != BSDE_OK) return rc;
    // the descriptors are rewritten (synchronously) for every candidate shape:
    // no kernel of the stream may still read them
    HIP_OK(hipStreamSynchronize(s));
    EventPair ev;
    if (!ev.create()) return BSDE_EDEVICE;
    hipEvent_t e0 = ev.e0, e1 = ev.e1;
    int tried = 0;
    for (Group &g : plan->groups) {
        std::vector<SweepConfig> cand;
        auto consider = [&](const Shape &q) {
            const SweepConfig c = fused_config(plan->inst, g.members, q.P, q.W, q.G, plan->max_lds);
            if (c.lds) cand.push_back(c);
        };
        if (g.f32)
            for (const Shape &q : kShapes32) consider(q);
        else
            for (const Shape &q : kShapes64) consider(q);
        if (group_gathers(plan->inst, g.members)) {
            cand.clear();
            double t = 0.0;
            if (in_windows(gather_config(plan->inst, g.members, plan->max_lds))) {
                for (const Shape &q : kLocatedShapes) {
                    const SweepConfig c = located_config(plan->inst, g.members, q, plan->max_lds);
                    if (c.lds) cand.push_back(c);
                }
                (void)best_located(plan->inst, g.members, plan->max_lds, t);
            }
            if (cand.empty() || gather_cost(plan->inst, g.members) < 1.3 * t)
                cand.push_back(SweepConfig{PATH_GATHER, 1, 1, 0});
        }
        if (group_exact(plan->inst, g.members)) cand.assign(1, toeplitz_config(plan->inst, g.members, plan->max_lds));
        // both kernels where neither is much the faster by estimate (a large batch
        // of small grids with wide windows is the direct kernel's)
        double fused_us = 0.0;
        if (!g.f32 && !cand.empty()) (void)best_fused(plan->inst, g.members, false, plan->max_lds, fused_us);
        if (cand.empty() || (!g.f32 && cand[0].path == PATH_FUSED &&
                             direct_cost(plan->inst, g.members) < 1.3 * fused_us)) {
            cand.push_back(direct_config(plan->inst, g.members, g.f32, 1));
            cand.push_back(direct_config(plan->inst, g.members, g.f32, 2));
        }
        float best = 0.0f;
        SweepConfig best_c = g.cfg;
        // Timed steps: the first, and three more spread over the group's
        // steps, so that a batch's shrinking set of active instances weighs
        // in.  The warm-up runs steps 0 and 1, after which every plane of
        // every ring slot holds finite data (initial layers, their splines
        // and the warm-up's output), so any step does the work of a real one;
        // the solve reloads the initial layers afterwards.
        int sample[4] = {0, g.max_steps / 4, g.max_steps / 2, (3 * g.max_steps) / 4};
        const int nsample = g.max_steps >= 8 ? 4 : 1;
        // Two passes over the candidates, each keeping its faster pass: the
        // first candidate timed would otherwise run while the clocks ramp up.
        std::vector<float> t(cand.size(), 0.0f);
        for (int pass = 0; pass < 2 && rc == BSDE_OK; ++pass) {
            for (size_t ci = 0; ci < cand.size(); ++ci) {
                rc = apply_config(*plan, g, cand[ci]);
                if (rc != BSDE_OK) break;
                rc = enqueue_step(*plan, g, w, 0, false, s, nullptr);  // warm-up
                if (rc == BSDE_OK && nsample > 1) rc = enqueue_step(*plan, g, w, 1, false, s, nullptr);
                if (rc != BSDE_OK) break;
                auto timed_steps = [&](hipStream_t q) {
                    bsde_status r2 = BSDE_OK;
                    for (int r = 0; r < reps && r2 == BSDE_OK; ++r)
                        for (int k = 0; k < nsample && r2 == BSDE_OK; ++k)
                            r2 = enqueue_step(*plan, g, w, sample[k], false, q, nullptr);
                    return r2;
                };
                // the timed steps run the way a solve runs: replayed from a
                // graph (launches from a graph and direct launches rank the
                // shapes differently), or directly when the plan does not use
                // graphs
                hipGraphExec_t exec = nullptr;
                if (plan->use_graphs) {
                    if (!plan->capture_stream &&
                        hipStreamCreateWithFlags(&plan->capture_stream, hipStreamNonBlocking) != hipSuccess) {
                        rc = BSDE_EDEVICE;
                        break;
                    }
                    hipStream_t cs = plan->capture_stream;
                    if (hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) != hipSuccess) {
                        rc = BSDE_EDEVICE;
                        break;
                    }
                    rc = timed_steps(cs);
                    hipGraph_t graph = nullptr;
                    const hipError_t ec = hipStreamEndCapture(cs, &graph);
                    if (rc == BSDE_OK && ec == hipSuccess &&
                        hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess)
                        rc = BSDE_EDEVICE;
                    if (graph) (void)hipGraphDestroy(graph);
                    if (rc == BSDE_OK && ec != hipSuccess) rc = BSDE_EDEVICE;
                    if (rc == BSDE_OK && hipGraphLaunch(exec, s) != hipSuccess) rc = BSDE_EDEVICE;
                    if (rc != BSDE_OK) {
                        if (exec) (void)hipGraphExecDestroy(exec);
                        break;
                    }
                }
                float ms = 0.0f;
                if (hipEventRecord(e0, s) != hipSuccess) rc = BSDE_EDEVICE;
                if (rc == BSDE_OK) rc = exec ? (hipGraphLaunch(exec, s) == hipSuccess ? BSDE_OK : BSDE_EDEVICE)
                                             : timed_steps(s);
                if (rc == BSDE_OK &&
                    (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                     hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
                    rc = BSDE_EDEVICE;
                if (exec) (void)hipGraphExecDestroy(exec);
                if (rc != BSDE_OK) break;
                if (pass == 0) ++tried;
                if (t[ci] == 0.0f || ms < t[ci]) t[ci] = ms;
            }
        }
        for (size_t ci = 0; ci < cand.size() && rc == BSDE_OK; ++ci) {
            if (best == 0.0f || t[ci] < best) {
                best = t[ci];
                best_c = cand[ci];
            }
        }
        if (rc == BSDE_OK) rc = apply_config(*plan, g, best_c);
        if (rc != BSDE_OK) break;
        if (rep && &g == &plan->groups[0]) {
            rep->path = best_c.path;
            rep->points_per_lane = best_c.P;
            rep->node_groups = best_c.G;
            rep->best_ms_per_step = best / (reps * nsample);
        }
    }
    if (rep) rep->candidates = tried;
    return rc;
}

}  // extern "C"
