// sweep.hip -- kernels of the backward sweep (arXiv:1909.13560, Section 2.2
// eq (20)-(21), Section 3.1 step 3, Section 3.2) and their host-side
// launchers, in the FP64 and the FP32 form.
//
// Every kernel serves a group of instances: the grid's tiles are numbered
// instance after instance, a device table maps a tile to its instance, and
// each block reads that instance's descriptor (a single solve is a group of
// one).  One launch per time step advances every instance still active by one
// layer; instances are sorted by their number of steps, so the active ones
// are a prefix of the group and the launch covers exactly their tiles.
//
// The sweep kernels that compute layer n from layers n+1..n+K:
//   sweep_fused  (fused.h) LDS windows of every layer, the spline of layer n+1
//                built in-kernel: one launch per step.
//   sweep_direct (windows too wide for LDS or, in FP64, so wide that only small
//                tiles fit a large grid; the E[y dW]/dt z form): records are
//                read straight from HBM/L2, P consecutive points per lane; the
//                natural spline of the new layer is a separate launch.
//   sweep_gather (state-dependent coefficients; in FP64 with windows for LDS they
//                take sweep_fused where that is the faster): nodes located per
//                point and read from HBM/L2.
#include "device_common.h"
#include "fused.h"
#include "kernels.h"

namespace bsde {

// Node records read straight from the layer in HBM (direct kernel).
template <bool F32>
struct GlobalWindow {
    using V = typename Prec<F32>::V;
    static constexpr int NA = Prec<F32>::NA;
    Slot<F32> lay;  // the layer
    int i0;         // the lane's first point
    template <int P>
    __device__ void fetch(int m, V (&r)[NA][P + 1]) const
    {
#pragma unroll
        for (int q = 0; q <= P; ++q) {
            const auto v = lay.val(i0 + m + q), mm = lay.der(i0 + m + q);
            if constexpr (F32) {
                r[0][q] = make_float4(v.x, v.y, mm.x, mm.y);
            } else {
                r[0][q] = v;
                r[1][q] = mm;
            }
        }
    }
};

template <int P, int DRV, bool F32, typename Src>
__device__ inline void layer_dispatch(const Src &src, const int *tm, int j, int l0, int LS,
                                      const SweepArgs &a, Acc<P> &acc, int lend)
// nodes l = l0, l0 + LS, ... < lend of layer j
{
    using Node = typename Prec<F32>::Node;
    const Driver<DRV, typename Prec<F32>::Raw> f(a.drv, (a.n + j) * a.dt);
    const int row = (j - 1) * a.L;
    const Node *nodes = node_recs(a.tab, static_cast<Node *>(nullptr)) + row;
    const bool last_y = j == a.Ky;
    if (j == 1 && a.zform) {
        if (last_y)
            layer_nodes<P, DRV, kNodeLastY | kNodeYW, F32>(src, nodes, tm + row, l0, LS, lend, f, acc);
        else
            layer_nodes<P, DRV, kNodeYW, F32>(src, nodes, tm + row, l0, LS, lend, f, acc);
        return;
    }
    if (last_y)
        layer_nodes<P, DRV, kNodeLastY, F32>(src, nodes, tm + row, l0, LS, lend, f, acc);
    else
        layer_nodes<P, DRV, 0, F32>(src, nodes, tm + row, l0, LS, lend, f, acc);
}

// ---------------------------------------------------------------------------
// Direct sweep: records from HBM/L2, P consecutive points per lane.
// Dynamic LDS: node table only.  The nodes are summed chunk by chunk
// (kDirectChunk nodes of one layer, each chunk from zero, the chunks added in
// order); on a small grid a tile's chunks are split over s.dsplit blocks
// (P = 1), which write the chunk sums for direct_finish.
// ---------------------------------------------------------------------------
template <int P, int DRV, bool F32, bool SPLIT>
__global__ void __launch_bounds__(kBlock) sweep_direct(const StepArgs s)
{
    static_assert(!SPLIT || P == 1, "split direct steps take one point per lane");
    const int S = SPLIT ? s.dsplit : 1;
    const int idx = xcd_tile(blockIdx.x, gridDim.x);
    const int tg = SPLIT ? idx / S : idx, sp = SPLIT ? idx - tg * S : 0;  // tile of the group, split
    const InstDesc &d = block_desc(s, tg);
    const SweepArgs a = bind_instance(d, s.ws, s.s, s.stats != 0);
    const int tile = tg - d.tile_base;
    __shared__ int tm[kMaxNodes];
    for (int i = threadIdx.x; i < a.K * a.L; i += kBlock) tm[i] = a.tab.m[i];
    __syncthreads();
    const int first = (tile * kBlock + (int)threadIdx.x) * P;
    const int i0 = min(first, a.nx - 1);  // lanes past the end read in bounds, store nothing
    Acc<P> acc;
#pragma unroll
    for (int q = 0; q < P; ++q) acc.Y[q] = acc.Z[q] = 0.0;
    const int nch = (a.L + kDirectChunk - 1) / kDirectChunk;  // chunks per layer
    for (int j = 1, c = 0; j <= a.K; ++j) {
        const GlobalWindow<F32> src{ring_slot<F32>(a, a.n + j), i0};
        for (int h = 0; h < nch; ++h, ++c) {
            if (SPLIT && c % S != sp) continue;
            Acc<P> ch;
#pragma unroll
            for (int q = 0; q < P; ++q) ch.Y[q] = ch.Z[q] = 0.0;
            layer_dispatch<P, DRV, F32>(src, tm, j, h * kDirectChunk, 1, a, ch,
                                              min(a.L, (h + 1) * kDirectChunk));
            if constexpr (SPLIT) {
                double *p = s.part + ((size_t)tg * s.dchunks + c) * 2 * kBlock;
                p[threadIdx.x] = ch.Y[0];
                p[kBlock + threadIdx.x] = ch.Z[0];
            } else {
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    acc.Y[q] += ch.Y[q];
                    acc.Z[q] += ch.Z[q];
                }
            }
        }
    }
    if constexpr (!SPLIT)
        finish_points<P, DRV, F32>(a, first, acc, (tile * kBlock + (int)threadIdx.x) >> 6);
}

// A split direct step: the chunk sums of a tile added in chunk order, then
// the implicit y equation (Picard) of its points.  Loads go out four chunks
// at a time.
template <int DRV, bool F32>
__global__ void __launch_bounds__(kBlock) direct_finish(const StepArgs s)
{
    const int tg = xcd_tile(blockIdx.x, gridDim.x);
    const InstDesc &d = block_desc(s, tg);
    const SweepArgs a = bind_instance(d, s.ws, s.s, s.stats != 0);
    const int tile = tg - d.tile_base, tid = threadIdx.x;
    const int C = direct_chunks(a.K, a.L);
    const double *p = s.part + (size_t)tg * s.dchunks * 2 * kBlock + tid;
    Acc<1> acc;
    acc.Y[0] = acc.Z[0] = 0.0;
    for (int c0 = 0; c0 < C; c0 += 4) {
        double vy[4], vz[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            vy[q] = c0 + q < C ? p[(size_t)(c0 + q) * 2 * kBlock] : 0.0;
            vz[q] = c0 + q < C ? p[(size_t)(c0 + q) * 2 * kBlock + kBlock] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (c0 + q < C) {
                acc.Y[0] += vy[q];
                acc.Z[0] += vz[q];
            }
    }
    finish_points<1, DRV, F32>(a, tile * kBlock + tid, acc, (tile * kBlock + tid) >> 6);
}

// ---------------------------------------------------------------------------
// Gather sweep: forward coefficients that depend on the state (eq (1)),
// affine in x or tabulated on the grid (and then also per time step).  The
// node of (j, l) for point x_i is one Euler step of X over j dt from t_n,
//   X = x_i + a(t_n, x_i) j dt + b(t_n, x_i) sqrt(2 j dt) a_l,
// so its cell and fraction differ from point to point: each lane locates
// its nodes (Section 3.2: floor on the uniform grid, the boundary value
// outside the truncated domain), forms the spline basis weights at the
// fraction and reads the two records from HBM/L2.  One point per lane; the
// natural spline of the new layer is a separate launch.
// ---------------------------------------------------------------------------
template <int DRV, bool F32>
__global__ void __launch_bounds__(kBlock) sweep_gather(const StepArgs s)
{
    using PR = Prec<F32>;
    using Node = typename PR::Node;
    using V = typename PR::V;
    const int idx = xcd_tile(blockIdx.x, gridDim.x);
    const InstDesc &d = block_desc(s, idx);
    const SweepArgs a = bind_instance(d, s.ws, s.s, s.stats != 0);
    const int tile = idx - d.tile_base;
    const int first = tile * kBlock + (int)threadIdx.x;
    const int i = min(first, a.nx - 1);  // lanes past the end compute in bounds, store nothing
    const double xi = a.x_min + i * a.dx;
    double ax, bx;
    if (a.ctab) {  // tabulated a(t_n, x_i), b(t_n, x_i)
        const double *row = a.ctab + (size_t)2 * (a.tab_steps > 1 ? a.n : 0) * a.nx;
        ax = row[i];
        bx = row[a.nx + i];
    } else {
        ax = fma(a.drift_x, xi, a.drift0);
        bx = fma(a.vol_x, xi, a.vol0);
    }
    const double dx26 = a.dx * a.dx / 6.0;
    Acc<1> acc;
    acc.Y[0] = acc.Z[0] = 0.0;
    for (int j = 1; j <= a.K; ++j) {
        const Slot<F32> g = ring_slot<F32>(a, a.n + j);
        const Driver<DRV, typename PR::Raw> f(a.drv, (a.n + j) * a.dt);
        const int row = (j - 1) * a.L;
        const Node *nodes = node_recs(a.tab, static_cast<Node *>(nullptr)) + row;
        const int nf = (j == a.Ky ? kNodeLastY : 0) | (j == 1 && a.zform ? kNodeYW : 0);
        if (F32) acc.Yf[0] = acc.Zf[0] = 0.0f;
        for (int l = 0; l < a.L; ++l) {
            const double X = xi + ax * (j * a.dt) + bx * a.tab.dw[row + l];
            const double sx = (X - a.x_min) / a.dx;
            int p = 0;
            double phi = 0.0;
            if (sx >= (double)(a.nx - 1)) {
                p = a.nx - 1;  // the last record; its right neighbour is a ghost, weight 0
            } else if (sx > 0.0) {
                p = min((int)floor(sx), a.nx - 2);
                phi = sx - p;
            }
            const double u = 1.0 - phi;
            Node c = load_node(nodes + l);
            c.B = phi;
            c.C = dx26 * (u * u * u - u);
            c.D = dx26 * (phi * phi * phi - phi);
            V r[PR::NA][2];
            GlobalWindow<F32>{g, p}.template fetch<1>(0, r);
            switch (nf) {
            case 0: node_accumulate<1, DRV, 0>(r, c, f, acc); break;
            case kNodeLastY: node_accumulate<1, DRV, kNodeLastY>(r, c, f, acc); break;
            case kNodeYW: node_accumulate<1, DRV, kNodeYW>(r, c, f, acc); break;
            default: node_accumulate<1, DRV, kNodeLastY | kNodeYW>(r, c, f, acc); break;
            }
        }
        if (F32) {
            acc.Y[0] += (double)acc.Yf[0];
            acc.Z[0] += (double)acc.Zf[0];
        }
    }
    finish_points<1, DRV, F32>(a, first, acc, (tile * kBlock + (int)threadIdx.x) >> 6);
}

// ---------------------------------------------------------------------------
// Standalone natural spline of one layer per instance: the initial layers
// (mode 0: layer n0 + 1 + s) and, on the direct path, the layer just computed
// (mode 1: layer n0 - s, skipped at n_stop, which no later step reads).
// ---------------------------------------------------------------------------
template <bool F32>
__global__ void __launch_bounds__(kBlock) spline_layer(const StepArgs s, int mode)
{
    using V = typename Prec<F32>::V;
    constexpr int WE = kSplineTile + 2 * kHalo, WS = WE + 2;
    static_assert(WE <= kSplineSlots, "spline tile exceeds the window layout");
    __shared__ V wsm[(F32 ? 1 : 2) * kSplineSlots];
    __shared__ double R[4 * WS];
    const int idx = xcd_tile(blockIdx.x, gridDim.x);
    const InstDesc &d = block_desc(s, idx);
    const SweepArgs a = bind_instance(d, s.ws, 0, false);
    const int tile = idx - d.spline_base;
    const int n = mode == 0 ? d.n0 + 1 + s.s : d.n0 - s.s;
    if (mode == 0 && s.s >= a.K) return;
    if (mode == 1 && n <= a.n_stop) return;
    const Slot<F32> g = ring_slot<F32>(a, n);
    const typename Prec<F32>::template Win<1> win{wsm};
    const int t0 = tile * kSplineTile;
    constexpr int U = (WS + kBlock - 1) / kBlock;
    SplineRaw<U, typename Prec<F32>::Raw> raw;
    spline_load<kBlock, U>(g, a.nx, t0, kSplineTile, raw);
    spline_window<kBlock, U, 1>(g, a.nx, t0, kSplineTile, win, R, WS, a.pcr, raw);
    const int kend = min(t0 + kSplineTile, a.nx);
    for (int k = t0 + (int)threadIdx.x; k < kend; k += kBlock) {
        const double2 dd = win.ders(k - t0 + kHalo);
        g.set_der(k, dd.x, dd.y);
    }
    if (tile == 0) {
        const auto e0 = g.val(0);
        for (int k = threadIdx.x; k < a.pad_l; k += kBlock) {
            g.set_val(k - a.pad_l, e0);
            g.set_der(k - a.pad_l, 0.0, 0.0);
        }
    }
    if (tile == d.spline_tiles - 1) {
        const auto e1 = g.val(a.nx - 1);
        for (int k = threadIdx.x; k < a.pad_r; k += kBlock) {
            g.set_val(a.nx + k, e1);
            g.set_der(a.nx + k, 0.0, 0.0);
        }
    }
}

// B-spline coefficients of the initial layers of the instances of a group
// (layer n0 + 1 + s), with their ghost records.
__global__ void __launch_bounds__(kBlock) coef_layer(const StepArgs s)
{
    constexpr int W = kSplineTile + 2;  // records t0 - 1 .. t0 + kSplineTile
    __shared__ double2 D[W + 2 * kHalo + 2 + kFirOver], A[W + 48 + kFirOver];
    const int idx = xcd_tile(blockIdx.x, gridDim.x);
    const InstDesc &d = block_desc(s, idx);
    const SweepArgs a = bind_instance(d, s.ws, 0, false);
    if (s.s >= a.K) return;
    const int tile = idx - d.spline_base, t0 = tile * kSplineTile, nx = a.nx, tid = threadIdx.x;
    const Slot<false> g = ring_slot<false>(a, d.n0 + 1 + s.s);
    const double2 end0 = layer_value(g, 0), end1 = layer_value(g, nx - 1);
    for (int e = tid; e < W + 2 * kHalo + 2; e += kBlock) {
        const int k = t0 - 2 - kHalo + e;
        D[e] = reflected_value(nx, k, layer_value(g, reflected_index(nx, k)), end0, end1);
    }
    __syncthreads();
    fir_pass_a<kBlock, 3>(W, D, A);
    __syncthreads();
    const double inv_b = a.pcr.inv_b;
    fir_pass_b<kBlock, 2>(W, A, [&](int e, double wy, double wz) {
        const int k = t0 - 1 + e;
        const bool own = (k >= t0 && k < min(t0 + kSplineTile, nx)) || k == -1 ||
                         (k == nx && tile == d.spline_tiles - 1);
        const double2 v = D[e + kHalo + 1];
        if (k == 0 || k == nx - 1) wy = wz = 0.0;  // an end value is its own coefficient
        if (own) g.set_der(k, fma(-inv_b, wy, v.x), fma(-inv_b, wz, v.y));
    });
    if (tile == 0) {
        const double2 e0 = g.val(0);
        for (int k = -2 - tid; k >= -a.pad_l; k -= kBlock) g.set_der(k, e0.x, e0.y);
    }
    if (tile == d.spline_tiles - 1) {
        const double2 e1 = g.val(nx - 1);
        for (int k = nx + 1 + tid; k < nx + a.pad_r; k += kBlock) g.set_der(k, e1.x, e1.y);
    }
}

// ---------------------------------------------------------------------------
// Input / output / statistics kernels
// ---------------------------------------------------------------------------
// Initial layers r = 0..K-1 (t_{N-K+1+r}) of the instances of a chunk into
// their rings (the records' y and z; the splines follow).
__global__ void __launch_bounds__(kBlock) scatter_layers(const ScatterChunk c, char *ws,
                                                         const InstDesc *desc)
{
    const int b = blockIdx.y;
    const InstDesc &d = desc[c.inst[b]];
    const SweepArgs a = bind_instance(d, ws, 0, false);
    const double *__restrict__ iy = c.iy[b];
    const double *__restrict__ iz = c.iz[b];
    for (int r = 0; r < a.K; ++r) {
        const int n = d.n0 + 1 + r;
        const Slot<false> g64 = ring_slot<false>(a, n);
        const Slot<true> g32 = ring_slot<true>(a, n);
        for (int i = blockIdx.x * kBlock + threadIdx.x; i < a.nx; i += gridDim.x * kBlock) {
            const double y = iy[(size_t)r * a.nx + i], z = iz[(size_t)r * a.nx + i];
            if (d.f32)
                store_fed_back(g32, a.npad, i, y, z, 0.0f, 0.0f);
            else
                g64.set_val(i, y, z);
        }
    }
}

// Layer n_stop (double precision, in the workspace) of the instances of a
// chunk to the caller's buffers, counting non-finite values.
__global__ void __launch_bounds__(kBlock) gather_layers(const GatherChunk c, char *ws,
                                                        const InstDesc *desc,
                                                        unsigned long long *nonfinite)
{
    const int b = blockIdx.y;
    const InstDesc &d = desc[c.inst[b]];
    const int nx = d.a.nx;
    const double *__restrict__ fy = reinterpret_cast<const double *>(ws + d.fin_off);
    const double *__restrict__ fz = fy + nx;
    double *__restrict__ y0 = c.y0[b];
    double *__restrict__ z0 = c.z0[b];
    unsigned int bad = 0;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < nx; i += gridDim.x * kBlock) {
        const double y = fy[i], z = fz[i];
        y0[i] = y;
        z0[i] = z;
        bad += (isfinite(y) && isfinite(z)) ? 0u : 1u;
    }
    bad = wave_sum_u32(bad);
    if (nonfinite && (threadIdx.x & 63) == 0 && bad) atomicAdd(nonfinite, (unsigned long long)bad);
}

// Checkpoint export: layers n_stop .. n_stop + K - 1 of one instance (still in
// its ring after a solve stopped at n_stop) into the initial-layer layout, row
// r = layer n_stop + r.  The FP32 form exports the stored value plus its
// residual, which a later scatter splits back into the same pair.
template <bool F32>
__global__ void __launch_bounds__(kBlock) export_layers(const InstDesc *desc, char *ws,
                                                        double *__restrict__ ly,
                                                        double *__restrict__ lz)
{
    const InstDesc &d = *desc;
    SweepArgs a = d.a;
    a.ring = ws + d.ring_off;
    const int r = blockIdx.y, nx = a.nx;
    const Slot<F32> g = ring_slot<F32>(a, a.n_stop + r);
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < nx; i += gridDim.x * kBlock) {
        const auto v = g.val(i);
        double y = v.x, z = v.y;
        if constexpr (F32) {
            const float2 e = fed_back_residual(g, a.npad, i);
            y += (double)e.x;
            z += (double)e.y;
        }
        ly[(size_t)r * nx + i] = y;
        lz[(size_t)r * nx + i] = z;
    }
}

hipError_t launch_export_layers(bool f32, const InstDesc *desc, int K, int nx, char *ws,
                                double *ly, double *lz, hipStream_t s)
{
    const dim3 grid((unsigned)std::min(1024, (nx + kBlock - 1) / kBlock), (unsigned)K);
    if (f32)
        hipLaunchKernelGGL(export_layers<true>, grid, dim3(kBlock), 0, s, desc, ws, ly, lz);
    else
        hipLaunchKernelGGL(export_layers<false>, grid, dim3(kBlock), 0, s, desc, ws, ly, lz);
    return hipGetLastError();
}

__global__ void __launch_bounds__(kBlock) clear_u64(unsigned long long *p, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)kBlock + threadIdx.x; i < n;
         i += (size_t)gridDim.x * kBlock)
        p[i] = 0ull;
}

// Statistics of one instance: totals[0] = max iterations, [1] = sum,
// [2] = unconverged.
__global__ void __launch_bounds__(kBlock)
reduce_stats(char *ws, const InstDesc *desc, unsigned long long *totals)
{
    __shared__ unsigned long long sm[3][kBlock];
    const InstDesc &d = desc[blockIdx.x];
    const int nw = d.nwaves;
    const unsigned long long *isum = reinterpret_cast<const unsigned long long *>(ws + d.stat_off);
    const unsigned long long *nonc = isum + nw;
    const unsigned int *imax = reinterpret_cast<const unsigned int *>(isum + 2 * nw);
    unsigned long long m = 0, s = 0, c = 0;
    for (int w = threadIdx.x; w < nw; w += kBlock) {
        m = max(m, (unsigned long long)imax[w]);
        s += isum[w];
        c += nonc[w];
    }
    sm[0][threadIdx.x] = m;
    sm[1][threadIdx.x] = s;
    sm[2][threadIdx.x] = c;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            sm[0][threadIdx.x] = max(sm[0][threadIdx.x], sm[0][threadIdx.x + o]);
            sm[1][threadIdx.x] += sm[1][threadIdx.x + o];
            sm[2][threadIdx.x] += sm[2][threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        totals[3 * blockIdx.x + 0] = sm[0][0];
        totals[3 * blockIdx.x + 1] = sm[1][0];
        totals[3 * blockIdx.x + 2] = sm[2][0];
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
namespace {

// One shape of the fused sweep: allow its dynamic LDS, or launch it.
template <int P, int WP, int G, int DRV, bool F32>
hipError_t fused_t(const StepArgs *a, int blocks, size_t lds, hipStream_t s)
{
    if (!a)
        return hipFuncSetAttribute(reinterpret_cast<const void *>(&sweep_fused<P, WP, G, DRV, F32>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((sweep_fused<P, WP, G, DRV, F32>), dim3(blocks), dim3(64 * WP * G), lds, s, *a);
    return hipGetLastError();
}

template <int P, int WP, int G, bool F32>
hipError_t fused_by_driver(int driver, const StepArgs *a, int blocks, size_t lds, hipStream_t s)
{
    switch (driver) {
    case BSDE_DRIVER_LINEAR: return fused_t<P, WP, G, BSDE_DRIVER_LINEAR, F32>(a, blocks, lds, s);
    case BSDE_DRIVER_BIDASK: return fused_t<P, WP, G, BSDE_DRIVER_BIDASK, F32>(a, blocks, lds, s);
    case BSDE_DRIVER_CUBIC: return fused_t<P, WP, G, BSDE_DRIVER_CUBIC, F32>(a, blocks, lds, s);
    default: return fused_t<P, WP, G, BSDE_DRIVER_EXP, F32>(a, blocks, lds, s);
    }
}

template <int P, int DRV, bool F32>
hipError_t launch_direct_t(const StepArgs &a, int blocks, size_t lds, hipStream_t s)
{
    if (a.dsplit == 1) {
        hipLaunchKernelGGL((sweep_direct<P, DRV, F32, false>), dim3(blocks), dim3(kBlock), lds, s, a);
        return hipGetLastError();
    }
    if constexpr (P == 1) {
        hipLaunchKernelGGL((sweep_direct<1, DRV, F32, true>), dim3(blocks * a.dsplit), dim3(kBlock),
                           lds, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((direct_finish<DRV, F32>), dim3(blocks), dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;  // split steps take one point per lane
}

template <int P, int DRV, bool F32>
hipError_t launch_gather_t(const StepArgs &a, int blocks, size_t, hipStream_t s)
{
    static_assert(P == 1, "one point per lane");
    hipLaunchKernelGGL((sweep_gather<DRV, F32>), dim3(blocks), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

#define BSDE_BY_DRIVER(F, TP, ...)                                     \
    switch (driver) {                                                  \
    case BSDE_DRIVER_LINEAR: return F<TP, BSDE_DRIVER_LINEAR, F32>(__VA_ARGS__); \
    case BSDE_DRIVER_BIDASK: return F<TP, BSDE_DRIVER_BIDASK, F32>(__VA_ARGS__); \
    case BSDE_DRIVER_CUBIC: return F<TP, BSDE_DRIVER_CUBIC, F32>(__VA_ARGS__);   \
    default: return F<TP, BSDE_DRIVER_EXP, F32>(__VA_ARGS__);                    \
    }

template <int P, bool F32>
hipError_t direct_by_driver(int driver, const StepArgs &a, int blocks, size_t lds, hipStream_t s)
{
    BSDE_BY_DRIVER(launch_direct_t, P, a, blocks, lds, s)
}

template <bool F32>
hipError_t gather_by_driver(int driver, const StepArgs &a, int blocks, hipStream_t s)
{
    BSDE_BY_DRIVER(launch_gather_t, 1, a, blocks, 0, s)
}

#undef BSDE_BY_DRIVER

// The shapes built: X(P, WP, G, forms), forms 1 FP64, 2 FP32, 3 both.  The plan
// chooses among kShapes64 and kShapes32; the others are for requests (BSDE_SWEEP).
#define BSDE_FUSED_SHAPES(X) \
    X(1, 4, 1, 3)            \
    X(1, 4, 2, 3)            \
    X(2, 4, 1, 3)            \
    X(2, 4, 2, 3)            \
    X(4, 4, 1, 3)            \
    X(4, 4, 2, 3)            \
    X(1, 1, 8, 1)            \
    X(2, 1, 8, 1)            \
    X(4, 1, 8, 1)            \
    X(4, 4, 4, 1)            \
    X(1, 2, 1, 2)            \
    X(1, 8, 1, 2)            \
    X(1, 16, 1, 2)

// a = NULL: allow the shape's dynamic LDS instead of launching it
hipError_t fused_shape(int P, int WP, int G, bool f32, int driver, const StepArgs *a, int blocks,
                       size_t lds, hipStream_t s)
{
#define BSDE_SHAPE(p, w, g, forms)                                                   \
    if (P == p && WP == w && G == g) {                                               \
        if constexpr ((forms) & 2)                                                   \
            if (f32) return fused_by_driver<p, w, g, true>(driver, a, blocks, lds, s); \
        if constexpr ((forms) & 1)                                                   \
            if (!f32) return fused_by_driver<p, w, g, false>(driver, a, blocks, lds, s); \
    }
    BSDE_FUSED_SHAPES(BSDE_SHAPE)
#undef BSDE_SHAPE
    return hipErrorInvalidValue;
}

}  // namespace

bool fused_supported(int P, int WP, int G, bool f32)
{
#define BSDE_SHAPE(p, w, g, forms) \
    if (P == p && WP == w && G == g && ((forms) & (f32 ? 2 : 1))) return true;
    BSDE_FUSED_SHAPES(BSDE_SHAPE)
#undef BSDE_SHAPE
    return false;
}
bool direct_p_supported(int P) { return P == 1 || P == 2 || P == 4; }

hipError_t launch_sweep_fused(int P, int WP, int G, bool F32, int driver, const StepArgs &a, int blocks,
                              size_t lds, hipStream_t s)
{
    return fused_shape(P, WP, G, F32, driver, &a, blocks, lds, s);
}

namespace {
template <int WP, int G, int DRV>
hipError_t located_t(const StepArgs *a, int blocks, size_t lds, hipStream_t s)
{
    if (!a)
        return hipFuncSetAttribute(reinterpret_cast<const void *>(&sweep_fused<1, WP, G, DRV, false, true>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((sweep_fused<1, WP, G, DRV, false, true>), dim3(blocks), dim3(64 * WP * G), lds, s, *a);
    return hipGetLastError();
}
template <int WP, int G>
hipError_t located_by_driver(int driver, const StepArgs *a, int blocks, size_t lds, hipStream_t s)
{
    switch (driver) {
    case BSDE_DRIVER_LINEAR: return located_t<WP, G, BSDE_DRIVER_LINEAR>(a, blocks, lds, s);
    case BSDE_DRIVER_BIDASK: return located_t<WP, G, BSDE_DRIVER_BIDASK>(a, blocks, lds, s);
    case BSDE_DRIVER_CUBIC: return located_t<WP, G, BSDE_DRIVER_CUBIC>(a, blocks, lds, s);
    default: return located_t<WP, G, BSDE_DRIVER_EXP>(a, blocks, lds, s);
    }
}
// 64-point tiles with eight node groups, or 256-point tiles with one
hipError_t located(int WP, int driver, const StepArgs *a, int blocks, size_t lds, hipStream_t s)
{
    return WP == 1 ? located_by_driver<1, 8>(driver, a, blocks, lds, s)
                   : located_by_driver<4, 1>(driver, a, blocks, lds, s);
}
}  // namespace

hipError_t launch_sweep_located(int WP, int driver, const StepArgs &a, int blocks, size_t lds, hipStream_t s)
{
    return located(WP, driver, &a, blocks, lds, s);
}

hipError_t set_located_lds_limit(int WP, int driver, size_t lds)
{
    return located(WP, driver, nullptr, 0, lds, nullptr);
}

hipError_t set_fused_lds_limit(int P, int WP, int G, bool F32, int driver, size_t lds)
{
    return fused_shape(P, WP, G, F32, driver, nullptr, 0, lds, nullptr);
}

hipError_t launch_sweep_direct(int P, bool F32, int driver, const StepArgs &a, int blocks,
                               size_t lds, hipStream_t s)
{
    switch (P) {
    case 1: return F32 ? direct_by_driver<1, true>(driver, a, blocks, lds, s)
                       : direct_by_driver<1, false>(driver, a, blocks, lds, s);
    case 2: return F32 ? direct_by_driver<2, true>(driver, a, blocks, lds, s)
                       : direct_by_driver<2, false>(driver, a, blocks, lds, s);
    case 4: return F32 ? direct_by_driver<4, true>(driver, a, blocks, lds, s)
                       : direct_by_driver<4, false>(driver, a, blocks, lds, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sweep_gather(bool F32, int driver, const StepArgs &a, int blocks, hipStream_t s)
{
    return F32 ? gather_by_driver<true>(driver, a, blocks, s)
               : gather_by_driver<false>(driver, a, blocks, s);
}

hipError_t launch_spline(bool f32, const StepArgs &a, int mode, int blocks, hipStream_t s)
{
    if (f32)
        hipLaunchKernelGGL(spline_layer<true>, dim3(blocks), dim3(kBlock), 0, s, a, mode);
    else
        hipLaunchKernelGGL(spline_layer<false>, dim3(blocks), dim3(kBlock), 0, s, a, mode);
    return hipGetLastError();
}

hipError_t launch_coef(const StepArgs &a, int blocks, hipStream_t s)
{
    hipLaunchKernelGGL(coef_layer, dim3(blocks), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_scatter(const ScatterChunk &c, char *ws, const InstDesc *desc, int blocks_x,
                          hipStream_t s)
{
    hipLaunchKernelGGL(scatter_layers, dim3(blocks_x, c.count), dim3(kBlock), 0, s, c, ws, desc);
    return hipGetLastError();
}

hipError_t launch_gather(const GatherChunk &c, char *ws, const InstDesc *desc, int blocks_x,
                         unsigned long long *nonfinite, hipStream_t s)
{
    hipLaunchKernelGGL(gather_layers, dim3(blocks_x, c.count), dim3(kBlock), 0, s, c, ws, desc,
                       nonfinite);
    return hipGetLastError();
}

hipError_t launch_clear(unsigned long long *p, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(clear_u64, dim3(64), dim3(kBlock), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_reduce_stats(char *ws, const InstDesc *desc, int count,
                               unsigned long long *totals, hipStream_t s)
{
    hipLaunchKernelGGL(reduce_stats, dim3(count), dim3(kBlock), 0, s, ws, desc, totals);
    return hipGetLastError();
}

}  // namespace bsde
