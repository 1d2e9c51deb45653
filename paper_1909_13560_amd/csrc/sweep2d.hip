// sweep2d.hip -- the backward sweep on a two-dimensional tensor grid
// (arXiv:1909.13560, eq (20)-(21); Section 5, Examples 4 and 5).
//
// The expectations over the L x L tensor Gauss-Hermite nodes use the tensor
// natural spline of each layer.  Its 16-term evaluation at a node
// (i0 + s0, i1 + s1) is regrouped by axes:
//   U(q) = A0 v(p, q)    + B0 v(p+1, q)    + C0 Mxx(p, q)   + D0 Mxx(p+1, q)
//   V(q) = A0 Myy(p, q)  + B0 Myy(p+1, q)  + C0 Mxxyy(p, q) + D0 Mxxyy(p+1, q)
//   S    = A1 U(q) + B1 U(q+1) + C1 V(q) + D1 V(q+1)      (p = i0 + m0, q = i1 + m1)
// With X = x + drift t + vol W and vol lower triangular, the axis-0 offset
// s0 depends on the axis-0 Gauss-Hermite index l0 only, so for one l0 the
// block evaluates (U, V) once per (tile row, window column) into LDS and
// every node l1 of that row costs one axis-1 evaluation per function.
//
// Two forms: sweep2d / sweep2d_ahead on value and derivative planes (the FP32
// form's spline, the bicubic in both forms), and sweep2b on planes of tensor
// B-spline coefficients (FP64 natural spline), further down.
#include "sweep2d.h"

namespace bsde {

namespace {

__device__ inline double f_linear2(const DriverParams &p, double y, double z1, double z2)
{
    return fma(p.p0, y, fma(p.p1, z1, fma(p.p2, z2, p.p3)));
}

__device__ inline size_t pidx(const Sweep2Args &a, int i0, int i1)
{
    return (size_t)(i0 + a.pad0) * a.npad1 + (size_t)(i1 + a.pad1);
}

// (U, V) of function f, tile row rr, window column cc in the LDS window:
// column slots of 3 functions, the even columns of a row first.
__device__ inline int uv_index(int half, int f, int rr, int cc)
{
    return ((rr * 2 + (cc & 1)) * half + (cc >> 1)) * 3 + f;
}

// Node record through the constant address space: the address is the same
// for the whole wavefront, so this compiles to scalar loads into SGPRs.
__device__ inline Node2 load_node2(const Node2 *p)
{
    const __attribute__((address_space(4))) Node2 *q =
        (const __attribute__((address_space(4))) Node2 *)p;
    Node2 n;
    n.B1 = q->B1;
    n.C1 = q->C1;
    n.D1 = q->D1;
    n.cfy = q->cfy;
    n.cfz1 = q->cfz1;
    n.cfz2 = q->cfz2;
    n.cz = q->cz;
    n.cy = q->cy;
    n.cyz1 = q->cyz1;
    n.cyz2 = q->cyz2;
    return n;
}

// Node flags: bit 0 the y expectation (layer j = K_y), bit 1 the y-hat terms
// of z^n (layer j = 1 of the z form E[y^{n+1} dW]/dt).
// CLAMP: the node's axis-1 cell q may leave the grid, and a cell that does not
// lie inside it evaluates to the value at its first point (the nearest grid
// line: the ghost records hold it), i.e. the interpolant at the coordinate
// clamped to the box.  The natural spline gets that from its ghost records
// alone (its second derivatives vanish at the ends); the bicubic's first
// derivatives do not, so its weights B1, C1, D1 are dropped there.
// A lane holds kCols2 = 2 adjacent columns c, c+1 (c even): the node of the
// second sits one record further, so the two read three (U, V) records per
// function, not four: window columns c+s, c+s+1, c+s+2, i.e. column slots
// c/2 + (s >> 1) and c/2 + (s >> 1) + 1 of the parity of s and one slot of
// the other parity (s, the node's window offset, is wavefront-uniform).
static_assert(kCols2 == 2, "the parity-split window serves two columns per lane");
template <int NF, bool CLAMP>
__device__ inline void node2_accumulate(const Sweep2Args &a, const double2 *uvl, const Node2 &nd,
                                        int s, int q, double (&Y)[kCols2],
                                        double (&Z1)[kCols2], double (&Z2)[kCols2])
// uvl: function 0 of the lane's column slot c/2 (even half of its tile row)
{
    const int h0 = ((s & 1) * a.half + (s >> 1)) * 3;              // records 0 and 2
    const int h1 = (((s + 1) & 1) * a.half + ((s + 1) >> 1)) * 3;  // record 1
    double2 p[3][kCols2 + 1];
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        p[f][0] = uvl[h0 + f];
        p[f][1] = uvl[h1 + f];
        p[f][2] = uvl[h0 + 3 + f];
    }
#pragma unroll
    for (int k = 0; k < kCols2; ++k) {
        double B1 = nd.B1, C1 = nd.C1, D1 = nd.D1;
        if (CLAMP && !(q + k >= 0 && q + k < a.n1 - 1)) B1 = C1 = D1 = 0.0;
        double h[3];
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            const double2 p0 = p[f][k], p1 = p[f][k + 1];
            h[f] = fma(B1, p1.x - p0.x, fma(C1, p0.y, fma(D1, p1.y, p0.x)));
        }
        const double fh = f_linear2(a.drv, h[0], h[1], h[2]);
        Y[k] = fma(nd.cfy, fh, Y[k]);
        if (NF & 1) Y[k] = fma(nd.cy, h[0], Y[k]);
        Z1[k] = fma(nd.cfz1, fh, fma(nd.cz, h[1], Z1[k]));
        Z2[k] = fma(nd.cfz2, fh, fma(nd.cz, h[2], Z2[k]));
        if (NF & 2) {
            Z1[k] = fma(nd.cyz1, h[0], Z1[k]);
            Z2[k] = fma(nd.cyz2, h[0], Z2[k]);
        }
    }
}

// The L nodes l1 of one axis-0 row of layer j, for the lane's points.  The
// node records come through scalar loads and the axis-1 offsets, one per
// lane in mv, through readlane, so the only per-node LDS reads are the
// (U, V) records; two nodes per iteration share one wait.
// uvl: the lane's slot in the window (see node2_accumulate), i1 its first
// grid column, so that a node's window offset is s = m1 - m1lo and its
// axis-1 cell q = m1 + i1.
template <int NF, bool CLAMP>
__device__ inline void row_nodes(const Sweep2Args &a, const double2 *uvl, const Node2 *ntab,
                                 int mv, int m1lo, int i1, double (&Y)[kCols2],
                                 double (&Z1)[kCols2], double (&Z2)[kCols2])
{
    int l1 = 0;
#pragma unroll 1
    for (; l1 + 1 < a.L; l1 += 2) {
        const Node2 n0 = load_node2(ntab + l1), n1 = load_node2(ntab + l1 + 1);
        const int m0 = __builtin_amdgcn_readlane(mv, l1), m1 = __builtin_amdgcn_readlane(mv, l1 + 1);
        node2_accumulate<NF, CLAMP>(a, uvl, n0, m0 - m1lo, m0 + i1, Y, Z1, Z2);
        node2_accumulate<NF, CLAMP>(a, uvl, n1, m1 - m1lo, m1 + i1, Y, Z1, Z2);
    }
    if (l1 < a.L) {
        const Node2 n0 = load_node2(ntab + l1);
        const int m0 = __builtin_amdgcn_readlane(mv, l1);
        node2_accumulate<NF, CLAMP>(a, uvl, n0, m0 - m1lo, m0 + i1, Y, Z1, Z2);
    }
}

template <bool CLAMP>
__device__ inline void row_nodes_nf(int nf, const Sweep2Args &a, const double2 *uvl,
                                    const Node2 *ntab, int mv, int m1lo, int i1,
                                    double (&Y)[kCols2], double (&Z1)[kCols2], double (&Z2)[kCols2])
{
    if (nf == 0)
        row_nodes<0, CLAMP>(a, uvl, ntab, mv, m1lo, i1, Y, Z1, Z2);
    else if (nf == 1)
        row_nodes<1, CLAMP>(a, uvl, ntab, mv, m1lo, i1, Y, Z1, Z2);
    else if (nf == 2)
        row_nodes<2, CLAMP>(a, uvl, ntab, mv, m1lo, i1, Y, Z1, Z2);
    else
        row_nodes<3, CLAMP>(a, uvl, ntab, mv, m1lo, i1, Y, Z1, Z2);
}

}  // namespace

// The FP32 form stores a value as fl(v + e) with e the residual carried from
// the layer it was computed from, and keeps the new residual (as in 1-D).
__device__ inline void store_fed_back2(float *val, float *res, size_t o, double v, float e)
{
    const double t = v + (double)e;
    const float q = (float)t;
    val[o] = q;
    res[o] = (float)(t - (double)q);
}

// Picard iteration of the implicit y equation at one point, from y; a fixed
// number of iterations ends early where an iterate repeats one of the two
// before it, with the value that the last iteration would give.
__device__ inline double picard2(const Sweep2Args &a, double y, double Yc, double z1, double z2,
                                 unsigned int &it, bool &conv)
{
    it = 0;
    conv = true;
    const unsigned int itmax = (unsigned int)a.picard_max;
    if (a.picard_tol > 0.0) {
        conv = false;
        while (it < itmax) {
            const double yn = fma(a.h0, f_linear2(a.drv, y, z1, z2), Yc);
            ++it;
            const double dy = fabs(yn - y);
            y = yn;
            if (dy <= a.picard_tol * fmax(1.0, fabs(y))) {
                conv = true;
                break;
            }
        }
    } else {
        double y2 = y;
        while (it < itmax) {
            const double yn = fma(a.h0, f_linear2(a.drv, y, z1, z2), Yc);
            ++it;
            if (yn == y || yn == y2) {
                if (yn == y || ((itmax - it) & 1u) == 0) y = yn;
                it = itmax;
                break;
            }
            y2 = y;
            y = yn;
        }
    }
    return y;
}

// The implicit y equation by Picard iteration from y^{n+1} and the stores, per
// point of the lane (row i0, columns t1 + c + k); idx: the tile, tid: the thread.
template <typename E>
__device__ inline void finish2d(const Sweep2Args &a, int idx, int tid, int i0, int t1, int c,
                                const double (&Y)[kCols2], const double (&Z1)[kCols2],
                                const double (&Z2)[kCols2])
{
    const int S = a.K + 1;
    const E *prev = plane2<E>(a, (a.n + 1) % S, 0);
    E *out = plane2<E>(a, a.n % S, 0);
    unsigned int it_max = 0, it_sum = 0, nonconv = 0;
#pragma unroll
    for (int k = 0; k < kCols2; ++k) {
        const int i1 = t1 + c + k;
        const bool valid = i0 < a.n0 && i1 < a.n1;
        const size_t o = pidx(a, min(i0, a.n0 - 1), min(i1, a.n1 - 1));
        double y = prev[o];
        unsigned int it;
        bool conv;
        y = picard2(a, y, Y[k], Z1[k], Z2[k], it, conv);
        if (valid) {
            if constexpr (std::is_same<E, float>::value) {
                // residuals of y^{n+K_y} (y recurrence) and of z^{n+1} (z recurrence)
                const float *ry = plane2<float>(a, (a.n + a.Ky) % S, 12);
                const float *rz = plane2<float>(a, (a.n + 1) % S, 13);
                float *res = plane2<float>(a, a.n % S, 12);
                store_fed_back2(out, res, o, y, ry[o]);
                store_fed_back2(out + 4 * a.plane, res + a.plane, o, Z1[k], rz[o]);
                store_fed_back2(out + 8 * a.plane, res + 2 * a.plane, o, Z2[k], rz[o + a.plane]);
            } else {
                out[o] = y;
                out[o + 4 * a.plane] = Z1[k];
                out[o + 8 * a.plane] = Z2[k];
            }
            if (a.n == a.n_stop) {
                const size_t np = (size_t)a.n0 * a.n1, kk = (size_t)i0 * a.n1 + i1;
                a.fin[kk] = y;
                a.fin[np + kk] = Z1[k];
                a.fin[2 * np + kk] = Z2[k];
            }
            it_max = max(it_max, it);
            it_sum += it;
            nonconv += conv ? 0u : 1u;
        }
    }
    if (a.st_iter_max) {
        it_max = wave_max_u32(it_max);
        it_sum = wave_sum_u32(it_sum);
        nonconv = wave_sum_u32(nonconv);
        if ((tid & 63) == 0) {
            const int w = idx * kWaves2 + tid / 64;
            a.st_iter_max[w] = max(a.st_iter_max[w], it_max);
            a.st_iter_sum[w] += it_sum;
            a.st_nonconv[w] += nonconv;
        }
    }
}

// One time step: layer n from layers n+1..n+K.  Block = kTile2R x kTile2C points.
// Dynamic LDS: (U, V) of 3 functions x kTile2R rows x 2 a.half columns.  E: the
// element type of the ring planes; the arithmetic is double in both forms.
// The occupancy hint holds the kernel at 89 VGPRs (five waves per SIMD, no
// scratch); left to itself the compiler takes 131 (three waves) for the
// parity-split window addressing.
template <typename E>
__global__ void __launch_bounds__(kThreads2) __attribute__((amdgpu_waves_per_eu(4)))
sweep2d(const Sweep2Args a)
{
    extern __shared__ double2 uv[];
    const int tiles1 = (a.n1 + kTile2C - 1) / kTile2C;
    const int idx = xcd_tile(blockIdx.x, gridDim.x);
    const int t0 = (idx / tiles1) * kTile2R, t1 = (idx % tiles1) * kTile2C;
    const int tid = threadIdx.x;
    constexpr int kLanesRow = kTile2C / kCols2;  // lanes per tile row
    const int r = __builtin_amdgcn_readfirstlane(tid / kLanesRow), c = (tid % kLanesRow) * kCols2;
    const int S = a.K + 1;
    double Y[kCols2], Z1[kCols2], Z2[kCols2];
#pragma unroll
    for (int k = 0; k < kCols2; ++k) Y[k] = Z1[k] = Z2[k] = 0.0;
    for (int j = 1; j <= a.K; ++j) {
        const E *slot = plane2<E>(a, (a.n + j) % S, 0);
        for (int l0 = 0; l0 < a.L; ++l0) {
            const int rowi = (j - 1) * a.L + l0;
            const Node2Row row = a.rows[rowi];
            const int W = kTile2C + row.m1hi - row.m1lo + 2;
            // the row's axis-1 offsets, one per lane (L <= 64)
            const int mv = a.m1[(size_t)rowi * a.L + min(tid & 63, a.L - 1)];
            // axis-0 evaluation at s0 for the tile rows and the window columns
            for (int e = tid; e < kTile2R * W; e += kThreads2) {
                const int rr = e / W, cc = e - rr * W;
                const int p = t0 + rr + row.m0;  // the node's axis-0 cell
                const size_t o = pidx(a, p, t1 + row.m1lo + cc);
                const size_t o1 = o + a.npad1;
                // a cell outside the grid evaluates to its first point's record
                // (clamped coordinate; see node2_accumulate).  For the natural
                // spline this changes nothing: there both differences and both
                // second derivatives in such a cell are exact zeros.
                const bool in = p >= 0 && p < a.n0 - 1;
                const double B0 = in ? row.B0 : 0.0, C0 = in ? row.C0 : 0.0, D0 = in ? row.D0 : 0.0;
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    const E *v = slot + (size_t)(4 * f) * a.plane;
                    const E *mxx = v + a.plane, *myy = v + 2 * a.plane, *mxy = v + 3 * a.plane;
                    const double v0 = v[o], y0 = myy[o];
                    const double U = fma(B0, (double)v[o1] - v0,
                                         fma(C0, (double)mxx[o], fma(D0, (double)mxx[o1], v0)));
                    const double V = fma(B0, (double)myy[o1] - y0,
                                         fma(C0, (double)mxy[o], fma(D0, (double)mxy[o1], y0)));
                    uv[uv_index(a.half, f, rr, cc)] = make_double2(U, V);
                }
            }
            __syncthreads();
            const Node2 *ntab = a.nodes + (size_t)rowi * a.L;
            const int nf = (j == a.Ky ? 1 : 0) | (j == 1 && a.zform ? 2 : 0);
            // the bicubic needs the per-node cell check only where the tile's
            // node cells can leave the grid along axis 1 (block-uniform)
            const bool clamp = a.interp == BSDE_INTERP_BICUBIC_FD &&
                               (t1 + row.m1lo < 0 || t1 + kTile2C + row.m1hi > a.n1 - 1);
            const double2 *uvl = uv + uv_index(a.half, 0, r, c);
            if (clamp)
                row_nodes_nf<true>(nf, a, uvl, ntab, mv, row.m1lo, t1 + c, Y, Z1, Z2);
            else
                row_nodes_nf<false>(nf, a, uvl, ntab, mv, row.m1lo, t1 + c, Y, Z1, Z2);
            __syncthreads();
        }
    }
    finish2d<E>(a, idx, tid, t0 + r, t1, c, Y, Z1, Z2);
}

// The same step for grids of few tiles, which leave a CU one or two blocks to
// cover the staging's latency with: the raw planes of the next node row are
// loaded into registers before the nodes of this one, and two windows in LDS
// take turns, so a row costs one barrier and no exposed load.  Wavefronts whose
// columns all lie beyond the grid stage and then wait.  Same operations in the
// same order, same results.  Time of a whole step (sweep, derivative passes),
// L = 8, K = 3, with sweep2d and with this kernel: FP32 spline 129 x 129
// 133 -> 101 us, 387 x 387 150 -> 139 us; FP64 bicubic 250 x 250 150 -> 114 us,
// but 387 x 387 171 -> 249 us: 256 registers leave room for one block a CU.
constexpr int kPre2 = (kWin2 + kThreads2 - 1) / kThreads2;  // window columns per thread
template <typename E>
__global__ void __launch_bounds__(kThreads2) sweep2d_ahead(const Sweep2Args a)
{
    static_assert(kTile2R == 1, "one grid row per tile");
    extern __shared__ double2 uv[];
    const int tiles1 = (a.n1 + kTile2C - 1) / kTile2C;
    const int idx = xcd_tile(blockIdx.x, gridDim.x);
    const int i0 = idx / tiles1, t1 = (idx % tiles1) * kTile2C;
    const int tid = threadIdx.x, c = tid * kCols2;
    const int cols = min(kTile2C, (a.n1 - t1 + 127) & ~127);  // columns of wavefronts in the grid
    const bool idle = t1 + (tid & ~63) * kCols2 >= a.n1;  // wavefront beyond the grid
    const int S = a.K + 1, nrows = a.K * a.L, wsize = 6 * a.half;
    double Y[kCols2], Z1[kCols2], Z2[kCols2];
#pragma unroll
    for (int k = 0; k < kCols2; ++k) Y[k] = Z1[k] = Z2[k] = 0.0;
    E raw[kPre2][24];  // planes of the three functions at cells p and p + 1
    int mvn = 0;
    auto ahead = [&](int rowi, int j) {
        const Node2Row *row = a.rows + rowi;
        const int m0 = const_load(&row->m0), m1lo = const_load(&row->m1lo), m1hi = const_load(&row->m1hi);
        mvn = a.m1[(size_t)rowi * a.L + min(tid & 63, a.L - 1)];
        const E *slot = plane2<E>(a, (a.n + j) % S, 0);
        const int W = cols + m1hi - m1lo + 2;
#pragma unroll
        for (int u = 0; u < kPre2; ++u) {
            const int e = tid + u * kThreads2;
            if (e < W) {
                const unsigned o = (unsigned)pidx(a, i0 + m0, t1 + m1lo + e);
#pragma unroll
                for (int q = 0; q < 12; ++q) {
                    const E *v = slot + (size_t)q * a.plane;
                    raw[u][2 * q] = v[o];
                    raw[u][2 * q + 1] = v[o + (unsigned)a.npad1];
                }
            }
        }
    };
    ahead(0, 1);
    int buf = 0;
    for (int j = 1; j <= a.K; ++j) {
        for (int l0 = 0; l0 < a.L; ++l0, buf ^= 1) {
            const int rowi = (j - 1) * a.L + l0;
            const Node2Row *row = a.rows + rowi;
            const int m1lo = const_load(&row->m1lo), m1hi = const_load(&row->m1hi);
            const int p = i0 + const_load(&row->m0);
            const bool in = p >= 0 && p < a.n0 - 1;
            const double B0 = in ? const_load(&row->B0) : 0.0, C0 = in ? const_load(&row->C0) : 0.0,
                         D0 = in ? const_load(&row->D0) : 0.0;
            const int W = cols + m1hi - m1lo + 2;
            const int mv = mvn;
            double2 *win = uv + buf * wsize;
#pragma unroll
            for (int u = 0; u < kPre2; ++u) {
                const int e = tid + u * kThreads2;
                if (e < W) {
#pragma unroll
                    for (int f = 0; f < 3; ++f) {  // v, Mxx, Myy, Mxxyy at cells p and p + 1
                        const E *q = raw[u] + 8 * f;
                        const double v0 = q[0], y0 = q[4];
                        const double U = fma(B0, (double)q[1] - v0,
                                             fma(C0, (double)q[2], fma(D0, (double)q[3], v0)));
                        const double V = fma(B0, (double)q[5] - y0,
                                             fma(C0, (double)q[6], fma(D0, (double)q[7], y0)));
                        win[uv_index(a.half, f, 0, e)] = make_double2(U, V);
                    }
                }
            }
            __syncthreads();
            if (rowi + 1 < nrows) ahead(rowi + 1, l0 + 1 < a.L ? j : j + 1);
            if (idle) continue;
            const Node2 *ntab = a.nodes + (size_t)rowi * a.L;
            const int nf = (j == a.Ky ? 1 : 0) | (j == 1 && a.zform ? 2 : 0);
            const bool clamp = a.interp == BSDE_INTERP_BICUBIC_FD &&
                               (t1 + m1lo < 0 || t1 + kTile2C + m1hi > a.n1 - 1);
            const double2 *uvl = win + uv_index(a.half, 0, 0, c);
            if (clamp)
                row_nodes_nf<true>(nf, a, uvl, ntab, mv, m1lo, t1 + c, Y, Z1, Z2);
            else
                row_nodes_nf<false>(nf, a, uvl, ntab, mv, m1lo, t1 + c, Y, Z1, Z2);
        }
    }
    finish2d<E>(a, idx, tid, i0, t1, c, Y, Z1, Z2);
}

// ---------------------------------------------------------------------------
// Tensor natural spline of a layer (FP32 planes): M_xx and M_yy of the values,
// then M_xxyy as the axis-1 spline of M_xx, then the ghost points.
// ---------------------------------------------------------------------------
namespace {

// second difference of line values at k, oddly extended about 0 and n-1
template <typename E>
__device__ inline double rt_line(const E *v, long stride, int n, int k)
{
    const int per = 2 * (n - 1);
    int kk = k % per;
    if (kk < 0) kk += per;
    double sign = 1.0;
    if (kk > n - 1) {
        kk = per - kk;
        sign = -1.0;
    }
    if (kk == 0 || kk == n - 1) return 0.0;
    const double vm = v[(long)(kk - 1) * stride], v0 = v[(long)kk * stride],
                 vp = v[(long)(kk + 1) * stride];  // the arithmetic is double
    return sign * ((vp - v0) - (v0 - vm));
}

__device__ inline double spline_line(const float *v, long stride, int n, int i,
                                     const SplineFilter &F, double s6)
{
    if (i == 0 || i == n - 1) return 0.0;
    double acc = 0.0;
    if (i >= 32 && i <= n - 33) {
        const float *p = v + (long)(i - 32) * stride;
#pragma unroll
        for (int k = 0; k < kPcrTaps + 2; ++k) acc = fma(F.d[k], (double)p[(long)k * stride], acc);
    } else {
        for (int k = 0; k < kPcrTaps; ++k) acc = fma(F.c[k], rt_line(v, stride, n, i + k - 31), acc);
    }
    return s6 * acc;
}

constexpr int kRun = 16;  // consecutive outputs per thread of the line passes
// The axis-0 passes take four: 17 loads per output (mostly L2 hits) instead of
// 5, but four times the threads, which is what covers the loads' latency
// (387 x 387: 35 -> 9 us).
constexpr int kRunCols = 4;

// Outputs i0 .. i0 + kRun - 1 (those < n) of the natural spline of one line
// of n >= kMinLine values: M_i = s6 sum_k d[k] v~_{i-32+k}.  Each value is
// loaded once and feeds every output within the filter's reach.  Beyond the
// line's ends the values are reflected through the end points,
// v~_{-j} = 2 v_0 - v_j and v~_{n-1+j} = 2 v_{n-1} - v_{n-1-j}: their second
// differences are then the odd extension the natural end conditions call
// for, so the values form holds at every point; M_0 = M_{n-1} = 0.
template <int kRun>
__device__ inline void line_run(const float *v, long stride, int n, int i0, double s6, float *out,
                                long ostride)
{
    constexpr SplineTaps T = spline_taps();
    constexpr int H = kPcrTaps / 2 + 1;  // values on each side of an output
    double acc[kRun];
#pragma unroll
    for (int r = 0; r < kRun; ++r) acc[r] = 0.0;
    if (i0 >= H && i0 + kRun - 1 + H <= n - 1) {  // clear of both ends
        const float *p = v + (long)(i0 - H) * stride;
#pragma unroll
        for (int m = 0; m < kRun + 2 * H; ++m) {
            const double x = p[(long)m * stride];
#pragma unroll
            for (int r = 0; r < kRun; ++r)
                if (m - r >= 0 && m - r <= 2 * H) acc[r] = fma(T.d[m - r], x, acc[r]);
        }
    } else {
        const double v0 = v[0], vn = v[(long)(n - 1) * stride];  // double arithmetic
#pragma unroll
        for (int m = 0; m < kRun + 2 * H; ++m) {
            const int k = i0 - H + m;
            // reflected index; clamped too for the loads of outputs past the
            // end of a partial run, which are not stored
            const int kk = min(max(k < 0 ? -k : (k > n - 1 ? 2 * (n - 1) - k : k), 0), n - 1);
            const double y = v[(long)kk * stride];
            const double x = k < 0 ? 2.0 * v0 - y : (k > n - 1 ? 2.0 * vn - y : y);
#pragma unroll
            for (int r = 0; r < kRun; ++r)
                if (m - r >= 0 && m - r <= 2 * H) acc[r] = fma(T.d[m - r], x, acc[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < kRun; ++r) {
        const int i = i0 + r;
        if (i < n) out[(long)i * ostride] = (float)((i == 0 || i == n - 1) ? 0.0 : s6 * acc[r]);
    }
}

// The same outputs for lines shorter than kMinLine, one at a time.
template <int kRun>
__device__ inline void line_run_short(const float *v, long stride, int n, int i0,
                                      const SplineFilter &F, double s6, float *out, long ostride)
{
    for (int i = i0; i < min(i0 + kRun, n); ++i)
        out[(long)i * ostride] = (float)spline_line(v, stride, n, i, F, s6);
}

}  // namespace

// M_xx of field blockIdx.y (y, z1, z2): lines along axis 0.  Thread t:
// column t % n1 (adjacent lanes read adjacent columns), rows from
// kRun * (t / n1).
template <int kRun>
__global__ void __launch_bounds__(256) spline2d_cols(const Sweep2Args a, int slot,
                                                     const SplineFilter F)
{
    const long t = blockIdx.x * 256L + threadIdx.x;
    if (t >= (long)a.n1 * ((a.n0 + kRun - 1) / kRun)) return;
    const int i1 = (int)(t % a.n1), i0 = (int)(t / a.n1) * kRun;
    float *col = plane2<float>(a, slot, 4 * blockIdx.y) + pidx(a, 0, i1);
    if (a.n0 >= kMinLine)
        line_run<kRun>(col, a.npad1, a.n0, i0, F.s6[0], col + a.plane, a.npad1);
    else
        line_run_short<kRun>(col, a.npad1, a.n0, i0, F, F.s6[0], col + a.plane, a.npad1);
}

// Lines along axis 1 of field blockIdx.y / 2: the values give M_yy
// (blockIdx.y even), M_xx gives M_xxyy (odd).  Thread t: row t % n0, columns
// from kRun * (t / n0), so that a wavefront takes one branch of line_run.
__global__ void __launch_bounds__(256) spline2d_rows(const Sweep2Args a, int slot,
                                                     const SplineFilter F)
{
    const long t = blockIdx.x * 256L + threadIdx.x;
    if (t >= (long)a.n0 * ((a.n1 + kRun - 1) / kRun)) return;
    const int i0 = (int)(t % a.n0), i1 = (int)(t / a.n0) * kRun;
    const int f = blockIdx.y >> 1, g = blockIdx.y & 1;
    float *row = plane2<float>(a, slot, 4 * f) + pidx(a, i0, 0);
    const float *src = row + (size_t)g * a.plane;
    float *dst = row + (size_t)(2 + g) * a.plane;
    if (a.n1 >= kMinLine)
        line_run<kRun>(src, 1, a.n1, i1, F.s6[1], dst, 1);
    else
        line_run_short<kRun>(src, 1, a.n1, i1, F, F.s6[1], dst, 1);
}

// Lines along axis 1 of at least kMinLine points, through LDS: a block
// stages kRowTile rows x (kRowCols + 64) values of its source plane with
// coalesced loads (reflected through the line ends as in line_run), then each
// thread streams the 80 values of one run of kRun outputs from LDS.  Same
// arithmetic, in the same order, as line_run.
constexpr int kRowTile = 16;                   // rows per block
constexpr int kRowCols = 256 / kRowTile * kRun;  // outputs per row per block
constexpr int kRowIn = kRowCols + 2 * (kPcrTaps / 2 + 1);  // staged values per row
constexpr int kRowStride = kRowIn + 1;          // LDS row pitch (odd: fewer bank conflicts)

__global__ void __launch_bounds__(256) spline2d_rows_lds(const Sweep2Args a, int slot,
                                                         const SplineFilter F)
{
    constexpr SplineTaps T = spline_taps();
    constexpr int H = kPcrTaps / 2 + 1;
    __shared__ double sm[kRowTile * kRowStride];
    const int tiles1 = (a.n1 + kRowCols - 1) / kRowCols;
    const int r0 = (int)(blockIdx.x / tiles1) * kRowTile, c0 = (int)(blockIdx.x % tiles1) * kRowCols;
    const int f = blockIdx.y >> 1, g = blockIdx.y & 1;
    const int n = a.n1;
    float *plane0 = plane2<float>(a, slot, 4 * f);
    const float *src = plane0 + (size_t)g * a.plane;
    float *dst = plane0 + (size_t)(2 + g) * a.plane;
    for (int e = threadIdx.x; e < kRowTile * kRowIn; e += 256) {
        const int rr = e / kRowIn, cc = e - rr * kRowIn;
        const int i0 = r0 + rr;
        if (i0 >= a.n0) continue;
        const float *v = src + pidx(a, i0, 0);
        const int k = c0 - H + cc;
        const int kk = min(max(k < 0 ? -k : (k > n - 1 ? 2 * (n - 1) - k : k), 0), n - 1);
        const double y = v[kk];
        sm[rr * kRowStride + cc] =
            k < 0 ? 2.0 * (double)v[0] - y : (k > n - 1 ? 2.0 * (double)v[n - 1] - y : y);
    }
    __syncthreads();
    const int r = threadIdx.x % kRowTile, q = threadIdx.x / kRowTile;
    const int i0 = r0 + r, j0 = c0 + q * kRun;
    if (i0 >= a.n0 || j0 >= n) return;
    const double *w = sm + r * kRowStride + q * kRun;
    double acc[kRun];
#pragma unroll
    for (int u = 0; u < kRun; ++u) acc[u] = 0.0;
#pragma unroll
    for (int m = 0; m < kRun + 2 * H; ++m) {
        const double x = w[m];
#pragma unroll
        for (int u = 0; u < kRun; ++u)
            if (m - u >= 0 && m - u <= 2 * H) acc[u] = fma(T.d[m - u], x, acc[u]);
    }
    float *out = dst + pidx(a, i0, 0);
    const double s6 = F.s6[1];
#pragma unroll
    for (int u = 0; u < kRun; ++u) {
        const int i = j0 + u;
        if (i < n) out[i] = (float)((i == 0 || i == n - 1) ? 0.0 : s6 * acc[u]);
    }
}

// The paper's own 2-D interpolation (Section 3.3): bicubic from the values
// and the first and mixed derivatives, the derivatives by fourth-order
// finite differences (central inside, one-sided at the two points next to
// each end).  They go into the planes of the tensor spline's second
// derivatives: f_x in M_xx, f_y in M_yy, f_xy in M_xxyy; the sweep kernel is
// the same, with the Hermite basis weights in the node tables.
template <typename E>
__device__ inline double fd4_at(const E *f, long st, int n, int i, double inv12h)
{
    double v;  // double arithmetic on the (possibly float) values
    if (i >= 2 && i <= n - 3)
        v = (double)f[(i - 2) * st] - 8.0 * f[(i - 1) * st] + 8.0 * f[(i + 1) * st] - f[(i + 2) * st];
    else if (i == 0)
        v = -25.0 * f[0] + 48.0 * f[st] - 36.0 * f[2 * st] + 16.0 * f[3 * st] - 3.0 * f[4 * st];
    else if (i == 1)
        v = -3.0 * f[0] - 10.0 * f[st] + 18.0 * f[2 * st] - 6.0 * f[3 * st] + f[4 * st];
    else if (i == n - 1)
        v = 25.0 * f[(n - 1) * st] - 48.0 * f[(n - 2) * st] + 36.0 * f[(n - 3) * st] -
            16.0 * f[(n - 4) * st] + 3.0 * f[(n - 5) * st];
    else
        v = 3.0 * f[(n - 1) * st] + 10.0 * f[(n - 2) * st] - 18.0 * f[(n - 3) * st] +
            6.0 * f[(n - 4) * st] - f[(n - 5) * st];
    return v * inv12h;
}

// f_x of field blockIdx.y along axis 0 (adjacent lanes on adjacent columns)
template <typename E>
__global__ void __launch_bounds__(256) fd2d_cols(const Sweep2Args a, int slot, double inv12h)
{
    const long t = blockIdx.x * 256L + threadIdx.x;
    if (t >= (long)a.n0 * a.n1) return;
    const int i0 = (int)(t / a.n1), i1 = (int)(t % a.n1);
    E *v = plane2<E>(a, slot, 4 * blockIdx.y);
    v[a.plane + pidx(a, i0, i1)] = (E)fd4_at(v + pidx(a, 0, i1), a.npad1, a.n0, i0, inv12h);
}

// Along axis 1 of field blockIdx.y / 2: f_y from the values (blockIdx.y
// even), f_xy from f_x (odd)
template <typename E>
__global__ void __launch_bounds__(256) fd2d_rows(const Sweep2Args a, int slot, double inv12h)
{
    const long t = blockIdx.x * 256L + threadIdx.x;
    if (t >= (long)a.n0 * a.n1) return;
    const int i0 = (int)(t / a.n1), i1 = (int)(t % a.n1);
    const int f = blockIdx.y >> 1, g = blockIdx.y & 1;
    E *v = plane2<E>(a, slot, 4 * f);
    const E *src = v + (size_t)g * a.plane;
    v[(size_t)(2 + g) * a.plane + pidx(a, i0, i1)] =
        (E)fd4_at(src + pidx(a, i0, 0), 1, a.n1, i1, inv12h);
}

// Ghost points: the data of the nearest grid point with the derivative
// planes across the crossed edge set to zero (clamped evaluation).
template <typename E>
__global__ void __launch_bounds__(256) ghosts2d(const Sweep2Args a, int slot, int npad0)
{
    const long i = blockIdx.x * 256L + threadIdx.x;
    if (i >= (long)npad0 * a.npad1) return;
    const int g0 = (int)(i / a.npad1) - a.pad0, g1 = (int)(i % a.npad1) - a.pad1;
    const bool in0 = g0 >= 0 && g0 < a.n0, in1 = g1 >= 0 && g1 < a.n1;
    if (in0 && in1) return;
    const size_t src = pidx(a, min(max(g0, 0), a.n0 - 1), min(max(g1, 0), a.n1 - 1));
    E *base = plane2<E>(a, slot, 0);
    for (int f = 0; f < 3; ++f) {
        E *v = base + (size_t)(4 * f) * a.plane;
        v[i] = v[src];
        v[a.plane + i] = in0 ? v[a.plane + src] : (E)0;
        v[2 * a.plane + i] = in1 ? v[2 * a.plane + src] : (E)0;
        v[3 * a.plane + i] = (E)0;
    }
}

template <typename E>
__global__ void __launch_bounds__(256) scatter2d(const Sweep2Args a, const double *__restrict__ iy,
                                                 const double *__restrict__ iz)
{
    const long np = (long)a.n0 * a.n1;
    const long i = blockIdx.x * 256L + threadIdx.x;
    const int r = blockIdx.y;
    if (i >= np) return;
    const int n = a.n + 1 + r;  // a.n = N - K: layers N-K+1 .. N
    E *base = plane2<E>(a, n % (a.K + 1), 0);
    const size_t o = pidx(a, (int)(i / a.n1), (int)(i % a.n1));
    const double v[3] = {iy[r * np + i], iz[(2L * r) * np + i], iz[(2L * r + 1) * np + i]};
    for (int f = 0; f < 3; ++f) {
        if constexpr (std::is_same<E, float>::value) {  // value and its rounding residual
            store_fed_back2(base + 4 * f * a.plane, base + (12 + f) * a.plane, o, v[f], 0.0f);
        } else {
            base[(size_t)a.vstep * f * a.plane + o] = v[f];
        }
    }
}

__global__ void __launch_bounds__(256) gather2d(const Sweep2Args a, double *__restrict__ y0,
                                                double *__restrict__ z0,
                                                unsigned long long *nonfinite)
{
    const long np = (long)a.n0 * a.n1;
    unsigned int bad = 0;
    for (long i = blockIdx.x * 256L + threadIdx.x; i < np; i += (long)gridDim.x * 256) {
        const double y = a.fin[i], z1 = a.fin[np + i], z2 = a.fin[2 * np + i];
        y0[i] = y;
        z0[i] = z1;
        z0[np + i] = z2;
        bad += (isfinite(y) && isfinite(z1) && isfinite(z2)) ? 0u : 1u;
    }
    bad = wave_sum_u32(bad);
    if (nonfinite && (threadIdx.x & 63) == 0 && bad) atomicAdd(nonfinite, (unsigned long long)bad);
}

// ---------------------------------------------------------------------------
// B-spline form (FP64, natural spline).
//
// A layer's tensor spline is S = sum_ab b_a(phi0) b_b(phi1) c(p-1+a, q-1+b).
// For one axis-0 node l0 the four source rows combine into one row of
// coefficients per function; with the linear driver the functions that the
// sums of eq (20) need are linear in them, so a column of the window holds
//   s0 = u = p0 y + p1 z1 + p2 z2,  s1 = C z1 + Gu u + Gy y,  s2 = C z2
// and a node l1 costs, per point, t = sum_b w_b s0 (Y += H t, Z2 += gu t),
// Z1 += sum w_b s1, Z2 += sum w_b s2: 14 operations, against 20 with values
// and second derivatives of y, z1, z2 and the driver per node.  The layer
// j = K_y (and z form E[y dW]/dt at j = 1) adds a pass over y alone.
//
// One wavefront works by itself: it stages the window of its 256 columns (four
// per lane: a node reads 7 coefficients for 4 points) and runs the row's
// nodes without any block barrier, so the wavefronts of a CU drift apart and
// one stages while others compute.  The block's four wavefronts take every
// fourth node row of the same tile and add their sums in LDS at the end
// (classes 0+2, 1+3).  Bound: FP64 issue and LDS reads about equally (42 B per
// node and point).
//
// Cells outside the grid: along axis 0 the row's weights (uniform) become
// those of the end row; beyond the natural end the coefficient continues as
// 2 c(0) - c(1), folded into the weights of the first rows.  Along axis 1 the
// window continues the end column's coefficient as a constant, which is the
// clamped evaluation except in the two cells next to the end, whose error is
// (c(1) - c(0)) b_3 outside and (c(1) - c(0)) b_0 inside: per node two columns
// of the tile's row, summed over a row's nodes on the host (corr_l, corr_r).
// ---------------------------------------------------------------------------
namespace {

__device__ inline Node2B load_node2b(const Node2B *p)
{
    Node2B n{};
    n.w0 = const_load(&p->w0);
    n.w1 = const_load(&p->w1);
    n.w2 = const_load(&p->w2);
    n.w3 = const_load(&p->w3);
    n.gu = const_load(&p->gu);
    n.gy = const_load(&p->gy);
    return n;
}

__device__ inline int slot4(int e) { return e + (e >> 2); }  // a pad slot per four columns

// seven consecutive columns from the lane's first at an offset res mod 4
template <int B, typename V>
__device__ inline void fetch7(const V *p, V (&r)[7])
{
#pragma unroll
    for (int q = 0; q < 7; ++q) r[q] = p[q + ((B + q) >> 2)];
}
template <typename V>
__device__ inline void fetch7(const V *p, int res, V (&r)[7])
{
    switch (res & 3) {
    case 0: fetch7<0>(p, r); asm volatile("; pattern 0"); break;
    case 1: fetch7<1>(p, r); asm volatile("; pattern 1"); break;
    case 2: fetch7<2>(p, r); asm volatile("; pattern 2"); break;
    default: fetch7<3>(p, r); asm volatile("; pattern 3"); break;
    }
}

// order the wavefront's own LDS writes and reads
__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kEdge2B = 4;  // columns 0, 1, n1 - 2, n1 - 1 kept beside the window

}  // namespace

size_t sweep2b_wave_lds(int spread)
{
    const int w = kTile2B + spread + 3;
    const int slots = w + w / 4 + 2;
    const size_t stage = (size_t)slots * (sizeof(double2) + sizeof(double)) + kEdge2B * 3 * sizeof(double);
    const size_t part = (size_t)kTile2B * 3 * sizeof(double);
    return (std::max(stage, part) + 15) / 16 * 16;
}

__global__ void __launch_bounds__(64 * kGroups2B) __attribute__((amdgpu_waves_per_eu(3)))
sweep2b(const Sweep2Args a)
{
    extern __shared__ double2 smem2b[];
    const int tiles1 = (a.n1 + kTile2B - 1) / kTile2B;
    const int idx = xcd_tile(blockIdx.x, gridDim.x);
    const int i0 = idx / tiles1, c0 = (idx % tiles1) * kTile2B;
    const int tid = threadIdx.x, lane = tid & 63;
    const int grp = __builtin_amdgcn_readfirstlane(tid >> 6);
    char *mine = reinterpret_cast<char *>(smem2b) + (size_t)grp * a.lds_wave;
    const int S = a.K + 1, n0 = a.n0, n1 = a.n1;
    double Y[4], Z1[4], Z2[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) Y[k] = Z1[k] = Z2[k] = 0.0;
    const int col = c0 + lane * 4;  // the lane's first column
    const bool near_l = c0 < a.nl, near_r = c0 + kTile2B > n1 - a.nr;
    const int nrows = a.K * a.L;
    // the node rows of this wavefront.  GUARD: no value that a node does not touch
    // is multiplied by a zero weight, which would spread a non-finite one (end
    // corrections of columns that have none, the rows beside the end row for cells
    // outside the grid along axis 0).  The guards in every pass cost 3-5 % on grids up
    // to 256^2 (16 nodes: 156 -> 161 us a step), so only a wavefront whose sums are not
    // finite makes the guarded pass, and then all of its rows again
    auto rows = [&](auto guard) {
        constexpr bool GUARD = decltype(guard)::value;
        // the row ahead: its first window columns (kPre per lane) are loaded while
        // the nodes of the row before are evaluated
        constexpr int kPre = 1;
        int nslot = a.n % S, njc = 0, nl0 = grp;  // layer and l0 of the row ahead
        const double *nq0 = nullptr;
        int nw0 = 0;
        double pf[kPre][12];
        auto load_column = [&](const double *q0, int q, double (&r)[12]) {
            // scalar row bases and one 32-bit column offset (a row is below 4 GiB)
            const unsigned o = (unsigned)q * 8u;
            const size_t st = (size_t)n1 * 8;
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                const char *v = reinterpret_cast<const char *>(q0 + (size_t)f * a.plane);
#pragma unroll
                for (int k = 0; k < 4; ++k) r[4 * f + k] = *reinterpret_cast<const double *>(v + k * st + o);
            }
        };
        auto column = [&](int w0, int e) { return min(max(w0 + e, 0), n1 - 1); };
        auto ahead = [&](int rowi) {  // loads for row rowi
            while (nl0 >= a.L || njc == 0) {  // rows are ordered by layer
                if (njc != 0) nl0 -= a.L;
                ++njc;
                nslot = nslot + 1 == S ? 0 : nslot + 1;
            }
            nl0 += kGroups2B;
            const Row2B *rp = a.rowsb + rowi;
            const int r0 = min(max(i0 + const_load(&rp->m0) - 1, 0), n0 - 4);
            nq0 = plane2<double>(a, nslot, 3) + (size_t)r0 * n1;
            nw0 = c0 + const_load(&rp->m1lo) - 1;
#pragma unroll
            for (int u = 0; u < kPre; ++u) load_column(nq0, column(nw0, lane + 64 * u), pf[u]);
        };
        if (grp < nrows) ahead(grp);
        for (int rowi = grp; rowi < nrows; rowi += kGroups2B) {
            const Row2B *rp = a.rowsb + rowi;
            const int m0 = const_load(&rp->m0), m1lo = const_load(&rp->m1lo), m1hi = const_load(&rp->m1hi);
            const bool extra = const_load(&rp->extra) != 0;
            const int W = kTile2B + (m1hi - m1lo) + 3;
            const int slots = W + (W >> 2) + 2;
            double2 *wa = reinterpret_cast<double2 *>(mine);      // (s0, s1)
            double *wb = reinterpret_cast<double *>(wa + slots);  // s2, then y in pass 2
            double *we = wb + slots;                              // end columns: s0, s1, s2 each
            const int mv = a.m1[(size_t)rowi * a.L + min(lane, a.L - 1)] - m1lo;
            // axis-0 weights on four rows r0 .. r0 + 3 inside the grid
            double b0 = const_load(&rp->b[0]), b1 = const_load(&rp->b[1]), b2 = const_load(&rp->b[2]),
                   b3 = const_load(&rp->b[3]);
            // (the loads take the rows min(max(p - 1, 0), n0 - 4) ..)
            const int p = i0 + m0;
            if (p < 0) {  // the value at the first row
                b0 = 1.0;
                b1 = b2 = b3 = 0.0;
            } else if (p > n0 - 2) {  // the value at the last row
                b3 = 1.0;
                b0 = b1 = b2 = 0.0;
            } else {
                if (p == 0) {  // c(-1) = 2 c(0) - c(1)
                    const double x = b0;
                    b0 = fma(2.0, x, b1);
                    b1 = b2 - x;
                    b2 = b3;
                    b3 = 0.0;
                }
                if (p == n0 - 2) {  // c(n0) = 2 c(n0 - 1) - c(n0 - 2); rows shift down by one
                    const double x = b3;
                    b3 = fma(2.0, x, b2);
                    b2 = b1 - x;
                    b1 = b0;
                    b0 = 0.0;
                }
            }
            const double *q0 = nq0;
            const int w0 = nw0;  // window column 0
            const double H = const_load(&rp->H), Gu = const_load(&rp->Gu), Gy = const_load(&rp->Gy),
                         C = const_load(&rp->C), ey = const_load(&rp->ey);
            const double p0 = a.drv.p0, p1 = a.drv.p1, p2 = a.drv.p2;
            auto combine = [&](const double *r) {
                if (GUARD && p < 0) return r[0];
                if (GUARD && p > n0 - 2) return r[3];
                return fma(b3, r[3], fma(b0, r[0], fma(b2, r[2], b1 * r[1])));
            };
            auto put = [&](int e, const double (&r)[12]) {
                const double y = combine(r), z1 = combine(r + 4), z2 = combine(r + 8);
                const double u = fma(p0, y, fma(p1, z1, p2 * z2));
                const double s1 = fma(C, z1, fma(Gu, u, Gy * y)), s2 = C * z2;
                if (e < W) {
                    wa[slot4(e)] = make_double2(u, s1);
                    wb[slot4(e)] = s2;
                } else if (e < W + kEdge2B) {  // the end columns
                    we[3 * (e - W)] = u;
                    we[3 * (e - W) + 1] = s1;
                    we[3 * (e - W) + 2] = s2;
                }
            };
            // element e of the staging: window column, then the four end columns
            auto staged = [&](int e) {
                const int x = min(e - W, kEdge2B - 1);
                return x < 0 ? column(w0, e) : x < 2 ? x : n1 - 4 + x;
            };
            wave_lds_fence();  // the last row's reads are done
#pragma unroll
            for (int u = 0; u < kPre; ++u) put(lane + 64 * u, pf[u]);
#pragma unroll 1
            for (int e = lane + 64 * kPre; e - lane < W + kEdge2B; e += 128) {
                double r[2][12];
#pragma unroll
                for (int u = 0; u < 2; ++u) load_column(q0, staged(e + 64 * u), r[u]);
#pragma unroll
                for (int u = 0; u < 2; ++u) put(e + 64 * u, r[u]);
            }
            wave_lds_fence();
            // corrections of the lane's columns: of the left end where the tile is
            // near both (the right one's then follow after the nodes)
            const double4 *ct = near_l ? a.corr_l + (size_t)rowi * a.nl : a.corr_r + (size_t)rowi * a.nr;
            const int cn = near_l ? a.nl : a.nr;
            double2 kc[4];
            if (near_l || near_r) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int c = near_l ? col + k : n1 - 1 - (col + k);
                    const double2 v = *reinterpret_cast<const double2 *>(ct + min(max(c, 0), cn - 1));
                    kc[k] = c >= 0 && c < cn ? v : make_double2(0.0, 0.0);
                }
            }
            if (rowi + kGroups2B < nrows) ahead(rowi + kGroups2B);
            const double2 *la = wa + slot4(lane * 4);
            const double *lb = wb + slot4(lane * 4);
            const Node2B *nodes = a.nodesb + (size_t)rowi * a.L;
#pragma unroll 1
            for (int l = 0; l < a.L; ++l) {
                const Node2B nd = load_node2b(nodes + l);
                const int off = __builtin_amdgcn_readlane(mv, l), so = off + (off >> 2);
                double2 ra[7];
                double rb[7];
                // (the comments keep the four patterns apart: merged into one, every
                // read would compute its address and lose its alignment)
                switch (off & 3) {
                case 0:
                    fetch7<0>(la + so, ra);
                    fetch7<0>(lb + so, rb);
                    asm volatile("; pattern 0");
                    break;
                case 1:
                    fetch7<1>(la + so, ra);
                    fetch7<1>(lb + so, rb);
                    asm volatile("; pattern 1");
                    break;
                case 2:
                    fetch7<2>(la + so, ra);
                    fetch7<2>(lb + so, rb);
                    asm volatile("; pattern 2");
                    break;
                default:
                    fetch7<3>(la + so, ra);
                    fetch7<3>(lb + so, rb);
                    asm volatile("; pattern 3");
                    break;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double t = fma(nd.w3, ra[k + 3].x,
                                         fma(nd.w0, ra[k].x, fma(nd.w2, ra[k + 2].x, nd.w1 * ra[k + 1].x)));
                    Y[k] = fma(H, t, Y[k]);
                    Z1[k] = fma(nd.w0, ra[k].y, Z1[k]);
                    Z1[k] = fma(nd.w1, ra[k + 1].y, Z1[k]);
                    Z1[k] = fma(nd.w2, ra[k + 2].y, Z1[k]);
                    Z1[k] = fma(nd.w3, ra[k + 3].y, Z1[k]);
                    double z = fma(nd.gu, t, Z2[k]);
                    z = fma(nd.w0, rb[k], z);
                    z = fma(nd.w1, rb[k + 1], z);
                    z = fma(nd.w2, rb[k + 2], z);
                    Z2[k] = fma(nd.w3, rb[k + 3], z);
                }
            }
            // corrections next to the ends of axis 1: x the sum of the weights, y
            // of the weights times gu
            auto correct = [&](const double2 (&c)[4], int i, int o) {  // end columns i (inner), o (outer)
                const double e0 = we[3 * i] - we[3 * o], e1 = we[3 * i + 1] - we[3 * o + 1],
                             e2 = we[3 * i + 2] - we[3 * o + 2];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (GUARD && c[k].x == 0.0) continue;
                    Y[k] = fma(-H * c[k].x, e0, Y[k]);
                    Z1[k] = fma(-c[k].x, e1, Z1[k]);
                    Z2[k] = fma(-c[k].y, e0, fma(-c[k].x, e2, Z2[k]));
                }
            };
            if (near_l || near_r) correct(kc, near_l ? 1 : 2, near_l ? 0 : 3);
            if (near_l && near_r) {
                double2 k2[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int d = n1 - 1 - (col + k);
                    const double2 v = *reinterpret_cast<const double2 *>(a.corr_r + (size_t)rowi * a.nr +
                                                                         min(max(d, 0), a.nr - 1));
                    k2[k] = d >= 0 && d < a.nr ? v : make_double2(0.0, 0.0);
                }
                correct(k2, 2, 3);
            }
            if (extra) {  // pass 2: the expectation of y
                wave_lds_fence();
#pragma unroll 1
                for (int e = lane; e - lane < W + kEdge2B; e += 256) {
                    double r[4][4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const unsigned o = (unsigned)staged(e + 64 * u) * 8u;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            r[u][k] = *reinterpret_cast<const double *>(reinterpret_cast<const char *>(q0) +
                                                                        k * (size_t)n1 * 8 + o);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int x = e + 64 * u;
                        const double y = combine(r[u]);
                        if (x < W)
                            wb[slot4(x)] = y;
                        else if (x < W + kEdge2B)
                            we[x - W] = y;
                    }
                }
                wave_lds_fence();
#pragma unroll 1
                for (int l = 0; l < a.L; ++l) {
                    const Node2B nd = load_node2b(nodes + l);
                    const int off = __builtin_amdgcn_readlane(mv, l), so = off + (off >> 2);
                    double rb[7];
                    fetch7(lb + so, off, rb);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const double t = fma(nd.w3, rb[k + 3],
                                             fma(nd.w0, rb[k], fma(nd.w2, rb[k + 2], nd.w1 * rb[k + 1])));
                        Y[k] = fma(ey, t, Y[k]);
                        Z2[k] = fma(nd.gy, t, Z2[k]);
                    }
                }
                // x the sum of the weights, z of the weights times gy
                auto correct_y = [&](const double4 *t, int n, bool left) {
                    const double e0 = left ? we[1] - we[0] : we[2] - we[3];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int c = left ? col + k : n1 - 1 - (col + k);
                        const double4 v = t[(size_t)rowi * n + min(max(c, 0), n - 1)];
                        const bool in = c >= 0 && c < n;
                        if (GUARD && (!in || v.x == 0.0)) continue;
                        Y[k] = fma(in ? -ey * v.x : 0.0, e0, Y[k]);
                        Z2[k] = fma(in ? -v.z : 0.0, e0, Z2[k]);
                    }
                };
                if (near_l) correct_y(a.corr_l, a.nl, true);
                if (near_r) correct_y(a.corr_r, a.nr, false);
            }
        }
    };
    rows(std::false_type());
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) sum += Y[k] + (Z1[k] + Z2[k]);
    if (__any(!isfinite(sum))) {
#pragma unroll
        for (int k = 0; k < 4; ++k) Y[k] = Z1[k] = Z2[k] = 0.0;
        rows(std::true_type());
    }
    // the groups' sums meet in LDS (each over its own window); thread t
    // finishes column t of the tile
    wave_lds_fence();
    double *part = reinterpret_cast<double *>(mine);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        part[lane * 4 + k] = Y[k];
        part[kTile2B + lane * 4 + k] = Z1[k];
        part[2 * kTile2B + lane * 4 + k] = Z2[k];
    }
    __syncthreads();
    double v[3];
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        double g[kGroups2B];
#pragma unroll
        for (int k = 0; k < kGroups2B; ++k)
            g[k] = reinterpret_cast<const double *>(reinterpret_cast<const char *>(smem2b) +
                                                    (size_t)k * a.lds_wave)[f * kTile2B + tid];
        v[f] = (g[0] + g[2]) + (g[1] + g[3]);
    }
    const double Yc = v[0] + a.lin_y, z1 = v[1] + a.lin_z1, z2 = v[2] + a.lin_z2;
    const int i1 = c0 + tid;
    const bool valid = i1 < n1;
    const size_t o = (size_t)i0 * n1 + min(i1, n1 - 1);
    double y = plane2<double>(a, (a.n + 1) % S, 0)[o];
    unsigned int it = 0;
    bool conv = true;
    y = picard2(a, y, Yc, z1, z2, it, conv);
    if (valid) {
        double *out = plane2<double>(a, a.n % S, 0);
        out[o] = y;
        out[o + a.plane] = z1;
        out[o + 2 * a.plane] = z2;
        if (a.n == a.n_stop) {
            const size_t np = (size_t)n0 * n1;
            a.fin[o] = y;
            a.fin[np + o] = z1;
            a.fin[2 * np + o] = z2;
        }
    }
    if (a.st_iter_max) {
        const unsigned int itm = wave_max_u32(valid ? it : 0u), its = wave_sum_u32(valid ? it : 0u);
        const unsigned int nc = wave_sum_u32(valid && !conv ? 1u : 0u);
        if (lane == 0) {
            const int w = idx * kGroups2B + grp;
            a.st_iter_max[w] = max(a.st_iter_max[w], itm);
            a.st_iter_sum[w] += its;
            a.st_nonconv[w] += nc;
        }
    }
}

// Coefficients of a layer: the values filtered along axis 0 into the tmp
// planes, these along axis 1 into the coefficient planes.  A thread computes
// kRunCols (axis 0) or kRun consecutive outputs of one line and streams its inputs once, as
// spline2d_cols; the taps give v - dx^2/6 M directly, and both end values of a
// line are their own coefficients (M = 0 there).
namespace {
// lines shorter than the filter's one-reflection reach: point by point
__device__ inline double coef_line(const double *v, long stride, int n, int i)
{
    constexpr SplineTaps T = spline_taps();
    const double x = v[(long)i * stride];
    if (i == 0 || i == n - 1) return x;
    double acc = 0.0;
    for (int k = 0; k < kPcrTaps; ++k) acc = fma(T.c[k], rt_line(v, stride, n, i + k - 31), acc);
    return fma(-T.inv_b, acc, x);
}
}  // namespace

__global__ void __launch_bounds__(256) coef2d_cols(const Sweep2Args a, int slot)
{
    constexpr SplineTaps T = spline_taps();
    constexpr int H = kPcrTaps / 2 + 1;
    const long t = blockIdx.x * 256L + threadIdx.x;
    const int n = a.n0, st = a.n1;
    if (t >= (long)st * ((n + kRunCols - 1) / kRunCols)) return;
    const int i1 = (int)(t % st), j0 = (int)(t / st) * kRunCols;
    const double *v = plane2<double>(a, slot, blockIdx.y) + i1;
    double *out = a.tmp + (size_t)blockIdx.y * a.plane + i1;
    if (n < kMinLine) {
        for (int i = j0; i < min(j0 + kRunCols, n); ++i) out[(long)i * st] = coef_line(v, st, n, i);
        return;
    }
    double acc[kRunCols];
#pragma unroll
    for (int r = 0; r < kRunCols; ++r) acc[r] = 0.0;
    const double v0 = v[0], vn = v[(long)(n - 1) * st];
    if (j0 >= H && j0 + kRunCols - 1 + H <= n - 1) {  // clear of both ends
        const double *p = v + (long)(j0 - H) * st;
#pragma unroll
        for (int m = 0; m < kRunCols + 2 * H; ++m) {
            const double x = p[(long)m * st];
#pragma unroll
            for (int r = 0; r < kRunCols; ++r)
                if (m - r >= 0 && m - r <= 2 * H) acc[r] = fma(T.e[m - r], x, acc[r]);
        }
    } else {
#pragma unroll
        for (int m = 0; m < kRunCols + 2 * H; ++m) {
            const int k = j0 - H + m;
            const int kk = min(max(k < 0 ? -k : (k > n - 1 ? 2 * (n - 1) - k : k), 0), n - 1);
            const double y = v[(long)kk * st];
            const double x = k < 0 ? 2.0 * v0 - y : (k > n - 1 ? 2.0 * vn - y : y);
#pragma unroll
            for (int r = 0; r < kRunCols; ++r)
                if (m - r >= 0 && m - r <= 2 * H) acc[r] = fma(T.e[m - r], x, acc[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < kRunCols; ++r) {
        const int i = j0 + r;
        if (i < n) out[(long)i * st] = i == 0 ? v0 : i == n - 1 ? vn : acc[r];
    }
}

__global__ void __launch_bounds__(256) coef2d_rows(const Sweep2Args a, int slot)
{
    constexpr SplineTaps T = spline_taps();
    constexpr int H = kPcrTaps / 2 + 1;
    __shared__ double sm[kRowTile * kRowStride];
    const int n = a.n1, tiles1 = (n + kRowCols - 1) / kRowCols;
    const int r0 = (int)(blockIdx.x / tiles1) * kRowTile, c0 = (int)(blockIdx.x % tiles1) * kRowCols;
    const double *src = a.tmp + (size_t)blockIdx.y * a.plane;
    double *dst = plane2<double>(a, slot, 3 + blockIdx.y);
    const bool short_line = n < kMinLine;
    if (!short_line) {
        for (int e = threadIdx.x; e < kRowTile * kRowIn; e += 256) {
            const int rr = e / kRowIn, cc = e - rr * kRowIn;
            const int i0 = r0 + rr;
            if (i0 >= a.n0) continue;
            const double *v = src + (size_t)i0 * n;
            const int k = c0 - H + cc;
            const int kk = min(max(k < 0 ? -k : (k > n - 1 ? 2 * (n - 1) - k : k), 0), n - 1);
            const double y = v[kk];
            sm[rr * kRowStride + cc] = k < 0 ? 2.0 * v[0] - y : (k > n - 1 ? 2.0 * v[n - 1] - y : y);
        }
    }
    __syncthreads();
    const int r = threadIdx.x % kRowTile, q = threadIdx.x / kRowTile;
    const int i0 = r0 + r, j0 = c0 + q * kRun;
    double acc[kRun];
    if (!short_line) {
        const double *w = sm + r * kRowStride + q * kRun;
#pragma unroll
        for (int u = 0; u < kRun; ++u) acc[u] = 0.0;
#pragma unroll
        for (int m = 0; m < kRun + 2 * H; ++m) {
            const double x = w[m];
#pragma unroll
            for (int u = 0; u < kRun; ++u)
                if (m - u >= 0 && m - u <= 2 * H) acc[u] = fma(T.e[m - u], x, acc[u]);
        }
#pragma unroll
        for (int u = 0; u < kRun; ++u)
            if (j0 + u == 0 || j0 + u == n - 1) acc[u] = w[u + H];
    } else {
        const double *v = src + (size_t)min(i0, a.n0 - 1) * n;
#pragma unroll
        for (int u = 0; u < kRun; ++u) acc[u] = j0 + u < n ? coef_line(v, 1, n, j0 + u) : 0.0;
    }
    // outputs through LDS, so that the stores are whole lines
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kRun; ++u) sm[r * kRowStride + q * kRun + u] = acc[u];
    __syncthreads();
    for (int e = threadIdx.x; e < kRowTile * kRowCols; e += 256) {
        const int rr = e / kRowCols, cc = e - rr * kRowCols;
        if (r0 + rr < a.n0 && c0 + cc < n) dst[(size_t)(r0 + rr) * n + c0 + cc] = sm[rr * kRowStride + cc];
    }
}

hipError_t set_sweep2b_lds_limit(size_t bytes)
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&sweep2b),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_sweep2b(const Sweep2Args &a, hipStream_t s)
{
    const int tiles = a.n0 * ((a.n1 + kTile2B - 1) / kTile2B);
    hipLaunchKernelGGL(sweep2b, dim3(tiles), dim3(64 * kGroups2B), (size_t)kGroups2B * a.lds_wave, s, a);
    return hipGetLastError();
}

hipError_t launch_coef2d(const Sweep2Args &a, int slot, hipStream_t s)
{
    const long tc = (long)a.n1 * ((a.n0 + kRunCols - 1) / kRunCols);
    hipLaunchKernelGGL(coef2d_cols, dim3((unsigned)((tc + 255) / 256), 3), dim3(256), 0, s, a, slot);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long tiles = (long)((a.n0 + kRowTile - 1) / kRowTile) * ((a.n1 + kRowCols - 1) / kRowCols);
    hipLaunchKernelGGL(coef2d_rows, dim3((unsigned)tiles, 3), dim3(256), 0, s, a, slot);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
size_t sweep2d_lds(int half) { return (size_t)3 * kTile2R * 2 * half * sizeof(double2); }

// Checkpoint export: layers n_stop .. n_stop + K - 1 into the initial-layer
// layout (y: K x n0 n1; z: K x 2 x n0 n1), the FP32 form as value plus residual.
template <typename E>
__global__ void __launch_bounds__(256) export2d(const Sweep2Args a, double *__restrict__ ly,
                                                double *__restrict__ lz)
{
    const long np = (long)a.n0 * a.n1;
    const long i = blockIdx.x * 256L + threadIdx.x;
    const int r = blockIdx.y;
    if (i >= np) return;
    const int slot = (a.n_stop + r) % (a.K + 1);
    const E *base = plane2<E>(a, slot, 0);
    const size_t o = pidx(a, (int)(i / a.n1), (int)(i % a.n1));
    double v[3];
    for (int f = 0; f < 3; ++f) {
        v[f] = base[(size_t)(a.vstep * f) * a.plane + o];
        if constexpr (std::is_same<E, float>::value) v[f] += (double)base[(size_t)(12 + f) * a.plane + o];
    }
    ly[r * np + i] = v[0];
    lz[(2L * r) * np + i] = v[1];
    lz[(2L * r + 1) * np + i] = v[2];
}

namespace {

template <typename E>
hipError_t launch_sweep2d_t(const Sweep2Args &a, hipStream_t s)
{
    const int tiles = ((a.n0 + kTile2R - 1) / kTile2R) * ((a.n1 + kTile2C - 1) / kTile2C);
    // The staging runs a row ahead where all blocks are on the chip at once with
    // the registers that takes (213 of the FP32 planes' loads: two blocks a CU;
    // 256 of the FP64 planes': one).  See sweep2d_ahead for both sides.
    constexpr int kAheadTiles = std::is_same<E, float>::value ? 512 : 256;
    if (tiles <= kAheadTiles) {
        hipLaunchKernelGGL(sweep2d_ahead<E>, dim3(tiles), dim3(kThreads2), 2 * sweep2d_lds(a.half), s, a);
    } else {
        hipLaunchKernelGGL(sweep2d<E>, dim3(tiles), dim3(kThreads2), sweep2d_lds(a.half), s, a);
    }
    return hipGetLastError();
}

template <typename E>
hipError_t launch_ghosts2d_t(const Sweep2Args &a, int slot, hipStream_t s)
{
    const int npad0 = (int)(a.plane / a.npad1);
    const int gb = (int)(((long)npad0 * a.npad1 + 255) / 256);
    hipLaunchKernelGGL(ghosts2d<E>, dim3(gb), dim3(256), 0, s, a, slot, npad0);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_spline2d(const Sweep2Args &a, int slot, const SplineFilter &f, hipStream_t s)
{
    const long tc = (long)a.n1 * ((a.n0 + kRunCols - 1) / kRunCols);
    hipLaunchKernelGGL(spline2d_cols<kRunCols>, dim3((unsigned)((tc + 255) / 256), 3), dim3(256), 0, s, a,
                       slot, f);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.n1 >= kMinLine) {
        const long tiles = (long)((a.n0 + kRowTile - 1) / kRowTile) * ((a.n1 + kRowCols - 1) / kRowCols);
        hipLaunchKernelGGL(spline2d_rows_lds, dim3((unsigned)tiles, 6), dim3(256), 0, s, a, slot,
                           f);
    } else {
        const long tr = (long)a.n0 * ((a.n1 + kRun - 1) / kRun);
        hipLaunchKernelGGL(spline2d_rows, dim3((unsigned)((tr + 255) / 256), 6), dim3(256), 0, s,
                           a, slot, f);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_ghosts2d_t<float>(a, slot, s);
}

namespace {

template <typename E>
hipError_t launch_fd2d_t(const Sweep2Args &a, int slot, double dx0, double dx1, hipStream_t s)
{
    const long np = (long)a.n0 * a.n1;
    const unsigned nb = (unsigned)((np + 255) / 256);
    hipLaunchKernelGGL(fd2d_cols<E>, dim3(nb, 3), dim3(256), 0, s, a, slot, 1.0 / (12.0 * dx0));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fd2d_rows<E>, dim3(nb, 6), dim3(256), 0, s, a, slot, 1.0 / (12.0 * dx1));
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_ghosts2d_t<E>(a, slot, s);
}

template <typename E>
hipError_t launch_scatter2d_t(const Sweep2Args &a, const double *iy, const double *iz,
                              hipStream_t s)
{
    const long np = (long)a.n0 * a.n1;
    hipLaunchKernelGGL(scatter2d<E>, dim3((unsigned)((np + 255) / 256), a.K), dim3(256), 0, s, a,
                       iy, iz);
    return hipGetLastError();
}

}  // namespace

hipError_t set_sweep2d_lds_limit(bool f32, size_t bytes)
{
    return hipFuncSetAttribute(f32 ? reinterpret_cast<const void *>(&sweep2d_ahead<float>)
                                   : reinterpret_cast<const void *>(&sweep2d_ahead<double>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_sweep2d(bool f32, const Sweep2Args &a, hipStream_t s)
{
    return f32 ? launch_sweep2d_t<float>(a, s) : launch_sweep2d_t<double>(a, s);
}

hipError_t launch_fd2d(bool f32, const Sweep2Args &a, int slot, double dx0, double dx1,
                       hipStream_t s)
{
    return f32 ? launch_fd2d_t<float>(a, slot, dx0, dx1, s)
               : launch_fd2d_t<double>(a, slot, dx0, dx1, s);
}

hipError_t launch_export2d(bool f32, const Sweep2Args &a, double *ly, double *lz, hipStream_t s)
{
    const long np = (long)a.n0 * a.n1;
    const dim3 grid((unsigned)((np + 255) / 256), (unsigned)a.K);
    if (f32)
        hipLaunchKernelGGL(export2d<float>, grid, dim3(256), 0, s, a, ly, lz);
    else
        hipLaunchKernelGGL(export2d<double>, grid, dim3(256), 0, s, a, ly, lz);
    return hipGetLastError();
}

hipError_t launch_scatter2d(bool f32, const Sweep2Args &a, const double *iy, const double *iz,
                            hipStream_t s)
{
    return f32 ? launch_scatter2d_t<float>(a, iy, iz, s) : launch_scatter2d_t<double>(a, iy, iz, s);
}

hipError_t launch_gather2d(const Sweep2Args &a, double *y0, double *z0,
                           unsigned long long *nonfinite, hipStream_t s)
{
    const long np = (long)a.n0 * a.n1;
    const int blocks = (int)std::min<long>(2048, (np + 255) / 256);
    hipLaunchKernelGGL(gather2d, dim3(blocks), dim3(256), 0, s, a, y0, z0, nonfinite);
    return hipGetLastError();
}

}  // namespace bsde
