// fused.h -- the fused sweep of the one-dimensional scheme: one launch per
// time step with the windows of all K layers in LDS (arXiv:1909.13560,
// Section 2.2 eq (20)-(21), Section 3.1 step 3, Section 3.2).
//
// A block owns a tile of 64 P WP consecutive grid points (P consecutive
// points per lane, WP wavefronts along the points) and has G groups of WP
// wavefronts that share the nodes.  It stages every layer's window (the
// records its nodes touch: the tile widened by the layer's node offsets) in
// LDS with all loads in flight at once: layer n+1's values come first, and both
// passes of its spline run on them, with a barrier after each, before the other
// layers' records are written to LDS.  The node loops of all K layers follow;
// then the groups' sums are added in a fixed order and the implicit y equation is
// solved, one point per thread.
//
// FP64 form: the spline is kept by its cubic B-spline coefficients
//   c_i = v_i - dx^2/6 M_i   (v = sum_k b_k(phi) c_{p-1+k}, k = 0..3),
// one (c_y, c_z) pair per grid point.  Against the value/second-derivative
// form (M) this halves the bytes of a window record (16 instead of 32 B) in
// HBM and LDS, and P consecutive points share P + 3 records of 16 B per node
// instead of P + 1 of 32 B: 28 B per node and point at P = 4 against 64 B at
// P = 1 in the M form, whose LDS reads took as long as its arithmetic.
// Outside the grid the interpolant is the boundary value (Section 3.2), which
// no B-spline coefficients reproduce next to the end (the slope jumps), so a
// node whose cells leave the grid at some point of the wavefront selects the
// boundary value point by point; the test is wave-uniform.
// FP32 form: records (y, z, M_y, M_z) in single precision, as its arithmetic
// keeps the exact record values apart (node_accumulate).
#pragma once

#include "device_common.h"

namespace bsde {

// Tile shape: WP wavefronts of P points per lane, G node groups.
template <int P, int WP, int G>
struct FusedShape {
    static constexpr int T = 64 * P * WP;
    static constexpr int NT = 64 * WP * G;
    static_assert(NT <= 1024, "block size");
};

// ---------------------------------------------------------------------------
// Natural spline of a window as a filter of the values.  The five rounds of
// the truncated parallel cyclic reduction act as a 17-tap stencil (rounds
// 1-3, second difference folded in) followed by a 7-tap stencil at stride 8
// (rounds 4-5).  Beyond the domain ends the values are continued by
// reflection through the end points, v(-k) = 2 v(0) - v(k) and likewise at
// N - 1, whose second differences are the odd extension that the natural end
// conditions call for, so the same filter holds at every record.
// ---------------------------------------------------------------------------
// Grid point whose value the reflected continuation at k uses, and the
// continuation from that value and the end values v0, v1.
__device__ inline int reflected_index(int nx, int k)
{
    if (k < 0) k = -k;
    if (k < nx) return k;  // one reflection at the left end, or none
    const int per = 2 * (nx - 1), b = k % per;
    return b > nx - 1 ? per - b : b;
}
__device__ inline double2 reflected_value(int nx, int k, const double2 &v, const double2 &v0,
                                          const double2 &v1)
{
    if (k >= 0 && k < nx) return v;
    int q = 0, b = k;
    if (k < -(nx - 1) || k > 2 * (nx - 1)) {  // further than one line length: whole periods first
        const int per = 2 * (nx - 1);
        q = k / per;
        b = k - q * per;
        if (b < 0) {
            b += per;
            --q;
        }
    }
    const double t = 2.0 * q;
    double2 r = v;
    if (b < 0) r = make_double2(2.0 * v0.x - v.x, 2.0 * v0.y - v.y);
    if (b > nx - 1) r = make_double2(2.0 * v1.x - v.x, 2.0 * v1.y - v.y);
    if (q != 0) r = make_double2(r.x + t * (v1.x - v0.x), r.y + t * (v1.y - v0.y));
    return r;
}
template <typename Slot>
__device__ inline double2 layer_value(const Slot &g, int k)
{
    const auto v = g.val(k);
    return make_double2(v.x, v.y);
}

// Outputs 0 .. W-1 of the filter belong to the records g0 .. g0 + W - 1.
// D[e] holds (y, z) of record g0 - kHalo - 1 + e, e < W + 2 kHalo + 2; A[e]
// the first pass at record g0 - 24 + e, e < W + 48.  Both arrays have room
// past that (kFirOver) for outputs that nothing reads.
// Pass A: kA consecutive outputs per thread, which share their reads; kA = 1
// where the block has a thread per output (the shortest chain of reads).
template <int NT, int kA>
__device__ inline void fir_pass_a(int W, const double2 *D, double2 *A)
{
    constexpr PcrFilters F = coef_filters();
    for (int t = threadIdx.x; kA * t < W + 48; t += NT) {
        const int e = kA * t;
        double vy[kA], vz[kA];
#pragma unroll
        for (int o = 0; o < kA; ++o) vy[o] = vz[o] = 0.0;
#pragma unroll
        for (int i = 0; i < kA + 16; ++i) {
            // bound the reads the scheduler hoists: all nineteen at once would
            // raise the register count of the whole kernel
            if (kA > 1 && i % 8 == 0) __builtin_amdgcn_sched_barrier(0);
            const double2 x = D[e + 1 + i];
#pragma unroll
            for (int o = 0; o < kA; ++o) {
                const int q = i - 8 - o;
                if (q >= -8 && q <= 8) {
                    const double w = F.fa[q < 0 ? -q : q];
                    vy[o] = fma(w, x.x, vy[o]);
                    vz[o] = fma(w, x.y, vz[o]);
                }
            }
        }
#pragma unroll
        for (int o = 0; o < kA; ++o) A[e + o] = make_double2(vy[o], vz[o]);
    }
}

// Pass B: kB outputs eight apart per thread; out(e, wy, wz) receives output
// e < W, with M = 6/dx^2 inv_b w (and c = v - inv_b w).
template <int NT, int kB, typename Out>
__device__ inline void fir_pass_b(int W, const double2 *A, Out out)
{
    constexpr PcrFilters F = coef_filters();
    for (int t = threadIdx.x;; t += NT) {
        const int e = (t & 7) + 8 * kB * (t >> 3);  // outputs e, e + 8, ...
        if (e >= W) break;
        double wy[kB], wz[kB];
#pragma unroll
        for (int o = 0; o < kB; ++o) wy[o] = wz[o] = 0.0;
#pragma unroll
        for (int i = 0; i < 6 + kB; ++i) {
            const double2 x = A[e + 8 * i];
#pragma unroll
            for (int o = 0; o < kB; ++o) {
                const int q = i - 3 - o;
                if (q >= -3 && q <= 3) {
                    const double w = F.fb[q < 0 ? -q : q];
                    wy[o] = fma(w, x.x, wy[o]);
                    wz[o] = fma(w, x.y, wz[o]);
                }
            }
        }
#pragma unroll
        for (int o = 0; o < kB; ++o)
            if (e + 8 * o < W) out(e + 8 * o, wy[o], wz[o]);
    }
}

// The FP32 form's passes: the same dependence as fir_pass_a / fir_pass_b, but
// every reduction round with the rounding it has on its own (intermediate
// values are recomputed, not stored).  A derivative that differs in its last
// bit can round to another single-precision value, and the rounding of the
// stored layers amplifies one such bit to the form's own error level, so the
// form keeps one sequence of operations.
__device__ inline double pcr_round(double kap, double lo, double mid, double hi)
{
#pragma clang fp contract(off)
    const double t = lo + hi;
    return fma(-kap, t, mid);
}

template <int NT>
__device__ inline void pcr_pass_a(int W, const double2 *D, double2 *A, const PcrCoef &c)
{
#pragma clang fp contract(off)
    for (int e = threadIdx.x; e < W + 48; e += NT) {
        double2 r[15], x1[7], x2[3];  // right-hand sides, rounds 1 and 2 around the output
#pragma unroll
        for (int i = 0; i < 15; ++i) {
            const double2 m = D[e + 1 + i], v = D[e + 2 + i], p = D[e + 3 + i];
            r[i] = make_double2(c.s6 * ((p.x - v.x) - (v.x - m.x)), c.s6 * ((p.y - v.y) - (v.y - m.y)));
        }
#pragma unroll
        for (int i = 0; i < 7; ++i)
            x1[i] = make_double2(pcr_round(c.kappa[0], r[2 * i].x, r[2 * i + 1].x, r[2 * i + 2].x),
                                 pcr_round(c.kappa[0], r[2 * i].y, r[2 * i + 1].y, r[2 * i + 2].y));
#pragma unroll
        for (int i = 0; i < 3; ++i)
            x2[i] = make_double2(pcr_round(c.kappa[1], x1[2 * i].x, x1[2 * i + 1].x, x1[2 * i + 2].x),
                                 pcr_round(c.kappa[1], x1[2 * i].y, x1[2 * i + 1].y, x1[2 * i + 2].y));
        A[e] = make_double2(pcr_round(c.kappa[2], x2[0].x, x2[1].x, x2[2].x),
                            pcr_round(c.kappa[2], x2[0].y, x2[1].y, x2[2].y));
    }
}

template <int NT, typename Out>
__device__ inline void pcr_pass_b(int W, const double2 *A, const PcrCoef &c, Out out)
{
#pragma clang fp contract(off)
    for (int e = threadIdx.x; e < W; e += NT) {
        double2 x[7], x4[3];
#pragma unroll
        for (int i = 0; i < 7; ++i) x[i] = A[e + 8 * i];
#pragma unroll
        for (int i = 0; i < 3; ++i)
            x4[i] = make_double2(pcr_round(c.kappa[3], x[2 * i].x, x[2 * i + 1].x, x[2 * i + 2].x),
                                 pcr_round(c.kappa[3], x[2 * i].y, x[2 * i + 1].y, x[2 * i + 2].y));
        out(e, pcr_round(c.kappa[4], x4[0].x, x4[1].x, x4[2].x) * c.inv_b,
            pcr_round(c.kappa[4], x4[0].y, x4[1].y, x4[2].y) * c.inv_b);
    }
}

// Bring [p, p + bytes) into the scalar cache, one 64-byte line in `stride`
// from line `line` on: the lines are touched together here, while the window
// loads are in flight, instead of one miss after the other where they are used.
__device__ inline void warm_scalar(const void *p, int bytes, int line, int stride)
{
    const char *q = static_cast<const char *>(p);
    const int last = (bytes - 1) & ~63;
#pragma unroll 1
    for (int o = line * 64; o < bytes; o += 8 * stride * 64) {
        unsigned x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            x[k] = const_load(reinterpret_cast<const unsigned *>(q + min(o + k * stride * 64, last)));
        asm volatile("" ::"s"(x[0]), "s"(x[1]), "s"(x[2]), "s"(x[3]), "s"(x[4]), "s"(x[5]), "s"(x[6]),
                     "s"(x[7]));
    }
}

// Descriptor values that a phase reads for itself, through the constant
// address space (scalar loads).  The pointer is made opaque first: values
// loaded earlier and kept over the node loops would take the scalar registers
// that the nodes' coefficients need.
__device__ inline const InstDesc *own_copy(const InstDesc *d)
{
    asm volatile("" : "+s"(d));
    return d;
}
template <int DRV>
__device__ inline SweepArgs driver_args(const InstDesc *d)
{
    SweepArgs a{};
    a.drv.p0 = const_load(&d->a.drv.p0);
    a.drv.p1 = const_load(&d->a.drv.p1);
    a.drv.p2 = const_load(&d->a.drv.p2);
    a.drv.p3 = const_load(&d->a.drv.p3);
    a.drv.p4 = const_load(&d->a.drv.p4);
    a.drv.inv3 = const_load(&d->a.drv.inv3);
    return a;
}

// ---------------------------------------------------------------------------
// Records of a window: element e of layer j at slot WinLayout<P>::slot(e).
// The lane's q-th record of a node is element lane_pt + off + q.
// ---------------------------------------------------------------------------
template <int P, int B, int NR, typename V>
__device__ inline void fetch_pattern(const V *p, V (&r)[NR])
{
#pragma unroll
    for (int q = 0; q < NR; ++q) r[q] = p[q + (WinLayout<P>::kPad ? (B + q) / P : 0)];
}

// p: the lane's record at the node's offset; res: that offset modulo P
template <int P, int NR, typename V>
__device__ inline void fetch_records(const V *p, int res, V (&r)[NR])
{
    if constexpr (!WinLayout<P>::kPad) {
        fetch_pattern<P, 0, NR>(p, r);
    } else if constexpr (P == 2) {
        // (the comments keep the patterns apart: merged into one, every read
        // would compute its address and lose its alignment)
        if (res & 1) {
            fetch_pattern<P, 1, NR>(p, r);
            asm volatile("; pattern 1");
        } else {
            fetch_pattern<P, 0, NR>(p, r);
            asm volatile("; pattern 0");
        }
    } else {
        switch (res & 3) {
        case 0: fetch_pattern<P, 0, NR>(p, r); asm volatile("; pattern 0"); break;
        case 1: fetch_pattern<P, 1, NR>(p, r); asm volatile("; pattern 1"); break;
        case 2: fetch_pattern<P, 2, NR>(p, r); asm volatile("; pattern 2"); break;
        default: fetch_pattern<P, 3, NR>(p, r); asm volatile("; pattern 3"); break;
        }
    }
}

// The driver at time t; c: (t, exp(t^2), exp(-t^2)) where the driver needs them.
template <int DRV, typename T>
__device__ inline Driver<DRV, T> make_driver(const SweepArgs &a, const double *c)
{
    if constexpr (DRV == BSDE_DRIVER_EXP)
        return Driver<DRV, T>(c);
    else
        return Driver<DRV, T>(a.drv, 0.0);
}

// FP32 form: source of layer_nodes.
template <int P>
struct LdsWindow {
    const float4 *lane;  // the lane's first record at the layer's lowest node offset
    int wlo;             // that offset
    template <int PP>
    __device__ void fetch(int m, float4 (&r)[1][PP + 1]) const
    {
        static_assert(PP == P, "window layout and fetch width differ");
        const int off = m - wlo;
        fetch_records<P, P + 1>(lane + off + (WinLayout<P>::kPad ? off / P : 0), off, r[0]);
    }
};

// The list of class c (nodes l = c mod 8 of all layers) in the tables, and the
// address that a lane holds for it (an empty list may start at the table's end:
// one entry more is allocated).
static_assert(kMaxOrder * 8 <= 64, "a class's node addresses fit the lanes of a wavefront");
__device__ inline void class_list(int K, int L, int c, int &start, int &cnt)
{
    start = K * (c * (L >> 3) + min(c, L & 7));
    cnt = K * ((L >> 3) + (c < (L & 7) ? 1 : 0));
}
__device__ inline int2 class_address(const int2 *addr, int start, int cnt, int lane)
{
    return addr[start + max(min(lane, cnt - 1), 0)];
}

// The nodes of one class (FP64 form): cnt consecutive table entries, whose
// addresses av (FusedHot::addr) the wavefront holds one per lane.  The loop
// carries little besides the arithmetic: on small grids a SIMD has two
// wavefronts, each of which issues one instruction of any kind in four clocks,
// so a loop that prefetched its coefficients a stage ahead (twice the scalar
// instructions) was slower than waiting for them.  Cells outside the grid: a
// bit per node says whether the node leaves the grid at some point of the
// wavefront; such a node selects the boundary values between the
// interpolation and the driver.  A second copy of the loop for the few
// wavefronts at the ends took twice the time per node there (code that no
// other block keeps in the instruction cache), and a launch ends with its
// slowest block.
template <int P, int DRV>
__device__ inline void class_nodes(const char *lane, const double2 *edge, const NodeRecB *recs, int cnt,
                                   const int2 &av, const SweepArgs &a, const double *drv, int first,
                                   int wfirst, int wlast, int nx, double (&Y)[P], double (&Z)[P])
// lane: the lane's record in LDS at offset 0; first: its first grid point;
// wfirst, wlast: the wavefront's first and last one
{
    const Driver<DRV, double> f = make_driver<DRV, double>(a, drv);
    const int mv = av.y >> 4;
    const unsigned long long crossing = __ballot(wfirst + mv < 0 || wlast + mv > nx - 2);
    auto fetch = [&](int k, double2 (&r)[P + 3]) {
        const int x = __builtin_amdgcn_readlane(av.x, k);
        fetch_records<P, P + 3>(reinterpret_cast<const double2 *>(lane + (x & ~15)), x, r);
    };
    auto node = [&](int k, const double2 (&r)[P + 3], const NodeRecB &c) {
        double yh[P], zh[P];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            yh[i] = fma(c.b3, r[i + 3].x, fma(c.b0, r[i].x, fma(c.b2, r[i + 2].x, c.b1 * r[i + 1].x)));
            zh[i] = fma(c.b3, r[i + 3].y, fma(c.b0, r[i].y, fma(c.b2, r[i + 2].y, c.b1 * r[i + 1].y)));
        }
        if ((crossing >> k) & 1) {
            const int y = __builtin_amdgcn_readlane(av.y, k), p0 = first + (y >> 4);
            const double2 *e = edge + 2 * ((y & 15) - 1);
            const double2 v0 = e[0], v1 = e[1];
#pragma unroll
            for (int i = 0; i < P; ++i) {
                yh[i] = p0 + i < 0 ? v0.x : p0 + i > nx - 2 ? v1.x : yh[i];
                zh[i] = p0 + i < 0 ? v0.y : p0 + i > nx - 2 ? v1.y : zh[i];
            }
        }
        const Driver<DRV, double> fj =
            DRV == BSDE_DRIVER_EXP
                ? make_driver<DRV, double>(a, drv + 3 * (__builtin_amdgcn_readlane(av.y, k) & 15))
                : f;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if constexpr (DRV == BSDE_DRIVER_LINEAR) {
                // the driver's coefficients are folded into the node weights (its
                // constant term into the descriptor's lin_y, lin_z)
                Y[i] = fma(c.w0, yh[i], fma(c.w1, zh[i], Y[i]));
                Z[i] = fma(c.w2, yh[i], fma(c.w3, zh[i], Z[i]));
            } else {
                // w3 is zero but for the layer K_y (a test costs more than the product)
                const double fh = fj(yh[i], zh[i]);
                Y[i] = fma(c.w0, fh, fma(c.w3, yh[i], Y[i]));
                Z[i] = fma(c.w1, fh, fma(c.w2, zh[i], Z[i]));
            }
        }
    };
    int k = 0;
#pragma unroll 1
    for (; k + 1 < cnt; k += 2) {
        const NodeRecB ca = load_node(recs + k), cb = load_node(recs + k + 1);
        double2 ra[P + 3], rb[P + 3];
        fetch(k, ra);
        if (P < 4) fetch(k + 1, rb);
        node(k, ra, ca);
        if (P == 4) {
            // four points per lane: one node's records in flight at a time
            // (28 registers each), so that the kernel keeps four wavefronts
            // per SIMD, which cover each other's waits
            __builtin_amdgcn_sched_barrier(0);
            fetch(k + 1, rb);
        }
        node(k + 1, rb, cb);
    }
    if (k < cnt) {
        const NodeRecB ca = load_node(recs + k);
        double2 ra[P + 3];
        fetch(k, ra);
        node(k, ra, ca);
    }
}

// The nodes of one class for state-dependent coefficients (one point per
// lane): the node of (j, l) sits s = i + (a(x_i) j dt + b(x_i) dW_l) / dx cells
// along the grid, so each lane locates its cell, forms the B-spline weights at
// its fraction and reads its four records.  Clamping s to the grid gives the
// boundary value beyond the ends: the natural spline ends at its end values.
// ENDS: such a node takes the boundary value itself (edge).  A wavefront whose
// sums are not finite runs the loop once more so: a non-finite record next to
// an end does not cancel in the boundary value.  (A selection or a branch in
// every node cost 4 to 12% on 2001 points, the check of the sums 1%.)
// recs: b0 = dW / dx, b1 = j dt / dx; av: LDS address of the record of grid
// point t0, layer; base: the block's LDS.
template <int DRV, bool ENDS>
__device__ inline void gather_nodes(const char *base, const double2 *edge, const NodeRecB *recs, int cnt,
                                    const int2 &av, const SweepArgs &a, const double *drv, double pos,
                                    double ax, double bx, int t0, int nx, double &Y, double &Z)
{
    const Driver<DRV, double> f = make_driver<DRV, double>(a, drv);
    const double top = nx - 1.0;
    auto fetch = [&](int k, const NodeRecB &c, double2 (&r)[4], double &ph, double &s) {
        s = fmin(fmax(fma(bx, c.b0, fma(ax, c.b1, pos)), 0.0), top);
        const int p = min((int)s, nx - 2);
        ph = s - p;
        const double2 *q =
            reinterpret_cast<const double2 *>(base + __builtin_amdgcn_readlane(av.x, k) + 16 * (p - 1 - t0));
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = q[i];
    };
    auto node = [&](int k, const NodeRecB &c, const double2 (&r)[4], double ph, double s) {
        const double u = 1.0 - ph, p2 = ph * ph, u2 = u * u;
        const double b0 = u2 * u * (1.0 / 6.0), b3 = p2 * ph * (1.0 / 6.0);
        const double b2 = fma(-0.5 * u2, 1.0 + ph, 2.0 / 3.0), b1 = (1.0 - b2) - (b0 + b3);  // (they sum to one)
        double yh = fma(b3, r[3].x, fma(b0, r[0].x, fma(b2, r[2].x, b1 * r[1].x)));
        double zh = fma(b3, r[3].y, fma(b0, r[0].y, fma(b2, r[2].y, b1 * r[1].y)));
        if constexpr (ENDS) {
            const double2 *e = edge + 2 * (__builtin_amdgcn_readlane(av.y, k) - 1);
            const double2 v0 = e[0], v1 = e[1];
            yh = s == 0.0 ? v0.x : s == top ? v1.x : yh;
            zh = s == 0.0 ? v0.y : s == top ? v1.y : zh;
        }
        if constexpr (DRV == BSDE_DRIVER_LINEAR) {
            Y = fma(c.w0, yh, fma(c.w1, zh, Y));
            Z = fma(c.w2, yh, fma(c.w3, zh, Z));
        } else {
            const Driver<DRV, double> fj =
                DRV == BSDE_DRIVER_EXP
                    ? make_driver<DRV, double>(a, drv + 3 * (__builtin_amdgcn_readlane(av.y, k) & 15))
                    : f;
            const double fh = fj(yh, zh);
            Y = fma(c.w0, fh, fma(c.w3, yh, Y));
            Z = fma(c.w1, fh, fma(c.w2, zh, Z));
        }
    };
    int k = 0;
#pragma unroll 1
    for (; k + 1 < cnt; k += 2) {
        const NodeRecB ca = load_node(recs + k), cb = load_node(recs + k + 1);
        double2 ra[4], rb[4];
        double pa, pb;
        double sa, sb;
        fetch(k, ca, ra, pa, sa);
        fetch(k + 1, cb, rb, pb, sb);
        node(k, ca, ra, pa, sa);
        node(k + 1, cb, rb, pb, sb);
    }
    if (k < cnt) {
        const NodeRecB ca = load_node(recs + k);
        double2 ra[4];
        double pa;
        double sa;
        fetch(k, ca, ra, pa, sa);
        node(k, ca, ra, pa, sa);
    }
}

// ---------------------------------------------------------------------------
// The sweep kernel.  Sums: the FP64 form adds the nodes of class l mod 8 over
// the layers K, ..., 2, 1 in each of eight classes; the classes k and k + 4,
// then k and k + 2, then k and k + 1 are added, in registers within a group
// and in LDS across groups, so every shape gives the same bits (a batch equals
// its instances solved alone).  A class has at most 48 nodes, so a wavefront
// holds the addresses of its list one per lane.  The FP32
// form adds all nodes in one sequence per point (its results depend on the
// order at the level of its own rounding), hence one group; more groups, on
// request, take whole layers.
// Dynamic LDS (byte offsets in the descriptor): the windows of the K layers,
// later the partial sums; D and A of the spline filter; boundary values; the
// driver's time factors.
// ---------------------------------------------------------------------------
// GATHER: state-dependent coefficients (FP64, one point per lane).
template <int P, int WP, int G, int DRV, bool F32, bool GATHER = false>
__global__ void __launch_bounds__(64 * WP * G) sweep_fused(const StepArgs s)
{
    static_assert(!GATHER || (P == 1 && !F32), "located nodes: one point per lane, double precision");
    using PR = Prec<F32>;
    using V = typename std::conditional<F32, float4, double2>::type;  // one window record
    constexpr int T = FusedShape<P, WP, G>::T, NT = FusedShape<P, WP, G>::NT;
    constexpr int C = !F32 && G >= 4 ? 8 / G : 1;  // node classes that a group sums apart
    constexpr int kLeft = F32 ? 0 : 1;             // records left of a node's cell
    constexpr int kU = 2;                          // window records per thread and layer in registers
    extern __shared__ char smem_fused[];
    char *smem = smem_fused;
    constexpr int kA = T <= 128 ? 1 : T <= 256 && G >= 4 ? 2 : 3, kB = T <= 256 && G >= 4 ? 1 : 2;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // wavefront -> (group, part of the tile); the parts rotate with the group,
    // so the wavefronts at a domain end (whose nodes take the selecting form)
    // spread over the SIMDs
    const int grp = wave / WP, wp = (wave + grp) % WP;
    const int idx = xcd_tile(blockIdx.x, gridDim.x);
    const InstDesc &d = block_desc(s, idx);
    const FusedHot h = d.hot;
    asm volatile("" ::"s"(h.nx), "s"(h.npad), "s"(h.win_lo[1]), "s"(h.win_hi[kMaxOrder]), "s"(h.lds_win[1]),
                 "s"(h.mod_magic));
    const int K = h.K, nx = h.nx, tile = idx - h.tile_base, t0 = tile * T;

    double2 *D = reinterpret_cast<double2 *>(smem + h.lds_d);
    double2 *A = reinterpret_cast<double2 *>(smem + h.lds_a);
    double2 *edge = reinterpret_cast<double2 *>(smem + h.lds_edge);
    double *drv = reinterpret_cast<double *>(smem + h.lds_drv);
    int *tm = reinterpret_cast<int *>(smem + h.lds_tm);
    // ring slot of layer n + j: n = n0 - s, so one small remainder serves all
    const int KP = K + 1, q0 = (int)((unsigned)(s.s_mod * h.mod_magic) >> 16);
    int nmod = h.n0_mod - (s.s_mod - q0 * KP);
    if (nmod < 0) nmod += KP;
    char *ring = s.ws + h.ring_off;
    auto slot = [&](int j) {
        const int r = nmod + j >= KP ? nmod + j - KP : nmod + j;
        char *base = ring + (size_t)r * ((size_t)kSlotPlanes<F32> * h.npad * sizeof(typename PR::E));
        return Slot<F32>{base, base + (size_t)h.npad * sizeof(typename PR::E), h.pad_l};
    };
    auto record = [&](const Slot<F32> &g, int k) {
        // located nodes are clamped to the grid and read one record beyond it at
        // most; their windows' bounds may lie further out than the ring's ghosts
        if constexpr (GATHER) k = min(max(k, -1), nx);
        if constexpr (F32) {
            const float2 v = g.val(k), m = g.der(k);
            return make_float4(v.x, v.y, m.x, m.y);
        } else {
            return g.der(k);  // B-spline coefficients
        }
    };

    // every load of the block first: layer n+1's values (the spline's input,
    // continued by reflection beyond the domain ends), then the windows, which
    // stay in flight while the spline is built
    const Slot<F32> g1 = slot(1);
    const int W1 = T + (h.win_hi[1] - h.win_lo[1]) + (F32 ? 1 : 3);
    const int r1 = t0 + h.win_lo[1] - kLeft;                 // window 1's first record
    const int WS = W1 + 2 * kHalo + 2, s0 = r1 - kHalo - 1;  // staged values of the filter
    const bool ends = s0 < 0 || s0 + WS > nx;                // block-uniform
    double2 raw[kU];
    V pre[kMaxOrder - 1][kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int e = tid + u * NT;
        if (e < WS) {
            raw[u] = layer_value(g1, ends ? reflected_index(nx, s0 + e) : s0 + e);
        }
    }
    double2 end0, end1;
    if (ends) {
        end0 = layer_value(g1, 0);
        end1 = layer_value(g1, nx - 1);
    }
#pragma unroll
    for (int jj = 0; jj < kMaxOrder - 1; ++jj) {
        const int j = jj + 2;
        if (j <= K) {
            const Slot<F32> g = slot(j);
            const int W = T + (h.win_hi[j] - h.win_lo[j]) + (F32 ? 1 : 3), lo = t0 + h.win_lo[j] - kLeft;
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int e = tid + u * NT;
                if (e < W) pre[jj][u] = record(g, lo + e);
            }
        }
    }
    constexpr int FP = T > NT ? T / NT : 1;  // points a thread finishes
    float2 res[FP];                          // FP32 form: residuals of the error feedback
    if constexpr (F32) {
        const Slot<true> gy = slot(h.Ky);
#pragma unroll
        for (int v = 0; v < FP; ++v) {
            const int i = min(t0 + tid + v * NT, nx - 1);
            res[v] = make_float2(fed_back_residual(gy, h.npad, i).x, fed_back_residual(g1, h.npad, i).y);
        }
    }
    // FP32: node offsets for LDS.  FP64: the lists of the group's classes and
    // their addresses, one per lane
    const int mfirst = F32 && tid < K * h.L ? h.m[tid] : 0;
    int list0[C], lcnt[C];
    int2 av[C];
    if constexpr (!F32) {
#pragma unroll
        for (int k = 0; k < C; ++k) {  // the group's first class if it takes them one by one
            class_list(K, h.L, grp + k * G, list0[k], lcnt[k]);
            av[k] = class_address(h.addr, list0[k], lcnt[k], lane);
        }
    }
    double cax = 0.0, cbx = 0.0;  // a(t_n, x_i), b(t_n, x_i) of the lane's point
    if constexpr (GATHER) {
        const int i = min(t0 + wp * 64 + lane, nx - 1);
        const double *tab = const_load(&d.a.ctab);
        if (tab) {
            const double *row =
                tab + (size_t)2 * (const_load(&d.a.tab_steps) > 1 ? h.n0 - s.s : 0) * nx;
            cax = row[i];
            cbx = row[nx + i];
        } else {
            const double xi = fma((double)i, const_load(&d.a.dx), const_load(&d.a.x_min));
            cax = fma(const_load(&d.a.drift_x), xi, const_load(&d.a.drift0));
            cbx = fma(const_load(&d.a.vol_x), xi, const_load(&d.a.vol0));
        }
    }
    double2 ev;  // boundary values (grid points 0 and N - 1) of the K layers
    if (!F32 && tid < 2 * K) {
        const auto v = slot(1 + (tid >> 1)).val((tid & 1) ? nx - 1 : 0);
        ev = make_double2(v.x, v.y);
    }
    if constexpr (F32)
        warm_scalar(h.rec32, K * h.L * (int)sizeof(NodeRec32), wave, WP * G);
    else
        warm_scalar(h.recb, K * h.L * (int)sizeof(NodeRecB), wave, WP * G);
    warm_scalar(&d, sizeof(InstDesc), wave, WP * G);
    if constexpr (DRV == BSDE_DRIVER_EXP) {
        if (tid <= K) {  // the driver's time factors of the layers n .. n + K
            const double t = (h.n0 - s.s + tid) * const_load(&d.a.dt);
            drv[3 * tid] = t;
            drv[3 * tid + 1] = exp(t * t);
            drv[3 * tid + 2] = exp(-t * t);
        }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int e = tid + u * NT;
        if (e < WS) D[e] = ends ? reflected_value(nx, s0 + e, raw[u], end0, end1) : raw[u];
    }
    for (int e = tid + kU * NT; e < WS; e += NT) {
        const double2 v = layer_value(g1, ends ? reflected_index(nx, s0 + e) : s0 + e);
        D[e] = ends ? reflected_value(nx, s0 + e, v, end0, end1) : v;
    }
    __syncthreads();
    PcrCoef pcr{};
    pcr.inv_b = const_load(&d.a.pcr.inv_b);
    if constexpr (F32) {
        pcr.s6 = const_load(&d.a.pcr.s6);
#pragma unroll
        for (int k = 0; k < kPcrRounds; ++k) pcr.kappa[k] = const_load(&d.a.pcr.kappa[k]);
    }
    if constexpr (F32)
        pcr_pass_a<NT>(W1, D, A, pcr);
    else
        fir_pass_a<NT, kA>(W1, D, A);
    __syncthreads();
    {
        V *w1 = reinterpret_cast<V *>(smem + h.lds_win[1]);
        if constexpr (F32) {
            pcr_pass_b<NT>(W1, A, pcr, [&](int e, double my, double mz) {
                const double2 v = D[e + kHalo + 1];
                const int k = r1 + e;
                const bool in = k > 0 && k < nx - 1;
                float4 r = make_float4((float)v.x, (float)v.y, in ? (float)my : 0.0f, in ? (float)mz : 0.0f);
                if (ends && (k < 0 || k >= nx)) {
                    const float2 b = g1.val(k < 0 ? 0 : nx - 1);
                    r.x = b.x;
                    r.y = b.y;
                }
                w1[WinLayout<P>::slot(e)] = r;
            });
        } else {
            const double inv_b = pcr.inv_b;
            fir_pass_b<NT, kB>(W1, A, [&](int e, double wy, double wz) {
                const double2 v = D[e + kHalo + 1];
                w1[WinLayout<P>::slot(e)] = make_double2(fma(-inv_b, wy, v.x), fma(-inv_b, wz, v.y));
            });
        }
    }
    // the other windows have arrived meanwhile
#pragma unroll
    for (int jj = 0; jj < kMaxOrder - 1; ++jj) {
        const int j = jj + 2;
        if (j <= K) {
            const Slot<F32> g = slot(j);
            const int W = T + (h.win_hi[j] - h.win_lo[j]) + (F32 ? 1 : 3), lo = t0 + h.win_lo[j] - kLeft;
            V *w = reinterpret_cast<V *>(smem + h.lds_win[j]);
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int e = tid + u * NT;
                if (e < W) w[WinLayout<P>::slot(e)] = pre[jj][u];
            }
            for (int e = tid + kU * NT; e < W; e += NT) w[WinLayout<P>::slot(e)] = record(g, lo + e);
        }
    }
    if constexpr (F32) {
        if (tid < K * h.L) tm[tid] = mfirst;
        for (int i = tid + NT; i < K * h.L; i += NT) tm[i] = h.m[i];
    }
    if (!F32 && tid < 2 * K) edge[tid] = ev;
    __syncthreads();
    {
        // the tile's part of the spline goes to HBM for the later steps, with
        // the ghost records beyond the domain ends
        const V *w1 = reinterpret_cast<V *>(smem + h.lds_win[1]);
        const int kend = min(t0 + T, nx);
        for (int k = t0 + tid; k < kend; k += NT) {
            const V r = w1[WinLayout<P>::slot(k - r1)];
            if constexpr (F32)
                g1.set_der(k, (double)r.z, (double)r.w);
            else
                g1.set_der(k, r.x, r.y);
        }
        if (tile == 0) {
            for (int k = -1 - tid; k >= -h.pad_l; k -= NT) {
                if constexpr (F32) {
                    g1.set_val(k, g1.val(0));
                    g1.set_der(k, 0.0, 0.0);
                } else {
                    const double2 r = k == -1 ? w1[WinLayout<P>::slot(-1 - r1)] : edge[0];
                    g1.set_der(k, r.x, r.y);
                }
            }
        }
        if (tile == h.ntiles - 1) {
            for (int k = nx + tid; k < h.npad - h.pad_l; k += NT) {
                if constexpr (F32) {
                    g1.set_val(k, g1.val(nx - 1));
                    g1.set_der(k, 0.0, 0.0);
                } else {
                    const double2 r = k == nx ? w1[WinLayout<P>::slot(nx - r1)] : edge[1];
                    g1.set_der(k, r.x, r.y);
                }
            }
        }
    }

    const int wfirst = t0 + wp * 64 * P;                    // the wavefront's points
    const int wlast = min(wfirst + 64 * P, nx) - 1;
    const char *lane_rec = smem + 16 * WinLayout<P>::slot((wp * 64 + lane) * P);
    const int first = wfirst + lane * P;
    double2 *part = reinterpret_cast<double2 *>(smem + h.lds_part);  // partial sums
    using F = Driver<DRV, typename PR::Raw>;
    const InstDesc *dn = own_copy(&d);  // the node phase's own values
    const int nK = const_load(&dn->hot.K), nL = const_load(&dn->hot.L), nKy = const_load(&dn->hot.Ky);
    const SweepArgs a = driver_args<DRV>(dn);
    double Y[C][P], Z[C][P];
#pragma unroll
    for (int k = 0; k < C; ++k)
#pragma unroll
        for (int q = 0; q < P; ++q) Y[k][q] = Z[k][q] = 0.0;
    if (wfirst < nx) {
        if constexpr (F32) {
            // layers in the order 2, ..., K, 1 rotated by the point's 8192-point
            // segment, a layer's nodes in order
            const int rot = ((t0 >> 13) & 3) % nK;
            Acc<P> acc;
#pragma unroll
            for (int q = 0; q < P; ++q) acc.Y[q] = acc.Z[q] = 0.0;
#pragma unroll 1
            for (int jj = 0; jj < nK; ++jj) {
                int q0 = jj + rot;
                q0 = q0 >= nK ? q0 - nK : q0;
                const int j = q0 + 1 < nK ? q0 + 2 : 1;
                if (G > 1 && jj % G != grp) continue;
                const int row = (j - 1) * nL;
                const F f = make_driver<DRV, float>(a, drv + 3 * j);
                const LdsWindow<P> src{
                    reinterpret_cast<const float4 *>(lane_rec + const_load(&dn->hot.lds_win[j])),
                    const_load(&dn->hot.win_lo[j])};
                const NodeRec32 *recs = const_load(&dn->hot.rec32) + row;
                if (j == nKy)
                    layer_nodes<P, DRV, kNodeLastY, true>(src, recs, tm + row, 0, 1, nL, f, acc);
                else
                    layer_nodes<P, DRV, 0, true>(src, recs, tm + row, 0, 1, nL, f, acc);
            }
#pragma unroll
            for (int q = 0; q < P; ++q) {
                Y[0][q] = acc.Y[q];
                Z[0][q] = acc.Z[q];
            }
        } else {
            const NodeRecB *recb = const_load(&dn->hot.recb);
            // the nodes of one list into y, z
            auto list_nodes = [&](const NodeRecB *recs, int n, const int2 &at, double (&y)[P], double (&z)[P]) {
                if constexpr (GATHER) {
                    const double pos = min(first, nx - 1);
                    gather_nodes<DRV, false>(smem, edge, recs, n, at, a, drv, pos, cax, cbx, t0, nx, y[0], z[0]);
                    if (__any(!isfinite(y[0] + z[0]))) {
                        y[0] = z[0] = 0.0;
                        gather_nodes<DRV, true>(smem, edge, recs, n, at, a, drv, pos, cax, cbx, t0, nx, y[0],
                                                z[0]);
                    }
                } else {
                    class_nodes<P, DRV>(lane_rec, edge, recs, n, at, a, drv, first, wfirst, wlast, nx, y, z);
                }
            };
            if constexpr (G < 4) {
                // four or eight classes one after the other: a class and its
                // partner are added as soon as both are there, in the order of
                // the other shapes' sums (s: the sums that wait for theirs)
                constexpr int NC = 8 / G;
                const int2 *addr = const_load(&dn->hot.addr);
                double sy[3][P], sz[3][P];
                int l0 = list0[0], cnt = lcnt[0];
                int2 an = av[0];
#pragma unroll 1
                for (int e = 0; e < NC; ++e) {
                    const NodeRecB *recs = recb + l0;
                    const int2 ac = an;
                    const int n = cnt;
                    if (e + 1 < NC) {  // the next class's addresses come during this one's nodes
                        const int r = e + 1;  // its bits reversed
                        const int c = NC == 8 ? ((r & 1) << 2) | (r & 2) | (r >> 2) : ((r & 1) << 1) | (r >> 1);
                        class_list(nK, nL, grp + c * G, l0, cnt);
                        an = class_address(addr, l0, cnt, lane);
                    }
#pragma unroll
                    for (int q = 0; q < P; ++q) Y[0][q] = Z[0][q] = 0.0;
                    list_nodes(recs, n, ac, Y[0], Z[0]);
                    auto meet = [&](int d) {
#pragma unroll
                        for (int q = 0; q < P; ++q) {
                            Y[0][q] = sy[d][q] + Y[0][q];
                            Z[0][q] = sz[d][q] + Z[0][q];
                        }
                    };
                    auto wait = [&](int d) {
#pragma unroll
                        for (int q = 0; q < P; ++q) {
                            sy[d][q] = Y[0][q];
                            sz[d][q] = Z[0][q];
                        }
                    };
                    if (!(e & 1)) {
                        wait(0);
                    } else {
                        meet(0);
                        if (!(e & 2)) {
                            wait(1);
                        } else {
                            meet(1);
                            if (NC == 8) {
                                if (!(e & 4))
                                    wait(2);
                                else
                                    meet(2);
                            }
                        }
                    }
                }
            } else {
#pragma unroll
                for (int k = 0; k < C; ++k) list_nodes(recb + list0[k], lcnt[k], av[k], Y[k], Z[k]);
            }
        }
    }

    auto class_sum = [&](int q) {  // the group's classes added pairwise, k and k + C/2 first
        double2 p[C];
#pragma unroll
        for (int k = 0; k < C; ++k) p[k] = make_double2(Y[k][q], Z[k][q]);
#pragma unroll
        for (int h = C / 2; h >= 1; h >>= 1)
#pragma unroll
            for (int k = 0; k < h; ++k) p[k] = make_double2(p[k].x + p[k + h].x, p[k].y + p[k + h].y);
        return p[0];
    };
    // the groups' sums meet in LDS; a thread finishes one point
    constexpr bool kDirectSums = G == 1 && P == 1;
    if constexpr (!kDirectSums) {
        if (h.lds_part == h.lds_win[1]) __syncthreads();  // over the windows: they are no longer read
#pragma unroll
        for (int q = 0; q < P; ++q)
            part[(size_t)grp * T + (wp * 64 + lane) * P + q] = class_sum(q);
        __syncthreads();
    }
    const InstDesc *de = own_copy(&d);  // the finish's own values
    SweepArgs fa = driver_args<DRV>(de);
    fa.h0 = const_load(&de->a.h0);
    fa.picard_max = const_load(&de->a.picard_max);
    fa.picard_tol = const_load(&de->a.picard_tol);
    const Driver<DRV, double> f0 = make_driver<DRV, double>(fa, drv);
    const int fnx = const_load(&de->hot.nx), fnpad = const_load(&de->hot.npad);
    // slot of layer n
    char *obase = s.ws + const_load(&de->hot.ring_off) +
                  (size_t)nmod * ((size_t)kSlotPlanes<F32> * fnpad * sizeof(typename PR::E));
    const Slot<F32> out{obase, obase + (size_t)fnpad * sizeof(typename PR::E), const_load(&de->hot.pad_l)};
    const bool last = const_load(&de->hot.n0) - s.s == const_load(&de->a.n_stop);
    double *fin_y = reinterpret_cast<double *>(s.ws + const_load(&de->fin_off)), *fin_z = fin_y + fnx;
#pragma unroll
    for (int v = 0; v < FP; ++v) {
        const int pt = tid + v * NT;
        const int i = t0 + pt;
        unsigned int it = 0;
        bool conv = true;
        const bool valid = pt < T && i < fnx;
        if (valid) {
            double2 sum;
            if constexpr (kDirectSums) {
                sum = class_sum(0);
            } else {
                double2 p[G];
#pragma unroll
                for (int g = 0; g < G; ++g) p[g] = part[(size_t)g * T + pt];
#pragma unroll
                for (int h = G / 2; h >= 1; h >>= 1)
#pragma unroll
                    for (int g = 0; g < h; ++g)
                        p[g] = make_double2(p[g].x + p[g + h].x, p[g].y + p[g + h].y);
                sum = p[0];
            }
            if constexpr (!F32 && DRV == BSDE_DRIVER_LINEAR) {
                sum.x += const_load(&de->lin_y);
                sum.y += const_load(&de->lin_z);
            }
            const double y = picard_solve(fa, f0, D[i - s0].x, sum.x, sum.y, it, conv);
            if constexpr (F32)
                store_fed_back(out, fnpad, i, y, sum.y, res[v].x, res[v].y);
            else
                out.set_val(i, y, sum.y);
            if (last) {
                fin_y[i] = y;
                fin_z[i] = sum.y;
            }
        }
        // per-wave statistics; a wavefront without a point of the grid has no slot
        if (s.stats && pt - lane < T && i - lane < fnx) {
            const unsigned int itm = wave_max_u32(it), its = wave_sum_u32(it);
            const unsigned int nc = wave_sum_u32(conv ? 0u : 1u);
            if (lane == 0) {
                const int w = i >> 6, nw = const_load(&de->nwaves);
                unsigned long long *sum =
                    reinterpret_cast<unsigned long long *>(s.ws + const_load(&de->stat_off));
                unsigned int *mx = reinterpret_cast<unsigned int *>(sum + 2 * nw);
                mx[w] = max(mx[w], itm);
                sum[w] += its;
                sum[nw + w] += nc;
            }
        }
    }
}

}  // namespace bsde
