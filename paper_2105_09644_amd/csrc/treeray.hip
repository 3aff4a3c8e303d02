// TreeRay/OnTheSpot on MI355X (gfx950): device kernels and the C ABI.
//
// Steps of one outer iteration (paper Sec. 2):
//   k_fill / k_deposit     point sources onto the leaf cells (Sec. 2.1, 2.7)
//   k_cell_quantities      eps, alpha, e of every cell (eqs. os:ems, os:abs, os:erd)
//   k_reduce_level         FP64 bottom-up node moments, one launch per tree level
//   k_pack                 node records for the sweep (FP64 or FP32, SoA)
//   k_walk                 the accepted nodes of every target and their pixel pairs
//   k_sweep                per target: node->ray mapping + per-ray
//                          On-the-Spot integration + sum over rays (Sec. 2.3-2.5)
//   k_select / k_delta     delta_cell with an exact radix-select median
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "chunk.h"
#include "kernels.h"
#include "tr_internal.h"

namespace tr {

// moment rows of the FP64 node arrays
enum { MO_EPS = 0, MO_ALPHA, MO_E, MO_V, MO_MASS, MO_MX, MO_MY, MO_MZ, MO_VX, MO_VY, MO_VZ, MO_MION, MO_COUNT };

// ---------------------------------------------------------------------------
// small utility kernels
// ---------------------------------------------------------------------------
__global__ void k_fill_f64(double *p, int64_t n, double v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_u64(unsigned long long *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// ---------------------------------------------------------------------------
// a1. Point sources onto leaf cells.  A source coordinate within 1e-9 finest
// cells of a cell face is moved onto it; the rate is split equally over every
// leaf cell whose closed cube contains the point.  One thread per source
// descends the tree from its domain's root.
// ---------------------------------------------------------------------------
__global__ void k_deposit(const double *__restrict__ xyz, const double *__restrict__ q,
                          const int32_t *__restrict__ sdom, int32_t n_src, const DomDev *__restrict__ doms,
                          const int4 *__restrict__ geo, const int2 *__restrict__ topo, double *ndot,
                          int32_t *err)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_src) return;
    const DomDev D = doms[sdom[s]];
    double u[3];
    for (int a = 0; a < 3; ++a) {
        double v = xyz[3 * s + a] / D.dx_cm;
        const double rn = floor(v + 0.5);
        if (fabs(v - rn) <= 1e-9) v = rn;
        u[a] = v;
    }
    int stack[160];
    int sp = 0;
    stack[sp++] = D.root;
    int cells[8];
    int nc = 0;
    while (sp > 0) {
        const int n = stack[--sp];
        const int4 g = geo[n];
        const double sz = (double)(g.w & kSizeMask);
        if (!(u[0] >= g.x && u[0] <= g.x + sz && u[1] >= g.y && u[1] <= g.y + sz && u[2] >= g.z &&
              u[2] <= g.z + sz))
            continue;
        const int2 tp = topo[n];
        if (tp.y == 0) {
            if (nc < 8) cells[nc] = tp.x;
            ++nc;
        } else {
            if (sp + tp.y > 160) { atomicOr(err, 4); return; }
            for (int c = 0; c < tp.y; ++c) stack[sp++] = tp.x + c;
        }
    }
    if (nc == 0 || nc > 8 || !(q[s] >= 0.0) || !isfinite(q[s])) {
        atomicOr(err, 1);
        return;
    }
    const double share = q[s] / (double)nc;
    for (int c = 0; c < nc; ++c) atomicAdd(&ndot[cells[c]], share);
}

// Sources as uniform spheres (Sec. 2.7): each leaf cell receives the rate
// times the fraction of the sphere's in-domain volume that lies inside it.
// Volume of a ball cut by a box = integral over z of the area of a disk cut
// by a rectangle; that area is exact, and the integral is split where the
// circle meets an edge line or a corner of the rectangle (the area's
// derivatives jump there) and taken on each piece after the substitution
// z = p + (q - p)(1 - cos(pi t))/2 with Gauss-Legendre nodes in t.
__constant__ double c_gl_t[kGlNodes], c_gl_w[kGlNodes];

// area of {x >= u, y >= v} inside the disk of radius r, for u, v >= 0
__device__ double disk_corner(double r, double u, double v)
{
    if (u * u + v * v >= r * r) return 0.0;
    const double r2 = r * r, x1 = sqrt(r2 - v * v);
    const double gu = u * sqrt(fmax(r2 - u * u, 0.0)) + r2 * asin(fmin(u / r, 1.0));
    const double g1 = x1 * v + r2 * asin(fmin(x1 / r, 1.0));
    return 0.5 * (g1 - gu) - v * (x1 - u);
}

// the same for any signs: a negative bound is reflected (the half-plane
// x >= u < 0 is twice x >= 0 less x >= -u)
__device__ double disk_quadrant(double r, double u, double v)
{
    if (u >= 0.0 && v >= 0.0) return disk_corner(r, u, v);
    if (v >= 0.0) return 2.0 * disk_corner(r, 0.0, v) - disk_corner(r, -u, v);
    if (u >= 0.0) return 2.0 * disk_corner(r, u, 0.0) - disk_corner(r, u, -v);
    return 2.0 * (2.0 * disk_corner(r, 0.0, 0.0) - disk_corner(r, 0.0, -v)) -
           (2.0 * disk_corner(r, -u, 0.0) - disk_corner(r, -u, -v));
}

__device__ double disk_rect(double r, double x0, double x1, double y0, double y1)
{
    return disk_quadrant(r, x0, y0) - disk_quadrant(r, x1, y0) - disk_quadrant(r, x0, y1) + disk_quadrant(r, x1, y1);
}

// volume of the ball (centre c, radius R) inside the box [lo, hi]
__device__ double ball_box(const double c[3], double R, const double lo[3], const double hi[3])
{
    const double za = fmax(lo[2], c[2] - R), zb = fmin(hi[2], c[2] + R);
    if (za >= zb || lo[0] >= c[0] + R || hi[0] <= c[0] - R || lo[1] >= c[1] + R || hi[1] <= c[1] - R) return 0.0;
    const double x0 = lo[0] - c[0], x1 = hi[0] - c[0], y0 = lo[1] - c[1], y1 = hi[1] - c[1];
    const double dist[8] = {fabs(x0), fabs(x1), fabs(y0), fabs(y1), sqrt(x0 * x0 + y0 * y0), sqrt(x1 * x1 + y0 * y0),
                            sqrt(x0 * x0 + y1 * y1), sqrt(x1 * x1 + y1 * y1)};
    double cut[18];
    int nc = 0;
    cut[nc++] = za;
    cut[nc++] = zb;
    for (int k = 0; k < 8; ++k) {
        if (dist[k] >= R) continue;
        const double h = sqrt(R * R - dist[k] * dist[k]);
        if (c[2] - h > za && c[2] - h < zb) cut[nc++] = c[2] - h;
        if (c[2] + h > za && c[2] + h < zb) cut[nc++] = c[2] + h;
    }
    for (int i = 1; i < nc; ++i)   // insertion sort of at most 18 heights
        for (int j = i; j > 0 && cut[j] < cut[j - 1]; --j) {
            const double t = cut[j];
            cut[j] = cut[j - 1];
            cut[j - 1] = t;
        }
    double v = 0.0;
    for (int k = 0; k + 1 < nc; ++k) {
        const double p = cut[k], q = cut[k + 1];
        if (!(q > p)) continue;
        double sum = 0.0;
        for (int i = 0; i < kGlNodes; ++i) {
            const double t = c_gl_t[i];
            const double z = p + (q - p) * 0.5 * (1.0 - cospi(t));
            const double h = z - c[2];
            const double r2 = R * R - h * h;
            if (r2 > 0.0) sum += c_gl_w[i] * disk_rect(sqrt(r2), x0, x1, y0, y1) * sinpi(t);
        }
        v += sum * (q - p) * 0.5 * kPi;
    }
    return v;
}

// One thread per source; pass 0 sums the in-domain volume, pass 1 deposits.
__global__ void k_deposit_spheres(const double *__restrict__ xyz, const double *__restrict__ q,
                                  const int32_t *__restrict__ sdom, int32_t n_src, const DomDev *__restrict__ doms,
                                  const int4 *__restrict__ geo, const int2 *__restrict__ topo, double radius_cm,
                                  double *ndot, int32_t *err)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_src) return;
    const DomDev D = doms[sdom[s]];
    const double R = radius_cm / D.dx_cm;
    double u[3];
    for (int a = 0; a < 3; ++a) u[a] = xyz[3 * s + a] / D.dx_cm;
    if (!(q[s] >= 0.0) || !isfinite(q[s])) {
        atomicOr(err, 1);
        return;
    }
    double total = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
        int stack[160];
        int sp = 0;
        stack[sp++] = D.root;
        while (sp > 0) {
            const int n = stack[--sp];
            const int4 g = geo[n];
            const int sz = g.w & kSizeMask;
            const double lo[3] = {(double)g.x, (double)g.y, (double)g.z};
            const double hi[3] = {lo[0] + sz, lo[1] + sz, lo[2] + sz};
            bool touch = true;
            for (int a = 0; a < 3; ++a) touch &= lo[a] < u[a] + R && hi[a] > u[a] - R;
            if (!touch) continue;
            const int2 tp = topo[n];
            if (tp.y == 0) {
                const double v = ball_box(u, R, lo, hi);
                if (v > 0.0) {
                    if (pass == 0) total += v;
                    else atomicAdd(&ndot[tp.x], q[s] * (v / total));
                }
            } else {
                if (sp + tp.y > 160) {
                    atomicOr(err, 4);
                    return;
                }
                for (int c = 0; c < tp.y; ++c) stack[sp++] = tp.x + c;
            }
        }
        if (pass == 0 && !(total > 0.0)) {
            atomicOr(err, 1);
            return;
        }
    }
}

// ---------------------------------------------------------------------------
// a2. Cell quantities in internal units (length: finest cell of the domain;
// rate: rate_unit, a power of two).  s = ndot - alpha_B n^2 dV is netted
// inside the cell: eps = max(s, 0), alpha = max(-s, 0).  E = F_prev dV.
// ---------------------------------------------------------------------------
__global__ void k_cell_quantities(int64_t n_cells, const double *__restrict__ n_h,
                                  const double *__restrict__ ndot, const double *__restrict__ f_prev,
                                  const int32_t *__restrict__ cell_node, const int32_t *__restrict__ cell_dom,
                                  const DomDev *__restrict__ doms, const int4 *__restrict__ geo, int32_t thin,
                                  double *__restrict__ M, int64_t nn, int32_t *err)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_cells) return;
    const int node = cell_node[c];
    const DomDev D = doms[cell_dom[c]];
    const int4 g = geo[node];
    const int sz = g.w & kSizeMask;
    const double dv = (double)sz * (double)sz * (double)sz;
    const double nh = n_h[c];
    double fp = f_prev ? f_prev[c] : 0.0;
    if (!(nh >= 0.0) || !isfinite(nh) || !(fp >= 0.0) || !isfinite(fp)) {
        atomicOr(err, 2);
    }
    const double s = ndot[c] / D.rate_unit - (thin ? 0.0 : D.alpha_int * nh * nh * dv);
    const double mass = nh * dv;
    M[MO_EPS * nn + node] = s > 0.0 ? s : 0.0;
    M[MO_ALPHA * nn + node] = s < 0.0 ? -s : 0.0;
    M[MO_E * nn + node] = (fp / D.flux_unit) * dv;
    M[MO_V * nn + node] = dv;
    M[MO_MASS * nn + node] = mass;
    const double cx = g.x + 0.5 * sz, cy = g.y + 0.5 * sz, cz = g.z + 0.5 * sz;
    M[MO_MX * nn + node] = mass * cx;
    M[MO_MY * nn + node] = mass * cy;
    M[MO_MZ * nn + node] = mass * cz;
    M[MO_VX * nn + node] = dv * cx;
    M[MO_VY * nn + node] = dv * cy;
    M[MO_VZ * nn + node] = dv * cz;
    // ionised gas: cells with a positive previous flux (the IF MAC's ionised mass)
    M[MO_MION * nn + node] = fp > 0.0 ? mass : 0.0;
}

// ---------------------------------------------------------------------------
// a3. Node moments: plain FP64 sums over the children (contiguous), one
// launch per level, deepest first.
// ---------------------------------------------------------------------------
__global__ void k_reduce_level(int64_t b, int64_t e, const int2 *__restrict__ topo, double *__restrict__ M,
                               int64_t nn)
{
    const int64_t n = b + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= e) return;
    const int2 tp = topo[n];
    if (tp.y == 0) return;
    for (int m = 0; m < MO_COUNT; ++m) {
        double s = 0.0;
        const double *row = M + m * nn + tp.x;
        for (int c = 0; c < tp.y; ++c) s += row[c];
        M[m * nn + n] = s;
    }
}

// Node records for the sweep, and the node flags of the IF and Src MACs
// (Sec. 2.4): an ionisation front when the ionised mass lies strictly between
// 1e-8 and 1 - 1e-8 of the mass, emission when eps_n > 0.
template <typename R, typename R4>
__global__ void k_pack(int64_t nn, const double *__restrict__ M, R4 *__restrict__ A, R4 *__restrict__ B,
                       int4 *__restrict__ geo)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= nn) return;
    const double m = M[MO_MASS * nn + n], v = M[MO_V * nn + n];
    {
        const double mi = M[MO_MION * nn + n], dif = 1e-8;
        int w = geo[n].w & ~(kIfBit | kSrcBit);
        if (dif * m < mi && mi < (1.0 - dif) * m) w |= kIfBit;
        if (M[MO_EPS * nn + n] > 0.0) w |= kSrcBit;
        geo[n].w = w;
    }
    double cx, cy, cz;
    if (m > 0.0) {
        cx = M[MO_MX * nn + n] / m;
        cy = M[MO_MY * nn + n] / m;
        cz = M[MO_MZ * nn + n] / m;
    } else {
        cx = M[MO_VX * nn + n] / v;
        cy = M[MO_VY * nn + n] / v;
        cz = M[MO_VZ * nn + n] / v;
    }
    R4 a, b;
    a.x = (R)cx; a.y = (R)cy; a.z = (R)cz; a.w = (R)M[MO_EPS * nn + n];
    b.x = (R)M[MO_ALPHA * nn + n]; b.y = (R)M[MO_E * nn + n]; b.z = (R)v; b.w = (R)0;
    A[n] = a;
    B[n] = b;
}

// ---------------------------------------------------------------------------
// The sweep
// ---------------------------------------------------------------------------
template <typename Real> struct R4T;
template <> struct R4T<float> { using T = float4; };
template <> struct R4T<double> { using T = double4; };

// One target of a chunk, written by k_walk for the sweep: doubled centre and
// size, domain, accepted nodes and those that emit, output index, moments.
struct TargetRec {
    int32_t tx, ty, tz, tsize;
    int32_t dom, n_acc, n_emit, pad;   // n_emit < 0: nothing to map (bad index, or queued for the fallback pass)
    int64_t out;
    double eps, alpha, e, v;
};

struct SweepArgs {
    const int4 *geo;
    const int4 *olo;
    const int4 *oext;
    const int2 *topo;
    const void *pA;          // Real4 (com.x, com.y, com.z, eps)
    const void *pB;          // Real4 (alpha, E, V, 0)
    const int32_t *cell_node;
    const int32_t *cell_dom;
    const DomDev *doms;
    const double *r64;       // evaluation points, finest-cell units, per domain
    const float *r32;
    const int64_t *targets;  // explicit target list, or NULL
    const int32_t *order;    // all cells in (domain, Morton) order
    int64_t n_cells;
    // the chunk of the work items [item0, item0 + n_chunk) whose walks are
    // listed: target i's accepted nodes at lists[i list_cap ..], each with where
    // its (pixel, count) pairs are, and the places of those that emit at
    // emit_at[i list_cap ..]
    int64_t item0;
    int32_t n_chunk, list_cap;
    int2 *lists;
    uint16_t *emit_at;
    TargetRec *rec;
    double *f_out;
    uint8_t *ion_out;
    int32_t *queue;          // [0] next item, [1] overflow flag
    unsigned long long *stats;  // [0] accepted, [1] tested, [2] guard recomputes, [3] rays marched in
                                // FP32, [4] of those marched again in FP64, [5] nodes from the table
    void *gbuf;              // ray buffers in global memory (when they do not fit in LDS)
    void *ebuf;              // split LDS buffers: the emission rows, rays x nr_max per workgroup
    unsigned char *mbuf;     // marks and ray numbers in device memory: mask_slab_bytes per workgroup
    int64_t mbuf_stride;
    int32_t split;           // 1: A, E, V rows in LDS (stride_k = 3 nr_max + 1), emission rows in ebuf
    double theta2, theta_if2, theta_src2;   // squared opening angles (0: criterion off)
    float guard_tol;
    int32_t f32;             // 1: float records (FP32C), 0: double
    int32_t nside, npix, subsample, nr_max, stride_k, zeta_g;
    int32_t int_wave;        // 1: a wave per ray (lanes = points); 0: a lane per ray
    int32_t int_group;       // > 0: a group of this many lanes per ray (slots = emitting points)
    int32_t int_fp32;        // 1 (FP32 buffers, groups): the FP32 march, FP64 again near a front
    float front_ratio;       // Phi / Phi_jj below which the FP32 march defers a ray to FP64
    int32_t eps_kernel;      // emission kernel (K_F1 .. K_G; 0 or K_F3: two-point W_f,3)
    int32_t periodic;        // 1: every node through its periodic copy closest to the target
    int32_t mass_gauss;      // 1: W_g for A, E, V and the self term; 0: W_p
    // walks too long for the lists: the item is queued in ovf and a second
    // launch (k_sweep_fallback) walks it with per-workgroup lists of gfmax /
    // gamax entries in device memory
    int32_t *ovf;
    int64_t ovf_cap;
    int32_t *glist;
    int32_t gfmax, gamax;
    int32_t rays;        // ray buffers of a workgroup: a target's rays that hold emission are mapped and
                         // integrated so many at a time
    // angular-weight table (NULL: none): for a node of 2^ri times the target's
    // size (ri < kAtabRatios) at offset o in target sizes from the target's
    // lower corner, |o_a| <= atab_w[ri], the entry
    // atab_idx[atab_base[ri] + ((o_x + w)(2w + 1) + o_y + w)(2w + 1) + o_z + w]
    // = (first pair / 4 << 6) | (pairs - 1), each pair in atab_pool = pixel | count << 16;
    // the pairs of the chunk's other nodes are in dyn_pool (kDynEntry set)
    const int32_t *atab_idx;
    const int32_t *atab_pool;
    int32_t atab_w[kAtabRatios], atab_base[kAtabRatios];
    int32_t *dyn_pool;
    int32_t dyn_units;   // its size in units of 4 pairs
};

// Ray buffer rows: eps, A (recombinations), E (previous flux x volume), V.

// Where ray k's rows live: A, E and V of point i at b[k stride + oa + (0, 1, 2) nrm + i],
// the emission at e[k estride + i].  Either one buffer with four rows per ray
// (e = b, estride = stride, oa = nrm), or, when four rows do not fit in LDS,
// the A, E, V rows in LDS and the emission rows (written by emitting nodes
// only) in a per-workgroup plane in device memory.
template <typename Real>
struct RayRows {
    Real *b, *e;
    int stride, estride, oa, nrm;
    __device__ Real &A(int k, int i) const { return b[(size_t)k * stride + oa + i]; }
    __device__ Real &E(int k, int i) const { return b[(size_t)k * stride + oa + nrm + i]; }
    __device__ Real &V(int k, int i) const { return b[(size_t)k * stride + oa + 2 * nrm + i]; }
    __device__ Real &eps(int k, int i) const { return e[(size_t)k * estride + i]; }
};

// Index into the angular table of a node whose cube has its (shifted) corner
// at (bx, by, bz), or -1: a cube of 1, 2, 4, ... target sizes within the
// table's window; offsets of its corner in target sizes (exact).
__device__ inline int table_key(const SweepArgs &a, int gw, int bx, int by, int bz, int tx, int ty, int tz, int tsize)
{
    const int size = gw & kSizeMask;
    if (!a.atab_idx || (gw & kPartialBit)) return -1;
    const int sh = __builtin_ctz((unsigned)tsize);   // (sizes are powers of two)
    const int ri = __builtin_ctz((unsigned)size) - sh;
    if ((unsigned)ri >= (unsigned)kAtabRatios) return -1;
    int w = a.atab_w[0], base = a.atab_base[0];
#pragma unroll
    for (int q = 1; q < kAtabRatios; ++q) {
        w = ri == q ? a.atab_w[q] : w;
        base = ri == q ? a.atab_base[q] : base;
    }
    const int kx = (bx - ((tx - tsize) >> 1)) >> sh, ky = (by - ((ty - tsize) >> 1)) >> sh,
              kz = (bz - ((tz - tsize) >> 1)) >> sh;
    const int nw = 2 * w + 1;   // (w = -1: this ratio is not tabulated)
    if (abs(kx) > w || abs(ky) > w || abs(kz) > w) return -1;
    return base + ((kx + w) * nw + (ky + w)) * nw + (kz + w);
}

// Accumulation into a ray buffer shared by the lanes and waves of a workgroup.
// AM: 1 a hardware atomic add, 2 (FP32 in LDS) an add by compare-and-swap on
// the value's bits: the same correctly rounded FP32 sum in some order.  An
// FP32 atomic add in LDS takes this chip 3 cycles a lane (195 for 64 lanes);
// three adds by compare-and-swap take 50 to 70 cycles for 64 lanes.
__device__ inline unsigned lds_swap(unsigned *q, unsigned expected, unsigned desired)
{
    __hip_atomic_compare_exchange_strong(q, &expected, desired, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
    return expected;   // what the word held
}
template <typename Real>
__device__ inline void buf_add(Real *p, Real v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Three adds at once (A, E, V of one ray point): wk x0, wk x1, wk x2.  In the
// compare-and-swap form the three reads and then the three swaps are in flight
// together, each sum rounded once.  Lanes that meet on a point meet on all
// three rows and lose there to the same lane, so the three are repeated
// together; one that is through adds zero.
template <typename Real, int AM>
__device__ inline void buf_add3(Real wk, Real *p0, Real x0, Real *p1, Real x1, Real *p2, Real x2)
{
    if constexpr (AM == 2 && sizeof(Real) == 4) {
        unsigned *q0 = (unsigned *)p0, *q1 = (unsigned *)p1, *q2 = (unsigned *)p2;
        unsigned o0 = __hip_atomic_load(q0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        unsigned o1 = __hip_atomic_load(q1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        unsigned o2 = __hip_atomic_load(q2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        for (;;) {
            const unsigned n0 = __float_as_uint(fmaf(wk, x0, __uint_as_float(o0)));
            const unsigned n1 = __float_as_uint(fmaf(wk, x1, __uint_as_float(o1)));
            const unsigned n2 = __float_as_uint(fmaf(wk, x2, __uint_as_float(o2)));
            const unsigned r0 = lds_swap(q0, o0, n0), r1 = lds_swap(q1, o1, n1), r2 = lds_swap(q2, o2, n2);
            const bool d0 = r0 == o0, d1 = r1 == o1, d2 = r2 == o2;
            if (d0 && d1 && d2) break;
            o0 = d0 ? n0 : r0;   // (a row that is through holds its sum now)
            o1 = d1 ? n1 : r1;
            o2 = d2 ? n2 : r2;
            x0 = d0 ? 0.0f : x0;
            x1 = d1 ? 0.0f : x1;
            x2 = d2 ? 0.0f : x2;
        }
    } else {
        buf_add<Real>(p0, wk * x0);
        buf_add<Real>(p1, wk * x1);
        buf_add<Real>(p2, wk * x2);
    }
}

// Periodic boundaries (Sec. 2.8): v is twice a node centre's offset from the
// target along an axis with period L finest cells; returns the multiple of L
// (in finest cells) that moves the offset into (-L/2, L/2], the closest copy.
__device__ inline int nearest_copy_shift(int v, int L)
{
    const int num = L - v, den = 2 * L;
    const int k = num >= 0 ? num / den : -((-num + den - 1) / den);   // floor(num / den)
    return k * L;
}

// Shift of a node to its periodic copy closest to the target (by the cube's centre); per NULL: none
__device__ inline void node_shift(const int *per, const int4 g, int tx, int ty, int tz, int sh[3])
{
    if (!per) return;
    const int size = g.w & kSizeMask;
    sh[0] = nearest_copy_shift(2 * g.x + size - tx, per[0]);
    sh[1] = nearest_copy_shift(2 * g.y + size - ty, per[1]);
    sh[2] = nearest_copy_shift(2 * g.z + size - tz, per[2]);
}

// Distance of a node's (shifted) mass centre from the target.  The marking and
// the mapping both take it, and the emission bracket below, and must end on the
// same two points bit for bit: emission mapped onto an unmarked point would be
// lost, and with split rows stay in the plane that only the march of the marked
// points clears.  So the fused operations are written out and the compiler adds
// none of its own.
template <typename Real, typename R4>
__device__ inline Real centre_distance(const R4 A, const int sh[3], int tx, int ty, int tz)
{
#pragma clang fp contract(off)
    const Real dx = (A.x + (Real)sh[0]) - (Real)0.5 * (Real)tx, dy = (A.y + (Real)sh[1]) - (Real)0.5 * (Real)ty,
               dz = (A.z + (Real)sh[2]) - (Real)0.5 * (Real)tz;
    return fsqrt(__builtin_elementwise_fma(dz, dz, __builtin_elementwise_fma(dy, dy, dx * dx)));
}

// Per ray, a mask of the points 1 .. N_R - 1 that received emission: ew words
// (1 for N_R <= 64, else 2) of 64 bits, bit i of word w for point 64 w + i.
__device__ inline void mask_or(unsigned long long *p, unsigned long long bits)
{
    __hip_atomic_fetch_or(p, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// marks points i0 (if e0) and i0 + 1 (if e1) of the ray whose mask starts at m
__device__ inline void mark_points(unsigned long long *m, int i0, bool e0, bool e1)
{
    const int i1 = i0 + 1;
    const unsigned long long b0 = e0 && i0 >= 1 ? 1ull << (i0 & 63) : 0ull;
    const unsigned long long b1 = e1 ? 1ull << (i1 & 63) : 0ull;
    if ((i0 >> 6) == (i1 >> 6)) {
        if (b0 | b1) mask_or(m + (i0 >> 6), b0 | b1);
    } else {
        if (b0) mask_or(m + (i0 >> 6), b0);
        if (b1) mask_or(m + (i1 >> 6), b1);
    }
}

// outermost marked point (0: none)
__device__ inline int mask_top(unsigned long long w0, unsigned long long w1)
{
    return w1 ? 127 - __clzll((long long)w1) : (w0 ? 63 - __clzll((long long)w0) : 0);
}

// radial kernels by kind: 5 W_p, 6 W_g (App. A.1, A.2)
enum { K_F1 = 1, K_F2 = 2, K_F3 = 3, K_F3N = 4, K_P = 5, K_G = 6 };
template <typename Real>
__device__ inline Real smooth_kernel(bool gauss, Real x)
{
    if (!gauss) return wp_kernel<Real>(x);
    x = x < (Real)0 ? -x : x;
    return x < (Real)0.86602540378443864676 ? (Real)exp((double)(-x * x)) : (Real)0;
}

// Phi (photon rate per steradian) lives in the eps slot of a point once the
// march has passed it; FP32 buffers keep it as a split double in the
// (eps, A) slots, both consumed by then.
__device__ inline double phi_load(const RayRows<double> &R, int k, int j) { return R.eps(k, j); }
__device__ inline void phi_store(const RayRows<double> &R, int k, int j, double v) { R.eps(k, j) = v; }
__device__ inline double phi_load(const RayRows<float> &R, int k, int j)
{
    const uint32_t lo = __float_as_uint(R.eps(k, j));
    const uint32_t hi = __float_as_uint(R.A(k, j));
    return __hiloint2double((int)hi, (int)lo);
}
__device__ inline void phi_store(const RayRows<float> &R, int k, int j, double v)
{
    R.eps(k, j) = __uint_as_float((uint32_t)__double2loint(v));
    R.A(k, j) = __uint_as_float((uint32_t)__double2hiint(v));
}

// 1/x in FP64 for the ray march (x > 0, finite): the hardware estimate (relative
// error below 2^-24 on this chip, measured) refined by one Newton step, which
// squares the error: a few 1e-15, far inside the FP64 form's 1e-10 bound, with
// two fewer dependent FMAs on the march's critical path
__device__ inline double drcp(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    return fma(r, fma(-x, r, 1.0), r);
}

// One ray (Sec. 2.5), one lane: march inwards from the outermost point that
// holds emission (top; nothing reaches the target from beyond it), all
// sources together.
// Per segment [r_i, r_{i+1}] and source j beyond it:
//   R = (alpha_i + alpha_{i+1})/2 dV_{i,j} zeta_s zeta_d zeta_g,
//   zeta_s zeta_d = F_{i+1,j} min(2/F_{i+1}, 1/Fbar_{i+1})   (zeta_d = 2 where Fbar = 0),
//   dV_{i,j} = (r_{i+1} - r_i)(A^2 + A B + B^2)/3, A = r_j - r_i, B = r_j - r_{i+1},
// and the source at r_{i+1} itself takes zeta_s = zeta_d = 1.
// Returns F_{0,k} in internal flux units.
template <typename Real>
__device__ double integrate_ray(const RayRows<Real> &R, int k, const double *r, const double *inv2r, int nr, int top,
                                int nside, int zeta_g, bool clear_eps)
{
    const double inv4pi = 1.0 / (4.0 * kPi);
    const double ns = (double)nside;
    uint64_t m0 = 0, m1 = 0;     // points j holding a live Phi_j
    double a1 = 0.0, fb1 = 0.0;  // alpha and previous flux at r_{i+1}
    // the point's buffer entries are fetched one step ahead
    Real nV = R.V(k, top), nA = R.A(k, top), nE = R.E(k, top), nEps = R.eps(k, top);
    for (int i = top; i >= 0; --i) {
        const double Vi = (double)nV, Ai = (double)nA, Ei = (double)nE, ei = (double)nEps;
        if (i > 0) {
            nV = R.V(k, i - 1);
            nA = R.A(k, i - 1);
            nE = R.E(k, i - 1);
            nEps = R.eps(k, i - 1);
        }
        double ai = 0.0, fbi = 0.0;
        if (Vi > 0.0) {
            const double rv = drcp(Vi);
            ai = Ai * rv;
            fbi = Ei * rv;
        }
        if (i <= nr - 2 && (m0 | m1)) {
            const double ri = r[i], ri1 = r[i + 1], seg = ri1 - ri;
            // F_{i+1}: flux at r_{i+1} from the sources beyond it
            double ftot = 0.0;
            for (int h = 0; h < 2; ++h) {
                uint64_t m = h ? m1 : m0;
                while (m) {
                    const int j = (h << 6) + __ffsll((unsigned long long)m) - 1;
                    m &= m - 1;
                    if (j >= i + 2) {
                        const double dd = r[j] - ri1;
                        ftot += phi_load(R, k, j) * drcp(dd * dd);
                    }
                }
            }
            double g = 0.0;
            if (ftot > 0.0) {
                g = 2.0 * drcp(ftot);
                if (fb1 > 0.0) g = fmin(g, drcp(fb1));
            }
            const double aseg = 0.5 * (ai + a1) * seg * (1.0 / 3.0);
            for (int h = 0; h < 2; ++h) {
                uint64_t m = h ? m1 : m0;
                while (m) {
                    const int j = (h << 6) + __ffsll((unsigned long long)m) - 1;
                    m &= m - 1;
                    double ph = phi_load(R, k, j);
                    const double rj = r[j];
                    const double A = rj - ri, B = rj - ri1;
                    double z = 1.0;
                    if (j >= i + 2) z = ph * drcp(B * B) * g;
                    if (zeta_g) z *= fmin(1.0, ns * A * inv2r[j]);
                    ph = fmax(0.0, ph - aseg * (A * A + A * B + B * B) * z);
                    phi_store(R, k, j, ph);
                    if (!(ph > 0.0)) {
                        if (j < 64) m0 &= ~(1ull << j);
                        else m1 &= ~(1ull << (j - 64));
                    }
                }
            }
        }
        if (i >= 1 && ei > 0.0) {
            phi_store(R, k, i, ei * inv4pi);
            if (i < 64) m0 |= 1ull << i;
            else m1 |= 1ull << (i - 64);
        }
        a1 = ai;
        fb1 = fbi;
    }
    double f0 = 0.0;
    for (int h = 0; h < 2; ++h) {
        uint64_t m = h ? m1 : m0;
        while (m) {
            const int j = (h << 6) + __ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            const double rj = r[j];
            f0 += phi_load(R, k, j) * drcp(rj * rj);
        }
    }
    // emission rows kept in device memory are left zero for the next target
    // (the march reused them for Phi)
    if (clear_eps)
        for (int i = 1; i <= top; ++i) R.eps(k, i) = (Real)0;
    return f0;
}

template <typename T>
__device__ inline T rdlane(T v, int l);

// value of point i held by lane i % 64 of the pair (v[0], v[1]); i uniform
__device__ inline double point_value(const double v[2], int i)
{
    return i < 64 ? rdlane(v[0], i) : rdlane(v[1], i - 64);
}

// The same march with a whole wave on one ray: lane p holds point p (and
// p + 64), so every source on the ray advances in the same step and the
// total flux F_{i+1} is a wave reduction.  Phi stays in registers.  Returns
// F_{0,k} (uniform) in internal flux units.
template <typename Real, int NH>
__device__ double integrate_ray_wave(const RayRows<Real> &R, int k, const double *r, const double *inv2r, int nr,
                                     int top, int nside, int zeta_g, bool clear_eps)
{
    const int lane = here(lane_id());   // (nothing derived from it is held between calls)
    const double inv4pi = 1.0 / (4.0 * kPi);
    const double ns = (double)nside;
    double al[2], fb[2], ph[2], rp[2], i2r[2], ep[2];
    bool live[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int p = lane + 64 * h;
        al[h] = fb[h] = ph[h] = ep[h] = rp[h] = i2r[h] = 0.0;
        live[h] = false;
        if (p < nr) {
            const double V = (double)R.V(k, p);
            if (V > 0.0) {
                const double rv = drcp(V);
                al[h] = (double)R.A(k, p) * rv;
                fb[h] = (double)R.E(k, p) * rv;
            }
            ep[h] = (double)R.eps(k, p);
            rp[h] = r[p];
            i2r[h] = inv2r[p];
        }
    }
    bool any = false;   // uniform: some source on the ray is still live
    for (int i = top; i >= 0; --i) {
        if (i <= nr - 2 && any) {
            const double ri = r[i], ri1 = r[i + 1];
            const double ai = point_value(al, i), ai1 = point_value(al, i + 1), fb1 = point_value(fb, i + 1);
            double f[2], fs = 0.0;
            f[1] = 0.0;
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                f[h] = 0.0;
                if (live[h] && lane + 64 * h >= i + 2) {
                    const double B = rp[h] - ri1;
                    f[h] = ph[h] * drcp(B * B);
                }
                fs += f[h];
            }
            const double ftot = wave_sum(fs);
            double g = 0.0;
            if (ftot > 0.0) {
                g = 2.0 * drcp(ftot);
                if (fb1 > 0.0) g = fmin(g, drcp(fb1));
            }
            const double aseg = 0.5 * (ai + ai1) * (ri1 - ri) * (1.0 / 3.0);
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                if (live[h]) {
                    const double A = rp[h] - ri, B = rp[h] - ri1;
                    double z = lane + 64 * h >= i + 2 ? f[h] * g : 1.0;
                    if (zeta_g) z *= fmin(1.0, ns * A * i2r[h]);
                    ph[h] = fmax(0.0, ph[h] - aseg * (A * A + A * B + B * B) * z);
                    live[h] = ph[h] > 0.0;
                }
            }
            any = __ballot(live[0] || live[1]) != 0ull;
        }
        if (i >= 1 && point_value(ep, i) > 0.0) {
            const int h = i >> 6;
            if (lane == (i & 63)) {
                ph[h] = ep[h] * inv4pi;
                live[h] = true;
            }
            any = true;
        }
    }
    double s = 0.0;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        if (live[h]) s += ph[h] * drcp(rp[h] * rp[h]);
        // emission rows kept in device memory are left zero for the next target (a bracket weight
        // that rounds to less than nothing leaves a negative entry)
        if (clear_eps && ep[h] != 0.0) R.eps(k, lane + 64 * h) = (Real)0;
    }
    return wave_sum(s);
}

// Slot sl of a group of G lanes gets the sl-th emitting point of its ray
// (from the ray's mask (w0, w1) of points 1 .. N_R - 1; -1: none); cnt
// returns the ray's number of emitting points.
template <int G>
__device__ inline int group_emitter(unsigned long long w0, unsigned long long w1, int sl, bool has_ray, int &cnt)
{
    const int c0 = (int)__popcll(w0);
    cnt = has_ray ? c0 + (int)__popcll(w1) : 0;
    if (sl >= cnt) return -1;
    return sl < c0 ? nth_set_bit(w0, sl) : 64 + nth_set_bit(w1, sl - c0);
}

// The same march with a group of G lanes per ray (G = 4 .. 64), so that a
// wave integrates 64/G rays at once: slot s of the group holds the ray's s-th
// emitting point j (in pixel-row order) with its Phi_j in a register, and
// F_{i+1} is a group sum.  Every lane of a group reads the same point's
// moments.  k / (w0, w1): this lane's ray (has_ray false: none) and its
// mask of emitting points; tmax: the largest outermost emitting point of the
// wave's rays (uniform).  A
// ray with more than G emitting points is left alone (n_over returns their
// number on its lanes, else 0; the caller integrates it with more lanes).
// Returns F_{0,k} in internal flux units on every lane of the group.  Call
// with every lane active.
template <typename Real, int G>
__device__ double integrate_rays_group(const RayRows<Real> &R, int k, unsigned long long w0, unsigned long long w1,
                                       bool has_ray, int tmax,
                                       const double *r, const double *inv2r, int nr, int nside, int zeta_g,
                                       int &n_over, bool clear_eps)
{
    const int lane = here(lane_id());   // (nothing derived from it is held between calls)
    const int sl = lane & (G - 1);
    const int g0 = lane - sl;   // first lane of the group
    const double inv4pi = 1.0 / (4.0 * kPi);
    const double ns = (double)nside;
    int cnt;
    const int j = group_emitter<G>(w0, w1, sl, has_ray, cnt);
    n_over = has_ray && cnt > G ? cnt : 0;
    const bool act = has_ray && cnt <= G;
    double rj = 0.0, i2rj = 0.0, epsj = 0.0;
    if (act && j > 0) {
        rj = r[j];
        i2rj = inv2r[j];
        epsj = (double)R.eps(k, j);
    }
    const double phjj = epsj * inv4pi;   // Phi_jj, emitted at r_j
    double ph = 0.0, a1 = 0.0, fb1 = 0.0;   // alpha and previous flux at r_{i+1}
    bool live = false;
    // every step is predicated (selects, no branches on lane values); the
    // moments are read one point ahead, beyond the ray's outermost emitting
    // point too (they meet no live source); r_{i+1} and B = r_j - r_{i+1} are
    // the previous step's r_i and A
    double ri1 = tmax + 1 < nr ? r[tmax + 1] : 0.0;
    double Bv = rj - ri1, B2 = Bv * Bv;
    Real nV = R.V(k, tmax), nA = R.A(k, tmax), nE = R.E(k, tmax);
    for (int i = tmax; i >= 0; --i) {
        const double Vi = (double)nV, Ai = (double)nA, Ei = (double)nE;
        if (i >= 1) {
            nV = R.V(k, i - 1);
            nA = R.A(k, i - 1);
            nE = R.E(k, i - 1);
        }
        const double rv = drcp(Vi);
        const double ai = Vi > 0.0 ? Ai * rv : 0.0;
        const double fbi = Vi > 0.0 ? Ei * rv : 0.0;
        const double ri = r[i];
        const double A = rj - ri, A2 = A * A;
        if (i <= nr - 2) {
            const bool far = live && j >= i + 2;
            const double f = far ? ph * drcp(B2) : 0.0;
            const double ftot = group_sum(f, G);   // F_{i+1} of the group's ray
            // min(2 / F_{i+1}, 1 / Fbar_{i+1}), used where f > 0 (so F_{i+1} > 0)
            const double g2 = 2.0 * drcp(ftot);
            const double g = fb1 > 0.0 ? fmin(g2, drcp(fb1)) : g2;
            const double aseg = 0.5 * (ai + a1) * (ri1 - ri) * (1.0 / 3.0);
            double z = far ? f * g : 1.0;
            if (zeta_g) z *= fmin(1.0, ns * A * i2rj);
            const double nph = ph - aseg * (A2 + A * Bv + B2) * z;
            const bool alive = live && nph > 0.0;
            ph = alive ? nph : 0.0;
            live = alive;
        }
        const bool born = act && i >= 1 && j == i;
        ph = born ? phjj : ph;
        live = live || born;
        a1 = ai;
        fb1 = fbi;
        ri1 = ri;
        Bv = A;
        B2 = A2;
    }
    // emission rows kept in device memory are left zero for the next target
    if (clear_eps && act && j > 0) R.eps(k, j) = (Real)0;
    return group_sum(live ? ph * drcp(rj * rj) : 0.0, G);
}

// The same march in FP32 (FP32C integration, Sec. 2.5), a group of G lanes
// per ray as above, for FP32 ray buffers:
//  - radial differences from exact integers: r_j - r_i = c (j^2 - i^2), so a
//    segment's volume dV_{i,j} carries no cancellation error;
//  - Phi_j is kept as an unevaluated FP32 pair (hi + lo): each loss R is
//    subtracted with its rounding error kept (Fast2Sum, exact while R <= Phi),
//    so Phi's error is only that of the R's themselves (a few ulp of each, at
//    most a few 1e-7 of the emitted Phi_jj in all);
//  - F_{0,k} = sum_j Phi_{0,j} / r_j^2 as a compensated group sum.
// Where the FP32 result is not safe to 1e-4 -- a live source whose Phi falls
// below front_ratio of its emitted Phi_jj, or dies in a step whose loss is
// within 1e-3 of what it had (a close call between dying and surviving), the
// regime of an ionisation front -- near is set on the group and the caller
// integrates that ray again in FP64.  Returns F_{0,k} as (hi, lo) on every
// lane of the group.  Call with every lane active.
template <int G>
__device__ void integrate_rays_group_f32(const RayRows<float> &R, int k, unsigned long long w0, unsigned long long w1,
                                         bool has_ray, int tmax,
                                         float rcoef, const double *inv2r, int nr, int nside, int zeta_g,
                                         float front_ratio, int &n_over, bool &near, float &f_hi, float &f_lo,
                                         bool clear_eps)
{
    const int lane = here(lane_id());   // (nothing derived from it is held between calls)
    const int sl = lane & (G - 1);
    const int g0 = lane - sl;
    const uint64_t gmask = G == 64 ? ~0ull : ((1ull << G) - 1ull);
    const float inv4pi = (float)(1.0 / (4.0 * kPi));
    const float ns = (float)nside;
    const float third = 1.0f / 3.0f;
    int cnt;
    const int j = group_emitter<G>(w0, w1, sl, has_ray, cnt);
    n_over = has_ray && cnt > G ? cnt : 0;
    const bool act = has_ray && cnt <= G;
    float i2rj = 0.0f, epsj = 0.0f, rj = 0.0f;
    const int j2 = j > 0 ? j * j : 0;
    if (act && j > 0) {
        i2rj = (float)inv2r[j];
        epsj = R.eps(k, j);
        rj = rcoef * (float)j2;
    }
    const float phjj = epsj * inv4pi;   // Phi_jj, emitted at r_j
    const float gz = ns * i2rj;         // zeta_g = min(1, gz (r_j - r_i))
    float ph = 0.0f, pl = 0.0f, a1 = 0.0f, fb1 = 0.0f;
    bool live = false, died = false;
    float bd = 0.0f, ld = 0.0f;   // at the source's death: its Phi before the step and the step's loss
    // every step is predicated (selects, no branches on lane values); the
    // moments are read one point ahead, beyond the ray's outermost emitting
    // point too (they meet no live source).  q = j^2 - i^2 exactly, so
    // A = r_j - r_i = c q, and B = r_j - r_{i+1} is the previous step's A.
    float q = (float)(j2 - (tmax + 1) * (tmax + 1));
    float Bv = rcoef * q, B2 = Bv * Bv;
    float nV = R.V(k, tmax), nA = R.A(k, tmax), nE = R.E(k, tmax);
    for (int i = tmax; i >= 0; --i) {
        const float Vi = nV, Ai = nA, Ei = nE;
        if (i >= 1) {
            nV = R.V(k, i - 1);
            nA = R.A(k, i - 1);
            nE = R.E(k, i - 1);
        }
        const float rv = __builtin_amdgcn_rcpf(Vi);
        const float ai = Vi > 0.0f ? Ai * rv : 0.0f;
        const float fbi = Vi > 0.0f ? Ei * rv : 0.0f;
        const float odd = (float)(2 * i + 1);
        q += odd;
        const float A = rcoef * q, A2 = A * A;
        if (i <= nr - 2) {
            const bool far = live && j >= i + 2;
            const float f = far ? (ph + pl) * __builtin_amdgcn_rcpf(B2) : 0.0f;
            const float ftot = group_sum(f, G);   // F_{i+1} of the group's ray
            // min(2 / F_{i+1}, 1 / Fbar_{i+1}); used where f > 0 (so F_{i+1} > 0), and
            // Fbar_{i+1} = 0 gives 1 / Fbar = +inf
            const float g = fminf(2.0f * __builtin_amdgcn_rcpf(ftot), __builtin_amdgcn_rcpf(fb1));
            const float aseg = 0.5f * (ai + a1) * (rcoef * odd) * third;
            float z = far ? f * g : 1.0f;
            if (zeta_g) z *= fminf(1.0f, A * gz);
            const float loss = aseg * (A2 + A * Bv + B2) * z;
            const float before = ph + pl;
            // ph - loss as sh + se, exactly while the source lives (|loss| <= ph:
            // Fast2Sum); a larger loss kills it whatever the rounding, and a near
            // tie is the close call marched again in FP64
            const float sh = ph - loss;
            const float se = -loss - (sh - ph);
            const float npl = pl + se;
            const bool alive = live && sh + npl > 0.0f;
            const bool dies = live && !alive;
            bd = dies ? before : bd;
            ld = dies ? loss : ld;
            died = died || dies;
            ph = alive ? sh : 0.0f;
            pl = alive ? npl : 0.0f;
            live = alive;
        }
        const bool born = act && i >= 1 && j == i;
        ph = born ? phjj : ph;
        live = live || born;
        a1 = ai;
        fb1 = fbi;
        Bv = A;
        B2 = A2;
    }
    // Phi only falls: a live source ended below front_ratio of Phi_jj, or a
    // source died from below that or in a close call between dying and
    // surviving (the step's loss within 1e-3 of what it had)
    const float frp = front_ratio * phjj;
    const bool flag = (live && ph + pl < frp) || (died && (bd < frp || ld < 1.001f * bd));
    float th = 0.0f, tl = 0.0f;
    if (live) {
        const float rr = __builtin_amdgcn_rcpf(rj * rj);
        th = ph * rr;
        tl = pl * rr;
    }
    group_csum(th, tl, G);
    f_hi = th;
    f_lo = tl;
    near = ((__ballot(flag) >> g0) & gmask) != 0ull;
    // emission rows kept in device memory are left zero for the next target
    // (a ray marched again in FP64 is cleared there)
    if (clear_eps && act && j > 0 && !near) R.eps(k, j) = 0.0f;
}

// The class of ray k (k >= np: none) from its mask of emitting points: 0 no
// emission, else ceil(log2) of its number of emitting points, at least lg0, 7
// beyond 64; tp returns its outermost emitting point.
__device__ inline int ray_class(const unsigned long long *emask, int ew, int np, int lg0, int k, int &tp)
{
    unsigned long long w0 = 0ull, w1 = 0ull;
    if (k < np) {
        w0 = emask[(size_t)k * ew];
        if (ew > 1) w1 = emask[(size_t)k * ew + 1];
    }
    tp = mask_top(w0, w1);
    const int cnt = (int)(__popcll(w0) + __popcll(w1));
    return cnt == 0 ? 0 : cnt > 64 ? 7 : max(lg0, 32 - __clz(cnt - 1));
}

// One batch of the group integration: 64 / G rays of G lanes each (myk < 0:
// no ray on this group; (m0, m1) the ray's mask of emitting points).  Adds the
// rays' F_{0,k} on their groups' first lanes: FP64 results into fsum, FP32
// marched ones (FP32 buffers with the FP32 march) into the compensated pair
// (cs_hi, cs_lo), a ray near an ionisation front marched again in FP64.
template <typename Real, int G>
__device__ __forceinline__ void march_batch(const SweepArgs &a, const RayRows<Real> &R, int myk, unsigned long long m0,
                                            unsigned long long m1, Real rcoef,
                                            const double *rd, const double *rd2, int nr, bool split, double &fsum,
                                            float &cs_hi, float &cs_lo, uint64_t &n_f32, uint64_t &n_f64)
{
    const int lane = here(lane_id());   // (nothing derived from it is held between calls)
    const bool has = myk >= 0;
    const int tmax = wave_max_nonneg(mask_top(m0, m1));
    const bool head = (lane & (G - 1)) == 0;
    int over = 0;   // zero: the ray's class holds its emitting points
    if constexpr (sizeof(Real) == 4) {
        if (a.int_fp32) {
            bool near = false;
            float fh = 0.0f, fl = 0.0f;
            integrate_rays_group_f32<G>(R, has ? myk : 0, m0, m1, has, tmax, rcoef, rd2, nr, a.nside, a.zeta_g,
                                        a.front_ratio, over, near, fh, fl, split);
            const bool ok = head && has;
            if (ok && !near) {
                float sh, se;
                two_sum(cs_hi, fh, sh, se);
                cs_hi = sh;
                cs_lo += se + fl;
            }
            n_f32 += __popcll(__ballot(ok));
            // the rays near an ionisation front, again in FP64
            const bool redo = has && near;
            if (__ballot(head && redo)) {
                const double f = integrate_rays_group<Real, G>(R, redo ? myk : 0, m0, m1, redo, tmax, rd, rd2, nr,
                                                               a.nside, a.zeta_g, over, split);
                if (head && redo) fsum += f;
                n_f64 += __popcll(__ballot(head && redo));
            }
            return;
        }
    }
    const double f = integrate_rays_group<Real, G>(R, has ? myk : 0, m0, m1, has, tmax, rd, rd2, nr, a.nside, a.zeta_g,
                                                   over, split);
    if (head && has) fsum += f;
}

template <typename T>
__device__ inline T rdlane(T v, int l)
{
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
    } else {
        const long long b = __builtin_bit_cast(long long, v);
        const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
        const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
        return __builtin_bit_cast(T, (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
    }
}

// W_f,1 and W_f,2 (App. A.3) on the bracket r_i <= d < r_{i+1}: both keep the
// flux at the target exact; W_f,1 takes u_{i+1}/u_i = (d - r_i)/(r_{i+1} - d),
// W_f,2 also makes the flux exact at r_{i-1} (i >= 2; it keeps W_f,3 when a
// weight would be negative).  Solved in FP64.
template <typename Real>
__device__ void two_point_variant(int ek, const Real *rt, int i, double d, Real &u0, Real &u1)
{
    const double ri = (double)rt[i], rn = (double)rt[i + 1];
    if (ek == K_F1) {
        const double rho = (d - ri) / (rn - d);
        const double ui = 1.0 / (d * d * (1.0 / (ri * ri) + rho / (rn * rn)));
        u0 = (Real)ui;
        u1 = (Real)(rho * ui);
        return;
    }
    if (i < 2) return;
    const double p = (double)rt[i - 1];
    const double a11 = 1.0 / (ri * ri), a12 = 1.0 / (rn * rn), b1 = 1.0 / (d * d);
    const double a21 = 1.0 / ((ri - p) * (ri - p)), a22 = 1.0 / ((rn - p) * (rn - p)), b2 = 1.0 / ((d - p) * (d - p));
    const double det = a11 * a22 - a12 * a21;
    const double ui = (b1 * a22 - a12 * b2) / det, un = (a11 * b2 - a21 * b1) / det;
    if (ui >= 0.0 && un >= 0.0) {
        u0 = (Real)ui;
        u1 = (Real)un;
    }
}

// N-point W_f,3 (App. A.3, eqs. eKernFC1, eKernFC2): over the points k >= 1
// inside the node's extent, |r_k - d| < sqrt(3)/2 h, weights a + b (k - le)
// with sum 1 and sum 1/r_k^2 = 1/d^2.  Leaves mode 0 (two-point) when fewer
// than two points qualify or a weight would be negative.  Solved in FP64.
template <typename Real>
__device__ void n_point_f3(const Real *rt, int l0, int h0, double d, double h, int &mode, int &le, int &ne, Real &ea,
                           Real &eb)
{
    const double half = 0.86602540378443864676 * h;
    int first = -1, n = 0;
    double s1 = 0, t0 = 0, t1 = 0;
    for (int k = l0 > 1 ? l0 : 1; k <= h0; ++k) {
        const double rk = (double)rt[k];
        if (fabs(rk - d) >= half) continue;
        if (first < 0) first = k;
        const double m = (double)(k - first), w = 1.0 / (rk * rk);
        s1 += m;
        t0 += w;
        t1 += m * w;
        ++n;
    }
    if (n < 2) return;
    const double det = (double)n * t1 - s1 * t0;
    const double av = (t1 - s1 / (d * d)) / det, bv = ((double)n / (d * d) - t0) / det;
    if (av < 0.0 || av + bv * (double)(n - 1) < 0.0) return;
    mode = 1;
    le = first;
    ne = n;
    ea = (Real)av;
    eb = (Real)bv;
}

// Weight of support point i (offset io from the support's first point) in the
// spread emission forms: 1 linear N-point W_f,3, 2 a smoothing kernel scaled by
// ea, 3 the mass fall-back split (fb on the first point, 1 - fb on the next).
template <typename Real>
__device__ inline Real emission_weight(int mode, int i, int io, int le, int ne, Real ea, Real eb, Real fb, Real rcoef,
                                       Real d, Real hinv, bool gauss)
{
    if (mode == 1) return (i >= le && i < le + ne) ? ea + eb * (Real)(i - le) : (Real)0;
    if (mode == 2) return smooth_kernel<Real>(gauss, (rcoef * (Real)(i * i) - d) * hinv) * ea;
    return io == 0 ? fb : (Real)1 - fb;
}

// W_f,3 (App. A.3): the bracket r_i <= d < r_{i+1}, i >= 1, and its two weights
// (beyond either end all on the end point).  Returns i.  The same bits wherever
// it is inlined (see centre_distance).
template <typename Real>
__device__ inline int emission_bracket(const Real *rt, int nr, Real rc_inv, Real d, Real &u0, Real &u1)
{
#pragma clang fp contract(off)
    u0 = 1;
    u1 = 0;
    if (d >= rt[nr - 1]) return nr - 1;
    if (!(d >= rt[1])) return 1;
    int k = (int)fsqrt(d * rc_inv);
    k = k < 1 ? 1 : (k > nr - 2 ? nr - 2 : k);
    while (k > 1 && rt[k] > d) --k;
    while (k < nr - 2 && rt[k + 1] <= d) ++k;
    const Real ai = frcp(rt[k] * rt[k]), an = frcp(rt[k + 1] * rt[k + 1]), ad = frcp(d * d);
    const Real dn = ad - an, di = frcp(ai - an);
    u0 = dn * di;
    u1 = __builtin_elementwise_fma(-dn, di, (Real)1);
    return k;
}

// A lane's place in the s^3 sub-point lattice of a node's box (lanes from s^3
// on have none).
struct Lattice {
    int s, ia, ib, ic;
    float ca, cb, cc;   // index + 1/2 + the fixed shift
    bool active;
    uint64_t mask;
    __device__ Lattice(int s_) : s(s_)
    {
        const int lane = lane_id();
        ia = lane / (s * s);
        ib = (lane / s) % s;
        ic = lane % s;
        ca = ((float)ia + 0.5f) + (float)kJit0;
        cb = ((float)ib + 0.5f) + (float)kJit1;
        cc = ((float)ic + 0.5f) + (float)kJit2;
        active = lane < s * s * s;
        mask = __ballot(active);
    }
};

// A node's box: its lower corner relative to the target and its sub-box steps
// in FP32, and the same as integers (corner, extent in finest cells).
struct Box {
    float o[3], step[3];
    int b[3], e[3];
};

// The pixels of a box's sub-points, by a whole wave (lane = sub-point): FP32
// with a guard band, FP64 inside it, so the FP64 classifier's pixel for every
// sub-point.  Returns the number of distinct pixels; lane q of kc holds the
// q-th and its sub-point count, pixel | count << 16.
__device__ __forceinline__ int classify_box(const Lattice &L, int ns, int npix, float guard_tol, const Box &box, int tx,
                                            int ty, int tz, int32_t *flag, uint64_t &guard_count, int &kc)
{
    const int lane = lane_id();
    const float vx = fmaf(L.ca, box.step[0], box.o[0]);
    const float vy = fmaf(L.cb, box.step[1], box.o[1]);
    const float vz = fmaf(L.cc, box.step[2], box.o[2]);
    bool unsure = false;
    int pix = ang2pix_f(ns, vx, vy, vz, guard_tol, unsure);
    unsure &= L.active;
    if (const uint64_t again = __ballot(unsure)) {
        guard_count += __popcll(again);
        if (unsure)
            pix = subpoint_pix_d(ns, L.s, box.b[0], box.b[1], box.b[2], box.e[0], box.e[1], box.e[2], tx, ty, tz, L.ia,
                                 L.ib, L.ic);
    }
    if ((unsigned)pix >= (unsigned)npix) {
        // cannot happen for a finite direction: reported, never written out of bounds
        atomicOr(flag, 4);
        pix = 0;
    }
    uint64_t left = L.mask;
    int nd = 0;
    while (left) {
        const int first = __ffsll((unsigned long long)left) - 1;
        const int k = __builtin_amdgcn_readlane(pix, first);
        const uint64_t m = __ballot(pix == k) & left;
        left &= ~m;
        const int v = k | ((int)__popcll(m) << 16);   // uniform
        kc = lane == nd ? v : kc;
        ++nd;
    }
    return nd;
}

// The box of a node for its sub-points; sh: the shift to its periodic copy.
__device__ inline Box node_box(const SweepArgs &a, int n, const int4 g, const int sh[3], int tx, int ty, int tz)
{
    Box box;
    const int size = g.w & kSizeMask;
    box.b[0] = g.x; box.b[1] = g.y; box.b[2] = g.z;
    box.e[0] = box.e[1] = box.e[2] = size;
    if (g.w & kPartialBit) {
        const int4 o = a.olo[n], e = a.oext[n];
        box.b[0] = o.x; box.b[1] = o.y; box.b[2] = o.z;
        box.e[0] = e.x; box.e[1] = e.y; box.e[2] = e.z;
    }
    const float inv_s = 1.0f / (float)a.subsample;
    const int tc[3] = {tx, ty, tz};
    for (int q = 0; q < 3; ++q) {
        box.b[q] += sh[q];
        box.o[q] = 0.5f * (float)(2 * box.b[q] - tc[q]);
        box.step[q] = (float)box.e[q] * inv_s;
    }
    return box;
}

// The (node, pixel) pairs of up to 64 nodes, node n on a lane, its pairs at
// entry (kNoEntry: none, or no node), laid end to end and handed out 64 at a
// time.  CLASSIFY (fallback pass): then those of the lanes in todo, node by
// node, each classified by the whole wave.
template <bool CLASSIFY>
struct PairStream {
    // node on lane l: its pairs start at off; lane q of perm holds the lane of
    // the q-th node with an entry, offc its start
    const int lane;
    unsigned entry;
    int n_ent, off, perm, offc, ptot, b;
    uint64_t todo;

    __device__ __forceinline__ PairStream(int lane_, unsigned entry_, uint64_t todo_) : lane(lane_), entry(entry_), b(0), todo(todo_)
    {
        const bool has = entry != kNoEntry;
        const uint64_t tmask = __ballot(has), nmask = uniform(~tmask);
        n_ent = (int)__popcll(tmask);
        off = wave_excl_scan_dpp(has ? (int)(entry & 63u) + 1 : 0, ptot);
        const int rank_t = bits_below(tmask), rank_n = n_ent + bits_below(nmask);
        perm = __builtin_amdgcn_ds_permute((has ? rank_t : rank_n) << 2, lane);
        offc = __shfl(off, perm, 64);
    }

    // The next pairs: node (its lane) and kc = pixel | count << 16 (pixel < 2^16,
    // count <= 64) on lanes below the returned number; 0: no more.
    __device__ __forceinline__ int next(const SweepArgs &a, int n, const int *per, int tx, int ty, int tz,
                                        uint64_t &guard_count, int &node, int &kc)
    {
        node = kc = 0;
        if (b < ptot) {
            // S: the positions 1 .. 63 where a node's pairs start, shifted by one; r0: the node of position 0
            const int rel = offc - b;
            const bool is_node = lane < n_ent;
            const int r0 = (int)__popcll(__ballot(is_node && rel <= 0)) - 1;
            const uint64_t bit = is_node && rel > 0 && rel < 64 ? 1ull << (rel - 1) : 0ull;
            const uint64_t S = ((uint64_t)(unsigned)wave_or((int)(bit >> 32)) << 32) | (unsigned)wave_or((int)bit);
            node = __shfl(perm, r0 + bits_below(S), 64);
            const unsigned en = (unsigned)__shfl((int)entry, node, 64);
            const int on = __shfl(off, node, 64);
            const int fill = ptot - b < 64 ? ptot - b : 64;
            if (lane < fill) {
                const int32_t *const pool = en & kDynEntry ? a.dyn_pool : a.atab_pool;
                kc = pool[(int)((en & ~kDynEntry) >> 6) * 4 + (b + lane - on)];
            }
            b += 64;
            return fill;
        }
        if constexpr (CLASSIFY) {
            if (todo == 0ull) return 0;
            node = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const int jn = rdlane(n, node);
            const int4 g = a.geo[jn];
            int sh[3] = {0, 0, 0};
            node_shift(per, g, tx, ty, tz, sh);
            return classify_box(Lattice(a.subsample), a.nside, a.npix, a.guard_tol, node_box(a, jn, g, sh, tx, ty, tz), tx,
                                ty, tz, &a.queue[1], guard_count, kc);
        }
        return 0;
    }
};

// The angular-table entry of the node on this lane (kNoEntry: none)
__device__ inline unsigned table_entry(const SweepArgs &a, const int4 g, const int sh[3], int tx, int ty, int tz, int tsize)
{
    const int key = table_key(a, g.w, g.x + sh[0], g.y + sh[1], g.z + sh[2], tx, ty, tz, tsize);
    return key >= 0 ? (unsigned)a.atab_idx[key] : kNoEntry;
}

// The points that the emitting nodes among cnt <= 64 (node n on lane < cnt,
// its pairs at entry; CLASSIFY: the angular table is still to be asked) put emission on, marked in the masks of all rays.  Nothing else is deposited
// yet: a ray without emission adds nothing to the flux, nor does what lies
// beyond a ray's outermost emitting point, so the mapping that follows skips
// both (with few sources most rays: 81% of the pairs on 64^3 N_side 4 with one
// source, 60% on 128^3 N_side 2 with 16).  rt: the evaluation points.
template <typename Real, bool CLASSIFY>
__device__ void mark_nodes(const SweepArgs &a, unsigned long long *emask, int ew, const int *per, const Real *rt, int nr,
                           Real rc_inv, int n, unsigned entry, int cnt, int tx, int ty, int tz, int tsize)
{
    using R4 = typename R4T<Real>::T;
    const int lane = here(lane_id());
    int mark = 0;   // the bracket's lower point, bit 8: emission there, bit 9: on the next
    if (lane < cnt) {
        const R4 A = ((const R4 *)a.pA)[n];
        int sh[3] = {0, 0, 0};
        if (per || CLASSIFY) {
            const int4 g = a.geo[n];
            node_shift(per, g, tx, ty, tz, sh);
            if (CLASSIFY) entry = table_entry(a, g, sh, tx, ty, tz, tsize);
        }
        if (A.w > (Real)0) {
            const Real d = centre_distance<Real>(A, sh, tx, ty, tz);
            Real u0, u1;
            mark = emission_bracket<Real>(rt, nr, rc_inv, d, u0, u1);
            mark |= (A.w * u0 != (Real)0 ? 256 : 0) | (A.w * u1 != (Real)0 ? 512 : 0);
        }
    }
    if (CLASSIFY && mark < 256) entry = kNoEntry;   // (the fallback pass lists all nodes)
    PairStream<CLASSIFY> ps(lane, entry, CLASSIFY ? __ballot(mark >= 256 && entry == kNoEntry) : 0ull);
    uint64_t guard_count = 0;   // (the mapping counts them)
    for (;;) {
        int node, kc;
        const int fill = ps.next(a, n, per, tx, ty, tz, guard_count, node, kc);
        if (fill == 0) break;
        const int m = __shfl(mark, node, 64);
        if (lane < fill && m >= 256)
            mark_points(emask + (size_t)(kc & 0xffff) * ew, m & 255, (m & 256) != 0, (m & 512) != 0);
    }
}

// Maps cnt <= 64 accepted nodes, node n on lane < cnt with its pairs at entry
// (CLASSIFY: the angular table is still to be asked), onto the target's rays
// that have a buffer; executed by a whole wave in two phases.
//  Phase 1, lane = node: loads the node, its mass-centre distance d, the
//   W_p normalisation over the evaluation points in its support and the W_f,3
//   bracket of its emission (App. A).
//  Phase 2, lane = (node, pixel) pair: the pairs of all the nodes; those on a
//   ray with a buffer (rinfo: its index << 8 | its outermost emitting point, 0
//   none) are collected 64 at a time, and each lane runs over its node's
//   support points up to that point and adds its pixel's share of A, E and V
//   to each.  A node has few pairs (mean 2.8 at N_side 2, 5.3 at N_side 4) and
//   few points with a weight (3 to 4), so one node at a time leaves most lanes
//   idle: 154 to 200 vector instructions per node, against 11 to 27 for the
//   same adds in pairs.
// The evaluation points are r_i = c i^2; the lanes recompute them in
// registers, so the loop over them makes no memory round trip besides its
// atomics.
// KV: the radial-kernel variants of App. A (otherwise two-point W_f,3 and
// W_p), whose emission may be spread; every ray has a buffer then, and cmask
// (by buffer) is marked here.
// LDSBUF false (buffers in device memory): a lane per point of a pair, the
// points of 64 pairs laid end to end: neighbouring lanes add to neighbouring
// points, so an atomic instruction touches a few cache lines and not 64 (W_p
// emission, every ray with a buffer: 48^3 N_side 2 FP64 50.6 ms, a lane per pair
// 104.8; 32^3 N_side 4 with 100 points 35.7 / 153.6, FP32C 29.1 / 158.9).
template <typename Real, int ATOMIC, bool LDSBUF, bool KV, bool CLASSIFY>
__device__ void map_nodes(const SweepArgs &a, const RayRows<Real> &R, const unsigned *rinfo, unsigned long long *cmask,
                          int ew, const int *per, const Real *rt, int nr, Real rc_inv, Real rcoef, int n,
                          unsigned entry, int cnt, int tx, int ty, int tz, int tsize, uint64_t &guard_count,
                          uint64_t &tab_count)
{
    using R4 = typename R4T<Real>::T;
    const int lane = here(lane_id());
    const Real xe = (Real)0.86602540378443864676;
    // ---------------- phase 1 ----------------
    int lo = 0, nsup = 0, ie = 1;
    Real d = 1, hinv = 1, wscale = 0, fb0 = 1, qa = 0, qe = 0, qv = 0, e0 = 0, e1 = 0;
    // emission spread over several points: mode 1 linear (a + b (i - le) on [le, le + ne)),
    // 2 a smoothing kernel scaled by ea, 3 the mass fall-back weights
    int emode = 0, le = 0, ne = 0;
    Real ea = 0, eb = 0, qeps = 0;
    const bool mg = KV && a.mass_gauss != 0;
    if (lane < cnt) {
        const int4 g = a.geo[n];
        const int size = g.w & kSizeMask;
        const R4 A = ((const R4 *)a.pA)[n];
        const R4 B = ((const R4 *)a.pB)[n];
        qa = B.x; qe = B.y; qv = B.z;
        int sh[3] = {0, 0, 0};
        node_shift(per, g, tx, ty, tz, sh);
        if (CLASSIFY) entry = table_entry(a, g, sh, tx, ty, tz, tsize);
        d = centre_distance<Real>(A, sh, tx, ty, tz);
        const Real h = (Real)size;
        hinv = frcp(h);   // a power of two: exact
        const Real rl = d - xe * h, rh = d + xe * h;
        // the points inside the support, and one beyond it on either side at most (a square
        // root that rounds across an integer loses none)
        const int l0 = rl > (Real)0 ? (int)fsqrt(rl * rc_inv) : 0;
        int h0 = (int)fsqrt(rh * rc_inv) + 1;
        h0 = h0 > nr - 1 ? nr - 1 : h0;
        Real sum = 0;
        int end = 0, npos = 0;   // the points with a weight (contiguous: the kernel is positive inside its support)
        Real fi = (Real)l0;
        for (int i = l0; i <= h0; ++i, fi += (Real)1) {
            const Real v = smooth_kernel<Real>(mg, (rcoef * (fi * fi) - d) * hinv);
            sum += v;
            const bool pos = v > (Real)0;
            end = pos ? i : end;
            npos += pos ? 1 : 0;
        }
        if (sum > (Real)0) {
            wscale = frcp(sum);
            lo = KV ? l0 : end - npos + 1;   // (an emission variant may use a point that rounding leaves outside)
            nsup = KV ? h0 - l0 + 1 : npos;
        } else if (d >= rt[nr - 1]) {   // no point in the support: linear split over the bracket
            lo = nr - 1;
            nsup = 1;
            fb0 = 1;
        } else {
            int ib = (int)fsqrt(d * rc_inv);
            ib = ib > nr - 2 ? nr - 2 : ib;
            while (ib > 0 && rt[ib] > d) --ib;
            while (ib < nr - 2 && rt[ib + 1] <= d) ++ib;
            lo = ib;
            nsup = 2;
            fb0 = (rt[ib + 1] - d) * frcp(rt[ib + 1] - rt[ib]);
        }
        qeps = A.w;
        const int ek = KV ? a.eps_kernel : 0;
        if (A.w > (Real)0 && (ek == K_P || ek == K_G)) {   // a smoothing kernel for the emission too
            if (sum > (Real)0) {
                Real es = 0;
                for (int i = l0; i <= h0; ++i) {
                    const Real v = smooth_kernel<Real>(ek == K_G, (rcoef * (Real)(i * i) - d) * hinv);
                    es += v;
                }
                emode = 2;
                ea = frcp(es);
            } else {
                emode = 3;
            }
        } else if (A.w > (Real)0) {   // W_f,3 bracket r_i <= d < r_{i+1}, i >= 1
            Real u0, u1;
            ie = emission_bracket<Real>(rt, nr, rc_inv, d, u0, u1);
            if ((ek == K_F1 || ek == K_F2) && d >= rt[1] && d < rt[nr - 1])
                two_point_variant(ek, rt, ie, (double)d, u0, u1);
            if (ek == K_F3N && sum > (Real)0)
                n_point_f3(rt, l0, h0, (double)d, (double)h, emode, le, ne, ea, eb);
            if (emode != 1) {
                e0 = A.w * u0;
                e1 = A.w * u1;
            }
        }
    }

    // ---------------- phase 2 ----------------
    const int nrm = a.nr_max;
    const Real inv_s3 = (Real)1 / (Real)(a.subsample * a.subsample * a.subsample);
    // each below 256; bit 24: the node emits (two-point emission weights e0, e1)
    const bool emits = e0 != (Real)0 || e1 != (Real)0;
    const int packed = lo | (nsup << 8) | (ie << 16) | (emits ? 1 << 24 : 0);
    const int epacked = emode | (le << 2) | (ne << 10);   // 2 + 8 + 8 bits
    const bool any_emits = __ballot(emits) != 0ull;
    // the W_p normalisation, or (no support point: linear split) minus the
    // bracket weight of the lower point
    const Real wsf = wscale > (Real)0 ? wscale : -fb0;
    PairStream<CLASSIFY> ps(lane, entry, CLASSIFY ? __ballot(lane < cnt && entry == kNoEntry) : 0ull);
    if (CLASSIFY) tab_count += ps.n_ent;
    // this lane's points i0 .. i0 + npt - 1 of a pair's support (buffer k, weight wk), by the whole wave
    auto add_points = [&](int node, int npk, int k, Real wk, int i0, int npt) {
        const int jlo = (npk & 255) + i0;
        const Real jd = __shfl(d, node, 64), jhinv = __shfl(hinv, node, 64), jwf = __shfl(wsf, node, 64);
        const Real ja = __shfl(qa, node, 64), je = __shfl(qe, node, 64), jv = __shfl(qv, node, 64);
        const int jep = KV ? __shfl(epacked, node, 64) : 0;
        const int jemode = jep & 3, jle = (jep >> 2) & 255, jne = (jep >> 10) & 255;
        Real jea = 0, jeb = 0, jqeps = 0;
        if (KV) {
            jea = __shfl(ea, node, 64);
            jeb = __shfl(eb, node, 64);
            jqeps = __shfl(qeps, node, 64);
        }
        const Real jfb = -jwf;   // the bracket weight when there is no W_p support
        Real *row = R.b + ((int)__umul24(k, R.stride) + R.oa + jlo);
        Real fi = (Real)jlo;
        for (int io = 0; io < npt; ++io, ++row, fi += (Real)1) {
            const Real ws = here(smooth_kernel<Real>(mg, (rcoef * (fi * fi) - jd) * jhinv) * jwf);
            const Real w = jwf > (Real)0 ? ws : (i0 + io == 0 ? jfb : (Real)1 - jfb);
            buf_add3<Real, ATOMIC>(wk, row, w * ja, row + nrm, w * je, row + 2 * nrm, w * jv);
            if (KV && jemode != 0) {   // the emission row
                const Real wq = emission_weight<Real>(jemode, jlo + io, i0 + io, jle, jne, jea, jeb, jfb, rcoef, jd, jhinv,
                                                      a.eps_kernel == K_G) * jqeps;
                if (wq != (Real)0) {
                    buf_add<Real>(&R.eps(k, jlo + io), wk * wq);
                    mark_points(cmask + (size_t)k * ew, jlo + io, true, false);
                }
            }
        }
    };
    // pairs collected so far, lanes below qfill: kc with the node's lane above it (pixel 16 bits, count 7, lane 6)
    int q = 0, qfill = 0;
    for (;;) {
        int node, kc;
        const int got = ps.next(a, n, per, tx, ty, tz, guard_count, node, kc);
        int batch = q, fill = qfill;
        if (got > 0) {
            // keep the pairs on a buffered ray that reach it below its outermost emitting point
            const unsigned ri = lane < got ? rinfo[kc & 0xffff] : 0u;
            const int pk = __shfl(packed, node, 64);
            const bool keep = ri != 0u && ((int)(ri & 255u) >= (pk & 255) || ((pk >> 24) & 1));
            const uint64_t km = __ballot(keep), nm = uniform(~km);
            const int nk = (int)__popcll(km);
            if (nk == 0) continue;
            // the kept ones follow those collected (all lanes take part: a rotation of a partition)
            const int rank_k = bits_below(km), rank_n = nk + bits_below(nm);
            const int moved = __builtin_amdgcn_ds_permute(((qfill + (keep ? rank_k : rank_n)) & 63) << 2, kc | (node << 23));
            batch = lane >= qfill ? moved : q;
            fill = qfill + nk;
            if (fill < 64) {
                q = batch;
                qfill = fill;
                continue;
            }
            q = moved;   // (what wrapped around, lanes below fill - 64)
            qfill = fill - 64;
            fill = 64;
        } else {
            if (fill == 0) break;
            qfill = 0;
        }
        // --- deposit: this lane's pair over its node's support points lo .. lo + npt - 1 ---
        const bool valid = lane < fill;
        node = (batch >> 23) & 63;
        kc = batch & 0x7fffff;
        const int npk = __shfl(packed, node, 64);
        const unsigned ri = valid ? rinfo[kc & 0xffff] : 0u;
        const int npt = valid ? min((npk >> 8) & 255, (int)(ri & 255u) - (npk & 255) + 1) : 0;
        const int k = (int)(ri >> 8);
        const Real wk = (Real)(kc >> 16) * inv_s3;
        if (any_emits) {
            // the pixel's share of the emission on the two bracket points (the spread forms
            // go with A, E, V below)
            const Real je0 = __shfl(e0, node, 64), je1 = __shfl(e1, node, 64);
            if (valid && ((npk >> 24) & 1)) {
                const int jie = (npk >> 16) & 255;
                Real *row = &R.eps(k, jie);
                if (je0 != (Real)0) buf_add<Real>(row, wk * je0);
                if (je1 != (Real)0) buf_add<Real>(row + 1, wk * je1);
                if (KV) mark_points(cmask + (size_t)k * ew, jie, je0 != (Real)0, je1 != (Real)0);
            }
        }
        if constexpr (LDSBUF) {
            add_points(node, npk, k, wk, 0, npt);
        } else {
            int tot;
            const int off = wave_excl_scan_dpp(max(npt, 0), tot);
            for (int b = 0; b < tot; b += 64) {
                // the pair of this lane's point: the last one that starts at or before it
                int src = 0;
#pragma unroll
                for (int h = 32; h > 0; h >>= 1) src = __shfl(off, src + h, 64) <= b + lane ? src + h : src;
                const int pn = __shfl(node, src, 64);
                add_points(pn, __shfl(packed, pn, 64), __shfl(k, src, 64), __shfl(wk, src, 64),
                           b + lane - __shfl(off, src, 64), b + lane < tot ? 1 : 0);
            }
        }
    }
}

// LDS flags of the per-target walk (acquire/release inside the workgroup)
__device__ inline int lds_load(const int *p) { return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP); }

// One node of a walk (Sec. 2.3, 2.4): a node containing the target is opened,
// every other leaf is accepted, other nodes are accepted when
// size^2 < theta^2 d^2 (geometric centre, doubled integer coordinates, the
// product taken in FP64).  Returns 1 accepted, 2 opened, 0 neither (the target
// itself); sh: the shift to the node's periodic copy.
__device__ inline int test_node(const SweepArgs &a, const int *per, const int4 g, bool leaf, int tx, int ty, int tz,
                                int sh[3])
{
    const int sz = g.w & kSizeMask;
    sh[0] = sh[1] = sh[2] = 0;
    const bool inside = (2 * g.x <= tx && tx < 2 * (g.x + sz)) && (2 * g.y <= ty && ty < 2 * (g.y + sz)) &&
                        (2 * g.z <= tz && tz < 2 * (g.z + sz));
    if (inside) return leaf ? 0 : 2;
    int vx = 2 * g.x + sz - tx, vy = 2 * g.y + sz - ty, vz = 2 * g.z + sz - tz;
    if (per) {
        sh[0] = nearest_copy_shift(vx, per[0]);
        sh[1] = nearest_copy_shift(vy, per[1]);
        sh[2] = nearest_copy_shift(vz, per[2]);
        vx += 2 * sh[0];
        vy += 2 * sh[1];
        vz += 2 * sh[2];
    }
    if (leaf) return 1;
    const double ddx = (double)vx, ddy = (double)vy, ddz = (double)vz;
    const double D2 = ddx * ddx + ddy * ddy + ddz * ddz;
    double th2 = a.theta2;   // lowered by the IF and Src MACs (Sec. 2.4)
    if ((g.w & kIfBit) && a.theta_if2 > 0.0) th2 = fmin(th2, a.theta_if2);
    if ((g.w & kSrcBit) && a.theta_src2 > 0.0) th2 = fmin(th2, a.theta_src2);
    return th2 * D2 > 4.0 * (double)sz * (double)sz ? 1 : 2;
}

// Queues work item `item` for the fallback pass; without room (or in that pass
// itself) the target fails: NaN and the overflow flag.  One lane.
__device__ inline void queue_overflow(const SweepArgs &a, bool fallback, int64_t item, int64_t out)
{
    if (!fallback && a.ovf) {
        const int q = atomicAdd(&a.queue[3], 1);
        if (q < a.ovf_cap) {
            a.ovf[q] = (int32_t)item;
            return;
        }
    }
    a.f_out[out] = __longlong_as_double(0x7ff8000000000000ll);
    if (a.ion_out) a.ion_out[out] = 0;
    atomicOr(&a.queue[1], 1);
}

// Breadth-first walks of a chunk's targets, a wave per target: one node per
// lane, ballot and prefix scan to append the accepted nodes to the target's
// list in device memory and the next frontier in LDS.  Each accepted node is
// listed with its (pixel, count) pairs: its entry in the angular table, or its
// sub-points are classified here and the pairs go to the chunk's pool, of
// which a wave takes 256 units of 4 pairs at a time.  A walk is a chain of
// dependent node reads (a level at a time), so it is bound by latency: in a
// kernel of its own many walks hide each other's (4 workgroups of 4 waves per
// compute unit: the frontiers' 32768 B are 33280 in the LDS granule of 1280, so
// a fifth does not fit, and launched it ran alone at the end with its share of
// the targets: sweeps of 128^3 N_side 2 FP32C 112.9 ms with 5 against 106.1 with
// 4, 64^3 N_side 4 10.7 / 10.1, adaptive 72.0 / 67.0), where inside the sweep one target's
// walk held up the others' barrier; and the sweep is rid of the classifier,
// whose FP64 guard costs it registers.
constexpr int kWalkWaves = 4;
__global__ __launch_bounds__(kWalkWaves * 64) void k_walk(SweepArgs a)
{
    __shared__ int front[kWalkWaves][2][kWalkFront];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.queue[0] = 0;   // the sweep of this chunk starts from its first target
    const uint64_t below = (1ull << lane) - 1ull;
    const Lattice L(a.subsample);
    uint64_t n_test = 0, n_acc = 0, n_tab = 0, n_guard = 0;
    int dpos = 0, dend = 0;   // the wave's part of the pool of pairs, in units
    for (int i = (int)blockIdx.x * kWalkWaves + wave; i < a.n_chunk; i += (int)gridDim.x * kWalkWaves) {
        const int64_t item = a.item0 + i;
        const int64_t cell = a.targets ? a.targets[item] : (int64_t)a.order[item];
        TargetRec r{};
        r.out = a.targets ? item : cell;
        if (cell < 0 || cell >= a.n_cells) {
            r.n_emit = -1;
            if (lane == 0) {
                a.f_out[r.out] = __longlong_as_double(0x7ff8000000000000ll);
                if (a.ion_out) a.ion_out[r.out] = 0;
                atomicOr(&a.queue[1], 2);
                a.rec[i] = r;
            }
            continue;
        }
        r.dom = uniform(a.cell_dom[cell]);
        const DomDev &D = a.doms[r.dom];
        const int tnode = uniform(a.cell_node[cell]);
        const int4 tg = a.geo[tnode];
        r.tsize = tg.w & kSizeMask;
        r.tx = 2 * tg.x + r.tsize;
        r.ty = 2 * tg.y + r.tsize;
        r.tz = 2 * tg.z + r.tsize;
        int per_ext[3] = {D.ext[0], D.ext[1], D.ext[2]};
        const int *per = a.periodic ? per_ext : nullptr;
        int2 *const list = a.lists + (size_t)i * a.list_cap;
        uint16_t *const emit_at = a.emit_at + (size_t)i * a.list_cap;
        int *cur = front[wave][0], *nxt = front[wave][1];
        if (lane == 0) cur[0] = D.root;
        int nfr = 1, na = 0, ne = 0;
        uint64_t t_test = 0, t_tab = 0, t_guard = 0;   // (a walk that does not fit is counted by the fallback pass)
        bool ovf = false;
        while (nfr > 0 && !ovf) {
            int nn = 0;
            for (int base = 0; base < nfr; base += 64) {
                const bool valid = base + lane < nfr;
                int n = 0, nch = 0, fc = 0;
                int4 g{};
                int sh[3] = {0, 0, 0};
                unsigned entry = kNoEntry;
                bool acc_it = false;
                if (valid) {
                    n = cur[base + lane];
                    g = a.geo[n];
                    const int2 tp = a.topo[n];
                    const int what = test_node(a, per, g, tp.y == 0, r.tx, r.ty, r.tz, sh);
                    acc_it = what == 1;
                    if (acc_it) entry = table_entry(a, g, sh, r.tx, r.ty, r.tz, r.tsize);
                    nch = what == 2 ? tp.y : 0;
                    fc = tp.x;
                }
                t_test += min(64, nfr - base);
                const uint64_t macc = __ballot(acc_it), me = __ballot(acc_it && (g.w & kSrcBit) != 0);
                int tot = 0;
                const int off = wave_excl_scan_dpp(nch, tot);
                const int ca = (int)__popcll(macc);
                if (na + ca > a.list_cap || nn + tot > kWalkFront) {
                    ovf = true;
                    break;
                }
                // the nodes without a table entry, one by one
                uint64_t todo = __ballot(acc_it && entry == kNoEntry);
                t_tab += ca - (int)__popcll(todo);
                while (todo) {
                    const int j = __ffsll((unsigned long long)todo) - 1;
                    todo &= todo - 1;
                    const int4 jg{rdlane(g.x, j), rdlane(g.y, j), rdlane(g.z, j), rdlane(g.w, j)};
                    const int jsh[3] = {rdlane(sh[0], j), rdlane(sh[1], j), rdlane(sh[2], j)};
                    int kc = 0;
                    const int nd = classify_box(L, a.nside, a.npix, a.guard_tol,
                                                node_box(a, rdlane(n, j), jg, jsh, r.tx, r.ty, r.tz), r.tx, r.ty, r.tz,
                                                &a.queue[1], t_guard, kc);
                    const int need = (nd + 3) >> 2;
                    if (dpos + need > dend) {
                        int q = 0;
                        if (lane == 0) q = atomicAdd(&a.queue[4], kDynBlock);
                        dpos = uniform(q);
                        dend = dpos + kDynBlock;
                        if (dpos < 0 || dend > a.dyn_units) {   // the pool is used up: the fallback pass
                            dpos = dend = 0;
                            ovf = true;
                            break;
                        }
                    }
                    if (lane < nd) a.dyn_pool[(size_t)dpos * 4 + lane] = kc;
                    if (lane == j) entry = kDynEntry | (unsigned)dpos << 6 | (unsigned)(nd - 1);
                    dpos += need;
                }
                if (ovf) break;
                if (acc_it) {
                    const int at = na + (int)__popcll(macc & below);
                    list[at] = int2{n, (int)entry};
                    if (g.w & kSrcBit) emit_at[ne + (int)__popcll(me & below)] = (uint16_t)at;
                }
                for (int c = 0; c < nch; ++c) nxt[nn + off + c] = fc + c;
                na += ca;
                ne += (int)__popcll(me);
                nn += tot;
            }
            int *t = cur;
            cur = nxt;
            nxt = t;
            nfr = nn;
        }
        r.n_acc = na;
        r.n_emit = ovf ? -1 : ne;
        if (!ovf) {
            n_acc += na;
            n_test += t_test;
            n_tab += t_tab;
            n_guard += t_guard;
        }
        if (lane == 0) {
            if (a.f32) {
                const float4 A = ((const float4 *)a.pA)[tnode], B = ((const float4 *)a.pB)[tnode];
                r.eps = A.w; r.alpha = B.x; r.e = B.y; r.v = B.z;
            } else {
                const double4 A = ((const double4 *)a.pA)[tnode], B = ((const double4 *)a.pB)[tnode];
                r.eps = A.w; r.alpha = B.x; r.e = B.y; r.v = B.z;
            }
            a.rec[i] = r;
            if (ovf) queue_overflow(a, false, item, r.out);
        }
    }
    if (lane == 0) {
        if (n_acc > 0) atomicAdd(&a.stats[0], (unsigned long long)n_acc);
        if (n_test > 0) atomicAdd(&a.stats[1], (unsigned long long)n_test);
        if (n_guard > 0) atomicAdd(&a.stats[2], (unsigned long long)n_guard);
        if (n_tab > 0) atomicAdd(&a.stats[5], (unsigned long long)n_tab);
    }
}

// Bytes of a workgroup's marks and ray numbers in device memory: the
// masks of all rays, of the rays with a buffer (in LDS when the buffers are), and the rays' buffers
__host__ __device__ inline size_t mask_slab_bytes(int npix, int rays, int ew, bool ldsbuf)
{
    return (((size_t)npix + (ldsbuf ? 0 : rays)) * 8 * ew + (size_t)npix * 4 + 255) / 256 * 256;
}

// LDS words of a sweep workgroup: its next work item, and (fallback pass) the
// shared walk's meetings, the next frontier's length (three by level), the
// accepted count, an overflow
enum { S_NEXT = 0, S_PMEET, S_PNEXT, S_PACC = S_PNEXT + 3, S_POVF, S_COUNT = 16 };

// Waits until this wave's device-memory stores have completed (vmcnt 0), so
// that an LDS flag written next publishes them to the workgroup's other waves
// (a workgroup-scope release does not wait for them).
__device__ inline void wait_stores() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// The walk of one target by the K waves of a workgroup, with its lists in
// device memory (fallback pass): the batches of 64 nodes of a level go round
// the waves, their appends to the next frontier and to the accepted list are
// reserved by LDS atomics, and the waves meet at an LDS counter after every
// level (all leave the loop at the same level).  The S_P words are zero and
// cur[0] = root before any starts.  Returns the accepted count (the same on
// every wave), or -1 after an overflow.
template <int K>
__device__ int walk_shared(const SweepArgs &a, int wave, const int *per, int tx, int ty, int tz, int *fr0, int *fr1,
                           int *acc, int *sc, int fmax, int amax, uint64_t &n_test)
{
    const int lane = lane_id();
    int *cur = fr0, *nxt = fr1;
    int nfr = 1;
    for (int lev = 0;; ++lev) {
        int *const next_count = &sc[S_PNEXT + lev % 3];
        // the counter of the level after next is free (read before the last meeting)
        if (wave == 0 && lane == 0) sc[S_PNEXT + (lev + 1) % 3] = 0;
        for (int base = 64 * wave; base < nfr; base += 64 * K) {
            const bool valid = base + lane < nfr;
            int n = 0, nch = 0, fc = 0;
            bool acc_it = false;
            if (valid) {
                n = cur[base + lane];
                const int2 tp = a.topo[n];
                int sh[3];
                const int what = test_node(a, per, a.geo[n], tp.y == 0, tx, ty, tz, sh);
                acc_it = what == 1;
                nch = what == 2 ? tp.y : 0;
                fc = tp.x;
            }
            n_test += min(64, nfr - base);
            const uint64_t macc = __ballot(acc_it);
            const int cacc = (int)__popcll(macc);
            int tot = 0;
            const int off = wave_excl_scan_dpp(nch, tot);
            int oa = 0, on = 0;
            if (lane == 0) {
                oa = cacc ? atomicAdd(&sc[S_PACC], cacc) : 0;
                on = tot ? atomicAdd(next_count, tot) : 0;
            }
            oa = __shfl(oa, 0, 64);
            on = __shfl(on, 0, 64);
            if (oa + cacc > amax || on + tot > fmax) {
                // nothing is written; all waves stop after this level's meeting
                if (lane == 0) sc[S_POVF] = lev + 1;
                continue;
            }
            if (acc_it) acc[oa + (int)__popcll(macc & ((1ull << lane) - 1ull))] = n;
            for (int c = 0; c < nch; ++c) nxt[on + off + c] = fc + c;
        }
        // meet the other waves: the level's appends are all written
        wait_stores();
        if (lane == 0) atomicAdd(&sc[S_PMEET], 1);
        while (lds_load(&sc[S_PMEET]) < K * (lev + 1)) __builtin_amdgcn_s_sleep(1);
        nfr = uniform(lds_load(next_count));
        // (an overflow of another wave's next level is not this level's)
        const int ov = uniform(lds_load(&sc[S_POVF]));
        if (ov != 0 && ov <= lev + 1) return -1;
        if (nfr == 0) return uniform(lds_load(&sc[S_PACC]));
        int *t = cur;
        cur = nxt;
        nxt = t;
    }
}

// One target as the sweep holds it (the same on every lane).
struct Target {
    int dom, tsize, tx, ty, tz, na, ne;   // accepted nodes and, of them, those that emit (< 0: nothing to map)
    int64_t o, list;                      // output index, first place in the lists
};

// The sweep of one launch over the listed targets of a chunk.  FALLBACK: the
// second pass over the items whose walks did not fit in the lists, walked here
// by the whole workgroup with lists in device memory.  WIDE: the marks and
// numbers of all rays in device memory, wherever the ray buffers are: 12 to 20
// bytes a ray, which from N_side 32 on (12288 rays) leave LDS no room for buffers
// or do not fit at all.
template <typename Real, int WAVES, bool LDSBUF, bool FALLBACK, bool KV, bool CAS = false, bool WIDE = false>
__device__ __forceinline__ void sweep_body(const SweepArgs &a)
{
    using R4 = typename R4T<Real>::T;
    constexpr int ATOMIC = CAS ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar loops over waves' work
    const int nrm = a.nr_max, npix = a.npix, rays = a.rays;
    const int ew = uniform(1 + (nrm > 64));   // words of a ray's mask of emitting points (1 or 2)
    const size_t buf_elems = (size_t)rays * a.stride_k;
    char *p = smem;
    unsigned long long *emask;   // the masks of all rays, marked before the mapping
    unsigned long long *cmask;   // those of the rays with a buffer
    unsigned *rinfo;             // per ray: its buffer << 8 | its outermost emitting point, 0: no buffer
    if constexpr (WIDE) {
        emask = (unsigned long long *)(a.mbuf + (size_t)blockIdx.x * (size_t)a.mbuf_stride);
        rinfo = (unsigned *)(emask + ((size_t)npix + (LDSBUF ? 0 : rays)) * ew);
    } else {
        emask = (unsigned long long *)p;
        p += (size_t)npix * ew * 8;
    }
    if constexpr (WIDE && !LDSBUF) {
        cmask = emask + (size_t)npix * ew;
    } else {
        cmask = (unsigned long long *)p;
        p += (size_t)rays * ew * 8;
    }
    Real *buf;
    if constexpr (LDSBUF) {
        buf = (Real *)p;
        p += ((buf_elems * sizeof(Real) + 15) / 16) * 16;
    } else {
        buf = (Real *)a.gbuf + (size_t)blockIdx.x * buf_elems;
    }
    // split: three rows (A, E, V) per ray in buf, the emission rows in device memory
    const bool split = LDSBUF && a.split != 0;
    Real *const eplane = split ? (Real *)a.ebuf + (size_t)blockIdx.x * rays * nrm : buf;
    const RayRows<Real> R{buf, eplane, a.stride_k, split ? nrm : a.stride_k, split ? 0 : nrm, nrm};
    Real *rt = (Real *)p;
    p += ((nrm * sizeof(Real) + 15) / 16) * 16;
    Real *wself = (Real *)p;
    p += ((nrm * sizeof(Real) + 15) / 16) * 16;
    double *rd = (double *)p;   // the evaluation points in FP64 for the integration
    p += nrm * sizeof(double);
    double *rd2 = (double *)p;  // 1 / (2 r_i)
    p += nrm * sizeof(double);
    double *red = (double *)p;
    p += WAVES * sizeof(double);
    int *sc = (int *)p;
    p += S_COUNT * sizeof(int);
    if constexpr (!WIDE) rinfo = (unsigned *)p;
    int *fr0 = nullptr;   // fallback: frontiers of gfmax entries, then gamax accepted nodes
    if (FALLBACK) fr0 = a.glist + (size_t)blockIdx.x * (2 * (size_t)a.gfmax + a.gamax);

    uint64_t n_acc = 0, n_test = 0, n_guard = 0, n_f32 = 0, n_f64 = 0, n_tab = 0, n_re = 0;   // (uniform)
    const int64_t n_items =
        FALLBACK ? min((int64_t)__hip_atomic_load(&a.queue[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), a.ovf_cap)
                 : a.n_chunk;
    int32_t *const next_item = &a.queue[FALLBACK ? 2 : 0];
    // the claim of the next item, by one thread after everyone has read the last one
    auto claim = [&]() {
        if (threadIdx.x == 0) sc[S_NEXT] = atomicAdd(next_item, 1);
    };
    claim();
    if (!FALLBACK && blockIdx.x == 0 && tid == 0) a.queue[4] = 0;   // the next chunk's walks start an empty pool of pairs
    for (int e = tid; e < npix * ew; e += WAVES * 64) emask[e] = 0ull;
    __syncthreads();
    int cached_dom = -1, cached_tsize = -1;   // whose radial tables the LDS holds
    Target t{};
    Real teps = 0;
    double flux_unit = 0, ftarget = 0;   // ftarget: this lane's share of the target's flux
    bool have = false;
    // One round: the emission marks of the next target (beside the last waves'
    // integration of the current one), the current one's flux, then the next
    // one's buffers, mapping and integration.
    for (;;) {
        // (the lane's number anew in each part: what is derived from it is not held in registers
        // through the others, where 80 a lane let 6 waves share a SIMD)
        const int tid = here((int)threadIdx.x), lane = tid & 63;
        const int64_t item = uniform(sc[S_NEXT]);   // the same on every lane: scalar loads below
        const bool more = item < n_items;
        Target x{};
        x.ne = -1;
        if (more) {
            if (!FALLBACK) {
                const TargetRec &r = a.rec[item];
                x.dom = uniform(r.dom);
                x.tsize = uniform(r.tsize);
                x.tx = uniform(r.tx);
                x.ty = uniform(r.ty);
                x.tz = uniform(r.tz);
                x.na = uniform(r.n_acc);
                x.ne = uniform(r.n_emit);
                x.o = r.out;
                x.list = item * a.list_cap;
            } else {
                const int64_t it = a.ovf[item];   // (its cell index was checked when it was queued)
                const int64_t cell = a.targets ? a.targets[it] : (int64_t)a.order[it];
                x.o = a.targets ? it : cell;
                x.dom = uniform(a.cell_dom[cell]);
                const int4 tg = a.geo[uniform(a.cell_node[cell])];
                x.tsize = tg.w & kSizeMask;
                x.tx = 2 * tg.x + x.tsize;
                x.ty = 2 * tg.y + x.tsize;
                x.tz = 2 * tg.z + x.tsize;
                // the walk, by all waves
                __syncthreads();
                if (tid == 0) {
                    for (int q = S_PMEET; q <= S_POVF; ++q) sc[q] = 0;
                    fr0[0] = a.doms[x.dom].root;
                }
                wait_stores();
                __syncthreads();
                int *const acc = fr0 + 2 * (size_t)a.gfmax;
                x.na = walk_shared<WAVES>(a, wave, a.periodic ? a.doms[x.dom].ext : nullptr, x.tx, x.ty, x.tz, fr0,
                                          fr0 + a.gfmax, acc, sc, a.gfmax, a.gamax, n_test);
                x.ne = x.na;   // (any of them may emit)
                n_acc += wave == 0 && x.na > 0 ? x.na : 0;
            }
            if (!KV) {
                // the points that will hold emission, by the waves from the last on (the first
                // are the last to leave the integration); at least 16 nodes on a wave
                const DomDev &D = a.doms[x.dom];
                const int share = min(64, max(16, (x.ne + WAVES - 1) / WAVES));
                const Real *rtg;
                if constexpr (sizeof(Real) == 4) rtg = a.r32 + D.r_off;
                else rtg = a.r64 + D.r_off;
                for (int e0 = (WAVES - 1 - wave) * share; e0 < x.ne; e0 += WAVES * share) {
                    const int cnt = min(share, x.ne - e0);
                    int2 v{0, (int)kNoEntry};
                    if (lane < cnt) {
                        if (FALLBACK) v.x = fr0[2 * (size_t)a.gfmax + e0 + lane];
                        else v = a.lists[x.list + a.emit_at[x.list + e0 + lane]];
                    }
                    mark_nodes<Real, FALLBACK>(a, emask, ew, a.periodic ? D.ext : nullptr, rtg, D.nr, (Real)D.rc_inv, v.x,
                                               (unsigned)v.y, cnt, x.tx, x.ty, x.tz, x.tsize);
                }
            }
        }
        if (have) {
            const double f = wave_sum(ftarget);
            if (lane == 0) red[wave] = f;
        }
        __syncthreads();
        if (have && tid == 0) {
            double f = 0.0;
            for (int w = 0; w < WAVES; ++w) f += red[w];
            const double rtp = 0.5 * (double)t.tsize;
            f += 3.0 * (double)teps / (4.0 * kPi * rtp * rtp);
            a.f_out[t.o] = f * flux_unit;
            if (a.ion_out) a.ion_out[t.o] = f > 0.0 ? 1 : 0;
        }
        if (!more) break;
        t = x;
        have = t.ne >= 0;
        ftarget = 0.0;
        if (!have) {   // a bad index, or a walk that did not fit
            if (FALLBACK && tid == 0) queue_overflow(a, true, item, t.o);
            claim();   // (everyone has read the last one)
            __syncthreads();
            continue;
        }
        const DomDev &D = a.doms[t.dom];
        const int nr = D.nr;
        const int *per = a.periodic ? D.ext : nullptr;
        const Real rc_inv = (Real)D.rc_inv;
        const Real rcoef = (Real)(1.0 / D.rc_inv);
        flux_unit = D.flux_unit;
        Real talpha, te, tv;
        if (!FALLBACK) {
            const TargetRec &r = a.rec[item];
            teps = (Real)r.eps;
            talpha = (Real)r.alpha;
            te = (Real)r.e;
            tv = (Real)r.v;
        } else {
            const int64_t it = a.ovf[item];
            const int tnode = uniform(a.cell_node[a.targets ? a.targets[it] : (int64_t)a.order[it]]);
            const R4 tA = ((const R4 *)a.pA)[tnode], tB = ((const R4 *)a.pB)[tnode];
            teps = tA.w;
            talpha = tB.x;
            te = tB.y;
            tv = tB.z;
        }

        // evaluation points and the self-term weights (W_p at d = 0, h = cell size):
        // kept in LDS while consecutive targets share the domain and cell size
        if (t.dom != cached_dom) {
            for (int i = tid; i < nr; i += WAVES * 64) {
                const double rv = a.r64[D.r_off + i];
                rd[i] = rv;
                rd2[i] = i > 0 ? 1.0 / (2.0 * rv) : 0.0;
                if constexpr (sizeof(Real) == 4) rt[i] = a.r32[D.r_off + i];
                else rt[i] = (Real)rv;
            }
            __syncthreads();
        }
        if (t.dom != cached_dom || t.tsize != cached_tsize) {
            if (wave == 0) {
                Real w0 = 0, w1 = 0;
                if (lane < nr) w0 = smooth_kernel<Real>(KV && a.mass_gauss != 0, rt[lane] / (Real)t.tsize);
                if (lane + 64 < nr) w1 = smooth_kernel<Real>(KV && a.mass_gauss != 0, rt[lane + 64] / (Real)t.tsize);
                const Real sum = wave_sum(w0 + w1);
                if (lane < nr) wself[lane] = w0 / sum;
                if (lane + 64 < nr) wself[lane + 64] = w1 / sum;
            }
            __syncthreads();
            cached_dom = t.dom;
            cached_tsize = t.tsize;
        }
        // The rays with emission (KV: all rays), as many at a time as there are buffers
        for (int r0 = 0;; r0 += rays) {
            const int tid = here((int)threadIdx.x), lane = tid & 63;
            // every wave numbers them (the same values); those of this pass get a buffer and a copy of their
            // mask (in device memory one wave writes each)
            int ns = 0;
            for (int base = 0; base < npix; base += 64) {
                const int k = base + lane;
                unsigned long long m0 = 0ull, m1 = 0ull;
                if (!KV && k < npix) {
                    m0 = emask[(size_t)k * ew];
                    if (ew > 1) m1 = emask[(size_t)k * ew + 1];
                }
                const int top = KV ? (k < npix ? nr - 1 : 0) : mask_top(m0, m1);
                const uint64_t on = __ballot(top > 0);
                const int i = ns + bits_below(on) - r0;
                ns += (int)__popcll(on);
                if (WIDE && (base >> 6) % WAVES != wave) continue;
                const bool mine = top > 0 && i >= 0 && i < rays;
                if (k < npix) rinfo[k] = mine ? (unsigned)(i << 8 | top) : 0u;
                if (mine) {
                    cmask[(size_t)i * ew] = m0;
                    if (ew > 1) cmask[(size_t)i * ew + 1] = m1;
                }
            }
            const int np = min(rays, ns - r0);
            const bool last = r0 + rays >= ns;
            // their buffers: zero emission, the target's own share of A, E, V, the same on every
            // ray (point lane, and lane + 64, of each row)
            {
                const Real inv_npix = (Real)1 / (Real)npix;
                const Real w0 = lane < nr ? wself[lane] * inv_npix : (Real)0;
                const Real w1 = lane + 64 < nr ? wself[lane + 64] * inv_npix : (Real)0;
                for (int k = wave; k < np; k += WAVES) {
                    Real *dst = buf + (size_t)k * a.stride_k + lane;
                    if (!split) {
                        if (lane < nrm) dst[0] = (Real)0;
                        if (lane + 64 < nrm) dst[64] = (Real)0;
                        dst += nrm;
                    }
                    if (lane < nrm) {
                        dst[0] = talpha * w0;
                        dst[nrm] = te * w0;
                        dst[2 * nrm] = tv * w0;
                    }
                    if (lane + 64 < nrm) {
                        dst[64] = talpha * w1;
                        dst[nrm + 64] = te * w1;
                        dst[2 * nrm + 64] = tv * w1;
                    }
                }
                // (the emission plane of split buffers is zero here: cleared when
                // allocated and, entry by entry, by the march that reads it)
            }
            __syncthreads();
            if (r0 == 0) claim();   // (visible to all after the mapping)
            // the next target's marks start from zero
            if (last)
                for (int e = tid; e < npix * ew; e += WAVES * 64) emask[e] = 0ull;

            // --- the waves map 64 nodes each at a time, from 64 WAVES consecutive ones of the walk
            // every WAVES-th: the nodes come level by level, so a wave's have supports of
            // similar length, but not side by side, where siblings would meet on the same
            // rays' points (3.3 lanes on one point at N_side 2 against 2.2).  Every nc-th node
            // of the whole walk on a wave met less (1.6) but made the loops over the support as
            // long as the largest node's: 128^3 N_side 2 149.5 against 143.2 ms, 64^3 N_side 4
            // 14.2 against 13.5 ms ---
            if (np > 0) {
                const int lane = here(lane_id());
                uint64_t p_guard = 0, p_tab = 0;
                for (int c = wave; c < t.na; c += 64 * WAVES) {
                    const int cnt = min(64, (t.na - c + WAVES - 1) / WAVES);
                    int2 v{0, (int)kNoEntry};
                    if (lane < cnt) {
                        if (FALLBACK) v.x = fr0[2 * (size_t)a.gfmax + c + WAVES * lane];
                        else v = a.lists[t.list + c + WAVES * lane];
                    }
                    map_nodes<Real, ATOMIC, LDSBUF, KV, FALLBACK>(a, R, rinfo, cmask, ew, per, rt, nr, rc_inv, rcoef, v.x,
                                                          (unsigned)v.y, cnt, t.tx, t.ty, t.tz, t.tsize, p_guard, p_tab);
                }
                if (r0 == 0) {   // (the same nodes in every pass)
                    n_guard += p_guard;
                    n_tab += p_tab;
                }
            }
            __syncthreads();

            // --- per-ray integration and the sum over rays (KV: rays without emission give 0) ---
            constexpr int IW = WAVES;
            double fsum = 0.0;
            float cs_hi = 0.0f, cs_lo = 0.0f;   // compensated FP32 sum of this lane's FP32-marched rays
            if (a.int_group > 0) {
                // Every emitting ray gets a group of lanes sized by its number of
                // emitting points: a power of two from the launch's group up to 64
                // (its class), more than 64 points a wave (class 7).  Rays of one
                // class share a batch of 64 / g rays of g lanes; the batches, widest
                // class first and pixel order within a class, are dealt round robin
                // over the waves.
                const int lane = here(lane_id());
                const int lg0 = 31 - __clz(a.int_group);
                int nb[6];   // batches of classes 2 .. 7 (class 7: a ray each)
                {
                    int n[6] = {0, 0, 0, 0, 0, 0};
                    for (int base = 0; base < np; base += 64) {
                        int tp;
                        const int c = ray_class(cmask, ew, np, lg0, base + lane, tp);
#pragma unroll
                        for (int q = 0; q < 6; ++q) n[q] += (int)__popcll(__ballot(c == q + 2));
                    }
                    int re = 0;
#pragma unroll
                    for (int q = 0; q < 6; ++q) {
                        nb[q] = q == 5 ? n[q] : (n[q] + (64 >> (q + 2)) - 1) >> (4 - q);
                        if (q + 2 > lg0) re += n[q];
                    }
                    n_re += wave == 0 ? re : 0;
                }
                const int n_batch = nb[0] + nb[1] + nb[2] + nb[3] + nb[4] + nb[5];
                for (int b = wave; b < n_batch; b += IW) {
                    int cls = -1, bi = b;
#pragma unroll
                    for (int q = 5; q >= 0; --q)
                        if (cls < 0) {
                            if (bi < nb[q]) cls = q + 2;
                            else bi -= nb[q];
                        }
                    const int ng = cls == 7 ? 1 : 64 >> cls;
                    // this lane's ray: the (bi ng + lane / g)-th of the class
                    const int want = bi * ng + (cls == 7 ? 0 : lane >> cls);
                    int myk = -1, mytp = 0, run = 0;
                    for (int base = 0; base < np && run < bi * ng + ng; base += 64) {
                        int tp;
                        const int c = ray_class(cmask, ew, np, lg0, base + lane, tp);
                        const uint64_t m = __ballot(c == cls);
                        const int n = (int)__popcll(m), w = want - run;
                        const bool mine = w >= 0 && w < n;
                        const int pos = mine ? nth_set_bit(m, w) : 0;
                        const int tv = __shfl(tp, pos, 64);
                        if (mine) {
                            myk = base + pos;
                            mytp = tv;
                        }
                        run += n;
                    }
                    if (cls == 7) {
                        const double fw = integrate_ray_wave<Real, 2>(R, myk, rd, rd2, nr, mytp, a.nside, a.zeta_g, split);
                        if (lane == 0) fsum += fw;
                        continue;
                    }
                    // the ray's mask, for its group's lanes to find their emitting points
                    unsigned long long m0 = 0ull, m1 = 0ull;
                    if (myk >= 0) {
                        m0 = cmask[(size_t)myk * ew];
                        if (ew > 1) m1 = cmask[(size_t)myk * ew + 1];
                    }
                    switch (cls) {
                        case 2: march_batch<Real, 4>(a, R, myk, m0, m1, rcoef, rd, rd2, nr, split, fsum, cs_hi, cs_lo, n_f32, n_f64); break;
                        case 3: march_batch<Real, 8>(a, R, myk, m0, m1, rcoef, rd, rd2, nr, split, fsum, cs_hi, cs_lo, n_f32, n_f64); break;
                        case 4: march_batch<Real, 16>(a, R, myk, m0, m1, rcoef, rd, rd2, nr, split, fsum, cs_hi, cs_lo, n_f32, n_f64); break;
                        case 5: march_batch<Real, 32>(a, R, myk, m0, m1, rcoef, rd, rd2, nr, split, fsum, cs_hi, cs_lo, n_f32, n_f64); break;
                        default: march_batch<Real, 64>(a, R, myk, m0, m1, rcoef, rd, rd2, nr, split, fsum, cs_hi, cs_lo, n_f32, n_f64); break;
                    }
                }
            } else if (a.int_wave) {
                // a wave per ray, the emitting rays dealt round robin over the waves
                int seen = 0;
                for (int base = 0; base < np; base += 64) {
                    int t = 0;
                    if (base + lane < np)
                        t = mask_top(cmask[(size_t)(base + lane) * ew], ew > 1 ? cmask[(size_t)(base + lane) * ew + 1] : 0ull);
                    uint64_t m = __ballot(t > 0);
                    while (m) {
                        const int l = __ffsll((unsigned long long)m) - 1;
                        m &= m - 1;
                        if (seen % IW == wave) {
                            const int tk = __builtin_amdgcn_readlane(t, l);
                            const double f =
                                nr > 64 ? integrate_ray_wave<Real, 2>(R, base + l, rd, rd2, nr, tk, a.nside, a.zeta_g, split)
                                        : integrate_ray_wave<Real, 1>(R, base + l, rd, rd2, nr, tk, a.nside, a.zeta_g, split);
                            if (lane == 0) fsum += f;
                        }
                        ++seen;
                    }
                }
            } else {
                // a lane per ray: ray k on lane k % 64 of wave (k / 64) % IW
                for (int k = wave * 64 + lane; k < np; k += 64 * IW) {
                    const int t = mask_top(cmask[(size_t)k * ew], ew > 1 ? cmask[(size_t)k * ew + 1] : 0ull);
                    if (t > 0) fsum += integrate_ray<Real>(R, k, rd, rd2, nr, t, a.nside, a.zeta_g, split);
                }
            }
            ftarget += fsum + ((double)cs_hi + (double)cs_lo);
            if (last) break;
            __syncthreads();   // the next pass takes the buffers
        }
    }
    // statistics
    if (lane == 0) {
        if (n_acc > 0) atomicAdd(&a.stats[0], (unsigned long long)n_acc);
        if (n_test > 0) atomicAdd(&a.stats[1], (unsigned long long)n_test);
        if (n_guard > 0) atomicAdd(&a.stats[2], (unsigned long long)n_guard);
        if (n_f32 > 0) atomicAdd(&a.stats[3], (unsigned long long)n_f32);
        if (n_f64 > 0) atomicAdd(&a.stats[4], (unsigned long long)n_f64);
        if (n_tab > 0) atomicAdd(&a.stats[5], (unsigned long long)n_tab);
        if (n_re > 0) atomicAdd(&a.stats[6], (unsigned long long)n_re);
    }
}

template <typename Real, int WAVES, bool LDSBUF>
__global__ __launch_bounds__(WAVES * 64, 4) void k_sweep(SweepArgs a)
{
    sweep_body<Real, WAVES, LDSBUF, false, false>(a);
}

template <typename Real, int WAVES, bool LDSBUF>
__global__ __launch_bounds__(WAVES * 64, 4) void k_sweep_fallback(SweepArgs a)
{
    sweep_body<Real, WAVES, LDSBUF, true, false>(a);
}

// the same with the radial-kernel variants (fewer launch shapes)
template <typename Real, int WAVES, bool LDSBUF>
__global__ __launch_bounds__(WAVES * 64, 4) void k_sweep_kv(SweepArgs a)
{
    sweep_body<Real, WAVES, LDSBUF, false, true>(a);
}

template <typename Real, int WAVES, bool LDSBUF>
__global__ __launch_bounds__(WAVES * 64, 4) void k_sweep_kv_fallback(SweepArgs a)
{
    sweep_body<Real, WAVES, LDSBUF, true, true>(a);
}

// FP32 ray buffers in LDS accumulated by compare-and-swap (4, 8 and 16 waves).
// With 4 waves per target 6 targets are resident: 6 waves per SIMD in 80
// registers (44 spilled, outside the inner loops) are faster than 4 without
// spills (120 against 134 ms on 128^3 at N_side 2): between its barriers a
// target's waves wait for memory and LDS, and only other targets fill that.
// With 8 waves 80 registers bring 3 targets instead of 2, but cost as much (93
// against 91 ms on the adaptive grid at N_side 4).
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64, WAVES == 4 ? 6 : 4) void k_sweep_cas(SweepArgs a)
{
    sweep_body<float, WAVES, true, false, false, true>(a);
}

template <int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_sweep_cas_fallback(SweepArgs a)
{
    sweep_body<float, WAVES, true, true, false, true>(a);
}

// Ray buffers in LDS, marks and ray numbers in device memory (4, 8 and 16
// waves; FP32 buffers by compare-and-swap).  Bound as k_sweep is, by the mapping;
// the marks (a few atomics and 12 to 20 B a ray and target) stay in L2.  1000 targets
// of 24^3, 4 sources: N_side 32 with 48 points FP32C 0.70 ms, FP64 1.47 ms (44.4 and
// 89.9 with passes over fixed pixel ranges, marks in LDS), 300 targets at N_side 64 0.90
// and 1.97 ms (84.5 and 171).
template <typename Real, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_sweep_wide(SweepArgs a)
{
    sweep_body<Real, WAVES, true, false, false, sizeof(Real) == 4, true>(a);
}

template <typename Real, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_sweep_wide_fallback(SweepArgs a)
{
    sweep_body<Real, WAVES, true, true, false, sizeof(Real) == 4, true>(a);
}

// both in device memory (8 waves): bound by the adds to L2.  The same at N_side 32, W_p
// emission (every ray has a buffer): FP32C 9.0 ms, FP64 13.3 ms.
template <typename Real, bool KV>
__global__ __launch_bounds__(512, 4) void k_sweep_wide_mem(SweepArgs a)
{
    sweep_body<Real, 8, false, false, KV, false, true>(a);
}

template <typename Real, bool KV>
__global__ __launch_bounds__(512, 4) void k_sweep_wide_mem_fallback(SweepArgs a)
{
    sweep_body<Real, 8, false, true, KV, false, true>(a);
}

// ---------------------------------------------------------------------------
// Angular-weight table (Sec. 2.3 "Mapping nodes onto rays").  A node's
// angular weights depend only on its box relative to the target; for nodes of
// 1, 2, 4, ... times the target's size they are tabulated once per context by
// offset, in units of the target's size, with the classifier the sweep itself
// uses: relative sub-point positions scale exactly with the size, so a table
// entry holds exactly what the sweep would compute for that node.  A wave
// takes a contiguous run of offsets: first (idx NULL) it counts their pairs (in
// units of 4), then, with the runs' first units known, it writes them.  A wave
// per offset classifies in FP32 with the FP64 guard band: 1.2 ms for 4.8
// million offsets where a thread per offset in FP64 took 1 ms for 0.6 million.
// For the larger nodes only the offsets where the walk accepts one are filled:
// not so near that it opens them, nor so far that it has accepted their parent.
// A larger leaf cell may be nearer, or the parent's angle smaller; such nodes
// are classified by the walk.
// ---------------------------------------------------------------------------
struct AtabGeom {
    int32_t w[kAtabRatios], base[kAtabRatios], nkeys;
    double near2, far2;   // from kAtabShell on: squared distances of the centre, in node sizes, inside which the
                          // walk opens a node and beyond which it has accepted its parent
};

__global__ __launch_bounds__(256) void k_atab(AtabGeom G, int ns, int s, float guard_tol, int run, int64_t *__restrict__ sums,
                                              int32_t *__restrict__ idx, int32_t *__restrict__ pool, int32_t *flag)
{
    const int wave = uniform((int)(blockIdx.x * 4 + (threadIdx.x >> 6))), lane = lane_id();
    const Lattice L(s);
    const float inv_s = 1.0f / (float)s;
    int64_t at = idx ? sums[wave] : 0;
    uint64_t guard = 0;
    const int end = min((wave + 1) * run, G.nkeys);
    for (int k0 = wave * run; k0 < end; k0 += 64) {
        // 64 offsets, one a lane
        const int key = k0 + lane;
        int ri = 0, w = G.w[0], k = key - G.base[0];
#pragma unroll
        for (int q = 1; q < kAtabRatios; ++q)
            if (G.w[q] >= 0 && key >= G.base[q]) {
                ri = q;
                w = G.w[q];
                k = key - G.base[q];
            }
        const int n = 2 * w + 1;
        const int oz = k % n - w, oy = (k / n) % n - w, ox = k / (n * n) - w;
        bool want = key < end;
        if (want && ri >= kAtabShell) {
            // twice the centre's offset from the target's, in target sizes
            const double cx = 2 * ox + (1 << ri) - 1, cy = 2 * oy + (1 << ri) - 1, cz = 2 * oz + (1 << ri) - 1;
            const double d2 = (cx * cx + cy * cy + cz * cz) / (double)(4 << (2 * ri));
            want = d2 >= G.near2 && d2 <= G.far2;
        }
        unsigned entry = kNoEntry;
        for (uint64_t todo = __ballot(want); todo; todo &= todo - 1) {
            const int j = __ffsll((unsigned long long)todo) - 1;
            const int jr = rdlane(ri, j);
            Box box;
            box.b[0] = rdlane(ox, j);
            box.b[1] = rdlane(oy, j);
            box.b[2] = rdlane(oz, j);
            for (int q = 0; q < 3; ++q) {
                box.e[q] = 1 << jr;
                // a unit target with its lower corner at the origin: twice its centre is (1, 1, 1)
                box.o[q] = 0.5f * (float)(2 * box.b[q] - 1);
                box.step[q] = (float)(1 << jr) * inv_s;
            }
            int kc = 0;
            const int nd = classify_box(L, ns, 12 * ns * ns, guard_tol, box, 1, 1, 1, flag, guard, kc);
            if (idx) {
                if (lane < nd) pool[at * 4 + lane] = kc;
                if (lane == j) entry = (unsigned)at << 6 | (unsigned)(nd - 1);
            }
            at += (nd + 3) >> 2;
        }
        if (idx && key < end) idx[key] = (int32_t)entry;
    }
    if (!idx && lane == 0) sums[wave] = at;
}

// ---------------------------------------------------------------------------
// a9. delta_cell per domain.  The median is the lower median of the domain's
// previous flux, found exactly by a radix select over the IEEE bit patterns
// (non-negative doubles order like their bits), 11 bits at a time: a pass
// reads every cell once, so the six passes and the final one are bound by
// memory (8M cells: 64 MB a pass, which stay in the last-level cache).  A
// block takes a contiguous run of cells, so it looks a domain up once and not
// for every cell, and counts in LDS, in four copies of the histogram (the top
// bits of neighbouring values are mostly equal, and lanes that meet on a bin
// are served one by one); the last block to finish picks every domain's bin.
// 8M cells of 7 domains: 1316 us with 8 bits a pass, a lookup per cell and a
// launch for every pick, 147 us now (189 us with 32 bins by lane in the pick; then two
// blocks a compute unit took 223 us and 512 threads a block 195 us: each block's fence
// writes an L2 back).
// ---------------------------------------------------------------------------
constexpr int kSelBits = 11, kSelBins = 1 << kSelBits, kSelPasses = 6, kSelCopies = 4, kSelThreads = 1024;
// The picks by the last block up to a domain a wave, beyond that in a launch of
// their own: with the last block alone 512 domains of 512 cells took 4.2 ms and 64
// of 4096 0.60 ms, now 0.15 and 0.09 ms; 16 domains have no more picks than the
// block has waves, and a launch after each of the six passes would cost more
constexpr int kSelPickWaves = kSelThreads / 64;
__host__ __device__ inline int select_shift(int pass) { return pass < 5 ? 64 - kSelBits * (pass + 1) : 0; }

// Cell ranges of the domains: from a context's records, or (the entry point
// without a context) at most kStaticDomains of them by value.
constexpr int kStaticDomains = 64;
struct DomByArray {
    const DomDev *doms;
    int32_t n;
    __device__ int64_t begin(int d) const { return doms[d].cell_off; }
};
struct DomByRanges {
    int32_t n;
    int64_t off[kStaticDomains + 1];   // domain d holds cells [off[d], off[d+1])
    __device__ int64_t begin(int d) const { return off[d]; }
};
template <typename Doms>
__device__ inline int domain_of(const Doms &D, int64_t c)
{
    int lo = 0, hi = D.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (D.begin(mid) <= c) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The radix select's state: per domain a histogram, the median's bit prefix,
// the rank still to skip and (for delta_cell) the running maximum; the number
// of blocks done with the pass.
struct SelectState {
    unsigned *hist;
    unsigned long long *prefix, *rank, *dmax;
    unsigned *done;
};

template <typename Doms>
__global__ void k_select_init(Doms D, int64_t n_cells, SelectState st)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (int64_t)D.n * kSelBins) st.hist[i] = 0;
    if (i == 0) *st.done = 0;
    if (i < D.n) {
        const int64_t n = (i + 1 < D.n ? D.begin((int)i + 1) : n_cells) - D.begin((int)i);
        st.rank[i] = (unsigned long long)((n - 1) / 2);   // lower median
        st.prefix[i] = 0ull;
        st.dmax[i] = 0ull;
    }
}

// A block's run of cells: [lo, hi)
__device__ inline void block_run(int64_t n_cells, int64_t &lo, int64_t &hi)
{
    int64_t per = (n_cells + gridDim.x - 1) / gridDim.x;
    per = (per + 63) / 64 * 64;
    lo = (int64_t)blockIdx.x * per;
    hi = lo + per < n_cells ? lo + per : n_cells;
}

// Sum of v over the lanes, and below: over the lanes below this one.  BIG: sums of
// 2^32 and more, in halves of 16 bits.
template <bool BIG>
__device__ inline unsigned long long wave_total(unsigned v, unsigned long long &below)
{
    int lo, hi = 0, h = 0;
    const int l = wave_excl_scan_dpp((int)(BIG ? v & 0xffffu : v), lo);
    if (BIG) h = wave_excl_scan_dpp((int)(v >> 16), hi);
    below = ((unsigned long long)(unsigned)h << 16) + (unsigned)l;
    return ((unsigned long long)(unsigned)hi << 16) + (unsigned)lo;
}

// The bin of domain d that holds its median, by a wave: 32 rows of 64 bins (whole
// cache lines, which other blocks wrote: four bins a lane took 8M cells of 7
// domains from 160 to 205 us; a row at a time 151, now 147), the row by the totals of pairs of rows, the bin by a
// scan of the row.  Leaves the histogram zero.
template <bool BIG>
__device__ inline void pick_bin(const SelectState &st, int d, int shift)
{
    constexpr int kRows = kSelBins / 64;
    const int lane = lane_id();
    unsigned *const hd = st.hist + (size_t)d * kSelBins + lane;
    unsigned v[kRows];
#pragma unroll
    for (int q = 0; q < kRows; ++q) v[q] = __hip_atomic_load(&hd[64 * q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long k = st.rank[d], below;
    int row = 0;
    unsigned mine = 0, next = 0;
    bool found = false;
#pragma unroll
    for (int q = 0; q < kRows; q += 2) {   // two rows at a time
        hd[64 * q] = 0;
        hd[64 * q + 64] = 0;
        const unsigned long long tot = BIG ? wave_total<BIG>(v[q], below) + wave_total<BIG>(v[q + 1], below)
                                           : wave_total<BIG>(v[q] + v[q + 1], below);
        if (!found) {   // (uniform)
            found = k < tot;
            row = q;
            mine = v[q];
            next = v[q + 1];
            k -= found ? 0 : tot;
        }
    }
    const unsigned long long tot = wave_total<BIG>(mine, below);
    if (k >= tot) {   // (uniform)
        k -= tot;
        ++row;
        mine = next;
        (void)wave_total<BIG>(mine, below);
    }
    if (k >= below && k < below + mine) {   // one lane
        st.rank[d] = k - below;
        st.prefix[d] |= (unsigned long long)(64 * row + lane) << shift;
    }
}

// The picks of more domains than the last block of k_select has waves
__global__ __launch_bounds__(256) void k_pick(int n_dom, int64_t n_cells, int pass, SelectState st)
{
    const int d = (int)blockIdx.x * 4 + uniform((int)(threadIdx.x >> 6));
    if (d >= n_dom) return;
    if (n_cells >> 32) pick_bin<true>(st, d, select_shift(pass));
    else pick_bin<false>(st, d, select_shift(pass));
}

template <typename Doms>
__global__ __launch_bounds__(kSelThreads) void k_select(Doms D, int64_t n_cells, const double *__restrict__ f, int pass,
                                                        SelectState st)
{
    __shared__ unsigned h[kSelCopies * kSelBins];
    __shared__ int is_last;
    const int tid = threadIdx.x, lane = tid & 63;
    const int shift = select_shift(pass), bits = pass < 5 ? kSelBits : 64 - 5 * kSelBits;
    const unsigned digit_mask = (1u << bits) - 1u;
    const unsigned long long above = pass == 0 ? 0ull : ~0ull << (shift + bits);
    for (int i = tid; i < kSelCopies * kSelBins; i += kSelThreads) h[i] = 0;
    __syncthreads();
    int64_t lo, hi;
    block_run(n_cells, lo, hi);
    unsigned *const mine = h + (lane & (kSelCopies - 1));   // copies interleaved: a bin's four counts in four banks
    for (int d = lo < hi ? domain_of(D, lo) : 0; lo < hi; ++d) {
        const int64_t de = d + 1 < D.n ? D.begin(d + 1) : n_cells;
        const int64_t end = de < hi ? de : hi;
        const unsigned long long prefix = st.prefix[d];
        auto count = [&](double v) {
            const unsigned long long key = (unsigned long long)__double_as_longlong(v);
            if ((key & above) == prefix) atomicAdd(&mine[kSelCopies * ((unsigned)(key >> shift) & digit_mask)], 1u);
        };
        int64_t c = lo + tid;
        for (; c + 3 * kSelThreads < end; c += 4 * kSelThreads) {
            const double v0 = f[c], v1 = f[c + kSelThreads], v2 = f[c + 2 * kSelThreads], v3 = f[c + 3 * kSelThreads];
            count(v0);
            count(v1);
            count(v2);
            count(v3);
        }
        for (; c < end; c += kSelThreads) count(f[c]);
        __syncthreads();
        for (int i = tid; i < kSelBins; i += kSelThreads) {
            unsigned v = 0;
            for (int q = 0; q < kSelCopies; ++q) {
                v += h[kSelCopies * i + q];
                h[kSelCopies * i + q] = 0;
            }
            if (v) atomicAdd(&st.hist[(size_t)d * kSelBins + i], v);
        }
        __syncthreads();
        lo = end;
    }
    if (D.n > kSelPickWaves) return;   // (k_pick follows)
    // the last block to get here picks the bins (its counts are all in: every
    // wave's adds have completed before its block's increment).  One thread
    // fences for its block: a device fence writes the XCD's L2 back, which
    // took 140 of a pass's 157 us when all 8 waves of 1024 blocks did it
    wait_stores();
    __syncthreads();
    if (tid == 0) {
        __threadfence();
        is_last = atomicAdd(st.done, 1u) == gridDim.x - 1;
        if (is_last) __threadfence();
    }
    __syncthreads();
    if (!is_last) return;
    const int d = uniform(tid >> 6);
    if (d < D.n) {
        if (n_cells >> 32) pick_bin<true>(st, d, shift);
        else pick_bin<false>(st, d, shift);
    }
    if (tid == 0) *st.done = 0;
}

template <typename Doms>
__global__ __launch_bounds__(kSelThreads) void k_delta(Doms D, int64_t n_cells, const double *__restrict__ fn,
                                                       const double *__restrict__ fo, SelectState st)
{
    __shared__ unsigned long long wmax[kSelThreads / 64];
    const int tid = threadIdx.x;
    int64_t lo, hi;
    block_run(n_cells, lo, hi);
    for (int d = lo < hi ? domain_of(D, lo) : 0; lo < hi; ++d) {
        const int64_t de = d + 1 < D.n ? D.begin(d + 1) : n_cells;
        const int64_t end = de < hi ? de : hi;
        const double m = __longlong_as_double((long long)st.prefix[d]);
        unsigned long long mx = 0;   // bits of a non-negative double order like the value
        for (int64_t c = lo + tid; c < end; c += kSelThreads) {
            const double old = fo[c];
            const double norm = old > m ? old : m;
            const double diff = fabs(fn[c] - old);
            double dl;
            if (norm > 0.0) dl = diff / norm;
            else dl = diff > 0.0 ? INFINITY : 0.0;
            if (!(dl == dl)) dl = INFINITY;
            const unsigned long long key = (unsigned long long)__double_as_longlong(dl);
            mx = key > mx ? key : mx;
        }
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long y = __shfl_xor(mx, o, 64);
            mx = y > mx ? y : mx;
        }
        if ((tid & 63) == 0) wmax[tid >> 6] = mx;
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < kSelThreads / 64; ++w) mx = wmax[w] > mx ? wmax[w] : mx;
            atomicMax(&st.dmax[d], mx);
        }
        __syncthreads();
        lo = end;
    }
}

// the per-domain maxima (bit patterns of non-negative doubles) as doubles
__global__ void k_store_delta(int n_dom, const unsigned long long *__restrict__ dmax, double *__restrict__ out)
{
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d < n_dom) out[d] = __longlong_as_double((long long)dmax[d]);
}

// Scratch of the entry point without allocation (tr_delta_noalloc): per
// domain a histogram, the median's bit prefix, the rank still to skip and
// the running maximum.  One copy per device, held until the
// process ends; every call on a device shares it.
constexpr size_t kStaticScratchWords = (size_t)kStaticDomains * (kSelBins / 2) + 3 * kStaticDomains + 1;
static __device__ __align__(256) unsigned long long scratch[kStaticScratchWords];

}  // namespace tr

// ===========================================================================
// Host side: the context and the C ABI
// ===========================================================================
using namespace tr;

struct tr_ctx {
    tr_params p{};
    hipStream_t stream = nullptr;
    int device = 0;
    int n_cu = 0;
    std::string err;
    // domains
    std::vector<DomTopo> topo;
    std::vector<DomDev> domh;
    int32_t n_dom = 0;
    int64_t n_cells = 0, n_nodes = 0;
    int32_t depth_max = 0, nr_max = 0;
    std::vector<int64_t> level_begin;   // global level ranges [L, L+1)
    // device arrays
    int4 *geo = nullptr, *olo = nullptr, *oext = nullptr;
    int2 *topo_d = nullptr;
    int32_t *cell_node = nullptr, *cell_dom = nullptr, *order = nullptr;
    DomDev *doms = nullptr;
    double *r64 = nullptr;
    float *r32 = nullptr;
    double *mom = nullptr;
    void *packA = nullptr, *packB = nullptr;
    double *ndot = nullptr;
    // sources
    std::vector<std::vector<double>> sxyz, sq;
    double *d_sxyz = nullptr, *d_sq = nullptr;
    int32_t *d_sdom = nullptr;
    int32_t n_src_dev = 0;
    bool src_dirty = true;
    double rate_unit = 1.0;
    // sweep state
    int32_t *queue = nullptr;
    unsigned long long *stats = nullptr;
    int32_t *err_flags = nullptr;
    void *gbuf = nullptr;
    size_t gbuf_bytes = 0;
    void *ebuf = nullptr;   // emission rows of split LDS buffers
    size_t ebuf_bytes = 0;
    unsigned char *mbuf = nullptr;   // marks and ray numbers that are not in LDS
    size_t mbuf_bytes = 0;
    int2 *lists = nullptr;               // the listed walks of a chunk of targets, their records, the pool
    uint16_t *emit_at = nullptr;         // of pairs of the nodes outside the angular table
    TargetRec *rec = nullptr;
    int32_t *dyn_pool = nullptr;
    int32_t dyn_units = 0;
    int64_t list_targets = 0, list_tried = 0;   // targets they hold, and that were asked for
    int32_t *glist = nullptr;            // walk lists of the fallback pass
    int32_t *ovf = nullptr;              // items queued for it
    int64_t ovf_cap = 0;
    // angular-weight table (built in tr_set_domains)
    int32_t *atab_idx = nullptr, *atab_pool = nullptr;
    AtabGeom atab{};
    // delta scratch
    unsigned int *hist = nullptr;
    unsigned long long *dprefix = nullptr, *drank = nullptr, *dmax = nullptr;   // (drank: a word more, the blocks done)
    double *solve_tmp = nullptr;
    int64_t solve_tmp_n = 0;
    // state
    bool built = false;
    tr_precision built_prec = TR_FP64;
    int32_t waves = 0, tpc = 0, bufmode = 0, intmode = 0, atommode = 0;   // user launch shape (0 = default)
    int32_t last_waves = 0, last_tpc = 0, last_lds = 0, last_intw = 0, last_cas = 0, last_int32 = 0;
    int tuned_waves[2] = {0, 0};         // per precision after tr_autotune
    int tuned_buf[2] = {0, 0};
    int tuned_int[2] = {0, 0};
    int tuned_atom[2] = {0, 0};
    float last_ms = 0.f;
    bool timed_valid = false;            // ev0/ev1 bracket a recorded sweep
    // one outer iteration captured as a hipGraph (tr_step)
    // (two cached graphs, so that an iteration alternating between two
    // buffers replays instead of capturing again)
    struct GraphSlot {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        const void *key[4] = {nullptr, nullptr, nullptr, nullptr};
        uint64_t used = 0;
    } gslot[2];
    uint64_t graph_clock = 0;
    hipStream_t cap_stream = nullptr;
    void *pinned = nullptr;              // host copies of the flags and deltas
    size_t pinned_bytes = 0;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    // the sweep kernels that this context has asked about: workgroups a compute unit by their registers
    std::vector<std::pair<const void *, int>> kernels;
};

namespace {

tr_status fail(tr_ctx *c, tr_status s, const std::string &m)
{
    if (c) c->err = m;
    return s;
}

#define HIPCHK(call)                                                                           \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return fail(c, TR_EHIP, std::string(#call) + ": " + hipGetErrorString(e_));        \
    } while (0)

template <typename T>
void dfree(T *&p)
{
    if (p) (void)hipFree((void *)p);
    p = nullptr;
}

void drop_slot(tr_ctx::GraphSlot &g)
{
    if (g.exec) (void)hipGraphExecDestroy(g.exec);
    if (g.graph) (void)hipGraphDestroy(g.graph);
    g = tr_ctx::GraphSlot();
}

void drop_graph(tr_ctx *c)
{
    for (auto &g : c->gslot) drop_slot(g);
}

void free_domains(tr_ctx *c)
{
    drop_graph(c);
    dfree(c->geo); dfree(c->olo); dfree(c->oext); dfree(c->topo_d);
    dfree(c->cell_node); dfree(c->cell_dom); dfree(c->order); dfree(c->doms);
    dfree(c->r64); dfree(c->r32); dfree(c->mom); dfree(c->packA); dfree(c->packB);
    dfree(c->ndot); dfree(c->d_sxyz); dfree(c->d_sq); dfree(c->d_sdom);
    dfree(c->hist); dfree(c->dprefix); dfree(c->drank); dfree(c->dmax);
    dfree(c->atab_idx); dfree(c->atab_pool);
    dfree(c->solve_tmp);
    dfree(c->gbuf);
    c->gbuf_bytes = 0;
    dfree(c->ebuf);
    c->ebuf_bytes = 0;
    dfree(c->mbuf);
    c->mbuf_bytes = 0;
    dfree(c->lists);
    dfree(c->emit_at);
    dfree(c->rec);
    dfree(c->dyn_pool);
    c->list_targets = c->list_tried = 0;
    dfree(c->glist);
    dfree(c->ovf);
    c->ovf_cap = 0;
    c->solve_tmp_n = 0;
    c->built = false;
}

tr_status check_params(tr_ctx *c, const tr_params &p)
{
    if (p.nside < 1 || p.nside > 64 || (p.nside & (p.nside - 1))) return fail(c, TR_EINVAL, "nside must be a power of two in [1, 64]");
    if (p.n_radial < 0 || p.n_radial == 1 || p.n_radial == 2 || p.n_radial > kMaxRadial)
        return fail(c, TR_EINVAL, "n_radial must be 0 or in [3, 128]");
    if (p.n_radial == 0 && !(p.eta_r > 0)) return fail(c, TR_EINVAL, "eta_r must be > 0");
    if (!(p.theta >= 0) || !std::isfinite(p.theta)) return fail(c, TR_EINVAL, "theta must be >= 0");
    if (!std::isfinite(p.theta_if) || !std::isfinite(p.theta_src))
        return fail(c, TR_EINVAL, "theta_if and theta_src must be finite");
    if (!(p.src_radius_cm >= 0) || !std::isfinite(p.src_radius_cm))
        return fail(c, TR_EINVAL, "src_radius_cm must be >= 0");
    if (p.eps_kernel < 0 || p.eps_kernel > 6) return fail(c, TR_EINVAL, "eps_kernel must be in [0, 6]");
    if (p.mass_kernel != 0 && p.mass_kernel != 5 && p.mass_kernel != 6)
        return fail(c, TR_EINVAL, "mass_kernel must be 0, 5 (W_p) or 6 (W_g)");
    if (!(p.alpha_b >= 0) || !std::isfinite(p.alpha_b)) return fail(c, TR_EINVAL, "alpha_b must be >= 0");
    if (p.subsample < 1 || p.subsample > 4) return fail(c, TR_EINVAL, "subsample must be in [1, 4]");
    if (p.max_iter < 0) return fail(c, TR_EINVAL, "max_iter must be >= 0");
    if (!(p.eps_lim >= 0)) return fail(c, TR_EINVAL, "eps_lim must be >= 0");
    if (p.precision != TR_FP64 && p.precision != TR_FP32C) return fail(c, TR_EINVAL, "unknown precision");
    return TR_OK;
}

inline unsigned grid1(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

template <typename T>
tr_status upload(tr_ctx *c, T *&dst, const std::vector<T> &src)
{
    dfree(dst);
    if (src.empty()) return TR_OK;
    if (hipMalloc((void **)&dst, src.size() * sizeof(T)) != hipSuccess) return fail(c, TR_ENOMEM, "hipMalloc failed");
    HIPCHK(hipMemcpyAsync(dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice, c->stream));
    return TR_OK;
}

tr_status dalloc(tr_ctx *c, void **p, size_t bytes)
{
    if (hipMalloc(p, bytes ? bytes : 16) != hipSuccess) return fail(c, TR_ENOMEM, "hipMalloc of " + std::to_string(bytes) + " bytes failed");
    return TR_OK;
}

// LDS bytes of one sweep workgroup with buffers for `rays` rays (must mirror the carve-up in sweep_body)
size_t sweep_lds_bytes(size_t real, int npix, int rays, int stride_k, int nrm, int waves, bool ldsbuf, bool wide)
{
    const size_t ew = nrm > 64 ? 2 : 1;
    size_t b = wide && !ldsbuf ? 0 : (size_t)rays * 8 * ew;
    if (ldsbuf) b += (((size_t)rays * stride_k * real + 15) / 16) * 16;
    b += 2 * (((size_t)nrm * real + 15) / 16) * 16;
    b += 2 * (size_t)nrm * 8;
    b += (size_t)waves * 8;
    b += S_COUNT * 4;
    if (!wide) b += (size_t)npix * (8 * ew + 4);
    return b;
}

constexpr size_t kLdsMax = 160 * 1024, kLdsGranule = 1280;
// From N_side 32 on marks and ray numbers do not fit in LDS (144 or 240 KB); beside
// ray buffers in LDS they leave it from N_side 16 on, where they take 36 or 60 KB
// of it (32^3 with 32 points, 1 / 2000 sources: FP32C 3.58 / 78.0 ms with the marks
// in LDS, 3.15 / 63.6 ms without, FP64 4.49 / 179 against 3.91 / 133; 100 points
// 9.65 / 256 against 5.18 / 200 and 13.3 / 557 against 10.8 / 432), not at N_side 8
// (9 or 15 KB: FP32C 1.43 / 15.2 ms against 1.73 / 15.5, FP64 1.97 / 27.8 against
// 1.85 / 26.5)
constexpr int kWidePix = 12 * 16 * 16, kWideMemPix = 12 * 32 * 32;
constexpr size_t kSlabBytes = (size_t)16 << 30;   // most for the ray buffers in device memory

using KernelFn = void (*)(SweepArgs);

template <typename Real>
KernelFn pick_kernel_kv(int waves, bool ldsbuf, bool fallback)
{
    if (waves == 4) {
        if (fallback) return ldsbuf ? (KernelFn)k_sweep_kv_fallback<Real, 4, true> : (KernelFn)k_sweep_kv_fallback<Real, 4, false>;
        return ldsbuf ? (KernelFn)k_sweep_kv<Real, 4, true> : (KernelFn)k_sweep_kv<Real, 4, false>;
    }
    if (waves == 8) {
        if (fallback) return ldsbuf ? (KernelFn)k_sweep_kv_fallback<Real, 8, true> : (KernelFn)k_sweep_kv_fallback<Real, 8, false>;
        return ldsbuf ? (KernelFn)k_sweep_kv<Real, 8, true> : (KernelFn)k_sweep_kv<Real, 8, false>;
    }
    return nullptr;
}

template <typename Real>
KernelFn pick_kernel_wide(int waves, bool fallback)
{
    if (waves == 4) return fallback ? (KernelFn)k_sweep_wide_fallback<Real, 4> : (KernelFn)k_sweep_wide<Real, 4>;
    if (waves == 8) return fallback ? (KernelFn)k_sweep_wide_fallback<Real, 8> : (KernelFn)k_sweep_wide<Real, 8>;
    return fallback ? (KernelFn)k_sweep_wide_fallback<Real, 16> : (KernelFn)k_sweep_wide<Real, 16>;
}

template <typename Real>
KernelFn pick_kernel_wide_mem(bool kv, bool fallback)
{
    if (kv) return fallback ? (KernelFn)k_sweep_wide_mem_fallback<Real, true> : (KernelFn)k_sweep_wide_mem<Real, true>;
    return fallback ? (KernelFn)k_sweep_wide_mem_fallback<Real, false> : (KernelFn)k_sweep_wide_mem<Real, false>;
}

KernelFn pick_kernel_cas(int waves, bool fallback)
{
    if (waves == 4) return fallback ? (KernelFn)k_sweep_cas_fallback<4> : (KernelFn)k_sweep_cas<4>;
    if (waves == 8) return fallback ? (KernelFn)k_sweep_cas_fallback<8> : (KernelFn)k_sweep_cas<8>;
    return fallback ? (KernelFn)k_sweep_cas_fallback<16> : (KernelFn)k_sweep_cas<16>;
}

template <typename Real>
KernelFn pick_kernel(int waves, bool ldsbuf, bool fallback)
{
#define TR_CASE(W)                                                                                      \
    case W:                                                                                             \
        if (fallback)                                                                                   \
            return ldsbuf ? (KernelFn)k_sweep_fallback<Real, W, true> : (KernelFn)k_sweep_fallback<Real, W, false>; \
        return ldsbuf ? (KernelFn)k_sweep<Real, W, true> : (KernelFn)k_sweep<Real, W, false>;
    switch (waves) {
        TR_CASE(1)
        TR_CASE(2)
        TR_CASE(4)
        TR_CASE(8)
        TR_CASE(16)
        default:
            return nullptr;
    }
#undef TR_CASE
}

struct LaunchPlan {
    KernelFn fn = nullptr, fn_fb = nullptr;
    int waves = 0, blocks = 0, per_cu = 0, stride_k = 0;
    int64_t chunk = 0;   // targets walked and listed at a time
    int64_t mbuf_stride = 0;
    size_t lds = 0;
    bool ldsbuf = true;
    bool cas = false;   // FP32 LDS buffers accumulated by compare-and-swap
    bool wide = false;  // marks and ray numbers in device memory
    bool split = false; // A, E, V rows in LDS, emission rows in device memory
    int rays = 0;       // ray buffers of a workgroup
    int intm = 1;   // integration: 1 a lane per ray, 2 a wave per ray, 3/4/5 a group of 4/8/16 lanes,
                    // 6/7/8 the same groups with the FP32 march (FP32 buffers only)
};

// lanes that integrate one ray in integration mode m
inline int lanes_per_ray(int m) { return m == 2 ? 64 : (m >= 3 ? 4 << ((m - 3) % 3) : 1); }

// Workgroups a compute unit by their LDS (the runtime's own figure leaves out the granule)
int targets_by_lds(size_t lds) { return (int)(kLdsMax / ((lds + kLdsGranule - 1) / kLdsGranule * kLdsGranule)); }

// Workgroups a compute unit by the kernel's registers, asked of the runtime once a
// context (as is the leave to use all of LDS): a plan asks about up to three kernels.
tr_status targets_by_registers(tr_ctx *c, KernelFn fn, int waves, int &n)
{
    for (const auto &k : c->kernels)
        if (k.first == (const void *)fn) {
            n = k.second;
            return TR_OK;
        }
    HIPCHK(hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax));
    HIPCHK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void *)fn, waves * 64, 0));
    c->kernels.emplace_back((const void *)fn, n);
    return TR_OK;
}

// Ray buffers: a target's rays that hold emission (KV: all) are mapped and integrated as
// many at a time as there are buffers.  Four rows per ray (odd stride: ray k of lane k hits
// distinct banks), or in FP32 the A, E, V rows in LDS and the emission rows in device memory
// where that holds more rays.  As many targets share a compute unit as the registers allow,
// fewer while that leaves a target less than `want` buffers: as many as rays that probably
// hold emission, between 16 and 32 (4 waves, targets a compute unit with 16 / with 32:
// 48^3 N_side 4, 64 points FP64 2 sources 4 / 2 targets 6.3 / 9.1 ms, 8 sources 14.6 / 12.8;
// 100 points FP32C 2 sources 6 / 3 targets 6.0 / 8.7, 16 sources 19.0 / 18.4; N_side 2, 64
// points FP64 2 sources 4 / 2 targets 5.7 / 8.3, 32 sources 12.5 / 11.4); below 16 for one
// target alone, all buffers are in device memory.
struct LdsFit {
    int targets = 0, rays = 0;   // a compute unit, a target
    bool split = false;
};

tr_status fit_lds(tr_ctx *c, KernelFn fn, bool f32, int npix, int nrm, int waves, int tpc_req, bool wide, bool may_split,
                  int want, LdsFit &F)
{
    const size_t real = f32 ? 4 : 8;
    const size_t fixed = sweep_lds_bytes(real, npix, 0, 0, nrm, waves, true, wide);
    if (fixed >= kLdsMax) return TR_OK;
    tr_status s = targets_by_registers(c, fn, waves, F.targets);
    if (s) return s;
    if (tpc_req > 0) F.targets = std::min(F.targets, tpc_req);
    for (; F.targets >= 1; --F.targets) {
        const size_t room = kLdsMax / (size_t)F.targets / kLdsGranule * kLdsGranule;
        auto fit = [&](int stride) {
            if (sweep_lds_bytes(real, npix, npix, stride, nrm, waves, true, wide) <= room) return npix;
            const size_t each = (size_t)stride * real + 8 * (nrm > 64 ? 2 : 1);
            return room <= fixed + 16 ? 0 : std::min(npix, (int)((room - fixed - 16) / each));
        };
        const int r4 = fit(4 * nrm + 1), r3 = may_split ? fit(3 * nrm + 1) : 0;
        F.split = r4 < npix && r3 > r4;
        F.rays = F.split ? r3 : r4;
        if (F.rays >= std::min(npix, F.targets > 1 ? want : 16)) break;
    }
    return TR_OK;
}

// Rays of a target that probably hold emission: a source puts it on as many rays as
// a node has pixels, about (1 + 0.34 N_side)^2, at random.  Sphere sources count one
// each: from most targets they are a few nodes.
double lit_rays(const tr_ctx *c, int npix)
{
    const double each = (1.0 + 0.34 * c->p.nside) * (1.0 + 0.34 * c->p.nside);
    return npix * (1.0 - std::exp(-each * c->n_src_dev / c->n_dom / npix));
}

int want_buffers(double lit) { return (int)std::min(32.0, std::max(16.0, lit)); }

// 4 or 8 waves per target where the caller leaves it open.  Several targets are
// resident, and the fewer waves share one the better their phases overlap (64^3
// N_side 2 FP32C: 6 targets of 4 waves 9.9 ms, 2 of 8 waves 13.6), as long as a
// target's rays with emission fit its share of the buffers; beyond that 8 waves
// on fewer targets save passes.  4 waves while those rays need 1.25 buffers at most
// (FP32 1.5; 0.75 where only 3 targets of 4 waves fit; never where fewer do), 4 / 8
// waves on either side (rays a buffer):
//   64^3 N_side 4, 32 points  FP32C 16 sources (1.2) 16.1 / 18.5 ms, 32 (1.9) 21.2 / 21.0
//                             FP64 8 (1.2) 15.5 / 17.8, 16 (2.0) 25.1 / 20.4
//   64^3 N_side 2, 32 points  FP64 32 (1.2) 15.8 / 18.0, 256 (1.4) 24.2 / 23.9, 2000 30.6 / 28.8
//   48^3 N_side 4, 64 points  FP32C 4 (0.5) 5.9 / 8.3, 16 (1.8) 10.8 / 9.9; FP64 (2 targets) 4 10.0 / 9.2
//   32^3 N_side 8, 32 points  FP32C 1 (0.3) 1.38 / 1.95, 8 (2.5) 2.94 / 2.49
//   48^3 N_side 4, a sphere of 8 / 12 cells: FP64 7.7 / 8.1 and 10.7 / 10.1, FP32C 6.0 / 7.4 and 7.8 / 9.2
tr_status default_waves(tr_ctx *c, bool f32, int npix, int nrm, int tpc_req, int &waves)
{
    const bool wide = npix >= kWidePix;
    const KernelFn fn = wide ? (f32 ? pick_kernel_wide<float>(4, false) : pick_kernel_wide<double>(4, false))
                             : f32 ? pick_kernel_cas(4, false) : pick_kernel<double>(4, true, false);
    const double lit = lit_rays(c, npix);
    LdsFit F;
    tr_status s = fit_lds(c, fn, f32, npix, nrm, 4, tpc_req, wide, f32, want_buffers(lit), F);
    if (s) return s;
    const double room = F.targets >= 4 ? (f32 ? 1.5 : 1.25) : F.targets == 3 ? 0.75 : 0.0;
    waves = lit <= room * F.rays || (F.rays == npix && F.targets >= 3) ? 4 : 8;
    return TR_OK;
}

tr_status plan_sweep(tr_ctx *c, int64_t n_items, int waves_req, int tpc_req, int buf_req, int int_req, LaunchPlan &L,
                     int atom_req = 0)
{
    const bool f32 = c->p.precision == TR_FP32C;
    const size_t real = f32 ? 4 : 8;
    const int npix = 12 * c->p.nside * c->p.nside;
    const int nrm = c->nr_max;
    tr_status s;
    int waves = waves_req;
    int bm = buf_req > 0 ? buf_req : c->tuned_buf[f32 ? 1 : 0];
    // the radial-kernel variants are built for 4 and 8 waves per target only
    const bool kv = !((c->p.eps_kernel == 0 || c->p.eps_kernel == 3) && (c->p.mass_kernel == 0 || c->p.mass_kernel == 5));
    if (waves <= 0) waves = c->tuned_waves[f32 ? 1 : 0];
    if (waves <= 0) {
        // A list of no more targets than a few a compute unit has nothing to overlap with: 8 waves
        // finish each sooner (64^3 N_side 4 FP32C, 4 sources, 4 / 8 waves: 256 targets 0.109 /
        // 0.097 ms, 1000 0.165 / 0.160, 2048 0.262 / 0.256, 4096 0.398 / 0.430).
        waves = 8;
        if (n_items > 4 * (int64_t)c->n_cu) {
            if (kv) {
                // All rays have buffers: 8 waves (FP64 4 / 8 waves: 48^3 N_side 2 10.4 / 9.4 ms, 24^3
                // N_side 8 11.7 / 8.9 ms, 32^3 N_side 4 with 100 points 30.6 / 24.1 ms; FP32C N_side 8
                // 10.9 / 9.9 ms; N_side 2 with buffers in device memory 55.0 / 50.0 ms), but in FP32 4
                // where few passes hold all rays (N_side 2 19.0 / 20.0 ms, N_side 4 9.7 / 10.1 ms, with
                // 100 points 27.4 / 26.4 ms).
                if (f32 && bm != 2 && npix * nrm <= 192 * 64) waves = 4;
            } else if (bm == 2) {
                // (32^3 N_side 4 with 4 sources FP32C 5.6 / 6.4 ms, 48^3 N_side 2 with 60 33.2 / 30.9 ms)
                if (c->n_src_dev <= 16 * c->n_dom) waves = 4;
            } else if ((s = default_waves(c, f32, npix, nrm, tpc_req, waves))) {
                return s;
            }
        }
    }
    if (kv) waves = waves <= 4 ? 4 : 8;
    L.waves = waves;
    if (kv) {
        L.fn = f32 ? pick_kernel_kv<float>(waves, bm != 2, false) : pick_kernel_kv<double>(waves, bm != 2, false);
    } else {
        L.fn = f32 ? pick_kernel<float>(waves, bm != 2, false) : pick_kernel<double>(waves, bm != 2, false);
    }
    if (!L.fn) return fail(c, TR_EINVAL, "waves per target must be 1, 2, 4, 8 or 16");
    // accumulation: compare-and-swap by default (FP32, LDS; 4 waves where they are the default pick)
    {
        const int am = atom_req > 0 ? atom_req : (c->atommode > 0 ? c->atommode : c->tuned_atom[f32 ? 1 : 0]);
        L.cas = f32 && bm != 2 && !kv &&
                (waves == 8 || waves == 16 ? (am > 0 ? am == 2 : true) : waves == 4 && (am > 0 ? am == 2 : waves_req <= 0));
        if (L.cas) L.fn = pick_kernel_cas(waves, false);
    }
    // the radial-kernel variants and 1 or 2 waves have their ray buffers in device memory (8 waves)
    // where marks and numbers do not fit in LDS
    L.wide = npix >= kWidePix && bm != 2 && !kv && waves >= 4;
    const bool lds_ok = bm != 2 && (npix < kWideMemPix || L.wide);
    if (L.wide) {
        L.cas = f32;
        L.fn = f32 ? pick_kernel_wide<float>(waves, false) : pick_kernel_wide<double>(waves, false);
    }
    const int stride4 = 4 * nrm + 1, stride3 = 3 * nrm + 1;
    LdsFit fit;
    const int want = kv ? 32 : want_buffers(lit_rays(c, npix));
    if (lds_ok && (s = fit_lds(c, L.fn, f32, npix, nrm, waves, tpc_req, L.wide, f32 && !kv, want, fit))) return s;
    L.split = fit.split;
    L.rays = fit.rays;
    L.ldsbuf = fit.targets >= 1;
    // With the radial-kernel variants every pass maps all nodes of the target again: device memory
    // where passes x points grow beyond these (24^3 FP64: N_side 8 with 64 points (1472) LDS 20.2,
    // device memory 23.8 ms; 100 points (1700) 34.9 / 30.8; N_side 16 with 32 points (2400) 22.2 /
    // 14.3; FP32C: N_side 8 with 64 points (704) 17.8 / 20.7; N_side 16 with 32 points (1184)
    // 13.6 / 12.6; N_side 8 with 100 points (1900) 29.4 / 24.3)
    if (L.ldsbuf && kv && bm != 1 && (npix + L.rays - 1) / L.rays * nrm > (f32 ? 1000 : 1600)) L.ldsbuf = false;
    if (bm == 1 && !L.ldsbuf) return fail(c, TR_EINVAL, "ray buffers do not fit in LDS for this N_PIX and N_R");
    if (!L.ldsbuf) {
        L.rays = std::min(npix, kWideMemPix);
        L.wide = npix >= kWideMemPix;
        L.split = false;
        L.cas = false;
        if (L.wide) L.waves = waves = 8;
        L.fn = L.wide ? (f32 ? pick_kernel_wide_mem<float>(kv, false) : pick_kernel_wide_mem<double>(kv, false))
               : kv   ? (f32 ? pick_kernel_kv<float>(waves, false, false) : pick_kernel_kv<double>(waves, false, false))
                      : (f32 ? pick_kernel<float>(waves, false, false) : pick_kernel<double>(waves, false, false));
    }
    L.fn_fb = L.wide ? (L.ldsbuf ? (f32 ? pick_kernel_wide<float>(waves, true) : pick_kernel_wide<double>(waves, true))
                                 : (f32 ? pick_kernel_wide_mem<float>(kv, true) : pick_kernel_wide_mem<double>(kv, true)))
                    : L.cas ? pick_kernel_cas(waves, true)
                    : kv ? (f32 ? pick_kernel_kv<float>(waves, L.ldsbuf, true) : pick_kernel_kv<double>(waves, L.ldsbuf, true))
                         : (f32 ? pick_kernel<float>(waves, L.ldsbuf, true) : pick_kernel<double>(waves, L.ldsbuf, true));
    L.stride_k = L.split ? stride3 : stride4;
    int occ = 0;
    L.lds = sweep_lds_bytes(real, npix, L.rays, L.stride_k, nrm, waves, L.ldsbuf, L.wide);
    if (L.lds > kLdsMax)
        return fail(c, TR_EINVAL, "sweep kernel does not fit on a compute unit (LDS " + std::to_string(L.lds) + " B)");
    int fb = 0;
    if ((s = targets_by_registers(c, L.fn, waves, occ)) || (s = targets_by_registers(c, L.fn_fb, waves, fb))) return s;
    occ = std::min(occ, targets_by_lds(L.lds));
    if (occ <= 0) return fail(c, TR_EINVAL, "sweep kernel does not fit on a compute unit (LDS " + std::to_string(L.lds) + " B)");
    L.per_cu = tpc_req > 0 ? std::min(tpc_req, occ) : occ;
    if (!L.ldsbuf)   // (N_side 32: 6 to 50 MB a workgroup)
        while (L.per_cu > 1 && (size_t)c->n_cu * L.per_cu * L.rays * L.stride_k * real > kSlabBytes) --L.per_cu;
    // integration: by default groups of at least 4 lanes per ray, so that a target's few
    // emitting rays share a wave (a ray with more emitting points gets a wider group): against
    // groups of at least 8 or 16 lanes 2 to 15% faster at N_side 4, equal at N_side 2
    const int im = int_req > 0 ? int_req : c->tuned_int[f32 ? 1 : 0];
    // (FP32 buffers march in FP32 by default, the FP64 form in FP64)
    L.intm = im > 0 ? im : 3 + (f32 ? 3 : 0);
    if (L.intm >= 6 && !f32) L.intm -= 3;
    L.chunk = std::min<int64_t>(n_items, kListTargets);
    // (a captured step graph holds these too.)  Where there is no memory for them, fewer targets at a
    // time, down to a few a compute unit: 36 KB a target, 1.2 GB for 32768
    if (c->list_tried < L.chunk) {
        drop_graph(c);
        auto take = [&](int64_t n) {
            dfree(c->lists);
            dfree(c->emit_at);
            dfree(c->rec);
            dfree(c->dyn_pool);
            // pairs outside the table: 4% of some 1000 nodes of about 3 (N_side 2) to 12 (N_side 8)
            // pairs; room for 1024 a target up to N_side 4, 4096 beyond, and a block for every wave
            c->dyn_units = (int32_t)std::min<int64_t>(
                (1 << 25) - 1, n * (c->p.nside <= 4 ? 256 : 1024) + (int64_t)c->n_cu * kWalkPerCu * kWalkWaves * kDynBlock);
            if (!dalloc(c, (void **)&c->lists, sizeof(int2) * (size_t)n * kListCap) &&
                !dalloc(c, (void **)&c->emit_at, sizeof(uint16_t) * (size_t)n * kListCap) &&
                !dalloc(c, (void **)&c->rec, sizeof(TargetRec) * (size_t)n) &&
                !dalloc(c, (void **)&c->dyn_pool, 16 * (size_t)c->dyn_units))
                return true;
            dfree(c->lists);
            dfree(c->emit_at);
            dfree(c->rec);
            dfree(c->dyn_pool);
            (void)hipGetLastError();
            return false;
        };
        c->list_tried = 0;
        c->list_targets = take_chunk(L.chunk, std::min<int64_t>(L.chunk, 4 * (int64_t)c->n_cu), take);
        if (c->list_targets == 0) return TR_ENOMEM;
        c->list_tried = L.chunk;
        if (c->list_targets < L.chunk) c->err.clear();
    }
    L.chunk = std::min(L.chunk, c->list_targets);
    L.blocks = (int)std::min<int64_t>((int64_t)c->n_cu * L.per_cu, L.chunk);
    if (!c->glist &&
        dalloc(c, (void **)&c->glist, sizeof(int32_t) * (size_t)c->n_cu * kFallbackPerCu * 3 * kGlobalList))
        return TR_ENOMEM;
    // a captured step graph holds the scratch pointers as kernel arguments:
    // it is dropped whenever one of them is reallocated below
    if (c->ovf_cap < n_items) {   // every item may need the second pass
        drop_graph(c);
        dfree(c->ovf);
        c->ovf_cap = 0;
        if (dalloc(c, (void **)&c->ovf, sizeof(int32_t) * (size_t)n_items)) return TR_ENOMEM;
        c->ovf_cap = n_items;
    }
    // per-workgroup slabs for the larger of the two grids (the second pass has
    // n_cu x min(per_cu, kFallbackPerCu) workgroups)
    const size_t nblk = (size_t)std::max<int64_t>(L.blocks, (int64_t)c->n_cu * std::min(L.per_cu, kFallbackPerCu));
    if (!L.ldsbuf) {
        const size_t need = nblk * L.rays * L.stride_k * real;
        if (need > c->gbuf_bytes) {
            drop_graph(c);
            dfree(c->gbuf);
            c->gbuf_bytes = 0;
            if (dalloc(c, &c->gbuf, need)) return TR_ENOMEM;
            c->gbuf_bytes = need;
        }
    }
    if (L.wide) {
        L.mbuf_stride = (int64_t)mask_slab_bytes(npix, L.rays, nrm > 64 ? 2 : 1, L.ldsbuf);
        const size_t need = nblk * (size_t)L.mbuf_stride;
        if (need > c->mbuf_bytes) {
            drop_graph(c);
            dfree(c->mbuf);
            c->mbuf_bytes = 0;
            if (dalloc(c, (void **)&c->mbuf, need)) return TR_ENOMEM;
            c->mbuf_bytes = need;
        }
    }
    if (L.split) {
        const size_t need = nblk * L.rays * nrm * real;
        if (need > c->ebuf_bytes) {
            drop_graph(c);
            dfree(c->ebuf);
            c->ebuf_bytes = 0;
            if (dalloc(c, &c->ebuf, need)) return TR_ENOMEM;
            c->ebuf_bytes = need;
            // the sweeps keep the plane zero between targets
            hipLaunchKernelGGL(k_fill_i32, dim3(grid1((int64_t)(need / 4))), dim3(256), 0, c->stream, (int32_t *)c->ebuf,
                               (int64_t)(need / 4), 0);
        }
    }
    return TR_OK;
}

float guard_tolerance(int nside);

tr_status launch_sweep(tr_ctx *c, const int64_t *targets, int64_t n, double *f_out, uint8_t *ion, bool timed,
                       int waves_req, int tpc_req, int buf_req, int int_req, int atom_req = 0)
{
    if (!c->built) return fail(c, TR_ESTATE, "tr_sweep needs tr_build first");
    if (c->built_prec != c->p.precision) return fail(c, TR_ESTATE, "precision changed since tr_build; build again");
    if (n == 0) return TR_OK;
    LaunchPlan L;
    tr_status s = plan_sweep(c, n, waves_req > 0 ? waves_req : c->waves, tpc_req > 0 ? tpc_req : c->tpc,
                             buf_req > 0 ? buf_req : c->bufmode, int_req > 0 ? int_req : c->intmode, L, atom_req);
    if (s) return s;
    SweepArgs a{};
    a.geo = c->geo;
    a.olo = c->olo;
    a.oext = c->oext;
    a.topo = c->topo_d;
    a.pA = c->packA;
    a.pB = c->packB;
    a.cell_node = c->cell_node;
    a.cell_dom = c->cell_dom;
    a.doms = c->doms;
    a.r64 = c->r64;
    a.r32 = c->r32;
    a.targets = targets;
    a.order = c->order;
    a.n_cells = c->n_cells;
    a.f_out = f_out;
    a.ion_out = ion;
    a.queue = c->queue;
    a.stats = c->stats;
    a.gbuf = c->gbuf;
    a.ebuf = c->ebuf;
    a.mbuf = c->mbuf;
    a.mbuf_stride = L.mbuf_stride;
    a.split = L.split ? 1 : 0;
    a.rays = L.rays;
    a.theta2 = c->p.theta * c->p.theta;
    a.theta_if2 = c->p.theta_if > 0.0 ? c->p.theta_if * c->p.theta_if : 0.0;
    a.theta_src2 = c->p.theta_src > 0.0 ? c->p.theta_src * c->p.theta_src : 0.0;
    a.guard_tol = guard_tolerance(c->p.nside);
    a.nside = c->p.nside;
    a.npix = 12 * c->p.nside * c->p.nside;
    a.subsample = c->p.subsample;
    a.f32 = c->p.precision == TR_FP32C ? 1 : 0;
    a.lists = c->lists;
    a.emit_at = c->emit_at;
    a.dyn_pool = c->dyn_pool;
    a.dyn_units = c->dyn_units;
    a.rec = c->rec;
    a.list_cap = kListCap;
    a.nr_max = c->nr_max;
    a.stride_k = L.stride_k;
    a.zeta_g = c->p.zeta_g;
    a.int_wave = L.intm == 2 ? 1 : 0;
    a.int_group = L.intm >= 3 ? lanes_per_ray(L.intm) : 0;
    a.int_fp32 = L.intm >= 6 ? 1 : 0;
    a.front_ratio = 1e-2f;
    a.eps_kernel = c->p.eps_kernel;
    a.periodic = c->p.periodic ? 1 : 0;
    a.mass_gauss = c->p.mass_kernel == 6 ? 1 : 0;
    a.ovf = c->ovf;
    a.ovf_cap = c->ovf_cap;
    a.glist = c->glist;
    a.gfmax = kGlobalList;
    a.gamax = kGlobalList;
    a.atab_idx = c->atab_idx;
    a.atab_pool = c->atab_pool;
    for (int q = 0; q < kAtabRatios; ++q) {
        a.atab_w[q] = c->atab.w[q];
        a.atab_base[q] = c->atab.base[q];
    }
    (void)hipGetLastError();   // a stale error of an earlier, unrelated call is not ours
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, c->stream, c->queue, (int64_t)8, 0);
    hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(64), 0, c->stream, c->stats, (int64_t)8);
    if (timed) HIPCHK(hipEventRecord(c->ev0, c->stream));
    // the targets a chunk at a time: their walks, then their mapping and integration
    for (int64_t i0 = 0; i0 < n; i0 += L.chunk) {
        a.item0 = i0;
        a.n_chunk = (int32_t)std::min<int64_t>(L.chunk, n - i0);
        const int wb = std::min((a.n_chunk + kWalkWaves - 1) / kWalkWaves, c->n_cu * kWalkPerCu);
        hipLaunchKernelGGL(k_walk, dim3(wb), dim3(kWalkWaves * 64), 0, c->stream, a);
        hipLaunchKernelGGL(L.fn, dim3(std::min(L.blocks, a.n_chunk)), dim3(L.waves * 64), L.lds, c->stream, a);
    }
    // the targets whose walks did not fit in the lists, again with longer lists per workgroup
    // (it ends at once when none was queued)
    {
        hipLaunchKernelGGL(L.fn_fb, dim3(c->n_cu * std::min(L.per_cu, kFallbackPerCu)), dim3(L.waves * 64), L.lds,
                           c->stream, a);
    }
    HIPCHK(hipGetLastError());
    if (timed) {
        HIPCHK(hipEventRecord(c->ev1, c->stream));
        c->timed_valid = true;
    }
    c->last_waves = L.waves;
    c->last_tpc = L.per_cu;
    c->last_lds = L.ldsbuf ? (L.split ? 2 : (L.rays < a.npix ? 3 : 1)) : 0;
    c->last_intw = lanes_per_ray(L.intm);
    c->last_int32 = L.intm >= 6 ? 1 : 0;
    c->last_cas = L.cas ? 1 : 0;
    return TR_OK;
}

tr_status upload_sources(tr_ctx *c)
{
    std::vector<double> xyz, q;
    std::vector<int32_t> dom;
    double qmax = 0;
    for (int d = 0; d < c->n_dom; ++d) {
        for (size_t s = 0; s < c->sq[d].size(); ++s) {
            for (int a = 0; a < 3; ++a) xyz.push_back(c->sxyz[d][3 * s + a]);
            q.push_back(c->sq[d][s]);
            dom.push_back(d);
            qmax = std::max(qmax, c->sq[d][s]);
        }
    }
    tr_status s;
    if ((s = upload(c, c->d_sxyz, xyz))) return s;
    if ((s = upload(c, c->d_sq, q))) return s;
    if ((s = upload(c, c->d_sdom, dom))) return s;
    c->n_src_dev = (int32_t)q.size();
    // internal rate unit: the power of two nearest the largest source rate
    c->rate_unit = std::ldexp(1.0, (int)std::lround(std::log2(std::max(qmax, 1.0))));
    for (int d = 0; d < c->n_dom; ++d) {
        DomDev &D = c->domh[d];
        D.rate_unit = c->rate_unit;
        D.flux_unit = c->rate_unit / (D.dx_cm * D.dx_cm);
        D.alpha_int = c->p.alpha_b * D.dx_cm * D.dx_cm * D.dx_cm / c->rate_unit;
    }
    HIPCHK(hipMemcpyAsync(c->doms, c->domh.data(), sizeof(DomDev) * c->n_dom, hipMemcpyHostToDevice, c->stream));
    c->src_dirty = false;
    return TR_OK;
}

// Gauss-Legendre nodes and weights on [0, 1] for the sphere deposit: the
// roots of P_n by Newton's method from Tricomi's initial estimates.
tr_status upload_gauss_legendre(tr_ctx *c)
{
    double t[kGlNodes], w[kGlNodes];
    const int n = kGlNodes;
    for (int i = 1; i <= n; ++i) {
        double x = (1.0 - 1.0 / (8.0 * n * n) + 1.0 / (8.0 * n * n * n)) * std::cos(kPi * (4 * i - 1) / (4.0 * n + 2.0));
        double d = 0.0;
        for (int it = 0; it < 50; ++it) {
            double pm = 1.0, p = x;   // P_0, P_1
            for (int k = 2; k <= n; ++k) {
                const double pn = ((2 * k - 1) * x * p - (k - 1) * pm) / k;
                pm = p;
                p = pn;
            }
            d = n * (pm - x * p) / (1.0 - x * x);   // P_n'
            const double step = p / d;
            x -= step;
            if (std::fabs(step) < 1e-17) break;
        }
        t[i - 1] = 0.5 * (1.0 + x);
        w[i - 1] = 1.0 / ((1.0 - x * x) * d * d);
    }
    HIPCHK(hipMemcpyToSymbol(HIP_SYMBOL(c_gl_t), t, sizeof(t)));
    HIPCHK(hipMemcpyToSymbol(HIP_SYMBOL(c_gl_w), w, sizeof(w)));
    return TR_OK;
}

// Guard band of the FP32 pixel classifier: 1e-5 N_side (at least 2e-5), several
// times the worst-case FP32 error of the pixel-edge quantities (a few 1e-7 N_side).
float guard_tolerance(int nside) { return 1e-5f * std::max(2.0f, (float)nside); }

// The angular-weight table of the context's N_side and s: for nodes of r = 1,
// 2, 4, ... 32 target sizes the offsets up to (2/theta + 1) r target sizes per
// axis (every node accepted at the smallest opening angle lies inside); nodes
// outside are classified by the walk.  Classifying a node takes about 180
// vector instructions of a wave more than reading its entry, and building an
// entry twice that: a ratio gets at most 32 entries per cell (a target accepts
// about 50 nodes of each of the middle ratios), so that the table has paid for
// itself within about two sweeps, at least 65536 and at most 16 million (theta
// 0.5 needs 1.8 million at r = 16 and 14.7 million at r = 32, 0.4 to 0.6 GB,
// which takes the walks of 128^3 from 55 to 33 ms, built in 8 ms (k_atab twice); r = 64 would take 8 times
// that for under 1% of the nodes).
tr_status build_angular_table(tr_ctx *c)
{
    const int s = c->p.subsample, ns = c->p.nside;
    double th = c->p.theta;
    if (c->p.theta_if > 0.0) th = std::min(th, c->p.theta_if);
    if (c->p.theta_src > 0.0) th = std::min(th, c->p.theta_src);
    th = std::max(th, 0.05);
    const double most = std::min(1.6e7, std::max(65536.0, 32.0 * (double)c->n_cells));
    int root = 1;   // nodes as large as the root are never accepted
    for (auto &t : c->topo) root = std::max(root, t.root_size);
    // accepted: size < theta d; its parent was not: its centre within 2 size / th, and the node's
    // within half the parent's diagonal of that (both with a margin)
    const double near = 0.999 / std::max(c->p.theta, 0.05), far = 1.001 * (2.0 / th + 0.8660254037844386);
    const double shell = 4.0 / 3.0 * kPi * (far * far * far - near * near * near);   // in node volumes
    for (int ratios = kAtabRatios; ratios > 0; --ratios) {
        AtabGeom G{};
        G.near2 = near * near;
        G.far2 = far * far;
        int64_t nk = 0;
        for (int q = 0; q < kAtabRatios; ++q) {
            G.base[q] = (int32_t)nk;
            G.w[q] = -1;
            if (q >= ratios || (1 << q) >= root) continue;
            double w = std::ceil((2.0 / th + 1.0) * (double)(1 << q));
            if (q < kAtabShell) w = std::min(w, std::floor((std::cbrt(most) - 1.0) / 2.0));
            const double keys = (2.0 * w + 1.0) * (2.0 * w + 1.0) * (2.0 * w + 1.0);
            if (q >= kAtabShell && (shell * (double)(1 << (3 * q)) > most || keys > 4e7)) continue;
            G.w[q] = (int)w;
            nk += (int64_t)keys;
        }
        G.nkeys = (int32_t)nk;
        if (nk == 0) return TR_OK;
        const int waves = 4 * (int)std::min<int64_t>((nk + 255) / 256, (int64_t)c->n_cu * 16);
        const int run = (int)((nk + waves - 1) / waves);
        int64_t *sums = nullptr;
        tr_status st;
        if ((st = dalloc(c, (void **)&sums, sizeof(int64_t) * (size_t)waves))) return st;
        auto launch = [&](int32_t *idx, int32_t *pool) {
            hipLaunchKernelGGL(k_atab, dim3(waves / 4), dim3(256), 0, c->stream, G, ns, s, guard_tolerance(ns), run, sums,
                               idx, pool, c->queue + 1);
        };
        launch(nullptr, nullptr);
        std::vector<int64_t> h((size_t)waves);
        if (hipMemcpyAsync(h.data(), sums, sizeof(int64_t) * (size_t)waves, hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
            hipStreamSynchronize(c->stream) != hipSuccess) {
            dfree(sums);
            return fail(c, TR_EHIP, "angular table: counting failed");
        }
        int64_t tot = 0;
        for (auto &v : h) {
            const int64_t n = v;
            v = tot;   // first unit (4 pairs) of each run
            tot += n;
        }
        if (tot >= 1ll << 25) {   // (first unit << 6) | (pairs - 1) below kDynEntry: without the largest ratio
            dfree(sums);
            continue;
        }
        if ((st = dalloc(c, (void **)&c->atab_pool, sizeof(int32_t) * 4 * (size_t)tot)) ||
            (st = dalloc(c, (void **)&c->atab_idx, sizeof(int32_t) * (size_t)nk))) {
            dfree(sums);
            dfree(c->atab_pool);
            dfree(c->atab_idx);
            if (ratios == 1) return st;
            (void)hipGetLastError();   // no memory for it: without the largest ratio
            c->err.clear();
            continue;
        }
        hipError_t e = hipMemcpyAsync(sums, h.data(), sizeof(int64_t) * (size_t)waves, hipMemcpyHostToDevice, c->stream);
        if (e == hipSuccess) {
            launch(c->atab_idx, c->atab_pool);
            e = hipStreamSynchronize(c->stream);
        }
        dfree(sums);
        if (e != hipSuccess) {
            dfree(c->atab_idx);
            dfree(c->atab_pool);
            return fail(c, TR_EHIP, std::string("angular table: ") + hipGetErrorString(e));
        }
        c->atab = G;
        return TR_OK;
    }
    return TR_OK;
}

tr_status read_flags(tr_ctx *c)
{
    int32_t f[2] = {0, 0};
    HIPCHK(hipMemcpyAsync(f, c->err_flags, sizeof(f), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(hipStreamSynchronize(c->stream));
    if (f[0] & 1) return fail(c, TR_EINVAL, "a source lies outside its domain or has a bad rate");
    if (f[0] & 2) return fail(c, TR_EINVAL, "n_h or f_prev holds a negative or non-finite value");
    if (f[0] & 4) return fail(c, TR_EINVAL, "source deposit stack overflow");
    return TR_OK;
}

// Device address of the static scratch, resolved once per device with that
// device current (the array's host-side name is only a stand-in for it).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

hipError_t static_scratch(int dev, void **out)
{
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

// message of the last call made without a context, per thread
thread_local std::string g_free_err;

tr_status fail_free(tr_status s, const std::string &m)
{
    g_free_err = m;
    return s;
}

}  // namespace

extern "C" {

tr_status tr_create(tr_ctx **out, const tr_params *p, void *stream)
{
    if (!out || !p) return TR_EINVAL;
    *out = nullptr;
    tr_ctx *c = new (std::nothrow) tr_ctx();
    if (!c) return TR_ENOMEM;
    tr_status s = check_params(c, *p);
    if (s) {
        delete c;
        return s;
    }
    c->p = *p;
    c->stream = (hipStream_t)stream;
    if (hipGetDevice(&c->device) != hipSuccess) {
        delete c;
        return TR_EHIP;
    }
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, c->device) != hipSuccess) {
        delete c;
        return TR_EHIP;
    }
    c->n_cu = prop.multiProcessorCount;
    void *sp = nullptr;
    if (static_scratch(c->device, &sp) != hipSuccess) {   // resolved here, outside any capture
        delete c;
        return TR_EHIP;
    }
    if (hipMalloc((void **)&c->queue, 64) != hipSuccess || hipMalloc((void **)&c->stats, 64) != hipSuccess ||
        hipMalloc((void **)&c->err_flags, 64) != hipSuccess || hipEventCreate(&c->ev0) != hipSuccess ||
        hipEventCreate(&c->ev1) != hipSuccess) {
        tr_destroy(c);
        return TR_ENOMEM;
    }
    // flags and counters start at zero (a sync before any launch reads them)
    if (hipMemset(c->queue, 0, 64) != hipSuccess || hipMemset(c->stats, 0, 64) != hipSuccess ||
        hipMemset(c->err_flags, 0, 64) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
        tr_destroy(c);
        return TR_EHIP;
    }
    if (upload_gauss_legendre(c) != TR_OK) {
        tr_destroy(c);
        return TR_EHIP;
    }
    *out = c;
    return TR_OK;
}

void tr_destroy(tr_ctx *c)
{
    if (!c) return;
    if (c->stream) (void)hipStreamSynchronize(c->stream);
    else (void)hipDeviceSynchronize();
    free_domains(c);
    dfree(c->queue);
    dfree(c->stats);
    dfree(c->err_flags);
    if (c->pinned) (void)hipHostFree(c->pinned);
    if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    if (c->ev0) (void)hipEventDestroy(c->ev0);
    if (c->ev1) (void)hipEventDestroy(c->ev1);
    delete c;
}

const char *tr_last_error(const tr_ctx *c) { return c ? c->err.c_str() : g_free_err.c_str(); }

tr_status tr_set_domains(tr_ctx *c, int32_t n_domains, const tr_domain *doms)
{
    if (!c) return TR_EINVAL;
    if (n_domains <= 0 || !doms) return fail(c, TR_EINVAL, "need at least one domain");
    HIPCHK(hipStreamSynchronize(c->stream));
    free_domains(c);
    c->topo.assign(n_domains, DomTopo());
    for (int d = 0; d < n_domains; ++d) {
        const std::string m = build_topology(doms[d], c->p, c->topo[d]);
        if (!m.empty()) return fail(c, TR_EINVAL, "domain " + std::to_string(d) + ": " + m);
    }
    c->n_dom = n_domains;
    c->depth_max = 0;
    c->nr_max = 0;
    for (auto &t : c->topo) {
        c->depth_max = std::max(c->depth_max, t.depth);
        c->nr_max = std::max(c->nr_max, t.n_radial);
    }
    // global node numbering: level-major, domains in order inside a level
    const int L = c->depth_max;
    std::vector<std::vector<int64_t>> off(L, std::vector<int64_t>(n_domains, 0));
    std::vector<std::vector<int64_t>> lbase(n_domains);   // local first index of each level
    c->level_begin.assign(L + 1, 0);
    int64_t g = 0;
    for (int l = 0; l < L; ++l) {
        c->level_begin[l] = g;
        for (int d = 0; d < n_domains; ++d) {
            off[l][d] = g;
            const auto &t = c->topo[d];
            if (l < t.depth) g += t.level_count[l];
        }
    }
    c->level_begin[L] = g;
    c->n_nodes = g;
    for (int d = 0; d < n_domains; ++d) {
        const auto &t = c->topo[d];
        int64_t b = 0;
        for (int l = 0; l < t.depth; ++l) {
            lbase[d].push_back(b);
            b += t.level_count[l];
        }
    }
    auto gidx = [&](int d, int64_t local) -> int64_t {
        const auto &lb = lbase[d];
        int l = (int)(std::upper_bound(lb.begin(), lb.end(), local) - lb.begin()) - 1;
        return off[l][d] + (local - lb[l]);
    };
    std::vector<int4> geo(g), olo(g), oext(g);
    std::vector<int2> topo(g);
    int64_t ncell = 0;
    for (auto &t : c->topo) ncell += t.n_cells;
    if (ncell > INT32_MAX) return fail(c, TR_EINVAL, "too many cells");
    c->n_cells = ncell;
    std::vector<int32_t> cnode(ncell), cdom(ncell), order(ncell);
    std::vector<double> r64;
    std::vector<float> r32;
    c->domh.assign(n_domains, DomDev());
    int64_t cbase = 0;
    for (int d = 0; d < n_domains; ++d) {
        const auto &t = c->topo[d];
        const int64_t nn = (int64_t)t.size.size();
        int64_t first_level_end = t.level_count.empty() ? 0 : 0;
        (void)first_level_end;
        for (int64_t i = 0; i < nn; ++i) {
            const int64_t gi = gidx(d, i);
            const int32_t sz = t.size[i];
            bool partial = false;
            for (int a = 0; a < 3; ++a)
                if (t.olo[3 * i + a] != t.lo[3 * i + a] || t.oext[3 * i + a] != sz) partial = true;
            geo[gi] = int4{t.lo[3 * i], t.lo[3 * i + 1], t.lo[3 * i + 2], sz | (partial ? kPartialBit : 0)};
            olo[gi] = int4{t.olo[3 * i], t.olo[3 * i + 1], t.olo[3 * i + 2], 0};
            oext[gi] = int4{t.oext[3 * i], t.oext[3 * i + 1], t.oext[3 * i + 2], 0};
            if (t.nchild[i] == 0) topo[gi] = int2{(int)(cbase + t.first[i]), 0};
            else topo[gi] = int2{(int)gidx(d, t.first[i]), t.nchild[i]};
        }
        for (int64_t q = 0; q < t.n_cells; ++q) {
            cnode[cbase + q] = (int32_t)gidx(d, t.cell_node[q]);
            cdom[cbase + q] = d;
            order[cbase + q] = (int32_t)(cbase + t.morton[q]);
        }
        DomDev &D = c->domh[d];
        D.root = (int32_t)gidx(d, 0);
        D.nr = t.n_radial;
        D.r_off = (int32_t)r64.size();
        D.cell_off = (int32_t)cbase;
        D.n_cells = (int32_t)t.n_cells;
        D.dx_cm = t.dx_cm;
        for (int q = 0; q < 3; ++q) D.ext[q] = t.ext[q];
        D.rate_unit = 1.0;
        D.flux_unit = 1.0 / (t.dx_cm * t.dx_cm);
        D.alpha_int = c->p.alpha_b * t.dx_cm * t.dx_cm * t.dx_cm;
        D.rc_inv = 1.0 / t.r_coef;
        for (double r : t.r_cells) {
            r64.push_back(r);
            r32.push_back((float)r);
        }
        cbase += t.n_cells;
    }
    tr_status s;
    if ((s = upload(c, c->geo, geo)) || (s = upload(c, c->olo, olo)) || (s = upload(c, c->oext, oext)) ||
        (s = upload(c, c->topo_d, topo)) || (s = upload(c, c->cell_node, cnode)) ||
        (s = upload(c, c->cell_dom, cdom)) || (s = upload(c, c->order, order)) || (s = upload(c, c->r64, r64)) ||
        (s = upload(c, c->r32, r32)) || (s = upload(c, c->doms, c->domh)))
        return s;
    if ((s = dalloc(c, (void **)&c->mom, sizeof(double) * MO_COUNT * (size_t)g))) return s;
    if ((s = dalloc(c, &c->packA, 32 * (size_t)g))) return s;
    if ((s = dalloc(c, &c->packB, 32 * (size_t)g))) return s;
    if ((s = dalloc(c, (void **)&c->ndot, sizeof(double) * (size_t)ncell))) return s;
    if ((s = dalloc(c, (void **)&c->hist, sizeof(unsigned int) * kSelBins * (size_t)n_domains))) return s;
    if ((s = dalloc(c, (void **)&c->dprefix, sizeof(unsigned long long) * n_domains))) return s;
    if ((s = dalloc(c, (void **)&c->drank, sizeof(unsigned long long) * (n_domains + 1)))) return s;
    if ((s = dalloc(c, (void **)&c->dmax, sizeof(unsigned long long) * n_domains))) return s;
    c->sxyz.assign(n_domains, {});
    c->sq.assign(n_domains, {});
    c->src_dirty = true;
    HIPCHK(hipStreamSynchronize(c->stream));
    if (c->p.subsample * c->p.subsample * c->p.subsample <= 64 && (s = build_angular_table(c))) return s;
    return TR_OK;
}

tr_status tr_cell_count(const tr_ctx *c, int32_t dom, int64_t *n)
{
    if (!c || !n) return TR_EINVAL;
    if (dom == -1) {
        *n = c->n_cells;
        return TR_OK;
    }
    if (dom < 0 || dom >= c->n_dom) return TR_EINVAL;
    *n = c->topo[dom].n_cells;
    return TR_OK;
}

tr_status tr_set_sources(tr_ctx *c, int32_t dom, int64_t n, const double *xyz, const double *q)
{
    if (!c) return TR_EINVAL;
    if (dom < 0 || dom >= c->n_dom) return fail(c, TR_EINVAL, "bad domain index");
    if (n < 0 || (n > 0 && (!xyz || !q))) return fail(c, TR_EINVAL, "bad source arrays");
    const auto &t = c->topo[dom];
    for (int64_t s = 0; s < n; ++s) {
        if (!(q[s] >= 0) || !std::isfinite(q[s])) return fail(c, TR_EINVAL, "source rates must be finite and >= 0");
        for (int a = 0; a < 3; ++a) {
            const double u = xyz[3 * s + a] / t.dx_cm;
            if (!std::isfinite(u) || u < -1e-9 || u > t.ext[a] + 1e-9)
                return fail(c, TR_EINVAL, "source " + std::to_string(s) + " lies outside domain " + std::to_string(dom));
        }
    }
    c->sxyz[dom].assign(xyz, xyz + 3 * n);
    c->sq[dom].assign(q, q + n);
    c->src_dirty = true;
    c->built = false;
    drop_graph(c);
    return TR_OK;
}

}  // extern "C"

namespace {

// Enqueues the tree build (no host synchronisation; capturable).
tr_status enqueue_build(tr_ctx *c, const double *n_h, const double *f_prev, int32_t thin)
{
    const int64_t nn = c->n_nodes, ncell = c->n_cells;
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, c->stream, c->err_flags, (int64_t)2, 0);
    hipLaunchKernelGGL(k_fill_f64, dim3(grid1(ncell)), dim3(256), 0, c->stream, c->ndot, ncell, 0.0);
    if (c->n_src_dev > 0)
    {
        if (c->p.src_radius_cm > 0.0)
            hipLaunchKernelGGL(k_deposit_spheres, dim3(grid1(c->n_src_dev, 64)), dim3(64), 0, c->stream, c->d_sxyz,
                               c->d_sq, c->d_sdom, c->n_src_dev, c->doms, c->geo, c->topo_d, c->p.src_radius_cm,
                               c->ndot, c->err_flags);
        else
            hipLaunchKernelGGL(k_deposit, dim3(grid1(c->n_src_dev, 64)), dim3(64), 0, c->stream, c->d_sxyz, c->d_sq,
                               c->d_sdom, c->n_src_dev, c->doms, c->geo, c->topo_d, c->ndot, c->err_flags);
    }
    hipLaunchKernelGGL(k_cell_quantities, dim3(grid1(ncell)), dim3(256), 0, c->stream, ncell, n_h, c->ndot, f_prev,
                       c->cell_node, c->cell_dom, c->doms, c->geo, thin, c->mom, nn, c->err_flags);
    for (int l = c->depth_max - 2; l >= 0; --l) {
        const int64_t b = c->level_begin[l], e = c->level_begin[l + 1];
        if (e > b)
            hipLaunchKernelGGL(k_reduce_level, dim3(grid1(e - b)), dim3(256), 0, c->stream, b, e, c->topo_d, c->mom, nn);
    }
    if (c->p.precision == TR_FP32C)
        hipLaunchKernelGGL((k_pack<float, float4>), dim3(grid1(nn)), dim3(256), 0, c->stream, nn, c->mom, (float4 *)c->packA,
                           (float4 *)c->packB, c->geo);
    else
        hipLaunchKernelGGL((k_pack<double, double4>), dim3(grid1(nn)), dim3(256), 0, c->stream, nn, c->mom,
                           (double4 *)c->packA, (double4 *)c->packB, c->geo);
    HIPCHK(hipGetLastError());
    return TR_OK;
}

// Enqueues delta_cell per domain into st.dmax (capturable, no errors checked).
template <typename Doms>
void launch_delta(const Doms &D, int64_t n_cells, const double *f_new, const double *f_old, const SelectState &st, int n_cu,
                  hipStream_t stream)
{
    const unsigned blocks = (unsigned)std::min<int64_t>((n_cells + 4 * kSelThreads - 1) / (4 * kSelThreads), 4 * (int64_t)n_cu);
    hipLaunchKernelGGL(k_select_init<Doms>, dim3(grid1((int64_t)D.n * kSelBins)), dim3(256), 0, stream, D, n_cells, st);
    for (int pass = 0; pass < kSelPasses; ++pass) {
        hipLaunchKernelGGL(k_select<Doms>, dim3(std::min(blocks, (unsigned)n_cu)), dim3(kSelThreads), 0, stream, D, n_cells, f_old, pass, st);
        if (D.n > kSelPickWaves) hipLaunchKernelGGL(k_pick, dim3(grid1(D.n, 4)), dim3(256), 0, stream, D.n, n_cells, pass, st);
    }
    hipLaunchKernelGGL(k_delta<Doms>, dim3(blocks), dim3(kSelThreads), 0, stream, D, n_cells, f_new, f_old, st);
}

tr_status enqueue_delta(tr_ctx *c, const double *f_new, const double *f_old)
{
    const SelectState st{c->hist, c->dprefix, c->drank, c->dmax, (unsigned *)(c->drank + c->n_dom)};
    launch_delta(DomByArray{c->doms, c->n_dom}, c->n_cells, f_new, f_old, st, c->n_cu, c->stream);
    HIPCHK(hipGetLastError());
    return TR_OK;
}

tr_status check_build_args(tr_ctx *c, const double *n_h)
{
    if (c->n_dom == 0) return fail(c, TR_ESTATE, "tr_build needs tr_set_domains first");
    if (!n_h) return fail(c, TR_EINVAL, "n_h is NULL");
    tr_status s;
    if (c->src_dirty && (s = upload_sources(c))) return s;
    return TR_OK;
}

}  // namespace

extern "C" {

tr_status tr_build(tr_ctx *c, const double *n_h, const double *f_prev, int32_t thin)
{
    if (!c) return TR_EINVAL;
    tr_status s;
    if ((s = check_build_args(c, n_h))) return s;
    (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
    if ((s = enqueue_build(c, n_h, f_prev, thin))) return s;
    if ((s = read_flags(c))) return s;
    c->built = true;
    c->built_prec = c->p.precision;
    return TR_OK;
}

tr_status tr_sweep(tr_ctx *c, double *f_out, uint8_t *ion)
{
    if (!c) return TR_EINVAL;
    if (!f_out) return fail(c, TR_EINVAL, "f_out is NULL");
    return launch_sweep(c, nullptr, c->n_cells, f_out, ion, true, 0, 0, 0, 0);
}

tr_status tr_sweep_targets(tr_ctx *c, const int64_t *targets, int64_t n, double *f_out, uint8_t *ion)
{
    if (!c) return TR_EINVAL;
    if (n < 0 || (n > 0 && (!targets || !f_out))) return fail(c, TR_EINVAL, "bad target list");
    return launch_sweep(c, targets, n, f_out, ion, true, 0, 0, 0, 0);
}

tr_status tr_delta(tr_ctx *c, const double *f_new, const double *f_old, double *delta_host)
{
    if (!c) return TR_EINVAL;
    if (!f_new || !f_old || !delta_host) return fail(c, TR_EINVAL, "NULL argument");
    if (c->n_dom == 0) return fail(c, TR_ESTATE, "no domains");
    (void)hipGetLastError();
    tr_status s;
    if ((s = enqueue_delta(c, f_new, f_old))) return s;
    const int nd = c->n_dom;
    std::vector<unsigned long long> dm(nd);
    HIPCHK(hipMemcpyAsync(dm.data(), c->dmax, sizeof(unsigned long long) * nd, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(hipStreamSynchronize(c->stream));
    for (int d = 0; d < nd; ++d) std::memcpy(&delta_host[d], &dm[d], 8);
    return TR_OK;
}

tr_status tr_step(tr_ctx *c, const double *n_h, const double *f_prev, double *f_out, uint8_t *ion, double *delta_host)
{
    if (!c) return TR_EINVAL;
    if (!f_prev || !f_out || !delta_host) return fail(c, TR_EINVAL, "NULL argument");
    if (f_prev == f_out) return fail(c, TR_EINVAL, "f_prev and f_out must be different buffers");
    tr_status s;
    if ((s = check_build_args(c, n_h))) return s;
    const int nd = c->n_dom;
    const void *key[4] = {n_h, f_prev, f_out, ion};
    tr_ctx::GraphSlot *slot = nullptr;
    for (auto &g : c->gslot) {
        bool same = g.exec != nullptr;
        for (int q = 0; q < 4 && same; ++q) same = key[q] == g.key[q];
        if (same) slot = &g;
    }
    (void)hipGetLastError();
    if (!slot) {
        slot = c->gslot[0].used <= c->gslot[1].used ? &c->gslot[0] : &c->gslot[1];
        drop_slot(*slot);
        // plan (and allocate) the sweep before capturing it
        LaunchPlan L;
        if ((s = plan_sweep(c, c->n_cells, c->waves, c->tpc, c->bufmode, c->intmode, L))) return s;
        if (!c->cap_stream) HIPCHK(hipStreamCreate(&c->cap_stream));
        const size_t host = 64 + sizeof(unsigned long long) * (size_t)nd;
        if (c->pinned_bytes < host) {   // (more domains than any step before: no captured graph writes the old one)
            if (c->pinned) (void)hipHostFree(c->pinned);
            c->pinned = nullptr;
            c->pinned_bytes = 0;
            HIPCHK(hipHostMalloc(&c->pinned, host));
            c->pinned_bytes = host;
        }
        hipStream_t user = c->stream;
        c->stream = c->cap_stream;
        HIPCHK(hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed));
        tr_status cs = enqueue_build(c, n_h, f_prev, 0);
        const bool built = c->built;
        const tr_precision bp = c->built_prec;
        c->built = true;
        c->built_prec = c->p.precision;
        if (!cs) cs = launch_sweep(c, nullptr, c->n_cells, f_out, ion, false, 0, 0, 0, 0);
        c->built = built;
        c->built_prec = bp;
        if (!cs) cs = enqueue_delta(c, f_out, f_prev);
        if (!cs && (hipMemcpyAsync(c->pinned, c->err_flags, 8, hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
                    hipMemcpyAsync((char *)c->pinned + 8, c->queue, 8, hipMemcpyDeviceToHost, c->stream) != hipSuccess))
            cs = fail(c, TR_EHIP, "capture of the flag copy failed");
        if (!cs && hipMemcpyAsync((char *)c->pinned + 64, c->dmax, sizeof(unsigned long long) * (size_t)nd,
                                  hipMemcpyDeviceToHost, c->stream) != hipSuccess)
            cs = fail(c, TR_EHIP, "capture of the delta copy failed");
        hipGraph_t g = nullptr;
        const hipError_t ee = hipStreamEndCapture(c->cap_stream, &g);
        c->stream = user;
        if (cs) {
            if (g) (void)hipGraphDestroy(g);
            return cs;
        }
        if (ee != hipSuccess) return fail(c, TR_EHIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(ee));
        slot->graph = g;
        HIPCHK(hipGraphInstantiate(&slot->exec, slot->graph, nullptr, nullptr, 0));
        for (int q = 0; q < 4; ++q) slot->key[q] = key[q];
    }
    slot->used = ++c->graph_clock;
    HIPCHK(hipGraphLaunch(slot->exec, c->stream));
    HIPCHK(hipStreamSynchronize(c->stream));
    c->timed_valid = false;   // no timed sweep in a step
    int32_t flags[4];
    std::memcpy(flags, c->pinned, 16);
    if (flags[3] & 4) return fail(c, TR_EHIP, "internal error: a HEALPix pixel index fell outside [0, N_PIX)");
    if (flags[3]) return fail(c, TR_EOVERFLOW, "a walk list overflowed; affected cells hold NaN");
    if (flags[0] & 1) return fail(c, TR_EINVAL, "a source lies outside its domain or has a bad rate");
    if (flags[0] & 2) return fail(c, TR_EINVAL, "n_h or f_prev holds a negative or non-finite value");
    if (flags[0] & 4) return fail(c, TR_EINVAL, "source deposit stack overflow");
    for (int d = 0; d < nd; ++d) std::memcpy(&delta_host[d], (char *)c->pinned + 64 + 8 * d, 8);
    c->built = true;
    c->built_prec = c->p.precision;
    return TR_OK;
}

tr_status tr_solve(tr_ctx *c, const double *n_h, double *f_out, uint8_t *ion, int32_t *iters_out, double *delta_out)
{
    if (!c) return TR_EINVAL;
    if (!n_h || !f_out) return fail(c, TR_EINVAL, "NULL argument");
    tr_status s;
    const int64_t ncell = c->n_cells;
    if (c->solve_tmp_n < ncell) {
        drop_graph(c);
        dfree(c->solve_tmp);
        if ((s = dalloc(c, (void **)&c->solve_tmp, sizeof(double) * (size_t)ncell))) return s;
        c->solve_tmp_n = ncell;
    }
    // F^0: the optically thin sweep
    if ((s = tr_build(c, n_h, nullptr, 1))) return s;
    if ((s = tr_sweep(c, f_out, ion))) return s;
    std::vector<double> dl(c->n_dom, 0.0);
    int32_t it = 0;
    double dmax = INFINITY;
    bool conv = false;
    // iterations alternate between f_out and the scratch field; each is one graph launch
    double *cur = f_out, *nxt = c->solve_tmp;
    while (it < c->p.max_iter) {
        if ((s = tr_step(c, n_h, cur, nxt, ion, dl.data()))) return s;
        std::swap(cur, nxt);
        ++it;
        dmax = 0;
        for (double v : dl) dmax = std::max(dmax, v);
        if (dmax < c->p.eps_lim) {
            conv = true;
            break;
        }
    }
    if (cur != f_out)
        HIPCHK(hipMemcpyAsync(f_out, cur, sizeof(double) * (size_t)ncell, hipMemcpyDeviceToDevice, c->stream));
    if (iters_out) *iters_out = it;
    if (delta_out) *delta_out = dmax;
    if ((s = tr_sync(c))) return s;
    if (!conv && c->p.max_iter > 0) return fail(c, TR_ENOCONV, "delta_cell did not fall below eps_lim");
    return TR_OK;
}

tr_status tr_set_precision(tr_ctx *c, tr_precision prec)
{
    if (!c) return TR_EINVAL;
    if (prec != TR_FP64 && prec != TR_FP32C) return fail(c, TR_EINVAL, "unknown precision");
    if (c->p.precision != prec) drop_graph(c);
    c->p.precision = prec;
    return TR_OK;
}

tr_status tr_set_launch(tr_ctx *c, int32_t waves, int32_t tpc, int32_t buffer, int32_t integration, int32_t atomics)
{
    if (!c) return TR_EINVAL;
    if (atomics < 0 || atomics > 2)
        return fail(c, TR_EINVAL, "atomics must be 0 (auto), 1 (hardware atomic adds) or 2 (compare-and-swap)");
    if (buffer < 0 || buffer > 2) return fail(c, TR_EINVAL, "buffer must be 0 (auto), 1 (LDS) or 2 (device memory)");
    if (integration < 0 || integration > 8)
        return fail(c, TR_EINVAL,
                    "integration must be 0 (auto), 1 (a lane per ray), 2 (a wave per ray), 3, 4, 5 (a group of 4, 8, "
                    "16 lanes per ray) or 6, 7, 8 (the same groups with the FP32 march)");
    if (!(waves == 0 || waves == 1 || waves == 2 || waves == 4 || waves == 8 || waves == 16))
        return fail(c, TR_EINVAL, "waves per target must be 0, 1, 2, 4, 8 or 16");
    if (tpc < 0) return fail(c, TR_EINVAL, "targets per CU must be >= 0");
    c->waves = waves;
    c->tpc = tpc;
    c->bufmode = buffer;
    c->intmode = integration;
    c->atommode = atomics;
    drop_graph(c);
    return TR_OK;
}

tr_status tr_autotune(tr_ctx *c, double *best_ms)
{
    if (!c) return TR_EINVAL;
    if (!c->built) return fail(c, TR_ESTATE, "tr_autotune needs tr_build first");
    c->tuned_int[c->p.precision == TR_FP32C ? 1 : 0] = 0;   // the first stages time the default forms
    c->tuned_atom[c->p.precision == TR_FP32C ? 1 : 0] = 0;
    // sample: every m-th cell in Morton order, enough to fill the chip a few times
    const int64_t want = std::min<int64_t>(c->n_cells, (int64_t)c->n_cu * 64);
    const int64_t step = std::max<int64_t>(1, c->n_cells / std::max<int64_t>(1, want));
    std::vector<int64_t> tg;
    std::vector<int32_t> ord(c->n_cells);
    HIPCHK(hipMemcpyAsync(ord.data(), c->order, sizeof(int32_t) * c->n_cells, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(hipStreamSynchronize(c->stream));
    for (int64_t i = 0; i < c->n_cells && (int64_t)tg.size() < want; i += step) tg.push_back(ord[i]);
    int64_t *dt = nullptr;
    double *fo = nullptr;
    tr_status s;
    if ((s = dalloc(c, (void **)&dt, sizeof(int64_t) * tg.size()))) return s;
    if ((s = dalloc(c, (void **)&fo, sizeof(double) * tg.size()))) { dfree(dt); return s; }
    HIPCHK(hipMemcpyAsync(dt, tg.data(), sizeof(int64_t) * tg.size(), hipMemcpyHostToDevice, c->stream));
    const int cand[5] = {1, 2, 4, 8, 16};
    double best = INFINITY;
    int bw = 0, bb = 0, bi = 0;
    // mean of two timed sweeps after one untimed; false if the shape does not run
    auto timed = [&](int w, int bm, int im, double &ms_out, int am = 0) {
        LaunchPlan L;
        if (plan_sweep(c, (int64_t)tg.size(), w, 0, bm, im, L, am) != TR_OK) return false;
        float ms = 0, tot = 0;
        for (int rep = 0; rep < 3; ++rep) {
            if (launch_sweep(c, dt, (int64_t)tg.size(), fo, nullptr, true, w, 0, bm, im, am) != TR_OK) return false;
            if (hipEventSynchronize(c->ev1) != hipSuccess) return false;
            (void)hipEventElapsedTime(&ms, c->ev0, c->ev1);
            if (rep > 0) tot += ms;
        }
        ms_out = tot / 2;
        return true;
    };
    // waves and buffer place with the default integration, then the integration form
    // (4 waves accumulate by compare-and-swap only when asked to)
    int ba = 0;
    for (int bm = 1; bm <= 2; ++bm)
        for (int w : cand) {
            const int am = w == 4 && bm == 1 && c->p.precision == TR_FP32C ? 2 : 0;
            double ms;
            if (timed(w, bm, 0, ms, am) && ms < best) {
                best = ms;
                bw = w;
                bb = bm;
                bi = 0;
                ba = am;
            }
        }
    if (bw > 0)
        for (int im : {1, 2, 3, 4, 5, 6, 7, 8}) {
            if (im >= 6 && c->p.precision != TR_FP32C) break;
            double ms;
            if (timed(bw, bb, im, ms, ba) && ms < best) {
                best = ms;
                bi = im;
            }
        }
    // and the accumulation form where there is a choice (FP32 buffers in LDS, 4, 8 or 16 waves)
    if (bw >= 4 && bb == 1 && c->p.precision == TR_FP32C)
        for (int am : {1, 2}) {
            double ms;
            if (timed(bw, bb, bi, ms, am) && ms < best) {
                best = ms;
                ba = am;
            }
        }
    dfree(dt);
    dfree(fo);
    c->err.clear();
    (void)hipGetLastError();
    drop_graph(c);   // trial plans may have reallocated the scratch a graph refers to
    if (bw == 0) return fail(c, TR_EHIP, "no launch shape ran");
    c->tuned_waves[c->p.precision == TR_FP32C ? 1 : 0] = bw;
    c->tuned_buf[c->p.precision == TR_FP32C ? 1 : 0] = bb;
    c->tuned_int[c->p.precision == TR_FP32C ? 1 : 0] = bi;
    c->tuned_atom[c->p.precision == TR_FP32C ? 1 : 0] = ba;
    if (best_ms) *best_ms = best;
    return TR_OK;
}

tr_status tr_get_stats(tr_ctx *c, tr_stats *out)
{
    if (!c || !out) return TR_EINVAL;
    std::memset(out, 0, sizeof(*out));
    unsigned long long st[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int32_t q[2] = {0, 0};
    HIPCHK(hipMemcpyAsync(st, c->stats, sizeof(st), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(hipMemcpyAsync(q, c->queue, sizeof(q), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(hipStreamSynchronize(c->stream));
    out->n_cells = c->n_cells;
    out->n_nodes = c->n_nodes;
    out->nodes_accepted = (int64_t)st[0];
    out->nodes_tested = (int64_t)st[1];
    out->guard_recomputes = (int64_t)st[2];
    out->n_radial_max = c->nr_max;
    out->depth_max = c->depth_max;
    out->waves_per_target = c->last_waves;
    out->targets_per_cu = c->last_tpc;
    out->buffer_in_lds = c->last_lds;
    out->integration_wave = c->last_intw;
    out->lds_cas = c->last_cas;
    out->integration_fp32 = c->last_int32;
    out->rays_fp32 = (int64_t)st[3];
    out->rays_fp64_again = (int64_t)st[4];
    out->nodes_tabulated = (int64_t)st[5];
    out->rays_regrouped = (int64_t)st[6];
    out->overflow = q[1];
    float ms = 0;
    if (c->timed_valid && hipEventElapsedTime(&ms, c->ev0, c->ev1) == hipSuccess) out->last_sweep_ms = ms;
    (void)hipGetLastError();
    return TR_OK;
}

tr_status tr_delta_noalloc(const double *f_new, const double *f_old, const int64_t *dom_offsets, int32_t n_domains,
                           double *delta_dev, void *stream)
{
    if (!f_new || !f_old || !dom_offsets || !delta_dev) return fail_free(TR_EINVAL, "NULL argument");
    if (n_domains < 1 || n_domains > kStaticDomains)
        return fail_free(TR_EINVAL, "n_domains must be in [1, " + std::to_string(kStaticDomains) +
                                        "]: the static scratch holds " + std::to_string(kStaticDomains) + " domains");
    DomByRanges R{};
    R.n = n_domains;
    if (dom_offsets[0] != 0) return fail_free(TR_EINVAL, "dom_offsets[0] must be 0");
    for (int d = 0; d <= n_domains; ++d) {
        R.off[d] = dom_offsets[d];
        if (d > 0 && dom_offsets[d] <= dom_offsets[d - 1])
            return fail_free(TR_EINVAL, "every domain needs at least one cell (dom_offsets strictly increasing)");
    }
    const int64_t ncell = R.off[n_domains];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail_free(TR_EHIP, "hipGetDevice failed");
    void *sp = nullptr;
    const hipError_t e = static_scratch(dev, &sp);
    if (e != hipSuccess) return fail_free(TR_EHIP, std::string("hipGetSymbolAddress: ") + hipGetErrorString(e));
    unsigned *hist = (unsigned *)sp;
    unsigned long long *prefix = (unsigned long long *)sp + (size_t)kStaticDomains * (kSelBins / 2);
    unsigned long long *rank = prefix + kStaticDomains, *dmax = rank + kStaticDomains;
    const SelectState sel{hist, prefix, rank, dmax, (unsigned *)(dmax + kStaticDomains)};
    hipStream_t st = (hipStream_t)stream;
    const int nd = n_domains;
    int n_cu = 0;
    if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return fail_free(TR_EHIP, "hipDeviceGetAttribute failed");
    (void)hipGetLastError();
    // the last call's contents stay in the scratch: everything read is set here first
    launch_delta(R, ncell, f_new, f_old, sel, n_cu, st);
    hipLaunchKernelGGL(k_store_delta, dim3(1), dim3(64), 0, st, nd, dmax, delta_dev);
    const hipError_t le = hipGetLastError();
    if (le != hipSuccess) return fail_free(TR_EHIP, std::string("launch failed: ") + hipGetErrorString(le));
    return TR_OK;
}

#ifndef TR_SOURCE_DIGEST
#define TR_SOURCE_DIGEST "unknown"
#endif
const char *tr_source_digest(void) { return TR_SOURCE_DIGEST; }

tr_status tr_sync(tr_ctx *c)
{
    if (!c) return TR_EINVAL;
    HIPCHK(hipStreamSynchronize(c->stream));
    HIPCHK(hipGetLastError());
    int32_t q[2] = {0, 0};
    HIPCHK(hipMemcpy(q, c->queue, sizeof(q), hipMemcpyDeviceToHost));
    if (q[1] & 4) return fail(c, TR_EHIP, "internal error: a HEALPix pixel index fell outside [0, N_PIX)");
    if (q[1] & 2) return fail(c, TR_EINVAL, "a target index lies outside [0, n_cells); those outputs hold NaN");
    if (q[1]) return fail(c, TR_EOVERFLOW, "a walk list overflowed; affected targets hold NaN");
    return TR_OK;
}

}  // extern "C"
