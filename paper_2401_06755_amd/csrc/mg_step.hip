// One two-phase time step of arXiv 2401.06755, Sec. 2.4 (Stages 1-4), with
// linear (p = 1) filters, or quadratic ConvFEM filters (p = 2) for the terms
// that the paper's linear/quadratic combination gives them, on gfx950.
//
// Every operator of the step is a 3x3x3 filter sum f(u; w) (Sec. 2.2.2) over a
// field whose halo is synthesised at load time from that field's boundary
// rule: a mirror with sign +1 or -1 per face, and for the hydrostatic pressure
// a bottom halo that adds g h rho (Sec. 2.3.3).  The filters are tensor
// products of the 1D linear-element vectors
//     M = h [1, 4, 1] / 6 (mass),  G = [-1, 0, 1] / 2 (first derivative),
//     K = [-1, 2, -1] / h (stiffness),
// evaluated separably: the linear filters by a z-march over LDS-staged planes
// (mg_step_linear.hip), the quadratic ones (5x5x5) here, in 8^3 blocks staged in
// LDS.  The three pressure solves, run by the multigrid hierarchy of this
// library with a fixed cycle count, take most of a step.
//
// Boundary rules on the tank box (Sec. 3.1: free-slip side and bottom walls,
// an outlet with zero pressure on top):
//   C, rho, mu, k and the scalars made from them: +mirror on all faces;
//   velocity component d: -mirror on the walls normal to d, except the top;
//   component d of a vector made from grad C: -mirror on both faces normal to d;
//   p_nh and its increment: +mirror, -mirror on top;
//   p_hs: +mirror on the sides, -mirror on top, mirror + g h rho on the bottom.
// In the Petrov-Galerkin formulas (Eqs. k-abs special case, k-square, a_psi,
// the normalisation and Eq. negativek) the gradient Psi_x is taken in
// derivative units, f(Psi; w_x) / m_l; the residuals use the filters as
// printed.  mu blends like Eq. rho.  The velocities take the isotropic
// coefficient of Eq. k_Psi-n; the volume fraction the anisotropic compressive
// coefficients of Sec. 2.3.5 with the linear detectors, evaluated with the
// new velocity.  The surface-tension source of the momentum residual takes the
// sign that the Stage-1 pressure balances (Eq. hydro-pressure): with the
// curvature div n of Eq. surface-tension-k, the pressure of Eq. ph_disc has the
// physical Laplace jump across a drop and gradient -s_t, so s_t enters the
// predictor as +f(s_t; w_m).
#include "mg_async.h"
#include "mg_step.h"

#include <cmath>
#include <cstring>
#include <string>

using namespace nn4mg;

namespace {

__device__ inline size_t at(const Grid &g, int i, int j, int k)
{
    return (size_t)i + (size_t)g.nx * ((size_t)j + (size_t)g.ny * (size_t)k);
}

// ------------------------------------------------------------------ kernels

// ---- one workgroup per 8^3 block (the quadratic kernels) ----
constexpr int SB = 8;                // block edge
constexpr int SBT = SB * SB * SB;    // threads: one cell each

// This thread's cell of the workgroup's block (the block at (i0, j0, k0)); a
// ragged block's threads beyond the grid work on their cell clamped into it
// and write nothing.
struct BCell {
    int i0, j0, k0, i, j, k;
    bool valid;
    size_t id;
};
__device__ inline BCell bcell(const Grid &g)
{
    BCell c;
    const int bxn = (g.nx + SB - 1) / SB, byn = (g.ny + SB - 1) / SB;
    const int lb = blockIdx.x, t = threadIdx.x;
    c.i0 = (lb % bxn) * SB;
    c.j0 = ((lb / bxn) % byn) * SB;
    c.k0 = (lb / bxn / byn) * SB;
    const int i = c.i0 + t % SB, j = c.j0 + (t / SB) % SB, k = c.k0 + t / (SB * SB);
    c.valid = i < g.nx && j < g.ny && k < g.nz;
    c.i = min(i, g.nx - 1);
    c.j = min(j, g.ny - 1);
    c.k = min(k, g.nz - 1);
    c.id = at(g, c.i, c.j, c.k);
    return c;
}

unsigned blocks_of(const Grid &g)
{
    return (unsigned)(((g.nx + SB - 1) / SB) * ((g.ny + SB - 1) / SB) * ((g.nz + SB - 1) / SB));
}

// u . grad C with the new velocity (input of the residual of Eq. a_psi for C).
__global__ __launch_bounds__(256) void advection_c_kernel(Grid g, C3 q, C3 Cd, double *out)
{
    const size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= g.n) return;
    out[id] = q.p[0][id] * Cd.p[0][id] + q.p[1][id] * Cd.p[1][id] + q.p[2][id] * Cd.p[2][id];
}

__global__ __launch_bounds__(256) void copy3_kernel(size_t n, C3 src, F3 dst)
{
    const size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= n) return;
    for (int d = 0; d < 3; ++d) dst.p[d][id] = src.p[d][id];
}

// ------------------------------------------------ quadratic ConvFEM (order 2)
// The 5 x 5 x 5 filters of the quadratic ConvFEM (Sec. 2.2.3: the stencils of
// the vertex and mid nodes of quadratic Lagrange elements summed and
// averaged) are tensor products of
//     M2 = h [-1, 4, 24, 4, -1] / 30,  G2 = [1, -8, 0, 8, -1] / 12,
//     K2 = [1, -16, 30, -16, 1] / (12 h),
// applied with two-cell halos (Sec. 2.3.3): halo cell -1-m takes interior
// cell m with the field's sign, and the bottom halo of p_hs adds
// (2m + 1) g h rho (the gradient -rho g extrapolated over (2m + 1) h).  They
// serve the momentum terms, the interface geometry and the volume-fraction
// advection (Table disc_combinations, "linear/quadratic"); the volume-fraction
// diffusion and the two pressure equations keep the linear filters.
//
// Each kernel runs one workgroup per 8^3 block of cells.  A filter factors
// into three 5-tap passes, along x, then y, then z, so the block stages a
// field once on its cells plus the two-cell halo (12^3, the field's boundary
// rule applied while staging) and runs the passes through LDS: about 5 fused
// multiply-adds per tap and output instead of 15, and one global load per
// staged cell instead of one per tap.  Every sum keeps the x-then-y-then-z
// order with the same weights.

struct V5 {
    double w[5];
};

// Index up to two cells outside folded onto the cell it mirrors; s flips on a
// crossed face whose bit is set in odd.
__device__ inline int fold2(int i, int n, unsigned odd, unsigned lo_bit, unsigned hi_bit, double &s)
{
    if (i < 0) {
        if (odd & lo_bit) s = -s;
        return -1 - i;
    }
    if (i >= n) {
        if (odd & hi_bit) s = -s;
        return 2 * n - 1 - i;
    }
    return i;
}

// Padded value of u at (i, j, k) with the two-cell halo of rule odd.
struct Tap2 {
    const double *u;
    unsigned odd;
    Grid g;
    __device__ double operator()(int i, int j, int k) const
    {
        double s = 1.0;
        i = fold2(i, g.nx, odd, 1u, 2u, s);
        j = fold2(j, g.ny, odd, 4u, 8u, s);
        k = fold2(k, g.nz, odd, 16u, 32u, s);
        return s * u[at(g, i, j, k)];
    }
};


constexpr int QB = SB;                // output block edge
constexpr int QT = SBT;               // threads: one output cell each
constexpr int QS = QB + 4;            // staged edge
constexpr int QSN = QS * QS * QS;     // staged cells
constexpr int QRN = QB * QS * QS;     // x-pass outputs per filter (8 x 12 x 12)
constexpr int QPN = QB * QB * QS;     // y-pass outputs per filter (8 x 8 x 12)

// The 1D weights of the quadratic filters and the mass of a cell, computed on
// the host and passed by value so they stay in scalar registers.
struct QW {
    V5 M, G, K;
    double ml;
};
QW quad_weights(double h)
{
    const double m[5] = {-1.0, 4.0, 24.0, 4.0, -1.0}, gw[5] = {1.0, -8.0, 0.0, 8.0, -1.0},
                 kw[5] = {1.0, -16.0, 30.0, -16.0, 1.0};
    QW w;
    for (int q = 0; q < 5; ++q) {
        w.M.w[q] = h * m[q] / 30.0;
        w.G.w[q] = gw[q] / 12.0;
        w.K.w[q] = kw[q] / (12.0 * h);
    }
    w.ml = h * h * h;
    return w;
}

struct QLds {
    double s[QSN];    // the staged field
    double r[2][QRN]; // x pass: the derivative (or K) filter and M
    double p[3][QPN]; // y pass: M on r[0], the derivative (or K) filter on r[1], M on r[1]
};

// Index up to two cells outside folded onto the cell it mirrors; indices further
// out (the halo of a ragged block's cells beyond the grid, which feed no output)
// are clamped into range.
__device__ inline int qfold(int i, int n)
{
    const int f = i < 0 ? -1 - i : (i >= n ? 2 * n - 1 - i : i);
    return min(max(f, 0), n - 1);
}

// The cells of the staged region that this thread stages: where each is read
// from (32 bits: the state of a grid of 2^32 cells is beyond the memory) and
// which faces its halo crosses (bits as in the boundary rules; for a cell
// below the bottom its mirror distance m in the bits from 8 on).  Worked out
// once per kernel: for every field anew it was most of the integer work.
struct QGeo {
    static constexpr int NR = (QSN + QT - 1) / QT;
    unsigned off[NR], face[NR];
};
__device__ inline QGeo qgeo(const Grid &g, int i0, int j0, int k0)
{
    QGeo o;
#pragma unroll
    for (int q = 0; q < QGeo::NR; ++q) {
        const int idx = min((int)threadIdx.x + q * QT, QSN - 1);
        const int i = i0 + idx % QS - 2, j = j0 + (idx / QS) % QS - 2, k = k0 + idx / (QS * QS) - 2;
        o.off[q] = (unsigned)at(g, qfold(i, g.nx), qfold(j, g.ny), qfold(k, g.nz));
        o.face[q] = (i < 0 ? 1u : 0u) | (i >= g.nx ? 2u : 0u) | (j < 0 ? 4u : 0u) | (j >= g.ny ? 8u : 0u) |
                    (k >= g.nz ? 32u : 0u) | (k < 0 ? 16u | (unsigned)(-1 - k) << 8 : 0u);
    }
    return o;
}

// Each staging functor splits into fetch (the global loads of a cell) and value
// (the staged value from the fetched raw data and the faces crossed), so the
// loads of the next field can be in flight while the current field's passes run.

// A field with the two-cell halo of rule odd.
struct QTap {
    const double *u;
    unsigned odd;
    typedef double Raw;
    __device__ Raw fetch(unsigned off, unsigned) const { return u[off]; }
    __device__ double value(Raw r, unsigned face) const { return (__popc(face & odd) & 1) ? -r : r; }
};

// p_hs: +mirror on the sides, -mirror on top, and below the bottom the mirror
// plus (2m + 1) g h rho of the mirrored cell (rho +mirror on the sides).
struct QPhs {
    const double *p, *rho;
    double gh;
    struct Raw {
        double p, r;
    };
    __device__ Raw fetch(unsigned off, unsigned face) const { return {p[off], (face & 16u) ? rho[off] : 0.0}; }
    __device__ double value(const Raw &o, unsigned face) const
    {
        if (face & 16u) return o.p + (double)(2 * (face >> 8) + 1) * gh * o.r;
        return (face & 32u) ? -o.p : o.p;
    }
};

template <typename A, typename B>
struct QPair {
    A a;
    B b;
    struct Raw {
        typename A::Raw a;
        typename B::Raw b;
    };
    __device__ Raw fetch(unsigned off, unsigned face) const { return {a.fetch(off, face), b.fetch(off, face)}; }
};
template <typename A, typename B>
struct QMul : QPair<A, B> {
    __device__ double value(const typename QPair<A, B>::Raw &r, unsigned face) const
    {
        return this->a.value(r.a, face) * this->b.value(r.b, face);
    }
};
// Sum of two fields, each with its own boundary rule.
template <typename A, typename B>
struct QSum : QPair<A, B> {
    __device__ double value(const typename QPair<A, B>::Raw &r, unsigned face) const
    {
        return this->a.value(r.a, face) + this->b.value(r.b, face);
    }
};

// A component of the surface tension plus w rho (rho +mirror at every face);
// rho is read only where w is not zero.
struct QForce {
    QTap st;
    const double *rho;
    double w;
    struct Raw {
        double st, r;
    };
    __device__ Raw fetch(unsigned off, unsigned face) const
    {
        return {st.fetch(off, face), w != 0.0 ? rho[off] : 0.0};
    }
    __device__ double value(const Raw &o, unsigned face) const
    {
        const double v = st.value(o.st, face);
        return w != 0.0 ? v + w * o.r : v;
    }
};

// The next field's staging in registers: fetch issues its loads, commit
// writes the staged values to LDS (after the current field's passes; the x
// pass, the only reader of the staged field, is then done on every thread).
template <typename V>
struct QNext {
    typename V::Raw r[QGeo::NR];
    __device__ void fetch(const V &v, const QGeo &G)
    {
#pragma unroll
        for (int q = 0; q < QGeo::NR; ++q) r[q] = v.fetch(G.off[q], G.face[q]);
    }
    __device__ void commit(QLds &L, const V &v, const QGeo &G) const
    {
#pragma unroll
        for (int q = 0; q < QGeo::NR; ++q) {
            const int idx = (int)threadIdx.x + q * QT;
            if (idx < QSN) L.s[idx] = v.value(r[q], G.face[q]);
        }
    }
};

// Stage field v on the block plus its two-cell halo.
template <typename V>
__device__ inline void qstage(QLds &L, const V &v, const QGeo &G)
{
    QNext<V> n;
    n.fetch(v, G);
    n.commit(L, v, G);
}

// The x and y passes of the staged field: wa is G (derivatives) or K
// (Laplacian); DER: also the passes only the derivatives or the Laplacian
// need (else the mass filter alone).  Barrier before each pass.
template <bool DER>
__device__ inline void qpasses(QLds &L, const V5 &wa, const V5 &wm)
{
    const int t = threadIdx.x;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < (QRN + QT - 1) / QT; ++r) {
        const int idx = t + r * QT;
        if (idx < QRN) {
            const int x = idx % QB, yz = idx / QB;  // y + QS z
            const double *row = L.s + x + QS * yz;
            double ra = 0.0, rm = 0.0;
#pragma unroll
            for (int a = 0; a < 5; ++a) {
                const double v = row[a];
                if (DER) ra += wa.w[a] * v;
                rm += wm.w[a] * v;
            }
            if (DER) L.r[0][idx] = ra;
            L.r[1][idx] = rm;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < (QPN + QT - 1) / QT; ++r) {
        const int idx = t + r * QT;
        if (idx < QPN) {
            const int x = idx % QB, y = (idx / QB) % QB, z = idx / (QB * QB);
            const int o = x + QB * (y + QS * z);
            double p0 = 0.0, p1 = 0.0, p2 = 0.0;
#pragma unroll
            for (int b = 0; b < 5; ++b) {
                if (DER) {
                    p0 += wm.w[b] * L.r[0][o + QB * b];
                    p1 += wa.w[b] * L.r[1][o + QB * b];
                }
                p2 += wm.w[b] * L.r[1][o + QB * b];
            }
            if (DER) {
                L.p[0][idx] = p0;
                L.p[1][idx] = p1;
            }
            L.p[2][idx] = p2;
        }
    }
    __syncthreads();
}

// The derivative filters d[0..2] = f(u; w_x, w_y, w_z) (DER) and the mass
// filter d[3] = f(u; w_m) of the staged field at this thread's cell.
template <bool DER>
__device__ inline void qderiv(QLds &L, const QW &F, double d[4])
{
    qpasses<DER>(L, F.G, F.M);
    const int t = threadIdx.x;
    const int o = (t % QB) + QB * ((t / QB) % QB + QB * (t / (QB * QB)));  // z-plane stride QB * QB
    double dx = 0.0, dy = 0.0, dz = 0.0, mm = 0.0;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        const int q = o + QB * QB * c;
        const double Mc = F.M.w[c];
        if (DER) {
            dx += Mc * L.p[0][q];
            dy += Mc * L.p[1][q];
            dz += F.G.w[c] * L.p[2][q];
        }
        mm += Mc * L.p[2][q];
    }
    d[0] = dx;
    d[1] = dy;
    d[2] = dz;
    d[3] = mm;
}

// f(u; w_lap) = f(u; K M M + M K M + M M K) of the staged field at this thread's cell.
__device__ inline double qlap(QLds &L, const QW &F)
{
    qpasses<true>(L, F.K, F.M);
    const int t = threadIdx.x;
    const int o = (t % QB) + QB * ((t / QB) % QB + QB * (t / (QB * QB)));
    double out = 0.0;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        const int q = o + QB * QB * c;
        out += F.M.w[c] * (L.p[0][q] + L.p[1][q]) + F.K.w[c] * L.p[2][q];
    }
    return out;
}

// rho, mu, grad C in derivative units and the unit normals, quadratic filters.
__global__ __launch_bounds__(QT) void props2_kernel(Grid g, Phys P, const QW F, const double *C, double *rho,
                                                    double *mu, F3 Cd, F3 nrm)
{
    __shared__ QLds L;
    const BCell X = bcell(g);
    const QGeo cells = qgeo(g, X.i0, X.j0, X.k0);
    const size_t id = X.id;
    double d[4];
    qstage(L, QTap{C, kEven}, cells);
    qderiv<true>(L, F, d);
    if (!X.valid) return;
    const double c0 = C[id];
    rho[id] = P.rho_l * c0 + P.rho_g * (1.0 - c0);
    mu[id] = P.mu_l * c0 + P.mu_g * (1.0 - c0);
    double gd[3];
    for (int e = 0; e < 3; ++e) gd[e] = d[e] / F.ml;
    const double l = sqrt(gd[0] * gd[0] + gd[1] * gd[1] + gd[2] * gd[2]);
    const double eps = 1e-7 / g.h;
    for (int e = 0; e < 3; ++e) {
        Cd.p[e][id] = gd[e];
        nrm.p[e][id] = gd[e] / (eps + l);
    }
}

// Curvature div n and the surface-tension vectors, quadratic filters.
__global__ __launch_bounds__(QT) void surface2_kernel(Grid g, const QW F, double sigma, C3 nrm, C3 Cd, F3 st)
{
    __shared__ QLds L;
    const BCell X = bcell(g);
    const QGeo cells = qgeo(g, X.i0, X.j0, X.k0);
    double kap = 0.0;
    for (int e = 0; e < 3; ++e) {
        double d[4];
        qstage(L, QTap{nrm.p[e], rule_grad(e)}, cells);
        qderiv<true>(L, F, d);
        kap += d[e];
    }
    kap /= F.ml;
    if (!X.valid) return;
    for (int e = 0; e < 3; ++e) st.p[e][X.id] = sigma * kap * Cd.p[e][X.id];
}

// adv_c = q . grad q_c, quadratic filters.
__global__ __launch_bounds__(QT) void advection2_kernel(Grid g, const QW F, C3 q, F3 adv)
{
    __shared__ QLds L;
    const BCell X = bcell(g);
    const QGeo cells = qgeo(g, X.i0, X.j0, X.k0);
    const size_t id = X.id;
    const double q0[3] = {q.p[0][id], q.p[1][id], q.p[2][id]};
    for (int c = 0; c < 3; ++c) {
        double d[4];
        qstage(L, QTap{q.p[c], rule_vel(c)}, cells);
        qderiv<true>(L, F, d);
        if (X.valid) adv.p[c][id] = q0[0] * (d[0] / F.ml) + q0[1] * (d[1] / F.ml) + q0[2] * (d[2] / F.ml);
    }
}

// Isotropic PG diffusivity of each component, quadratic filters (the residual
// filter of Eq. a_psi is w_m / m_l - E with the quadratic mass).
__global__ __launch_bounds__(QT) void pg_velocity2_kernel(Grid g, const QW F, C3 q, C3 adv, const double *rho,
                                                          const double *mu, F3 kq)
{
    __shared__ QLds L;
    const BCell X = bcell(g);
    const QGeo cells = qgeo(g, X.i0, X.j0, X.k0);
    const size_t id = X.id;
    const double eps_k = 1e-7, a_kabs = 1.0 / 16.0, a_ksq = 4.0, h = g.h;
    const double u = q.p[0][id], v = q.p[1][id], w = q.p[2][id];
    for (int c = 0; c < 3; ++c) {
        double d[4], am[4];
        qstage(L, QTap{q.p[c], rule_vel(c)}, cells);
        qderiv<true>(L, F, d);
        const double px = d[0] / F.ml, py = d[1] / F.ml, pz = d[2] / F.ml;
        qstage(L, QTap{adv.p[c], kEven}, cells);
        qderiv<false>(L, F, am);
        const double a = 2.0 * (am[3] / F.ml - adv.p[c][id]);
        const double G = fabs(px) + fabs(py) + fabs(pz);
        const double kabs = a_kabs * h * fabs(a) / (eps_k + G / 3.0);
        const double g2 = px * px + py * py + pz * pz;
        const double advabs = fabs(u * px) + fabs(v * py) + fabs(w * pz);
        const double ksq = a_ksq * a * a * h / (eps_k + advabs / 3.0 * g2);
        const double kmax = h * (fabs(u) + fabs(v) + fabs(w));
        const double m = fmin(kmax, fmin(kabs, ksq));
        if (X.valid) kq.p[c][id] = rho[id] * m + mu[id];
    }
}

// One predictor iteration with the quadratic filters: s_c = rho m_l adv_c +
// f_lap(q_c, k_c) + f(p_hs + p_nh; w_c) + f(s_t,c; w_m) [- f(-g rho; w_m) for
// c = z], the same residual as the linear march.  The filters are linear, so the
// two pressures are summed while they are staged, and so are the surface tension
// and the weight: 13 filtered fields.  Bound by its LDS passes at one workgroup
// of 8 waves per compute unit (184 registers; held to 128 for a second workgroup
// it spills 42, and the step takes 2.75 ms).  With 15 fields and the halo worked
// out for each, 190 us at 80 x 64 x 160; now 152 us (the step 2.75 and 2.65 ms).
__global__ __launch_bounds__(QT) void momentum2_kernel(Grid g, Phys P, const QW F, C3 qn, const double *p_hs,
                                                       const double *p_nh, const double *rho, C3 qh, C3 kq, C3 st,
                                                       C3 adv, F3 qt, F3 qnext)
{
    __shared__ QLds L;
    const BCell X = bcell(g);
    const QGeo cells = qgeo(g, X.i0, X.j0, X.k0);
    const size_t id = X.id;
    const double r0 = rho[id];
    double gp[4];
    // each field's loads are issued before the previous field's passes
    using TP = QSum<QPhs, QTap>;
    using TM = QMul<QTap, QTap>;
    {
        const TP fp{{QPhs{p_hs, rho, P.g * g.h}, QTap{p_nh, kOddTop}}};
        QNext<TP> n0;
        n0.fetch(fp, cells);
        n0.commit(L, fp, cells);
    }
    {
        const TM m0{{QTap{kq.p[0], kEven}, QTap{qh.p[0], rule_vel(0)}}};
        QNext<TM> n1;
        n1.fetch(m0, cells);
        qderiv<true>(L, F, gp);
        n1.commit(L, m0, cells);
    }
#pragma unroll 1
    for (int c = 0; c < 3; ++c) {
        const QTap tq{qh.p[c], rule_vel(c)}, tk{kq.p[c], kEven};
        const QForce ts{QTap{st.p[c], rule_grad(c)}, rho, c == 2 ? P.g : 0.0};
        const double q0 = qh.p[c][id], kc = kq.p[c][id];
        // Eq. k-T: 1/2 [f(k q; w) + k f(q; w) - q f(k; w)]; f(k q) is staged
        double lkq, lq, lk;
        {
            QNext<QTap> n;
            n.fetch(tq, cells);
            lkq = qlap(L, F);
            n.commit(L, tq, cells);
        }
        {
            QNext<QTap> n;
            n.fetch(tk, cells);
            lq = qlap(L, F);
            n.commit(L, tk, cells);
        }
        {
            QNext<QForce> n;
            n.fetch(ts, cells);
            lk = qlap(L, F);
            n.commit(L, ts, cells);
        }
        double s = 0.5 * (lkq + kc * lq - q0 * lk);
        s += gp[c];
        double t4[4];
        {
            // the next component's product field
            const int cn = c < 2 ? c + 1 : c;
            const TM mn{{QTap{kq.p[cn], kEven}, QTap{qh.p[cn], rule_vel(cn)}}};
            QNext<TM> n;
            if (c < 2) n.fetch(mn, cells);
            qderiv<false>(L, F, t4);
            if (c < 2) n.commit(L, mn, cells);
        }
        s += t4[3];
        s += r0 * F.ml * adv.p[c][id];
        const double qnc = qn.p[c][id];
        const double tt = (-s / F.ml + r0 * qnc / P.dt) / (r0 / P.dt);
        if (X.valid) {
            qt.p[c][id] = tt;
            qnext.p[c][id] = 0.5 * (qnc + tt);
        }
    }
}

// Volume-fraction diffusivities with the quadratic advection residual and the
// detectors of Eqs. Sx-quad..Sz-quad (the smallest of three products of
// successive differences along each axis).
__global__ __launch_bounds__(QT) void pg_volume_fraction2_kernel(Grid g, const QW F, double dt, const double *C,
                                                                 C3 Cd, C3 q, const double *advc, F3 kd)
{
    __shared__ QLds L;
    const BCell X = bcell(g);
    const QGeo cells = qgeo(g, X.i0, X.j0, X.k0);
    const size_t id = X.id;
    const int i = X.i, j = X.j, k = X.k;
    const double Kp = 300.0, Km = 300.0, beta = 0.1, eps_x = 1e-4, Kpos = 3.0, eps_k = 1e-7, h = g.h;
    const double kmin = 1e-4 / dt * h * h, kclamp = 0.05 / dt * h * h;
    double am[4];
    qstage(L, QTap{advc, kEven}, cells);
    qderiv<false>(L, F, am);
    if (!X.valid) return;
    const double a = 2.0 * (am[3] / F.ml - advc[id]);
    const Tap2 tc{C, kEven, g};
    const double c0 = C[id];
    double S[3];
    for (int d = 0; d < 3; ++d) {
        double c[5];
        for (int o = -2; o <= 2; ++o)
            c[o + 2] = tc(i + (d == 0 ? o : 0), j + (d == 1 ? o : 0), k + (d == 2 ? o : 0));
        S[d] = (c[2] - c[1]) * (c[3] - c[2]);
        const double s1 = (c[1] - c[0]) * (c[2] - c[1]), s3 = (c[3] - c[2]) * (c[4] - c[3]);
        if (s1 < S[d]) S[d] = s1;
        if (s3 < S[d]) S[d] = s3;
    }
    if (c0 > 0.95 || c0 < 0.05) S[0] = S[1] = S[2] = -1.0;
    const double cx = Cd.p[0][id], cy = Cd.p[1][id], cz = Cd.p[2][id];
    const double u = q.p[0][id], v = q.p[1][id], w = q.p[2][id];
    const double g2 = cx * cx + cy * cy + cz * cz;
    const double proj = (u * cx + v * cy + w * cz) / (eps_x + g2);
    const double us = cx * proj, vs = cy * proj, ws = cz * proj;
    const double kneg = -beta * (u * u + v * v + w * w) / (eps_x + g2 * (fabs(us) + fabs(vs) + fabs(ws)) / 3.0);
    const double G = fabs(cx) + fabs(cy) + fabs(cz);
    const double kabs = (1.0 / 16.0) * h * fabs(a) / (eps_k + G / 3.0);
    for (int d = 0; d < 3; ++d) {
        const double wp = -fmax(-1.0, fmin(0.0, Kp * S[d]));
        const double wm = fmin(1.0, fmax(0.0, Km * S[d]));
        const double kk = wp * (Kpos * kabs) + wm * (kneg / h);
        kd.p[d][id] = fmax(-kmin, fmin(kclamp, kk));
    }
}

C3 c3(double *const p[3]) { return C3{{p[0], p[1], p[2]}}; }
F3 f3(double *const p[3]) { return F3{{p[0], p[1], p[2]}}; }

}  // namespace

// ------------------------------------------------------------------ host side

struct nn4mg_stepper {
    Grid g{};
    nn4mg_step_params p{};
    hipStream_t s = nullptr;
    nn4mg_t P = nullptr;       // constant-coefficient pressure hierarchy
    double *mem = nullptr;     // all work fields, one allocation
    double *rho, *mu, *Cd[3], *nrm[3], *st[3], *b, *px, *qa[3], *qb[3], *qt[3], *adv[3], *kq[3], *tmp;
    double *red = nullptr;     // per-block partials of sum C, then the volume (last entry)
    int nred = 0;
    hipEvent_t ev[4]{};        // step start / end, solve start / end
    // the step's solves are enqueued without waiting: per solve a start/end
    // event pair and a pinned slot for its state header, read after the step
    static constexpr int kSolves = 8;  // 1 + n_corr <= 8
    hipEvent_t sev[2 * kSolves]{};
    unsigned char *hdr = nullptr;
    bool pending[kSolves]{};
};

namespace {

constexpr int kFields = 29;

int hip_fail(hipError_t e, const char *what)
{
    std::string m = std::string(what) + ": " + hipGetErrorString(e);
    return set_error(NN4MG_EDEVICE, m.c_str());
}

#define STEP_TRY(expr, what)                          \
    do {                                              \
        hipError_t e_ = (expr);                       \
        if (e_ != hipSuccess) return hip_fail(e_, what); \
    } while (0)

dim3 cells_grid(const Grid &g) { return dim3((unsigned)((g.n + 255) / 256)); }

// Fixed-cycle solve of A x = b on the pressure hierarchy; the work pair (b, px)
// is the same for every solve.  The solve is enqueued with nothing waited for on
// the host (its status, residual and time are read by collect_solves after the
// step); hierarchies that need the host inside the solve (singular ones) take
// the synchronous solve.
int pressure_solve(nn4mg_stepper *S, int slot, int cycles, nn4mg_step_info *info, float *ms_mg)
{
    STEP_TRY(hipEventRecord(S->sev[2 * slot], S->s), "hipEventRecord");
    int rc = solve_fixed_enqueue(S->P, S->b, S->px, cycles, S->hdr + (size_t)slot * solve_header_bytes());
    if (rc == NN4MG_OK) {
        STEP_TRY(hipEventRecord(S->sev[2 * slot + 1], S->s), "hipEventRecord");
        S->pending[slot] = true;
        if (info) info->solves = slot + 1;
        return NN4MG_OK;
    }
    if (rc != NN4MG_EINVAL) return rc;
    nn4mg_info si;
    rc = nn4mg_solve(S->P, S->b, S->px, 0.0, cycles, 1, &si);
    if (rc != NN4MG_OK && rc != NN4MG_ENOTCONV) return rc;
    STEP_TRY(hipEventRecord(S->sev[2 * slot + 1], S->s), "hipEventRecord");
    STEP_TRY(hipEventSynchronize(S->sev[2 * slot + 1]), "hipEventSynchronize");
    float ms = 0.0f;
    STEP_TRY(hipEventElapsedTime(&ms, S->sev[2 * slot], S->sev[2 * slot + 1]), "hipEventElapsedTime");
    *ms_mg += ms;
    if (info) {
        info->relres[slot] = si.relres;
        info->solves = slot + 1;
    }
    return NN4MG_OK;
}

// After the step's stream has drained: the status, final residual and device
// time of every solve enqueued without waiting.
int collect_solves(nn4mg_stepper *S, nn4mg_step_info *info, float *ms_mg)
{
    int status = NN4MG_OK;
    for (int slot = 0; slot < nn4mg_stepper::kSolves; ++slot) {
        if (!S->pending[slot]) continue;
        S->pending[slot] = false;
        double relres = 0.0;
        const int rc = solve_fixed_result(S->hdr + (size_t)slot * solve_header_bytes(), &relres);
        if (rc != NN4MG_OK && status == NN4MG_OK) status = rc;
        float ms = 0.0f;
        STEP_TRY(hipEventElapsedTime(&ms, S->sev[2 * slot], S->sev[2 * slot + 1]), "hipEventElapsedTime");
        *ms_mg += ms;
        if (info) info->relres[slot] = relres;
    }
    return status;
}

// sum C h^3 over the grid into S->red[S->nred] (fixed-order block partials)
int enqueue_volume(nn4mg_stepper *S, const double *C)
{
    const double h = S->g.h;
    STEP_TRY(launch_sum_partials(C, S->g.n, nullptr, 1, S->red, S->s), "sum partials");
    STEP_TRY(launch_reduce(S->red, S->nred, h * h * h, S->red + S->nred, S->s), "reduce");
    return NN4MG_OK;
}

int check_params(const nn4mg_step_params *p)
{
    if (!p) return set_error(NN4MG_EINVAL, "params is NULL");
    if (!(p->rho_l > 0.0) || !(p->rho_g > 0.0)) return set_error(NN4MG_EINVAL, "densities must be > 0");
    if (!(p->mu_l >= 0.0) || !(p->mu_g >= 0.0)) return set_error(NN4MG_EINVAL, "viscosities must be >= 0");
    if (!(p->dt > 0.0)) return set_error(NN4MG_EINVAL, "dt must be > 0");
    if (!std::isfinite(p->g) || !std::isfinite(p->sigma_t)) return set_error(NN4MG_EINVAL, "g, sigma_t must be finite");
    if (p->mg_cycles < 1 || p->mg_cycles > 511) return set_error(NN4MG_EINVAL, "mg_cycles must be in [1, 511]");
    if (p->mg_cycles_nh < 0 || p->mg_cycles_nh > 511) return set_error(NN4MG_EINVAL, "mg_cycles_nh must be in [0, 511]");
    if (p->order < 0 || p->order > 2) return set_error(NN4MG_EINVAL, "order must be 0, 1 or 2");
    for (int i = 0; i < 3; ++i)
        if (p->reserved[i] != 0) return set_error(NN4MG_EINVAL, "reserved fields must be zero");
    if (p->n_corr < 0 || p->n_corr > 7) return set_error(NN4MG_EINVAL, "n_corr must be in [0, 7]");
    if (p->n_vel_iter < 1 || p->n_vel_iter > 64) return set_error(NN4MG_EINVAL, "n_vel_iter must be in [1, 64]");
    return NN4MG_OK;
}

}  // namespace

extern "C" {

void nn4mg_step_params_default(nn4mg_step_params *p)
{
    if (!p) return;
    std::memset(p, 0, sizeof(*p));
    p->rho_l = 1000.0;
    p->rho_g = 1.0;
    p->mu_l = 1e-3;
    p->mu_g = 1.8e-5;
    p->g = 9.81;
    p->sigma_t = 0.07;
    p->dt = 1e-4;
    p->mg_cycles = 20;
    p->n_corr = 2;
    p->n_vel_iter = 2;
}

int nn4mg_step_destroy(nn4mg_step_t S)
{
    if (!S) return NN4MG_OK;
    if (S->s) (void)hipStreamSynchronize(S->s);
    else (void)hipDeviceSynchronize();
    if (S->P) nn4mg_destroy(S->P);
    if (S->mem) (void)hipFree(S->mem);
    if (S->red) (void)hipFree(S->red);
    for (auto &e : S->ev)
        if (e) (void)hipEventDestroy(e);
    for (auto &e : S->sev)
        if (e) (void)hipEventDestroy(e);
    if (S->hdr) (void)hipHostFree(S->hdr);
    delete S;
    return NN4MG_OK;
}

int nn4mg_step_create(int nx, int ny, int nz, double h, const nn4mg_step_params *p, void *hip_stream,
                      nn4mg_step_t *out)
{
    if (!out) return set_error(NN4MG_EINVAL, "out is NULL");
    *out = nullptr;
    int rc = check_params(p);
    if (rc) return rc;
    if (nx < 4 || ny < 4 || nz < 4) return set_error(NN4MG_EINVAL, "grid dims must be >= 4");
    // the quadratic filters index a cell's neighbourhood with 32-bit offsets
    if ((double)nx * ny * nz >= 2147483648.0) return set_error(NN4MG_EINVAL, "grid must have fewer than 2^31 cells");
    if (!(h > 0.0)) return set_error(NN4MG_EINVAL, "h must be > 0");
    // pressure: zero-normal-derivative walls, zero pressure on the top outlet
    nn4mg_config cfg;
    nn4mg_config_default(&cfg, nx, ny, nz, h);
    for (int f = 0; f < 5; ++f) cfg.bc[f] = NN4MG_BC_NEUMANN0;
    cfg.bc[5] = NN4MG_BC_DIRICHLET0;
    nn4mg_stepper *S = new nn4mg_stepper();
    S->g = Grid{nx, ny, nz, h, (size_t)nx * ny * nz};
    S->p = *p;
    S->s = (hipStream_t)hip_stream;
    if ((rc = nn4mg_setup(&cfg, nullptr, hip_stream, &S->P))) {
        S->P = nullptr;
        nn4mg_step_destroy(S);
        return rc;
    }
    const size_t n = S->g.n;
    hipError_t e = hipMalloc((void **)&S->mem, (size_t)kFields * n * sizeof(double));
    if (e != hipSuccess) {
        (void)hipGetLastError();
        S->mem = nullptr;
        nn4mg_step_destroy(S);
        return set_error(NN4MG_ENOMEM, "step work fields: hipMalloc failed");
    }
    double *q = S->mem;
    auto take = [&]() {
        double *r = q;
        q += n;
        return r;
    };
    S->rho = take();
    S->mu = take();
    for (int d = 0; d < 3; ++d) S->Cd[d] = take();
    for (int d = 0; d < 3; ++d) S->nrm[d] = take();
    for (int d = 0; d < 3; ++d) S->st[d] = take();
    S->b = take();
    S->px = take();
    for (int d = 0; d < 3; ++d) S->qa[d] = take();
    for (int d = 0; d < 3; ++d) S->qb[d] = take();
    for (int d = 0; d < 3; ++d) S->qt[d] = take();
    for (int d = 0; d < 3; ++d) S->adv[d] = take();
    for (int d = 0; d < 3; ++d) S->kq[d] = take();
    S->tmp = take();
    S->nred = sum_blocks(n);
    if ((e = hipMalloc((void **)&S->red, (size_t)(S->nred + 1) * sizeof(double))) != hipSuccess) {
        (void)hipGetLastError();
        S->red = nullptr;
        nn4mg_step_destroy(S);
        return set_error(NN4MG_ENOMEM, "step reduction buffer: hipMalloc failed");
    }
    for (auto &ev : S->ev)
        if ((e = hipEventCreate(&ev)) != hipSuccess) {
            ev = nullptr;
            nn4mg_step_destroy(S);
            return hip_fail(e, "hipEventCreate");
        }
    for (auto &ev : S->sev)
        if ((e = hipEventCreate(&ev)) != hipSuccess) {
            ev = nullptr;
            nn4mg_step_destroy(S);
            return hip_fail(e, "hipEventCreate");
        }
    if ((e = hipHostMalloc((void **)&S->hdr, nn4mg_stepper::kSolves * solve_header_bytes(), hipHostMallocDefault)) !=
        hipSuccess) {
        (void)hipGetLastError();
        S->hdr = nullptr;
        nn4mg_step_destroy(S);
        return set_error(NN4MG_ENOMEM, "step solve headers: hipHostMalloc failed");
    }
    // launch shapes of the pressure hierarchy, tuned once for this grid on the
    // stepper's own (zeroed) solve pair; every solve of the stepper uses them
    if ((e = launch_fill(S->b, n, 0.0, (hipStream_t)hip_stream)) != hipSuccess ||
        (e = launch_fill(S->px, n, 0.0, (hipStream_t)hip_stream)) != hipSuccess) {
        nn4mg_step_destroy(S);
        return hip_fail(e, "fill");
    }
    if ((rc = nn4mg_autotune(S->P, S->b, S->px, nullptr, 0))) {
        nn4mg_step_destroy(S);
        return rc;
    }
    *out = S;
    return NN4MG_OK;
}

int nn4mg_step(nn4mg_step_t S, double *C, double *u, double *v, double *w, double *p_hs, double *p_nh,
               nn4mg_step_info *info)
{
    if (!S || !C || !u || !v || !w || !p_hs || !p_nh) return set_error(NN4MG_EINVAL, "NULL argument");
    if (info) {
        std::memset(info, 0, sizeof(*info));
        info->volume = std::nan("");  // until the step completes
    }
    const Grid g = S->g;
    const nn4mg_step_params &p = S->p;
    const Phys P{p.rho_l, p.rho_g, p.mu_l, p.mu_g, p.g, p.sigma_t, p.dt};
    const hipStream_t s = S->s;
    const dim3 grid = cells_grid(g), blk(256);
    // the block-staged kernels: one workgroup per 8^3 block
    const dim3 bgrid(blocks_of(g)), bblk(SBT);
    const QW qw = quad_weights(g.h);
    double *q[3] = {u, v, w};
    float ms_mg = 0.0f;
    int rc;

    const bool quad = p.order == 2;
    for (bool &pend : S->pending) pend = false;  // nothing left over from a step that failed midway
    STEP_TRY(hipEventRecord(S->ev[0], s), "hipEventRecord");
    if (quad) {
        hipLaunchKernelGGL(props2_kernel, bgrid, bblk, 0, s, g, P, qw, (const double *)C, S->rho, S->mu,
                           f3(S->Cd), f3(S->nrm));
        hipLaunchKernelGGL(surface2_kernel, bgrid, bblk, 0, s, g, qw, p.sigma_t, c3(S->nrm), c3(S->Cd),
                           f3(S->st));
    } else {
        STEP_TRY(step_props(g, P, C, S->rho, S->mu, f3(S->Cd), f3(S->nrm), s), "props");
        STEP_TRY(step_surface(g, p.sigma_t, c3(S->nrm), c3(S->Cd), f3(S->st), s), "surface");
    }

    // Stage 1: hydrostatic + surface-tension pressure, warm-started from p_hs
    STEP_TRY(step_rhs_hydrostatic(g, p.g, c3(S->st), S->rho, S->b, s), "hydrostatic right-hand side");
    STEP_TRY(hipGetLastError(), "step kernels");
    STEP_TRY(hipMemcpyAsync(S->px, p_hs, g.n * sizeof(double), hipMemcpyDeviceToDevice, s), "hipMemcpyAsync");
    if ((rc = pressure_solve(S, 0, p.mg_cycles, info, &ms_mg))) return rc;
    STEP_TRY(hipMemcpyAsync(p_hs, S->px, g.n * sizeof(double), hipMemcpyDeviceToDevice, s), "hipMemcpyAsync");

    // Stage 2: velocity predictor iterations, q^ from q^n
    double **cur = S->qa, **nxt = S->qb;
    hipLaunchKernelGGL(copy3_kernel, grid, blk, 0, s, g.n, c3(q), f3(cur));
    for (int it = 0; it < p.n_vel_iter; ++it) {
        if (quad) {
            hipLaunchKernelGGL(advection2_kernel, bgrid, bblk, 0, s, g, qw, c3(cur), f3(S->adv));
            hipLaunchKernelGGL(pg_velocity2_kernel, bgrid, bblk, 0, s, g, qw, c3(cur), c3(S->adv),
                               (const double *)S->rho,
                               (const double *)S->mu, f3(S->kq));
            hipLaunchKernelGGL(momentum2_kernel, bgrid, bblk, 0, s, g, P, qw, c3(q), (const double *)p_hs,
                               (const double *)p_nh, (const double *)S->rho, c3(cur), c3(S->kq), c3(S->st),
                               c3(S->adv), f3(S->qt), f3(nxt));
            double **t = cur;
            cur = nxt;
            nxt = t;
            continue;
        }
        STEP_TRY(step_advection(g, c3(cur), f3(S->adv), s), "advection");
        STEP_TRY(step_pg_velocity(g, c3(cur), c3(S->adv), S->rho, S->mu, f3(S->kq), s), "velocity diffusivity");
        STEP_TRY(step_momentum(g, P, c3(q), p_hs, p_nh, S->rho, c3(cur), c3(S->kq), c3(S->st), c3(S->adv), f3(S->qt),
                               f3(nxt), s), "momentum");
        double **t = cur;
        cur = nxt;
        nxt = t;
    }
    STEP_TRY(hipGetLastError(), "step kernels");

    // Stage 3: non-hydrostatic corrections; the corrected velocity lands in q
    double **qin = S->qt;
    for (int it = 0; it < p.n_corr; ++it) {
        STEP_TRY(step_rhs_nonhydrostatic(g, p.dt, c3(qin), S->rho, S->b, s), "non-hydrostatic right-hand side");
        STEP_TRY(launch_fill(S->px, g.n, 0.0, s), "fill");
        if ((rc = pressure_solve(S, 1 + it, p.mg_cycles_nh > 0 ? p.mg_cycles_nh : p.mg_cycles, info, &ms_mg)))
            return rc;
        STEP_TRY(step_correct(g, p.dt, S->px, S->rho, c3(qin), f3(q), p_nh, s), "correction");
        qin = q;
    }
    if (p.n_corr == 0) hipLaunchKernelGGL(copy3_kernel, grid, blk, 0, s, g.n, c3(S->qt), f3(q));

    // Stage 4: volume fraction with the new velocity
    hipLaunchKernelGGL(advection_c_kernel, grid, blk, 0, s, g, c3(q), c3(S->Cd), S->tmp);
    if (quad)
        hipLaunchKernelGGL(pg_volume_fraction2_kernel, bgrid, bblk, 0, s, g, qw, p.dt, (const double *)C,
                           c3(S->Cd), c3(q), (const double *)S->tmp, f3(S->kq));
    else
        STEP_TRY(step_pg_volume_fraction(g, p.dt, C, c3(S->Cd), c3(q), S->tmp, f3(S->kq), s),
                 "volume-fraction diffusivity");
    STEP_TRY(step_volume_fraction(g, p.dt, C, c3(S->kq), S->tmp, S->b, s), "volume fraction");
    STEP_TRY(hipMemcpyAsync(C, S->b, g.n * sizeof(double), hipMemcpyDeviceToDevice, s), "hipMemcpyAsync");
    STEP_TRY(hipGetLastError(), "step kernels");
    STEP_TRY(hipEventRecord(S->ev[1], s), "hipEventRecord");
    // the volume of fluid after the step, sum C h^3 (the integral of C^{n+1})
    double vol = 0.0;
    if ((rc = enqueue_volume(S, C))) return rc;
    STEP_TRY(hipMemcpyAsync(&vol, S->red + S->nred, sizeof(double), hipMemcpyDeviceToHost, s), "hipMemcpyAsync");
    STEP_TRY(hipStreamSynchronize(s), "hipStreamSynchronize");
    if ((rc = collect_solves(S, info, &ms_mg))) return rc;
    if (info) {
        float ms = 0.0f;
        STEP_TRY(hipEventElapsedTime(&ms, S->ev[0], S->ev[1]), "hipEventElapsedTime");
        info->ms_total = ms;
        info->ms_mg = ms_mg;
        info->volume = vol;
    }
    if (!std::isfinite(vol)) return set_error(NN4MG_EBREAKDOWN, "non-finite volume fraction after the step");
    return NN4MG_OK;
}

int nn4mg_step_run(nn4mg_step_t S, int nsteps, double *C, double *u, double *v, double *w, double *p_hs, double *p_nh,
                   double *volume, int *steps_done, nn4mg_step_info *info)
{
    if (!S || !C || !u || !v || !w || !p_hs || !p_nh) return set_error(NN4MG_EINVAL, "NULL argument");
    if (nsteps < 0) return set_error(NN4MG_EINVAL, "nsteps must be >= 0");
    if (steps_done) *steps_done = 0;
    int rc;
    if (volume) {
        if ((rc = enqueue_volume(S, C))) return rc;
        STEP_TRY(hipMemcpyAsync(volume, S->red + S->nred, sizeof(double), hipMemcpyDeviceToHost, S->s),
                 "hipMemcpyAsync");
        STEP_TRY(hipStreamSynchronize(S->s), "hipStreamSynchronize");
    }
    nn4mg_step_info si;
    for (int n = 0; n < nsteps; ++n) {
        rc = nn4mg_step(S, C, u, v, w, p_hs, p_nh, &si);
        if (info) *info = si;
        if (volume && (rc == NN4MG_OK || rc == NN4MG_EBREAKDOWN)) volume[n + 1] = si.volume;  // NaN if it stopped early
        if (rc) return rc;
        if (steps_done) *steps_done = n + 1;
    }
    return NN4MG_OK;
}

}  // extern "C"
