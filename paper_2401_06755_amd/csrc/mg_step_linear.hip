// The time step's operators with linear filters (arXiv 2401.06755, Sec. 2.4),
// on gfx950.
//
// Every operator is a sum of 3x3x3 filters f(u; w) (Sec. 2.2.2), tensor
// products of the 1D linear-element vectors
//     M = h [1, 4, 1] / 6,  G = [-1, 0, 1] / 2,  K = [-1, 2, -1] / h,
// on fields whose halo is a mirror with a sign per face (and, for the
// hydrostatic pressure, a bottom halo that adds g h rho).  All of them run in
// one z-march: a workgroup of 256 threads owns a column of 32 x 8 RY cells;
// each plane of its input fields goes to LDS once, with a one-cell ring, the
// boundary rule applied on the way (and sums or products of fields formed
// there); each thread forms the in-plane sums of its RY cells from the rows
// they share, and a running sum per filter carries them from plane to plane.
// What bounds a plane step is its round of loads, so the next plane's are
// issued before the current one is summed, into registers.
//
// One thread per cell gathering 27 values of every field (through L1, or from
// LDS for the velocity terms) was bound by those gathers and their address
// arithmetic.  us per launch at 128^3 then and now: properties 40, 25; surface
// 99, 37; hydrostatic right-hand side 108, 22; advection 79, 33; velocity
// diffusivity 139, 60; momentum 293, 122 (three launches); non-hydrostatic
// right-hand side 130, 28; correction 46, 36; volume-fraction diffusivity 57, 34;
// volume fraction 113, 28.  At about 3.4 us per field read or written (a large
// copy's rate) these are 1.0 to 1.7 times their traffic.
#include "mg_device.h"
#include "mg_step.h"

namespace nn4mg {

namespace {

constexpr int LX = 32;       // cells of a tile along x
constexpr int LT = 256;      // threads
constexpr int LPX = LX + 2;  // staged row

template <int RY>
struct LTile {
    static constexpr int TY = LT / LX * RY;
    static constexpr int PN = LPX * (TY + 2);
    static constexpr int NS = (PN + LT - 1) / LT;  // staged cells per thread
};

__device__ __forceinline__ double signed_by(double v, unsigned crossed, unsigned odd)
{
    return (__popc(crossed & odd) & 1) ? -v : v;
}

// The rows of a staged plane that a thread's RY cells reach, reduced along x:
// m = l + 4 c + r, g = r - l, k = 2 c - l - r (unscaled).
template <int RY>
struct Rows {
    double l[RY + 2], c[RY + 2], r[RY + 2];
    __device__ __forceinline__ Rows(const double *p, int base)
    {
#pragma unroll
        for (int j = 0; j < RY + 2; ++j) {
            l[j] = p[base + j * LPX];
            c[j] = p[base + j * LPX + 1];
            r[j] = p[base + j * LPX + 2];
        }
    }
    __device__ __forceinline__ double m(int j) const { return fma(4.0, c[j], l[j] + r[j]); }
    __device__ __forceinline__ double g(int j) const { return r[j] - l[j]; }
    __device__ __forceinline__ double k(int j) const { return fma(2.0, c[j], -(l[j] + r[j])); }
    __device__ __forceinline__ double mid(int q) const { return c[q + 1]; }
    // in-plane sums of cell q, the first letter along x
    __device__ __forceinline__ double mm(int q) const { return fma(4.0, m(q + 1), m(q) + m(q + 2)); }
    __device__ __forceinline__ double gm(int q) const { return fma(4.0, g(q + 1), g(q) + g(q + 2)); }
    __device__ __forceinline__ double mg(int q) const { return m(q + 2) - m(q); }
    __device__ __forceinline__ double km(int q) const { return fma(4.0, k(q + 1), k(q) + k(q + 2)); }
    __device__ __forceinline__ double mk(int q) const { return fma(2.0, m(q + 1), -(m(q) + m(q + 2))); }
    // corner sum, and 2 x cross sum + corner sum (mg_stencil.hip's D and X)
    __device__ __forceinline__ double corners(int q) const { return (l[q] + r[q]) + (l[q + 2] + r[q + 2]); }
    __device__ __forceinline__ double other(int q) const
    {
        return fma(2.0, (c[q] + c[q + 2]) + (l[q + 1] + r[q + 1]), corners(q));
    }
};

// Filters along z as running sums: push(s) takes plane z's in-plane sum and
// returns the filter of the cell one plane below (unscaled).
struct ZM {
    double p = 0.0, r = 0.0;
    __device__ __forceinline__ double push(double s)
    {
        const double o = r + s;
        r = fma(4.0, s, p);
        p = s;
        return o;
    }
};
struct ZG {
    double p = 0.0, pp = 0.0;
    __device__ __forceinline__ double push(double s)
    {
        const double o = s - pp;
        pp = p;
        p = s;
        return o;
    }
};
struct ZK {
    double p = 0.0, r = 0.0;
    __device__ __forceinline__ double push(double s)
    {
        const double o = r - s;
        r = fma(2.0, s, -p);
        p = s;
        return o;
    }
};
// S = 2 D(z) + o(z - 1) + o(z + 1) of the linear-element Laplacian.
struct ZS {
    double q = 0.0, o = 0.0;
    __device__ __forceinline__ double push(double D, double on)
    {
        const double S = q + on;
        q = fma(2.0, D, o);
        o = on;
        return S;
    }
};
struct ZC {  // the cell's own value, one plane below
    double c = 0.0;
    __device__ __forceinline__ double push(double v)
    {
        const double o = c;
        c = v;
        return o;
    }
};
// The three derivative filters of one field.
struct ZD {
    ZM x, y;
    ZG z;
    template <int RY>
    __device__ __forceinline__ void push(const Rows<RY> &w, int q, double (&d)[3])
    {
        d[0] = x.push(w.gm(q));
        d[1] = y.push(w.mg(q));
        d[2] = z.push(w.mm(q));
    }
};

// Scales of the unscaled sums: w_d / m_l; w_m / m_l; w_d; w_m; w_dd^PG.
__device__ __forceinline__ double s_dml(double h) { return 1.0 / (72.0 * h); }
constexpr double kMassMl = 1.0 / 216.0;
__device__ __forceinline__ double s_d(double h) { return h * h / 72.0; }
__device__ __forceinline__ double s_mass(double h) { return h * h * h / 216.0; }
__device__ __forceinline__ double s_pg(double h) { return h / 36.0; }

// An operator K: NL loads per staged cell, NF fields staged from them, and per
// plane step the thread's cells: load, commit, plane (with the output cells of
// the plane below when emit).
template <class K>
__global__ __launch_bounds__(LT) void march_kernel(const Grid g, int tiles_x, int tiles_y, int zc, const K op)
{
    constexpr int RY = K::RY, NS = LTile<RY>::NS, PN = LTile<RY>::PN, TY = LTile<RY>::TY;
    __shared__ double sm[2][K::NF * PN];
    const int lb = xcd_remap(blockIdx.x, gridDim.x);
    const int bx = lb % tiles_x, rest = lb / tiles_x;
    const int by = rest % tiles_y, bz = rest / tiles_y;
    const int i0 = bx * LX, j0 = by * TY, z0 = bz * zc;
    const int z1 = min(z0 + zc, g.nz);
    const size_t plane = (size_t)g.nx * g.ny;
    const int t = threadIdx.x, li = t % LX, lj = t / LX;

    int off[NS];
    unsigned bits[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int c = min(t + s * LT, PN - 1);
        const int py = c / LPX, px = c - py * LPX;
        const int gi = i0 + px - 1, gj = j0 + py - 1;
        const int ci = min(max(gi, 0), g.nx - 1), cj = min(max(gj, 0), g.ny - 1);
        bits[s] = (gi < 0 ? 1u : (gi >= g.nx ? 2u : 0u)) | (gj < 0 ? 4u : (gj >= g.ny ? 8u : 0u));
        off[s] = ci + g.nx * cj;
    }
    size_t gb[RY];
    bool ok[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int i = i0 + li, j = j0 + RY * lj + r;
        ok[r] = i < g.nx && j < g.ny;
        gb[r] = (size_t)min(i, g.nx - 1) + (size_t)g.nx * (size_t)min(j, g.ny - 1);
    }
    const int base = RY * lj * LPX + li;
    typename K::State st[RY];

    double raw[NS][K::NL];
    auto fetch = [&](int z) {
        const size_t pl = plane * (size_t)min(max(z, 0), g.nz - 1);
#pragma unroll
        for (int s = 0; s < NS; ++s) op.load(raw[s], pl + (size_t)off[s], z);
    };
    fetch(z0 - 1);
    int buf = 0;
    for (int z = z0 - 1; z <= z1; ++z) {
        const unsigned zbit = z < 0 ? 16u : (z >= g.nz ? 32u : 0u);
        double *b = sm[buf];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int c = t + s * LT;
            double v[K::NF];
            op.commit(v, raw[s], bits[s] | zbit);
            if (c < PN) {
#pragma unroll
                for (int f = 0; f < K::NF; ++f) b[f * PN + c] = v[f];
            }
        }
        __syncthreads();
        if (z < z1) fetch(z + 1);
        // the two buffers alternate, so the next plane's commit may overtake
        // this plane's reads by at most one barrier
        size_t id[RY];
        const size_t pl = plane * (size_t)max(z - 1, 0);
#pragma unroll
        for (int r = 0; r < RY; ++r) id[r] = pl + gb[r];
        op.plane(g, st, b, base, z - 1, z > z0, ok, id);
        buf ^= 1;
    }
}

// Chunks of planes per workgroup: the fewest rounds of 512 workgroups (two per
// compute unit) times steps, two of which precede the first output.
template <class K>
hipError_t run(const Grid &g, const K &op, hipStream_t s)
{
    const int tx = (g.nx + LX - 1) / LX, ty = (g.ny + LTile<K::RY>::TY - 1) / LTile<K::RY>::TY;
    int zc = 1;
    double best = 1e300;
    for (int c = 1; c <= g.nz && c <= 128; ++c) {
        const long long w = (long long)tx * ty * ((g.nz + c - 1) / c), rest = w % 512;
        const double cost = ((double)(w / 512) + (rest == 0 ? 0.0 : rest <= 256 ? 0.7 : 1.0)) * (c + 2);
        if (cost < best) {
            best = cost;
            zc = c;
        }
    }
    const dim3 grid((unsigned)(tx * ty * ((g.nz + zc - 1) / zc)));
    hipLaunchKernelGGL(march_kernel<K>, grid, dim3(LT), 0, s, g, tx, ty, zc, op);
    return hipGetLastError();
}

// ------------------------------------------------------------------ operators

struct Props {
    static constexpr int RY = 2, NL = 1, NF = 1, PN = LTile<RY>::PN;
    struct State {
        ZD d;
        ZC c;
    };
    Phys P;
    const double *C;
    double *rho, *mu;
    F3 Cd, nrm;
    __device__ __forceinline__ void load(double (&v)[NL], size_t o, int) const { v[0] = C[o]; }
    __device__ __forceinline__ void commit(double (&v)[NF], const double (&l)[NL], unsigned) const { v[0] = l[0]; }
    __device__ __forceinline__ void plane(const Grid &g, State (&st)[RY], const double *b, int base, int, bool emit,
                                          const bool (&ok)[RY], const size_t (&id)[RY]) const
    {
        const Rows<RY> w(b, base);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            double d[3];
            st[r].d.push(w, r, d);
            const double c0 = st[r].c.push(w.mid(r));
            if (!emit || !ok[r]) continue;
            rho[id[r]] = P.rho_l * c0 + P.rho_g * (1.0 - c0);
            mu[id[r]] = P.mu_l * c0 + P.mu_g * (1.0 - c0);
            const double sc = s_dml(g.h);
            for (int e = 0; e < 3; ++e) d[e] *= sc;
            const double len = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]) + 1e-7 / g.h;
            for (int e = 0; e < 3; ++e) {
                Cd.p[e][id[r]] = d[e];
                nrm.p[e][id[r]] = d[e] / len;
            }
        }
    }
};

struct Surface {
    static constexpr int RY = 2, NL = 3, NF = 3, PN = LTile<RY>::PN;
    struct State {
        ZM x, y;
        ZG z;
    };
    double sigma;
    C3 nrm, Cd;
    F3 st_;
    __device__ __forceinline__ void load(double (&v)[NL], size_t o, int) const
    {
        for (int e = 0; e < 3; ++e) v[e] = nrm.p[e][o];
    }
    __device__ __forceinline__ void commit(double (&v)[NF], const double (&l)[NL], unsigned x) const
    {
        for (int e = 0; e < 3; ++e) v[e] = signed_by(l[e], x, rule_grad(e));
    }
    __device__ __forceinline__ void plane(const Grid &g, State (&st)[RY], const double *b, int base, int, bool emit,
                                          const bool (&ok)[RY], const size_t (&id)[RY]) const
    {
        double cd[RY][3], s[RY];
#pragma unroll
        for (int r = 0; r < RY; ++r)
            for (int e = 0; e < 3; ++e) cd[r][e] = Cd.p[e][id[r]];
        {
            const Rows<RY> w(b, base);
#pragma unroll
            for (int r = 0; r < RY; ++r) s[r] = st[r].x.push(w.gm(r));
        }
        {
            const Rows<RY> w(b + PN, base);
#pragma unroll
            for (int r = 0; r < RY; ++r) s[r] += st[r].y.push(w.mg(r));
        }
        const Rows<RY> w(b + 2 * PN, base);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            s[r] += st[r].z.push(w.mm(r));
            if (!emit || !ok[r]) continue;
            const double kap = sigma * (s[r] * s_dml(g.h));
            for (int e = 0; e < 3; ++e) st_.p[e][id[r]] = kap * cd[r][e];
        }
    }
};

// sum_d f(s_t,d; w_d) + f(g rho; w_z): the last two terms share the filter w_z,
// so their sum is staged as one field.
struct RhsHydrostatic {
    static constexpr int RY = 2, NL = 4, NF = 3, PN = LTile<RY>::PN;
    using State = Surface::State;
    double grav;
    C3 st_;
    const double *rho;
    double *out;
    __device__ __forceinline__ void load(double (&v)[NL], size_t o, int) const
    {
        for (int e = 0; e < 3; ++e) v[e] = st_.p[e][o];
        v[3] = rho[o];
    }
    __device__ __forceinline__ void commit(double (&v)[NF], const double (&l)[NL], unsigned x) const
    {
        for (int e = 0; e < 3; ++e) v[e] = signed_by(l[e], x, rule_grad(e));
        v[2] = fma(grav, l[3], v[2]);
    }
    // f(lift; w_lap) at a bottom cell, lift the plane g h rho below it
    __device__ double lift(const Grid &g, size_t id) const
    {
        const int i = (int)(id % (size_t)g.nx), j = (int)(id / (size_t)g.nx);
        double m[3], k[3];
        for (int q = 0; q < 3; ++q) {
            const size_t row = (size_t)g.nx * (size_t)min(max(j + q - 1, 0), g.ny - 1);
            const double l = rho[row + (size_t)max(i - 1, 0)], c = rho[row + (size_t)i];
            const double r = rho[row + (size_t)min(i + 1, g.nx - 1)];
            m[q] = fma(4.0, c, l + r);
            k[q] = fma(2.0, c, -(l + r));
        }
        const double km = fma(4.0, k[1], k[0] + k[2]), mk = fma(2.0, m[1], -(m[0] + m[2]));
        const double mm = fma(4.0, m[1], m[0] + m[2]);
        return grav * g.h * s_pg(g.h) * ((km + mk) - mm);
    }
    __device__ __forceinline__ void plane(const Grid &g, State (&st)[RY], const double *b, int base, int z, bool emit,
                                          const bool (&ok)[RY], const size_t (&id)[RY]) const
    {
        double s[RY];
        {
            const Rows<RY> w(b, base);
#pragma unroll
            for (int r = 0; r < RY; ++r) s[r] = st[r].x.push(w.gm(r));
        }
        {
            const Rows<RY> w(b + PN, base);
#pragma unroll
            for (int r = 0; r < RY; ++r) s[r] += st[r].y.push(w.mg(r));
        }
        const Rows<RY> w(b + 2 * PN, base);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            s[r] += st[r].z.push(w.mm(r));
            if (!emit || !ok[r]) continue;
            double v = s[r] * s_d(g.h);
            if (z == 0) v -= lift(g, id[r]);
            out[id[r]] = v;
        }
    }
};

struct Advection {
    static constexpr int RY = 1, NL = 3, NF = 3, PN = LTile<RY>::PN;
    struct State {
        ZD d[3];
        ZC c[3];
    };
    C3 q;
    F3 adv;
    __device__ __forceinline__ void load(double (&v)[NL], size_t o, int) const
    {
        for (int e = 0; e < 3; ++e) v[e] = q.p[e][o];
    }
    __device__ __forceinline__ void commit(double (&v)[NF], const double (&l)[NL], unsigned x) const
    {
        for (int e = 0; e < 3; ++e) v[e] = signed_by(l[e], x, rule_vel(e));
    }
    __device__ __forceinline__ void plane(const Grid &g, State (&st)[RY], const double *b, int base, int, bool emit,
                                          const bool (&ok)[RY], const size_t (&id)[RY]) const
    {
        double d[3][RY][3], q0[RY][3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const Rows<RY> w(b + c * PN, base);
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                st[r].d[c].push(w, r, d[c][r]);
                q0[r][c] = st[r].c[c].push(w.mid(r));
            }
        }
        const double sc = s_dml(g.h);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            if (!emit || !ok[r]) continue;
            for (int c = 0; c < 3; ++c) {
                const double *e = d[c][r];
                adv.p[c][id[r]] = sc * (q0[r][0] * e[0] + q0[r][1] * e[1] + q0[r][2] * e[2]);
            }
        }
    }
};

// k_c = rho min(k_max, k_abs, k_sq) + mu (Eqs. efficient-kabs-special-case,
// k-square with h_Psi = h, max-k; residual a_Psi of Eq. a_psi, alpha_a = 2).
struct PgVelocity {
    static constexpr int RY = 1, NL = 6, NF = 6, PN = LTile<RY>::PN;
    struct State {
        ZD d[3];
        ZC c[3], a[3];
        ZM m[3];
    };
    C3 q, adv;
    const double *rho, *mu;
    F3 kq;
    __device__ __forceinline__ void load(double (&v)[NL], size_t o, int) const
    {
        for (int e = 0; e < 3; ++e) v[e] = q.p[e][o];
        for (int e = 0; e < 3; ++e) v[3 + e] = adv.p[e][o];
    }
    __device__ __forceinline__ void commit(double (&v)[NF], const double (&l)[NL], unsigned x) const
    {
        for (int e = 0; e < 3; ++e) v[e] = signed_by(l[e], x, rule_vel(e));
        for (int e = 3; e < 6; ++e) v[e] = l[e];
    }
    __device__ __forceinline__ void plane(const Grid &g, State (&st)[RY], const double *b, int base, int, bool emit,
                                          const bool (&ok)[RY], const size_t (&id)[RY]) const
    {
        const double rho0 = rho[id[0]], mu0 = mu[id[0]];
        double d[3][3], q0[3], res[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const Rows<RY> w(b + c * PN, base);
            st[0].d[c].push(w, 0, d[c]);
            q0[c] = st[0].c[c].push(w.mid(0));
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const Rows<RY> w(b + (3 + c) * PN, base);
            const double mass = st[0].m[c].push(w.mm(0));
            res[c] = fma(kMassMl, mass, -st[0].a[c].push(w.mid(0)));
        }
        if (!emit || !ok[0]) return;
        const double h = g.h, sc = s_dml(h);
        const double kmax = h * (fabs(q0[0]) + fabs(q0[1]) + fabs(q0[2]));
        for (int c = 0; c < 3; ++c) {
            const double a = 2.0 * res[c];
            const double px = sc * d[c][0], py = sc * d[c][1], pz = sc * d[c][2];
            const double G = fabs(px) + fabs(py) + fabs(pz);
            const double kabs = (1.0 / 16.0) * h * fabs(a) / (1e-7 + G / 3.0);
            const double g2 = px * px + py * py + pz * pz;
            const double advabs = fabs(q0[0] * px) + fabs(q0[1] * py) + fabs(q0[2] * pz);
            const double ksq = 4.0 * a * a * h / (1e-7 + advabs / 3.0 * g2);
            kq.p[c][id[0]] = rho0 * fmin(kmax, fmin(kabs, ksq)) + mu0;
        }
    }
};

// Component c of s = rho m_l adv + f_lap(q, k) + f(p_hs + p_nh; w_c) +
// f(s_t; w_m) [+ f(g rho; w_m) for z].  Both pressures have the same halo rule
// (the lifted bottom halo of p_hs added while staging), and the two mass terms
// the same filter, so either pair is staged as its sum.  One launch per
// component: all three at once would need ten staged fields and the registers
// of their running sums, one workgroup per compute unit.
template <int COMP>
struct Momentum {
    static constexpr int RY = 2, NL = COMP == 2 ? 6 : 5, NF = 4, PN = LTile<RY>::PN;
    struct Dz {
        ZG z;
        template <int R>
        __device__ __forceinline__ double push(const Rows<R> &w, int q)
        {
            return z.push(w.mm(q));
        }
    };
    struct Dx {
        ZM x;
        template <int R>
        __device__ __forceinline__ double push(const Rows<R> &w, int q)
        {
            return x.push(COMP == 0 ? w.gm(q) : w.mg(q));
        }
    };
    struct State {
        typename std::conditional<COMP == 2, Dz, Dx>::type p;
        ZM t;
        ZS q, k, kq;
        ZC q0, k0;
    };
    Phys P;
    const double *qn, *p_hs, *p_nh, *rho, *q, *k, *st_, *adv;
    double *qt, *qnext;
    double gh;
    __device__ __forceinline__ void load(double (&v)[NL], size_t o, int z) const
    {
        v[0] = p_hs[o];
        v[1] = p_nh[o];
        v[2] = st_[o];
        v[3] = q[o];
        v[4] = k[o];
        if constexpr (COMP == 2)
            v[5] = rho[o];
        if (z < 0) v[0] = fma(gh, rho[o], v[0]);  // lifted bottom halo (rho +mirror)
    }
    __device__ __forceinline__ void commit(double (&v)[NF], const double (&l)[NL], unsigned x) const
    {
        v[0] = signed_by(l[0] + l[1], x, kOddTop);
        v[1] = signed_by(l[2], x, rule_grad(COMP));
        if constexpr (COMP == 2) v[1] = fma(P.g, l[5], v[1]);
        v[2] = signed_by(l[3], x, rule_vel(COMP));
        v[3] = l[4];
    }
    __device__ __forceinline__ void plane(const Grid &g, State (&st)[RY], const double *b, int base, int, bool emit,
                                          const bool (&ok)[RY], const size_t (&id)[RY]) const
    {
        double r0[RY], a0[RY], q0n[RY], s[RY];
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            r0[r] = rho[id[r]];
            a0[r] = adv[id[r]];
            q0n[r] = qn[id[r]];
        }
        const double h = g.h, ml = h * h * h;
        {
            const Rows<RY> w(b, base);
#pragma unroll
            for (int r = 0; r < RY; ++r) s[r] = s_d(h) * st[r].p.push(w, r);
        }
        {
            const Rows<RY> w(b + PN, base);
#pragma unroll
            for (int r = 0; r < RY; ++r) s[r] = fma(s_mass(h), st[r].t.push(w.mm(r)), s[r]);
        }
        Rows<RY> v(b + 2 * PN, base);
        const Rows<RY> kk(b + 3 * PN, base);
        double Sq[RY], Sk[RY], qc[RY], kc[RY];
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            Sq[r] = st[r].q.push(v.corners(r), v.other(r));
            Sk[r] = st[r].k.push(kk.corners(r), kk.other(r));
            qc[r] = st[r].q0.push(v.mid(r));
            kc[r] = st[r].k0.push(kk.mid(r));
        }
#pragma unroll
        for (int j = 0; j < RY + 2; ++j) {
            v.l[j] *= kk.l[j];
            v.c[j] *= kk.c[j];
            v.r[j] *= kk.r[j];
        }
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            const double Sp = st[r].kq.push(v.corners(r), v.other(r));
            if (!emit || !ok[r]) continue;
            // Eq. (k-T) in link form
            const double lap = fma(32.0, kc[r], Sk[r]) * qc[r] - kc[r] * Sq[r] - Sp;
            const double sum = fma(h / 24.0, lap, s[r]) + r0[r] * ml * a0[r];
            const double t = q0n[r] - sum * (P.dt / (ml * r0[r]));
            qt[id[r]] = t;
            qnext[id[r]] = 0.5 * (q0n[r] + t);
        }
    }
};

// (1/dt) sum_d [q~_d f(rho; w_d) - f(rho q~_d; w_d)]; the products are formed
// while staging.
struct RhsNonhydrostatic {
    static constexpr int RY = 2, NL = 4, NF = 4, PN = LTile<RY>::PN;
    struct State {
        ZM x, y;
        ZG z;
        ZD rho;
    };
    double dt;
    C3 q;
    const double *rho;
    double *out;
    __device__ __forceinline__ void load(double (&v)[NL], size_t o, int) const
    {
        for (int e = 0; e < 3; ++e) v[e] = q.p[e][o];
        v[3] = rho[o];
    }
    __device__ __forceinline__ void commit(double (&v)[NF], const double (&l)[NL], unsigned x) const
    {
        for (int e = 0; e < 3; ++e) v[e] = signed_by(l[e] * l[3], x, rule_vel(e));
        v[3] = l[3];
    }
    __device__ __forceinline__ void plane(const Grid &g, State (&st)[RY], const double *b, int base, int, bool emit,
                                          const bool (&ok)[RY], const size_t (&id)[RY]) const
    {
        double q0[RY][3], s[RY];
#pragma unroll
        for (int r = 0; r < RY; ++r)
            for (int e = 0; e < 3; ++e) q0[r][e] = q.p[e][id[r]];
        {
            const Rows<RY> w(b, base);
#pragma unroll
            for (int r = 0; r < RY; ++r) s[r] = st[r].x.push(w.gm(r));
        }
        {
            const Rows<RY> w(b + PN, base);
#pragma unroll
            for (int r = 0; r < RY; ++r) s[r] += st[r].y.push(w.mg(r));
        }
        {
            const Rows<RY> w(b + 2 * PN, base);
#pragma unroll
            for (int r = 0; r < RY; ++r) s[r] += st[r].z.push(w.mm(r));
        }
        const Rows<RY> w(b + 3 * PN, base);
        const double sc = s_d(g.h) / dt;
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            double d[3];
            st[r].rho.push(w, r, d);
            if (!emit || !ok[r]) continue;
            out[id[r]] = sc * ((q0[r][0] * d[0] + q0[r][1] * d[1] + q0[r][2] * d[2]) - s[r]);
        }
    }
};

struct Correct {
    static constexpr int RY = 2, NL = 1, NF = 1, PN = LTile<RY>::PN;
    struct State {
        ZD d;
        ZC c;
    };
    double dt;
    const double *dp, *rho;
    C3 qin;
    F3 qout;
    double *p_nh;
    __device__ __forceinline__ void load(double (&v)[NL], size_t o, int) const { v[0] = dp[o]; }
    __device__ __forceinline__ void commit(double (&v)[NF], const double (&l)[NL], unsigned x) const
    {
        v[0] = signed_by(l[0], x, kOddTop);
    }
    __device__ __forceinline__ void plane(const Grid &g, State (&st)[RY], const double *b, int base, int, bool emit,
                                          const bool (&ok)[RY], const size_t (&id)[RY]) const
    {
        const Rows<RY> w(b, base);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            double d[3];
            st[r].d.push(w, r, d);
            const double c0 = st[r].c.push(w.mid(r));
            if (!emit || !ok[r]) continue;
            const double f = dt * s_dml(g.h) / rho[id[r]];
            for (int e = 0; e < 3; ++e) qout.p[e][id[r]] = fma(-f, d[e], qin.p[e][id[r]]);
            p_nh[id[r]] += c0;
        }
    }
};

struct PgVolumeFraction {
    static constexpr int RY = 2, NL = 2, NF = 2, PN = LTile<RY>::PN;
    struct State {
        ZM m;
        ZC a, cx, cy;  // advection; the detectors' products along x and y
        double cm = 0.0, c0 = 0.0;  // C two planes and one plane below
    };
    double dt;
    const double *C;
    C3 Cd, q;
    const double *advc;
    F3 kd;
    __device__ __forceinline__ void load(double (&v)[NL], size_t o, int) const
    {
        v[0] = advc[o];
        v[1] = C[o];
    }
    __device__ __forceinline__ void commit(double (&v)[NF], const double (&l)[NL], unsigned) const
    {
        v[0] = l[0];
        v[1] = l[1];
    }
    __device__ __forceinline__ void plane(const Grid &g, State (&st)[RY], const double *b, int base, int, bool emit,
                                          const bool (&ok)[RY], const size_t (&id)[RY]) const
    {
        const double Kp = 300.0, Km = 300.0, beta = 0.1, eps_x = 1e-4, Kpos = 3.0, eps_k = 1e-7, h = g.h;
        const double kmin = 1e-4 / dt * h * h, kclamp = 0.05 / dt * h * h;
        const Rows<RY> w(b, base), c(b + PN, base);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            const double mass = st[r].m.push(w.mm(r));
            const double adv = st[r].a.push(w.mid(r));
            const double cc = c.mid(r), cm = st[r].cm, c0 = st[r].c0;
            double S[3];
            S[0] = st[r].cx.push((cc - c.l[r + 1]) * (c.r[r + 1] - cc));
            S[1] = st[r].cy.push((cc - c.c[r]) * (c.c[r + 2] - cc));
            S[2] = (c0 - cm) * (cc - c0);
            st[r].cm = c0;
            st[r].c0 = cc;
            if (!emit || !ok[r]) continue;
            if (c0 > 0.95 || c0 < 0.05) S[0] = S[1] = S[2] = -1.0;
            const double a = 2.0 * fma(kMassMl, mass, -adv);
            const double cx = Cd.p[0][id[r]], cy = Cd.p[1][id[r]], cz = Cd.p[2][id[r]];
            const double u = q.p[0][id[r]], v = q.p[1][id[r]], ww = q.p[2][id[r]];
            const double g2 = cx * cx + cy * cy + cz * cz;
            const double proj = adv / (eps_x + g2);  // advc is u . grad C
            const double us = cx * proj, vs = cy * proj, ws = cz * proj;
            const double kneg = -beta * (u * u + v * v + ww * ww) /
                                (eps_x + g2 * (fabs(us) + fabs(vs) + fabs(ws)) / 3.0);
            const double G = fabs(cx) + fabs(cy) + fabs(cz);
            const double kabs = (1.0 / 16.0) * h * fabs(a) / (eps_k + G / 3.0);
            for (int d = 0; d < 3; ++d) {
                const double wp = -fmax(-1.0, fmin(0.0, Kp * S[d]));
                const double wm = fmin(1.0, fmax(0.0, Km * S[d]));
                const double kk = wp * (Kpos * kabs) + wm * (kneg / h);
                kd.p[d][id[r]] = fmax(-kmin, fmin(kclamp, kk));
            }
        }
    }
};

// C - dt s_C / m_l, s_C = m_l u . grad C + sum_d f_d(C, k_d; w_dd^PG), with
// f_d = 1/2 [f(k_d C) + k_d f(C) - C f(k_d)] (Eq. k-Txx).
struct VolumeFraction {
    static constexpr int RY = 1, NL = 4, NF = 4, PN = LTile<RY>::PN;
    struct State {
        ZM cx, cy, kx, ky, px, py;
        ZK cz, kz, pz;
        ZC c, k[3];
    };
    double dt;
    const double *C;
    C3 kd;
    const double *advc;
    double *out;
    __device__ __forceinline__ void load(double (&v)[NL], size_t o, int) const
    {
        v[0] = C[o];
        for (int e = 0; e < 3; ++e) v[1 + e] = kd.p[e][o];
    }
    __device__ __forceinline__ void commit(double (&v)[NF], const double (&l)[NL], unsigned) const
    {
        for (int e = 0; e < 4; ++e) v[e] = l[e];
    }
    __device__ __forceinline__ void plane(const Grid &g, State (&st)[RY], const double *b, int base, int, bool emit,
                                          const bool (&ok)[RY], const size_t (&id)[RY]) const
    {
        const double a0 = advc[id[0]];
        State &S = st[0];
        const Rows<RY> c(b, base);
        const double fcx = S.cx.push(c.km(0)), fcy = S.cy.push(c.mk(0)), fcz = S.cz.push(c.mm(0));
        const double c0 = S.c.push(c.mid(0));
        double s = 0.0;
        auto part = [&](int e, auto &zk, auto &zp, double fc, auto &&in_plane) {
            Rows<RY> k(b + (1 + e) * PN, base);
            const double fk = zk.push(in_plane(k));
            const double k0 = S.k[e].push(k.mid(0));
#pragma unroll
            for (int j = 0; j < RY + 2; ++j) {
                k.l[j] *= c.l[j];
                k.c[j] *= c.c[j];
                k.r[j] *= c.r[j];
            }
            const double fp = zp.push(in_plane(k));
            s += fp + k0 * fc - c0 * fk;
        };
        part(0, S.kx, S.px, fcx, [](const Rows<RY> &w) { return w.km(0); });
        part(1, S.ky, S.py, fcy, [](const Rows<RY> &w) { return w.mk(0); });
        part(2, S.kz, S.pz, fcz, [](const Rows<RY> &w) { return w.mm(0); });
        if (!emit || !ok[0]) return;
        const double h = g.h;
        out[id[0]] = c0 - dt * fma(0.5 / (36.0 * h * h), s, a0);
    }
};

}  // namespace

hipError_t step_props(const Grid &g, const Phys &P, const double *C, double *rho, double *mu, F3 Cd, F3 nrm,
                      hipStream_t s)
{
    return run(g, Props{P, C, rho, mu, Cd, nrm}, s);
}

hipError_t step_surface(const Grid &g, double sigma, C3 nrm, C3 Cd, F3 st, hipStream_t s)
{
    return run(g, Surface{sigma, nrm, Cd, st}, s);
}

hipError_t step_rhs_hydrostatic(const Grid &g, double grav, C3 st, const double *rho, double *b, hipStream_t s)
{
    return run(g, RhsHydrostatic{grav, st, rho, b}, s);
}

hipError_t step_advection(const Grid &g, C3 q, F3 adv, hipStream_t s) { return run(g, Advection{q, adv}, s); }

hipError_t step_pg_velocity(const Grid &g, C3 q, C3 adv, const double *rho, const double *mu, F3 kq, hipStream_t s)
{
    return run(g, PgVelocity{q, adv, rho, mu, kq}, s);
}

hipError_t step_momentum(const Grid &g, const Phys &P, C3 qn, const double *p_hs, const double *p_nh,
                         const double *rho, C3 q, C3 kq, C3 st, C3 adv, F3 qt, F3 qnext, hipStream_t s)
{
    const double gh = P.g * g.h;
    auto one = [&](auto c) {
        constexpr int c_ = decltype(c)::value;
        return run(g, Momentum<c_>{P, qn.p[c_], p_hs, p_nh, rho, q.p[c_], kq.p[c_], st.p[c_], adv.p[c_], qt.p[c_],
                                   qnext.p[c_], gh}, s);
    };
    hipError_t e = one(std::integral_constant<int, 0>{});
    if (e == hipSuccess) e = one(std::integral_constant<int, 1>{});
    if (e == hipSuccess) e = one(std::integral_constant<int, 2>{});
    return e;
}

hipError_t step_rhs_nonhydrostatic(const Grid &g, double dt, C3 qt, const double *rho, double *b, hipStream_t s)
{
    return run(g, RhsNonhydrostatic{dt, qt, rho, b}, s);
}

hipError_t step_correct(const Grid &g, double dt, const double *dp, const double *rho, C3 qin, F3 qout, double *p_nh,
                        hipStream_t s)
{
    return run(g, Correct{dt, dp, rho, qin, qout, p_nh}, s);
}

hipError_t step_pg_volume_fraction(const Grid &g, double dt, const double *C, C3 Cd, C3 q, const double *advc, F3 kd,
                                   hipStream_t s)
{
    return run(g, PgVolumeFraction{dt, C, Cd, q, advc, kd}, s);
}

hipError_t step_volume_fraction(const Grid &g, double dt, const double *C, C3 kd, const double *advc, double *Cnew,
                                hipStream_t s)
{
    return run(g, VolumeFraction{dt, C, kd, advc, Cnew}, s);
}

}  // namespace nn4mg
