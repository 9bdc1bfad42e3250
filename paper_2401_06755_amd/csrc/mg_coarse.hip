// The coarsest level's matrix and its inverse, on the device (gfx950).
//
// The sawtooth cycle of Fig. multi-grid (arXiv 2401.06755, Sec. 2.4) ends in
// an exact solve with the FP64 inverse of the coarsest matrix (n <= 512
// unknowns).  The matrix is the linear-element operator in the link form of
// Eq. (k-T), Sec. 2.2.4,
//     (A x)_i = sum over edge and corner neighbours s of 2 c_s k_is (x_i - x_s),
//     c_edge = h/12, c_corner = h/24, k_is = (k_i + k_s) / 2,
// with the halo neighbours folded back into the grid by the boundary rules
// (Sec. 2.3.3), plus mean(diag) / n in every entry for singular problems.  It
// is symmetric positive definite, so Gauss-Jordan elimination needs no
// pivoting, and its pivots are the squares of the Cholesky factor's diagonal:
// one that is not positive says that the matrix is not positive definite.
// The inverse is symmetrised as it is stored: the cycle reads its columns as
// rows, and flexible CG expects a symmetric preconditioner.
//
// A new coefficient replaces the inverse, so this is on the path of every time
// step with a changing density.  Formed on the host (a copy of k out, Cholesky
// and n triangular solves on one core, a copy back) a coefficient update plus
// 20 cycles at 96 x 64 x 160 (n = 240) took 9.56 ms, and with the inverse formed
// here and nothing else changed 2.57 ms (now 1.88).  40 served solves of 32^3 ..
// 128^3, whose worker formed one inverse per request: 59.7 and 54.0 ms (now 44.5).
#include "mg_internal.h"

namespace nn4mg {

namespace {

constexpr int kLinks = 20;     // 12 edge and 8 corner neighbours
constexpr int kNT1 = 1024;     // threads of the one-workgroup form
constexpr int kMaxRows = 6;    // rows and columns per thread there
constexpr int kOneMax = 32 * kMaxRows;
constexpr int kB = 32;         // block edge of the blocked form
constexpr int kNTB = 256;

__device__ __forceinline__ int cfold(int i, int n, int lo, int hi, double &s)
{
    if (i < 0) {
        if (lo == BC_P) return i + n;
        if (lo == BC_D) s = -s;
        return -1 - i;
    }
    if (i >= n) {
        if (hi == BC_P) return i - n;
        if (hi == BC_D) s = -s;
        return 2 * n - 1 - i;
    }
    return i;
}

// Link l (0 .. 19) of row c: the column it reaches (folded) and its value in
// that column; returns what it adds to the diagonal.  A link that folds back
// onto its own cell counts there alone: nothing through a mirroring wall, so
// the diagonal of an operator that is zero comes out as zero.
__device__ __forceinline__ double link(const CoarseArgs &a, int c, int l, int &q, double &v)
{
    // the 27 offsets in x, y, z order without the centre and the faces
    constexpr signed char at[kLinks] = {0, 1, 2, 3, 5, 6, 7, 8, 9, 11, 15, 17, 18, 19, 20, 21, 23, 24, 25, 26};
    const int o = at[l];
    const int dx = o % 3 - 1, dy = (o / 3) % 3 - 1, dz = o / 9 - 1;
    const int i = c % a.nx, t = c / a.nx;
    const int j = t % a.ny, k = t / a.ny;
    double s = 1.0;
    const int fi = cfold(i + dx, a.nx, a.bc[0], a.bc[1], s);
    const int fj = cfold(j + dy, a.ny, a.bc[2], a.bc[3], s);
    const int fk = cfold(k + dz, a.nz, a.bc[4], a.bc[5], s);
    q = fi + a.nx * (fj + a.ny * fk);
    const double cs = (dx != 0 && dy != 0 && dz != 0) ? a.h / 24.0 : a.h / 12.0;
    const double w = 2.0 * cs * (a.k ? 0.5 * (a.k[c] + a.k[q]) : 1.0);
    v = q == c ? 0.0 : -s * w;
    return q == c ? (1.0 - s) * w : w;
}

// Entry of column j in a row whose links and diagonal are given.
__device__ __forceinline__ double entry(const short *q, const double *v, double diag, int i, int j)
{
    double m = i == j ? diag : 0.0;
#pragma unroll
    for (int l = 0; l < kLinks; ++l) m += q[l] == j ? v[l] : 0.0;
    return m;
}

// n <= 192: matrix and elimination in one workgroup, the matrix in registers
// (32 x 32 threads, R x R entries each, rows and columns cyclic), one step per
// unknown: the pivot's row and column go through LDS in two alternating
// buffers, so a step has one barrier.  What bounds it is the chain of n steps
// (a barrier and an LDS round trip each), not the n^3 operations.
template <int R>
__global__ __launch_bounds__(kNT1) void inverse_one_kernel(const CoarseArgs a)
{
    __shared__ short lq[32 * R][kLinks];
    __shared__ double lval[32 * R][kLinks];
    __shared__ double ldiag[32 * R];
    __shared__ double col[2][32 * R], row[2][32 * R];
    const int n = a.n, t = threadIdx.x, tx = t & 31, ty = t >> 5;
    for (int f = t; f < n * kLinks; f += kNT1) {
        const int c = f / kLinks, l = f - c * kLinks;
        int q;
        double v;
        (void)link(a, c, l, q, v);
        lq[c][l] = (short)q;
        lval[c][l] = v;
    }
    if (t < n) {
        double d = 0.0;
        for (int l = 0; l < kLinks; ++l) {
            int q;
            double v;
            d += link(a, t, l, q, v);
        }
        ldiag[t] = d;
    }
    __syncthreads();
    double shift = 0.0;
    if (a.singular) {  // mean of the diagonal over n
        for (int i = 0; i < n; ++i) shift += ldiag[i];
        shift /= (double)n;
        shift /= (double)n;
    }
    double m[R][R];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int s = 0; s < R; ++s) {
            const int i = ty + 32 * r, j = tx + 32 * s;
            m[r][s] = (i < n && j < n) ? entry(lq[i], lval[i], ldiag[i], i, j) + shift : (i == j ? 1.0 : 0.0);
        }
    bool bad = false;
    for (int p = 0; p < n; ++p) {
        const int b = p & 1, lp = p & 31, rp = p >> 5;
#pragma unroll
        for (int s = 0; s < R; ++s) {
            if (s != rp) continue;
            if (tx == lp) {
#pragma unroll
                for (int r = 0; r < R; ++r) col[b][ty + 32 * r] = m[r][s];
            }
            if (ty == lp) {
#pragma unroll
                for (int r = 0; r < R; ++r) row[b][tx + 32 * r] = m[s][r];
            }
        }
        __syncthreads();
        const double piv = row[b][p], d = 1.0 / piv;
        if (!(piv > 0.0)) bad = true;
        double hs[R];
#pragma unroll
        for (int s = 0; s < R; ++s) hs[s] = (tx + 32 * s) == p ? 1.0 : row[b][tx + 32 * s];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = ty + 32 * r;
            const double g = i == p ? -d : col[b][i] * d;
#pragma unroll
            for (int s = 0; s < R; ++s) {
                const double o = (i == p || (tx + 32 * s) == p) ? 0.0 : m[r][s];
                m[r][s] = fma(-g, hs[s], o);
            }
        }
    }
    if (bad && t == 0) a.flag[1] = 1;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int s = 0; s < R; ++s) {
            const int i = ty + 32 * r, j = tx + 32 * s;
            if (i < n && j < n) a.ainv[(size_t)i * n + j] = m[r][s];
        }
    __syncthreads();
    // symmetrised: each pair of entries by the thread of the upper one
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int s = 0; s < R; ++s) {
            const int i = ty + 32 * r, j = tx + 32 * s;
            if (i >= j || j >= n) continue;
            const double v = 0.5 * (m[r][s] + a.ainv[(size_t)j * n + i]);
            a.ainv[(size_t)i * n + j] = v;
            a.ainv[(size_t)j * n + i] = v;
        }
}

// n > 192: the matrix in memory, one workgroup per row.
__global__ __launch_bounds__(kNTB) void matrix_kernel(const CoarseArgs a)
{
    __shared__ short lq[kLinks];
    __shared__ double lval[kLinks], ldiag, red[kNTB / 64];
    const int n = a.n, i = blockIdx.x, t = threadIdx.x;
    double shift = 0.0;
    if (a.singular) {
        double d = 0.0;
        for (int c = t; c < n; c += kNTB)
            for (int l = 0; l < kLinks; ++l) {
                int q;
                double v;
                d += link(a, c, l, q, v);
            }
        for (int off = 32; off > 0; off >>= 1) d += __shfl_down(d, off);
        if ((t & 63) == 0) red[t >> 6] = d;
    }
    if (t < kLinks) {
        int q;
        double v;
        (void)link(a, i, t, q, v);
        lq[t] = (short)q;
        lval[t] = v;
    } else if (t == 64) {
        double d = 0.0;
        for (int l = 0; l < kLinks; ++l) {
            int q;
            double v;
            d += link(a, i, l, q, v);
        }
        ldiag = d;
    }
    __syncthreads();
    if (a.singular) shift = ((red[0] + red[1]) + (red[2] + red[3])) / (double)n / (double)n;
    for (int j = t; j < n; j += kNTB) a.ainv[(size_t)i * n + j] = entry(lq, lval, ldiag, i, j) + shift;
}

// ---- blocked Gauss-Jordan in place: 32 x 32 blocks, 256 threads per block
// (thread (ty, tx) holds rows ty + 8 r of column tx).  Step p takes two
// launches: the trailing blocks A_ij -= A_ip (A_pp^-1 A_pj), then the panels
// A_pj = A_pp^-1 A_pj and A_ip = -A_ip A_pp^-1.  Every workgroup inverts A_pp
// for itself, so A_pp stays as it is until the next step's trailing launch,
// whose workgroup of that block puts its inverse there (no launch reads a
// block that another workgroup of it writes).

// Block (bi, bj), identity outside the matrix, into registers.
__device__ __forceinline__ void load_block(const CoarseArgs &a, int bi, int bj, double (&m)[4])
{
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5, j = bj * kB + tx;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = bi * kB + ty + 8 * r;
        m[r] = (i < a.n && j < a.n) ? a.ainv[(size_t)i * a.n + j] : (i == j ? 1.0 : 0.0);
    }
}

__device__ __forceinline__ void store_block(const CoarseArgs &a, int bi, int bj, const double (&m)[4])
{
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5, j = bj * kB + tx;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = bi * kB + ty + 8 * r;
        if (i < a.n && j < a.n) a.ainv[(size_t)i * a.n + j] = m[r];
    }
}

__device__ __forceinline__ void to_lds(const double (&m)[4], double (*s)[kB + 1])
{
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
    for (int r = 0; r < 4; ++r) s[ty + 8 * r][tx] = m[r];
}

// m := x y for blocks in LDS.
__device__ __forceinline__ void product(const double (*x)[kB + 1], const double (*y)[kB + 1], double (&m)[4])
{
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
    for (int r = 0; r < 4; ++r) m[r] = 0.0;
#pragma unroll 4
    for (int k = 0; k < kB; ++k) {
        const double v = y[k][tx];
#pragma unroll
        for (int r = 0; r < 4; ++r) m[r] = fma(x[ty + 8 * r][k], v, m[r]);
    }
}

// m := its block's inverse (as inverse_one_kernel's elimination).
__device__ __forceinline__ void invert_block(double (&m)[4], double (*buf)[2][kB], int *flag)
{
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    bool bad = false;
#pragma unroll 1
    for (int p = 0; p < kB; ++p) {
        double(*bp)[kB] = buf[p & 1];
        if (tx == p) {
#pragma unroll
            for (int r = 0; r < 4; ++r) bp[0][ty + 8 * r] = m[r];
        }
        if (ty == (p & 7)) {
            const int r = p >> 3;
            bp[1][tx] = r == 0 ? m[0] : r == 1 ? m[1] : r == 2 ? m[2] : m[3];
        }
        __syncthreads();
        const double piv = bp[1][p], d = 1.0 / piv;
        if (!(piv > 0.0)) bad = true;
        const double hs = tx == p ? 1.0 : bp[1][tx];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = ty + 8 * r;
            const double g = i == p ? -d : bp[0][i] * d;
            m[r] = fma(-g, hs, (i == p || tx == p) ? 0.0 : m[r]);
        }
    }
    if (bad && threadIdx.x == 0) flag[1] = 1;
}

// last = 1: the last diagonal block's inverse, and the whole inverse symmetrised
// (the workgroup of an upper block averages it with the block across the diagonal).
__global__ __launch_bounds__(kNTB) void trailing_kernel(const CoarseArgs a, int p, int last)
{
    __shared__ double s0[kB][kB + 1], s1[kB][kB + 1], s2[kB][kB + 1];
    __shared__ double buf[2][2][kB];
    double m[4], u[4];
    const int bi = blockIdx.y, bj = blockIdx.x;
    if (last) {
        if (bi > bj) return;
        load_block(a, bi, bj, m);
        if (bi == p && bj == p) invert_block(m, buf, a.flag);
        if (bi == bj)
            to_lds(m, s1);
        else {
            load_block(a, bj, bi, u);
            to_lds(u, s1);
        }
        __syncthreads();
        const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
        for (int r = 0; r < 4; ++r) m[r] = 0.5 * (m[r] + s1[tx][ty + 8 * r]);
        store_block(a, bi, bj, m);
        if (bi == bj) return;
        to_lds(m, s0);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) u[r] = s0[tx][ty + 8 * r];
        store_block(a, bj, bi, u);
        return;
    }
    if (bi == p || bj == p) return;
    load_block(a, bi, p, u);
    to_lds(u, s1);
    load_block(a, p, bj, u);
    to_lds(u, s2);
    load_block(a, bi, bj, m);
    load_block(a, p, p, u);
    if (bi == p - 1 && bj == p - 1) {
        invert_block(m, buf, a.flag);
        __syncthreads();
    }
    invert_block(u, buf, a.flag);
    to_lds(u, s0);
    __syncthreads();
    product(s0, s2, u);  // A_pp^-1 A_pj
    __syncthreads();
    to_lds(u, s0);
    __syncthreads();
    product(s1, s0, u);
#pragma unroll
    for (int r = 0; r < 4; ++r) m[r] -= u[r];
    store_block(a, bi, bj, m);
}

__global__ __launch_bounds__(kNTB) void panel_kernel(const CoarseArgs a, int p, int nb)
{
    __shared__ double s0[kB][kB + 1], s1[kB][kB + 1];
    __shared__ double buf[2][2][kB];
    const int b = (int)blockIdx.x % nb;
    const bool column = (int)blockIdx.x >= nb;
    if (b == p) return;
    double m[4], u[4];
    load_block(a, column ? b : p, column ? p : b, m);
    load_block(a, p, p, u);
    to_lds(m, s1);
    invert_block(u, buf, a.flag);
    to_lds(u, s0);
    __syncthreads();
    if (column) {
        product(s1, s0, m);
#pragma unroll
        for (int r = 0; r < 4; ++r) m[r] = -m[r];
        store_block(a, b, p, m);
    } else {
        product(s0, s1, m);
        store_block(a, p, b, m);
    }
}

}  // namespace

// One workgroup up to 192 unknowns (the matrix in its registers); above, in
// blocks over the chip: the one-workgroup form would need more registers than
// its 1024 threads have.
hipError_t launch_coarse_inverse(const CoarseArgs &a, hipStream_t s)
{
    if (a.n < 1 || a.n > 512 || a.n != a.nx * a.ny * a.nz || !a.ainv || !a.flag) return hipErrorInvalidValue;
    if (a.n <= kOneMax) {
        const dim3 g(1), t(kNT1);
        switch ((a.n + 31) / 32) {
        case 1: hipLaunchKernelGGL(inverse_one_kernel<1>, g, t, 0, s, a); break;
        case 2: hipLaunchKernelGGL(inverse_one_kernel<2>, g, t, 0, s, a); break;
        case 3: hipLaunchKernelGGL(inverse_one_kernel<3>, g, t, 0, s, a); break;
        case 4: hipLaunchKernelGGL(inverse_one_kernel<4>, g, t, 0, s, a); break;
        case 5: hipLaunchKernelGGL(inverse_one_kernel<5>, g, t, 0, s, a); break;
        default: hipLaunchKernelGGL(inverse_one_kernel<6>, g, t, 0, s, a); break;
        }
        return hipGetLastError();
    }
    const int nb = (a.n + kB - 1) / kB;
    hipLaunchKernelGGL(matrix_kernel, dim3(a.n), dim3(kNTB), 0, s, a);
    for (int p = 0; p < nb; ++p) {
        hipLaunchKernelGGL(trailing_kernel, dim3(nb, nb), dim3(kNTB), 0, s, a, p, 0);
        hipLaunchKernelGGL(panel_kernel, dim3(2 * nb), dim3(kNTB), 0, s, a, p, nb);
    }
    hipLaunchKernelGGL(trailing_kernel, dim3(nb, nb), dim3(kNTB), 0, s, a, nb - 1, 1);
    return hipGetLastError();
}

}  // namespace nn4mg
