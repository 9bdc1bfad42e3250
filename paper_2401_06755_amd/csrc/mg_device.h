// Device helpers shared by the z-marching stencil kernels (not part of the C-ABI).
#pragma once

#include "mg_internal.h"

#include <type_traits>

namespace nn4mg {
namespace {

struct NoK {};

template <typename KT>
struct HasK {
    static constexpr bool value = true;
};
template <>
struct HasK<NoK> {
    static constexpr bool value = false;
};

// Storage type of a prefetched coefficient value (the value as loaded).
template <typename T, typename KT>
struct KStore {
    using type = KT;
};
template <typename T>
struct KStore<T, NoK> {
    using type = T;
};

template <typename T, typename KT>
__device__ __forceinline__ T kconv(typename KStore<T, KT>::type v)
{
    if constexpr (std::is_same<KT, __half>::value)
        return (T)__half2float(v);
    else if constexpr (std::is_same<KT, NoK>::value)
        return (T)0;
    else
        return (T)v;
}

// 1/d: hardware reciprocal refined by Newton steps (two in FP64).
__device__ __forceinline__ double recip(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    return r;
}
__device__ __forceinline__ float recip(float d)
{
    float r = __builtin_amdgcn_rcpf(d);
    return fmaf(fmaf(-d, r, 1.0f), r, r);
}

// ---- one Jacobi update, operation by operation.  Both forms of the two-sweep
// pass (the z-march and the blocks) go through these functions, with every
// fused multiply-add written out and none left to the compiler, so a cell's
// result is the same bit for bit whichever form a level takes.  Pairs of products
// are fused in the order that costs no product of its own: an instruction less
// per row than products shared between rows.

// k y summed over a pair of cells.
template <typename T>
__device__ __forceinline__ T pair_prod(T k0, T v0, T k1, T v1)
{
#pragma clang fp contract(off)
    const T p = k1 * v1;
    return fma(k0, v0, p);
}

// Corner and cross sums of a plane from its three rows: side pairs h, centres m.
template <typename T>
__device__ __forceinline__ T corner_sum(T ha, T hc)
{
    return ha + hc;
}
template <typename T>
__device__ __forceinline__ T cross_sum(T ma, T mc, T hb)
{
    return (ma + mc) + hb;
}
// The same of the product: the centres' coefficients and values, side pair p.
template <typename T>
__device__ __forceinline__ T cross_prod(T ka, T va, T kc, T vc, T p)
{
    return pair_prod(ka, va, kc, vc) + p;
}
// What a plane adds to the cell of a neighbouring plane: 2 X + D.
template <typename T>
__device__ __forceinline__ T neighbour_plane(T D, T X)
{
    return fma((T)2, X, D);
}

// y + omega (b - A y) / D with the sums S of y, k and k y; cw = -h/12,
// om_w0 = omega / (8h/3), icv = 24/h.
template <typename T>
__device__ __forceinline__ T jacobi_const(T y0, T Sx, T bb, T cw, T om_w0)
{
    return fma(om_w0, fma(-cw, fma((T)-32, y0, Sx), bb), y0);
}
template <typename T>
__device__ __forceinline__ T jacobi_nodal(T y0, T k0, T Sx, T Sk, T Sp, T bb, T om, T icv)
{
#pragma clang fp contract(off)
    const T Dg = fma((T)32, k0, Sk);
    const T ks = k0 * Sx;
    const T Ays = fma(Dg, y0, -ks) - Sp;
    const T w = om * fma(bb, icv, -Ays);
    return fma(w, recip(Dg), y0);
}

// Cell-centred linear interpolation along one axis: 3/4 near + 1/4 far.
template <typename T>
__device__ __forceinline__ T lerp31(T near, T far)
{
#pragma clang fp contract(off)
    const T f = (T)0.25 * far;
    return fma((T)0.75, near, f);
}

// Halo index -> interior index, flipping the sign across a Dirichlet-zero
// wall.  Indices beyond the one-cell halo (ragged tiles) are clamped into
// range; their values are never used by a valid output.
__device__ __forceinline__ int fold(int i, int n, int lo, int hi, int &sgn)
{
    if (i < 0) {
        if (lo == BC_P) {
            i += n;
            return i < 0 ? 0 : i;
        }
        if (lo == BC_D) sgn = -sgn;
        i = -1 - i;
        return i < n ? i : n - 1;
    }
    if (i >= n) {
        if (hi == BC_P) {
            i -= n;
            return i < n ? i : n - 1;
        }
        if (hi == BC_D) sgn = -sgn;
        i = 2 * n - 1 - i;
        return i >= 0 ? i : 0;
    }
    return i;
}

// Blocks are dispatched round-robin over the 8 XCDs (block b on XCD b % 8).
// Give each XCD a contiguous range of tiles so neighbouring tiles, which share
// halo lines, share that XCD's L2.
__device__ __forceinline__ int xcd_remap(int b, int nb)
{
    const int q = nb >> 3, r = nb & 7;
    const int x = b & 7, k = b >> 3;
    return (x < r) ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

}  // namespace
}  // namespace nn4mg
