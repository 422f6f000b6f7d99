// sem_geom_body.h -- geometry of the trilinear map along one column of an
// element's points, shared by the operator and the set-up kernels.
#pragma once

#include "sem_internal.h"

namespace sem {
namespace {

// a * b + c with one rounding.
template <typename T>
__device__ __forceinline__ T fmadd(T a, T b, T c) {
    if constexpr (sizeof(T) == 4) return __builtin_fmaf(a, b, c);
    else return __builtin_fma(a, b, c);
}

template <typename T>
struct Vec3 {
    T x, y, z;
};
template <typename T>
__device__ __forceinline__ Vec3<T> cross(const Vec3<T> &a, const Vec3<T> &b) {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
template <typename T>
__device__ __forceinline__ T dot3(const Vec3<T> &a, const Vec3<T> &b) {
    return a.x * b.x + a.y * b.y + a.z * b.z;
}
template <typename T>
__device__ __forceinline__ Vec3<T> axpy3(T s, const Vec3<T> &a, const Vec3<T> &b) {
    return {b.x + s * a.x, b.y + s * a.y, b.z + s * a.z};   // b + s a
}
template <typename T>
__device__ __forceinline__ Vec3<T> add3(const Vec3<T> &a, const Vec3<T> &b) {
    return {a.x + b.x, a.y + b.y, a.z + b.z};
}

// Per-thread constants of the trilinear map along one (i, j) column.
// Along the column only gamma varies, and
//   x_xi(gamma) = A0 + gamma A1,  x_eta(gamma) = B0 + gamma B1,  x_gamma = C,
// so the cofactor rows r0 = x_eta x x_gamma, r1 = x_gamma x x_xi,
// r2 = x_xi x x_eta and |J| = x_xi . r0 are low-degree polynomials in gamma.
template <typename T>
struct ColumnGeom {
    Vec3<T> R00, R01, R10, R11, R20, R21, R22;
    T d0, d1, d2, wij;
};

// The 12 edge vectors of an element from its 8 vertices, in the order the
// column geometry uses them: along xi (v1 - v0, v3 - v2, v5 - v4, v7 - v6),
// along eta (v2 - v0, v3 - v1, v6 - v4, v7 - v5), along gamma (v4 - v0,
// v5 - v1, v6 - v2, v7 - v3); ed[t * 3 + d].  The host builds the same
// FP32 array per element (Mesh::edge32) with the same subtractions.
template <typename T, typename VertPtr>
__device__ __forceinline__ void element_edges(VertPtr ve, T (&ed)[36]) {
    constexpr int kA[12] = {1, 3, 5, 7, 2, 3, 6, 7, 4, 5, 6, 7};
    constexpr int kB[12] = {0, 2, 4, 6, 0, 1, 4, 5, 0, 1, 2, 3};
#pragma unroll
    for (int t = 0; t < 12; ++t)
#pragma unroll
        for (int d = 0; d < 3; ++d) ed[t * 3 + d] = ve[kA[t] * 3 + d] - ve[kB[t] * 3 + d];
}

template <typename T, typename EdgePtr>
__device__ __forceinline__ ColumnGeom<T> column_geom_edges(EdgePtr ed, T xi_i, T eta_j, T wij) {
    const T fi0 = T(0.5) * (T(1) - xi_i), fi1 = T(0.5) * (T(1) + xi_i);
    const T fj0 = T(0.5) * (T(1) - eta_j), fj1 = T(0.5) * (T(1) + eta_j);
    T A0[3], A1[3], B0[3], B1[3], Cc[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        // Every product-sum here is an explicit fused multiply-add: the
        // edges may sit in scalar registers (matrix-core operator) or come
        // out of subtractions (VALU operator), and both must round alike.
        // d/dxi at (eta_j, gamma corner c)
        const T a0 = T(0.5) * fmadd(ed[0 * 3 + d], fj0, ed[1 * 3 + d] * fj1);
        const T a1 = T(0.5) * fmadd(ed[2 * 3 + d], fj0, ed[3 * 3 + d] * fj1);
        // d/deta at (xi_i, gamma corner c)
        const T b0 = T(0.5) * fmadd(ed[4 * 3 + d], fi0, ed[5 * 3 + d] * fi1);
        const T b1 = T(0.5) * fmadd(ed[6 * 3 + d], fi0, ed[7 * 3 + d] * fi1);
        A0[d] = T(0.5) * (a0 + a1);
        A1[d] = T(0.5) * (a1 - a0);
        B0[d] = T(0.5) * (b0 + b1);
        B1[d] = T(0.5) * (b1 - b0);
        const T c4 = fmadd(ed[9 * 3 + d] * fi1, fj0, ed[8 * 3 + d] * fi0 * fj0);
        const T c6 = fmadd(ed[10 * 3 + d] * fi0, fj1, c4);
        Cc[d] = T(0.5) * fmadd(ed[11 * 3 + d] * fi1, fj1, c6);
    }
    const Vec3<T> a0{A0[0], A0[1], A0[2]}, a1{A1[0], A1[1], A1[2]};
    const Vec3<T> b0{B0[0], B0[1], B0[2]}, b1{B1[0], B1[1], B1[2]};
    const Vec3<T> c{Cc[0], Cc[1], Cc[2]};
    ColumnGeom<T> g;
    g.R00 = cross(b0, c);
    g.R01 = cross(b1, c);
    g.R10 = cross(c, a0);
    g.R11 = cross(c, a1);
    g.R20 = cross(a0, b0);
    g.R21 = add3(cross(a0, b1), cross(a1, b0));
    g.R22 = cross(a1, b1);
    g.d0 = dot3(a0, g.R00);
    g.d1 = dot3(a0, g.R01) + dot3(a1, g.R00);
    g.d2 = dot3(a1, g.R01);
    g.wij = wij;
    return g;
}

template <typename T, typename VertPtr>
__device__ __forceinline__ ColumnGeom<T> column_geom(VertPtr ve, T xi_i, T eta_j, T wij) {
    T ed[36];
    element_edges<T>(ve, ed);
    return column_geom_edges<T>(ed, xi_i, eta_j, wij);
}

}  // namespace
}  // namespace sem
