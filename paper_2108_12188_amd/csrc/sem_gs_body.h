// sem_gs_body.h -- device code of the gather-scatter shared by the
// single-mesh and the batched kernels.
#pragma once

#include "sem_internal.h"

namespace sem {
namespace gsb {

constexpr int kGsThreads = 256;
constexpr int kXcds = 8;                          // MI355X: 8 XCDs, blocks dealt round-robin

// groups per thread for a group size: about 8 copies per thread in flight
__host__ __device__ constexpr int gs_per_thread(int M) { return M >= 8 ? 1 : (M >= 4 ? 2 : 4); }
__host__ __device__ constexpr int64_t gs_per_block(int M) {
    return (int64_t)kGsThreads * gs_per_thread(M);
}

template <int M>
struct alignas(M * 4 <= 16 ? M * 4 : 16) IdxVec {
    int32_t v[M];
};

// What a gather-scatter reads and writes at a local index; kMask: the groups
// on the Dirichlet boundary become zero.  A bit per group in group order marks
// them; its word loads with the indices and only selects the result, so that no
// load waits for it.
template <typename T>
struct InPlace {
    using Value = T;
    static constexpr bool kMask = false;
    T *__restrict__ w;
    __device__ __forceinline__ T load(int32_t q) const { return w[q]; }
    __device__ __forceinline__ void store(int32_t q, T s) const { w[q] = s; }
};
template <typename T>
struct InPlaceMasked : InPlace<T> {
    static constexpr bool kMask = true;
    const uint32_t *__restrict__ zero;
};

// b = mask(QQ^T (B f)): a group's products are rounded before they are summed
// (no contraction to a fused multiply-add), as a product vector in memory is.
template <typename T>
struct MassSource {
    using Value = double;
    static constexpr bool kMask = true;
    const double *__restrict__ B;
    const double *__restrict__ f;
    T *__restrict__ b;
    const uint32_t *__restrict__ zero;
    __device__ __forceinline__ double load(int32_t q) const {
#pragma clang fp contract(off)
        return B[q] * f[q];
    }
    __device__ __forceinline__ void store(int32_t q, double s) const { b[q] = (T)s; }
};

template <typename A>
__device__ __forceinline__ uint32_t mask_word(const A &a, int64_t zo, int64_t g) {
    if constexpr (A::kMask) return a.zero[zo + (g >> 5)];
    else return 0;
}

// Groups of a compile-time size M: every lane first issues the index loads
// of all its groups, then all value loads, so each lane keeps
// kGsPerThread * M independent loads in flight (groups are disjoint, so the
// stores of one group never alias the loads of another).
template <int M, typename A>
__device__ __forceinline__ void gs_groups_fixed(const int32_t *__restrict__ ib, int64_t g0,
                                                int64_t ng, int64_t zo, const A &a) {
    using V = typename A::Value;
    constexpr int kGsPerThread = gs_per_thread(M);
    int32_t q[kGsPerThread][M];
    bool ok[kGsPerThread];
    uint32_t zw[kGsPerThread];
#pragma unroll
    for (int it = 0; it < kGsPerThread; ++it) {
        const int64_t g = g0 + (int64_t)it * kGsThreads;
        ok[it] = g < ng;
        zw[it] = A::kMask ? mask_word(a, zo, ok[it] ? g : ng - 1) : 0;
        if (ok[it]) {
            const IdxVec<M> *src = reinterpret_cast<const IdxVec<M> *>(ib + g * M);
            const IdxVec<M> iv = *src;
#pragma unroll
            for (int t = 0; t < M; ++t) q[it][t] = iv.v[t];
        } else {
#pragma unroll
            for (int t = 0; t < M; ++t) q[it][t] = 0;
        }
    }
    V v[kGsPerThread][M];
#pragma unroll
    for (int it = 0; it < kGsPerThread; ++it) {
#pragma unroll
        for (int t = 0; t < M; ++t) v[it][t] = ok[it] ? a.load(q[it][t]) : V(0);
    }
#pragma unroll
    for (int it = 0; it < kGsPerThread; ++it) {
        if (!ok[it]) continue;
        V s = v[it][0];
#pragma unroll
        for (int t = 1; t < M; ++t) s += v[it][t];
        // every group of a thread has the same bit (a step is 256 groups)
        if (A::kMask && (zw[it] >> (g0 & 31) & 1)) s = V(0);
#pragma unroll
        for (int t = 0; t < M; ++t) a.store(q[it][t], s);
    }
}

template <typename A>
__device__ __forceinline__ void gs_groups_any(const int32_t *__restrict__ ib, int M, int64_t g0,
                                              int64_t ng, int64_t zo, const A &a) {
    for (int it = 0; it < gs_per_thread(M); ++it) {
        const int64_t g = g0 + (int64_t)it * kGsThreads;
        if (g >= ng) break;
        const int32_t *gi = ib + g * M;
        typename A::Value s = 0;
        if (!(mask_word(a, zo, g) >> (g & 31) & 1)) {
            s = a.load(gi[0]);
            for (int t = 1; t < M; ++t) s += a.load(gi[t]);
        }
        for (int t = 0; t < M; ++t) a.store(gi[t], s);
    }
}

// Sums only: out[g] = sum of the copies of group g (ascending local index,
// the order of gs_groups_fixed); w is read, not written.  Loads of all of a
// lane's groups are issued before any sum, as in gs_groups_fixed.
template <typename T, int M>
__device__ __forceinline__ void gs_sums_fixed(const int32_t *__restrict__ ib, int64_t g0,
                                              int64_t ng, const T *__restrict__ w,
                                              T *__restrict__ out) {
    constexpr int kGsPerThread = gs_per_thread(M);
    int32_t q[kGsPerThread][M];
    bool ok[kGsPerThread];
#pragma unroll
    for (int it = 0; it < kGsPerThread; ++it) {
        const int64_t g = g0 + (int64_t)it * kGsThreads;
        ok[it] = g < ng;
        if (ok[it]) {
            const IdxVec<M> iv = *reinterpret_cast<const IdxVec<M> *>(ib + g * M);
#pragma unroll
            for (int t = 0; t < M; ++t) q[it][t] = iv.v[t];
        } else {
#pragma unroll
            for (int t = 0; t < M; ++t) q[it][t] = 0;
        }
    }
    T v[kGsPerThread][M];
#pragma unroll
    for (int it = 0; it < kGsPerThread; ++it)
#pragma unroll
        for (int t = 0; t < M; ++t) v[it][t] = ok[it] ? w[q[it][t]] : T(0);
#pragma unroll
    for (int it = 0; it < kGsPerThread; ++it) {
        if (!ok[it]) continue;
        T s = v[it][0];
#pragma unroll
        for (int t = 1; t < M; ++t) s += v[it][t];
        out[g0 + (int64_t)it * kGsThreads] = s;
    }
}

template <typename T>
__device__ __forceinline__ void gs_sums_any(const int32_t *__restrict__ ib, int M, int64_t g0,
                                            int64_t ng, const T *__restrict__ w,
                                            T *__restrict__ out) {
    for (int it = 0; it < gs_per_thread(M); ++it) {
        const int64_t g = g0 + (int64_t)it * kGsThreads;
        if (g >= ng) break;
        const int32_t *gi = ib + g * M;
        T s = w[gi[0]];
        for (int t = 1; t < M; ++t) s += w[gi[t]];
        out[g] = s;
    }
}

// One logical block lb of a mesh's group sums over the classes with
// M >= mmin (3: the groups of more than two copies of the full class list;
// 2: every class of the edge-node list of the table-free gather).  The
// copies of class c's groups are read from w at the indices
// idx[cls.io[c] - io0 ...] (gs_idx and the local w, or the compact edge
// array and its positions); the sums go to out + (groups of the classes
// with M >= mmin before c).
template <typename T>
__device__ __forceinline__ void gs_sums_logical_block(const GsClasses &cls, int64_t lb,
                                                      const int32_t *__restrict__ idx,
                                                      int64_t io0, const T *__restrict__ w,
                                                      T *__restrict__ out, int mmin = 3) {
    int c = 0;
    while (c + 1 < cls.ncls && lb >= cls.blk0[c + 1]) ++c;
    int64_t goff = 0;
    for (int q = 0; q < c; ++q)
        if (cls.M[q] >= mmin) goff += cls.ng[q];
    const int M = cls.M[c];
    const int64_t g0 = (lb - cls.blk0[c]) * gs_per_block(M) + threadIdx.x;
    const int32_t *ib = idx + (cls.io[c] - io0);
    const int64_t ng = cls.ng[c];
    switch (M) {
        case 2: gs_sums_fixed<T, 2>(ib, g0, ng, w, out + goff); break;
        case 4: gs_sums_fixed<T, 4>(ib, g0, ng, w, out + goff); break;
        case 8: gs_sums_fixed<T, 8>(ib, g0, ng, w, out + goff); break;
        default: gs_sums_any<T>(ib, M, g0, ng, w, out + goff); break;
    }
}

// The logical block at position lb of a gather-scatter launch (uniform
// across the block), in the class-major block numbering after the mesh's
// block order, if it has one.
template <typename A>
__device__ __forceinline__ void gs_logical_block(const GsClasses &cls, int64_t lb,
                                                 const int32_t *__restrict__ idx, const A &a) {
    if (cls.lb_order) lb = cls.lb_order[lb];
    int c = 0;
    while (c + 1 < cls.ncls && lb >= cls.blk0[c + 1]) ++c;
    const int M = cls.M[c];
    const int64_t g0 = (lb - cls.blk0[c]) * gs_per_block(M) + threadIdx.x;
    const int32_t *ib = idx + cls.io[c];
    const int64_t ng = cls.ng[c], zo = cls.zo[c];
    switch (M) {
        case 2: gs_groups_fixed<2>(ib, g0, ng, zo, a); break;
        case 4: gs_groups_fixed<4>(ib, g0, ng, zo, a); break;
        case 8: gs_groups_fixed<8>(ib, g0, ng, zo, a); break;
        default: gs_groups_any(ib, M, g0, ng, zo, a); break;
    }
}

}  // namespace gsb
}  // namespace sem
