// sem_reduce.h -- deterministic reductions: every reduction kernel writes
// one FP64 partial per block; a one-block finalize kernel that follows in
// stream order sums the partials in index order.  (No grid-wide fences: on
// a chip whose L2 caches are private to each XCD an agent-scope fence per
// block costs an L2 write-back per block.)
#pragma once

#include <hip/hip_runtime.h>

#include "sem_internal.h"

namespace sem {

constexpr int kFinalizeThreads = 1024;

// s_waitcnt immediate (gfx9 encoding): lgkmcnt(0) alone
constexpr int kWaitLgkmcnt0 = 0xC07F;

// Barrier for LDS traffic only: the wave's own LDS accesses complete
// before it, but global loads and stores -- and staging loads, which
// write LDS -- keep flying across it (a fenced __syncthreads would wait for
// all of them).  The memory clobber keeps the compiler from moving any
// memory access across the barrier.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_s_waitcnt(kWaitLgkmcnt0);
    __asm__ volatile("s_barrier" ::: "memory");
}

// Sum of one double per thread in a fixed order; the result is valid in
// thread 0 only.  Every thread of the block must call it.
__device__ __forceinline__ double block_sum_f64(double v, double *red /* >= 16 */) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int wid = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[wid] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        for (int q = 0; q < nw; ++q) s += red[q];
    }
    __syncthreads();
    return s;
}

// Fixed-order sum of partial[0..cnt) by one block: thread t sums the
// entries t, t + blockDim, ... in order, then the block sums the threads.
// The loads of a batch of kBatch entries are issued before they are added,
// so the one block keeps many loads in flight.
__device__ __forceinline__ double sum_partials(const double *partial, int64_t cnt, double *red) {
    constexpr int kBatch = 8;
    double v = 0.0;
    const int64_t step = (int64_t)blockDim.x * kBatch;
    for (int64_t q0 = threadIdx.x; q0 < cnt; q0 += step) {
        double t[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int64_t q = q0 + (int64_t)u * blockDim.x;
            t[u] = q < cnt ? partial[q] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) v += t[u];
    }
    return block_sum_f64(v, red);
}

// Sum of one double per lane of a wave in a fixed order, valid in every lane:
// within rows of 16 lanes, then across the four rows, by data-parallel lane
// moves, which need no LDS round trip.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_add_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, kCtrl, kRowMask, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, kRowMask, 0xf, false);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double wave_sum_f64(double v) {
    v = dpp_add_f64<0x111, 0xf>(v);      // row_shr 1, 2, 4, 8: lane 15 of a row
    v = dpp_add_f64<0x112, 0xf>(v);      // holds the row's sum (lanes without a
    v = dpp_add_f64<0x114, 0xf>(v);      // source add 0)
    v = dpp_add_f64<0x118, 0xf>(v);
    v = dpp_add_f64<0x142, 0xa>(v);      // lane 15 to the next row: rows 1 and 3
    v = dpp_add_f64<0x143, 0xc>(v);      // lane 31 to rows 2 and 3
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, 63);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The same kind of sum by the first nthr threads of a block (a multiple of
// 64), valid in every thread: in a fixed order that depends on nthr only.
// A block of one wave (kOneWave, nthr = 64) needs no LDS.  In two parts, so
// that the first loads can fly while others are issued.  Threads past the
// end read the last entry (no load under a condition, which the compiler
// would wait for) and add 0.
template <bool kOneWave = false>
struct PartialSum {
    static constexpr int kBatch = kOneWave ? 16 : 8;
    double x[kBatch];
    __device__ __forceinline__ void load(const double *partial, int cnt, int nthr, int k0) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int q = k0 + u * nthr + (int)threadIdx.x;
            x[u] = partial[q < cnt ? q : cnt - 1];
        }
    }
    // after load(..., 0)
    __device__ __forceinline__ double finish(const double *partial, int cnt, int nthr,
                                             double *red /* >= 16 */) {
        const int t = (int)threadIdx.x;
        double v = 0.0;
        for (int k0 = 0;;) {                                       // uniform
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                v += k0 + u * nthr + t < cnt && t < nthr ? x[u] : 0.0;
            k0 += nthr * kBatch;
            if (k0 >= cnt) break;
            load(partial, cnt, nthr, k0);
        }
        v = wave_sum_f64(v);
        if constexpr (kOneWave) return v;
        if ((t & 63) == 0) red[t >> 6] = v;
        lds_barrier();
        double s = 0.0;
        for (int q = 0; q < (nthr >> 6); ++q) s += red[q];
        lds_barrier();
        return s;
    }
};
static_assert(64 * PartialSum<true>::kBatch == kInlineVecBlocksMfma &&
                  128 * PartialSum<false>::kBatch == kInlineVecBlocksMfma,
              "the matrix-core blocks (N = 7: 64 threads, N = 9: 128) read the partials in one round");
template <bool kOneWave = false>
__device__ __forceinline__ double sum_partials_all(const double *partial, int cnt, int nthr,
                                                   double *red) {
    PartialSum<kOneWave> p;
    p.load(partial, cnt, nthr, 0);
    return p.finish(partial, cnt, nthr, red);
}

// The changing part of a state, read in one go.
__device__ __forceinline__ CgStep load_step(const CgState *st) {
    return {st->rho, st->rr, st->alpha, st->beta, st->pw, st->iter, st->stop, st->x_lag,
            st->rho_pending};
}
__device__ __forceinline__ void store_step(CgState *st, const CgStep &s) {
    st->rho = s.rho;
    st->rr = s.rr;
    st->alpha = s.alpha;
    st->beta = s.beta;
    st->pw = s.pw;
    st->iter = s.iter;
    st->stop = s.stop;
    st->x_lag = s.x_lag;
    st->rho_pending = s.rho_pending;
}

// The rho step of Algorithm 1 after a completed update: rho_i = rho, beta_i =
// rho_i / rho_{i-1}, the iteration count and the stopping test (rr =
// <r, r, c>).  The history entry is the caller's.
__device__ __forceinline__ void rho_step(CgStep &s, double rho, double rr, double thresh,
                                         int max_iter, int fixed) {
    s.beta = rho / s.rho;
    s.rho = rho;
    s.rr = rr;
    s.rho_pending = 0;
    s.iter = s.iter + 1;
    s.stop = !isfinite(rho) || !isfinite(rr) ? 3
             : !fixed && rr <= thresh        ? 1
             : s.iter >= max_iter            ? 2
                                             : 0;
}

}  // namespace sem
