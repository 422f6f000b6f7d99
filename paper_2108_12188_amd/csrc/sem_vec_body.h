// sem_vec_body.h -- device code of the Algorithm 1 vector update and the
// one-block finalize steps, shared by the single-mesh and batched kernels.
#pragma once

#include "sem_internal.h"
#include "sem_reduce.h"

namespace sem {
namespace vecb {

constexpr int kVecThreads = 256;
#ifndef SEM_VEC_MAX_BLOCKS
#define SEM_VEC_MAX_BLOCKS 4096
#endif
constexpr int kVecMaxBlocks = SEM_VEC_MAX_BLOCKS;
// packs of 4 points a thread of the gather update keeps in flight per step
#ifndef SEM_UPD_PACKS
#define SEM_UPD_PACKS 2
#endif
constexpr int kUpdPacks = SEM_UPD_PACKS;
// the same for the table-free gather, whose records already keep loads in
// flight (one pack per step measured faster there); the per-thread packs
// and their order are those of every K, so both forms agree bitwise
#ifndef SEM_UPD_STRUCT_PACKS
#define SEM_UPD_STRUCT_PACKS 1
#endif
constexpr int kUpdStructPacks = SEM_UPD_STRUCT_PACKS;

// Blocks are dealt to the 8 XCDs round-robin (block b on XCD b mod 8): the
// vector updates give each XCD a contiguous range of the logical blocks
// instead (a bijection on [0, vgrid); the last vgrid mod 8 blocks keep
// their place), so that the face partners a block reads in neighbouring
// elements were mostly brought in through the same L2.  The ρ partial of a
// block stays at its own index vb.
__device__ __forceinline__ int64_t xcd_block(int64_t vb, int64_t vgrid) {
    const int64_t full = vgrid & ~int64_t(7);
    if (vb >= full) return vb;
    return (vb & 7) * (full >> 3) + (vb >> 3);
}

template <typename T>
struct alignas(4 * sizeof(T)) Pack4 {
    T v[4];
};
struct alignas(4) Code4 {
    uint8_t v[4];
};

__device__ __forceinline__ void weights_lds(double *cw) {
    // weight 1/m for every code (m in the low bits; exact for powers of two)
    const int m = threadIdx.x & kMultMask;
    cw[threadIdx.x] = m ? 1.0 / (double)m : 0.0;
    __syncthreads();
}

// [x += alpha p;] r -= alpha mask(w); rho_i = <r, r, c>  (Algorithm 1:
// mask, fused updates and reduction; the operator leaves w unmasked).
// WithX = false leaves x to the next operator launch (single-mesh solves).
// PC: also z = minv r, partial <- <r, z, c>, partial2 <- <r, r, c>.
// Virtual block vb of a grid of vgrid blocks; the partial goes to
// partial[vb].
template <typename T, bool WithX, bool PC = false>
__device__ __forceinline__ void update_body(int64_t n, T *__restrict__ x, T *__restrict__ r,
                                            const T *__restrict__ p, const T *__restrict__ w,
                                            const uint8_t *__restrict__ mcode, CgState *st,
                                            double *partial, int64_t vb, int64_t vgrid,
                                            PcArgs<T> pc = PcArgs<T>{}) {
    // the state's loads go out with the block's set-up; a stopped state
    // returns before the first store to global memory (uniform)
    const int stopped = st->stop;
    const T a = (T)st->alpha;
    __shared__ double cw[kVecThreads];
    __shared__ double red[16];
    weights_lds(cw);
    if (stopped) return;
    double acc = 0.0, acc2 = 0.0;
    const int64_t n4 = n >> 2;
    const int64_t stride = vgrid * blockDim.x;
    const int64_t tid = xcd_block(vb, vgrid) * blockDim.x + threadIdx.x;
    for (int64_t q = tid; q < n4; q += stride) {
        Pack4<T> rv = reinterpret_cast<const Pack4<T> *>(r)[q];
        const Pack4<T> wv = reinterpret_cast<const Pack4<T> *>(w)[q];
        const Code4 mv = reinterpret_cast<const Code4 *>(mcode)[q];
        if constexpr (WithX) {
            Pack4<T> xv = reinterpret_cast<const Pack4<T> *>(x)[q];
            const Pack4<T> pv = reinterpret_cast<const Pack4<T> *>(p)[q];
#pragma unroll
            for (int t = 0; t < 4; ++t) xv.v[t] += a * pv.v[t];
            reinterpret_cast<Pack4<T> *>(x)[q] = xv;
        }
        Pack4<T> mi{}, zv{};
        if constexpr (PC) mi = reinterpret_cast<const Pack4<T> *>(pc.minv)[q];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const T wm = (mv.v[t] & kDirichletBit) ? T(0) : wv.v[t];
            rv.v[t] -= a * wm;
            const double rd = (double)rv.v[t];
            if constexpr (PC) {
                zv.v[t] = mi.v[t] * rv.v[t];
                acc += rd * (double)zv.v[t] * cw[mv.v[t]];
                acc2 += rd * rd * cw[mv.v[t]];
            } else {
                acc += rd * rd * cw[mv.v[t]];
            }
        }
        reinterpret_cast<Pack4<T> *>(r)[q] = rv;
        if constexpr (PC) reinterpret_cast<Pack4<T> *>(pc.z)[q] = zv;
    }
    for (int64_t q = 4 * n4 + tid; q < n; q += stride) {
        const uint8_t c = mcode[q];
        if constexpr (WithX) x[q] += a * p[q];
        const T rn = r[q] - a * ((c & kDirichletBit) ? T(0) : w[q]);
        r[q] = rn;
        if constexpr (PC) {
            const T zn = pc.minv[q] * rn;
            pc.z[q] = zn;
            acc += (double)rn * (double)zn * cw[c];
            acc2 += (double)rn * (double)rn * cw[c];
        } else {
            acc += (double)rn * (double)rn * cw[c];
        }
    }
    const double s = block_sum_f64(acc, red);
    if (threadIdx.x == 0) partial[vb] = s;
    if constexpr (PC) {
        const double s2 = block_sum_f64(acc2, red);
        if (threadIdx.x == 0) pc.partial2[vb] = s2;
    }
}

// Where the sums over the copies are formed inside the update: per local
// point the partner of a pair point, the group rank of a point in a larger
// group, else the point's own index (see Mesh::gsrc).
struct GatherMap {
    const int32_t *gsrc;         // [n]
};

// Code of a pair point off the Dirichlet boundary: m = 2, flag clear.
constexpr uint8_t kPairCode = 2;

__host__ __device__ __forceinline__ bool is_group_code(uint8_t code) {
    return (code & kMultMask) > 2 && !(code & kDirichletBit);
}

// The one value point l loads besides its own: its partner's w (pairs), its
// group's sum (larger groups), else its own w again.
template <typename T>
__host__ __device__ __forceinline__ const T *gather_source(const T *w, const T *gsum,
                                                           uint8_t code, int32_t lk, int64_t l) {
    const bool group = is_group_code(code);
    const T *base = group ? gsum : w;
    const int64_t off = (code == kPairCode || group) ? (int64_t)(uint32_t)lk : l;
    return base + off;
}

// mask(QQ^T w)_l: a pair adds its partner's value (a + b == b + a in IEEE
// arithmetic, so both copies get the sum the gather-scatter forms); a point
// of a larger group takes the group's sum (formed in the gather-scatter's
// order); points with m = 1 keep their own value, Dirichlet points get 0.
// src: the value at gather_source.
template <typename T>
__host__ __device__ __forceinline__ T copies_sum(T own, uint8_t code, T src) {
    // selects, not branches: src is consumed on every path
    const T pair_sum = own + src;
    T v = code == kPairCode ? pair_sum : own;
    v = is_group_code(code) ? src : v;
    return (code & kDirichletBit) ? T(0) : v;
}

// update_body<T, false> with w replaced by QQ^T w (w itself is not
// modified).  Same grid, same per-thread order and the same sums as
// gather-scatter + update_body, so the results are bitwise those of the
// two-pass form.  All loads are unconditional: two packs (q, q + stride)
// per step, each costing two dependent rounds of loads (r, w, the codes and
// the 4 gather-table entries of a pack, then the 4 gathered values), all
// loads of both packs issued before any result is used; the sum of r^2/m
// still runs pack by pack in the thread's order q, q + stride, ...
template <typename T, bool PC = false>
__device__ __forceinline__ void update_gather_body(int64_t n, T *__restrict__ r,
                                                   const T *__restrict__ w,
                                                   const T *__restrict__ gsum,
                                                   const uint8_t *__restrict__ mcode,
                                                   const GatherMap &gm, CgState *st,
                                                   double *partial, int64_t vb, int64_t vgrid,
                                                   PcArgs<T> pc = PcArgs<T>{},
                                                   int packs = kVecThreads) {
    // the state's loads go out with the block's set-up; a stopped state
    // returns before the first store to global memory (uniform)
    const int stopped = st->stop;
    const T a = (T)st->alpha;
    __shared__ double cw[kVecThreads];
    __shared__ double red[16];
    weights_lds(cw);
    if (stopped) return;
    double acc = 0.0, acc2 = 0.0;
    const int64_t n4 = n >> 2;
    // threads past the block's packs have none (then n is a multiple of 4)
    const int64_t stride = vgrid * packs;
    const int64_t tid = (int)threadIdx.x < packs ? xcd_block(vb, vgrid) * packs + threadIdx.x : n4;
    constexpr int K = kUpdPacks;
    for (int64_t q = tid; q < n4; q += K * stride) {
        int64_t qq[K];
        bool live[K];
#pragma unroll
        for (int h = 0; h < K; ++h) {
            live[h] = q + h * stride < n4;
            qq[h] = live[h] ? q + h * stride : q;
        }
        int32_t lk[K][4];
        Pack4<T> rv[K], wv[K];
        Code4 mv[K];
#pragma unroll
        for (int h = 0; h < K; ++h) {
            const int4 g4 = reinterpret_cast<const int4 *>(gm.gsrc)[qq[h]];
            lk[h][0] = g4.x, lk[h][1] = g4.y, lk[h][2] = g4.z, lk[h][3] = g4.w;
            rv[h] = reinterpret_cast<const Pack4<T> *>(r)[qq[h]];
            wv[h] = reinterpret_cast<const Pack4<T> *>(w)[qq[h]];
            mv[h] = reinterpret_cast<const Code4 *>(mcode)[qq[h]];
        }
        T src[K][4];
#pragma unroll
        for (int h = 0; h < K; ++h)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                src[h][t] = *gather_source<T>(w, gsum, mv[h].v[t], lk[h][t],
                                              (int64_t)(4 * qq[h] + t));
        // a pack past the end (!live) repeats the first: it stores the same
        // values and adds exactly 0 to the sums (every result is consumed on
        // every path, so no load of this step is still pending when the next
        // step reuses its registers)
#pragma unroll
        for (int h = 0; h < K; ++h) {
            Pack4<T> mi{}, zv{};
            if constexpr (PC) mi = reinterpret_cast<const Pack4<T> *>(pc.minv)[qq[h]];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const T wg = copies_sum<T>(wv[h].v[t], mv[h].v[t], src[h][t]);
                rv[h].v[t] -= a * wg;
                const double rd = (double)rv[h].v[t];
                if constexpr (PC) {
                    zv.v[t] = mi.v[t] * rv[h].v[t];
                    acc += live[h] ? rd * (double)zv.v[t] * cw[mv[h].v[t]] : 0.0;
                    acc2 += live[h] ? rd * rd * cw[mv[h].v[t]] : 0.0;
                } else {
                    acc += live[h] ? rd * rd * cw[mv[h].v[t]] : 0.0;
                }
            }
            reinterpret_cast<Pack4<T> *>(r)[qq[h]] = rv[h];
            if constexpr (PC) reinterpret_cast<Pack4<T> *>(pc.z)[qq[h]] = zv;
        }
    }
    for (int64_t q = 4 * n4 + tid; q < n; q += stride) {
        const uint8_t c = mcode[q];
        const int32_t lk = gm.gsrc[q];
        const T wg = copies_sum<T>(w[q], c, *gather_source<T>(w, gsum, c, lk, q));
        const T rn = r[q] - a * wg;
        r[q] = rn;
        if constexpr (PC) {
            const T zn = pc.minv[q] * rn;
            pc.z[q] = zn;
            acc += (double)rn * (double)zn * cw[c];
            acc2 += (double)rn * (double)rn * cw[c];
        } else {
            acc += (double)rn * (double)rn * cw[c];
        }
    }
    const double s = block_sum_f64(acc, red);
    if (threadIdx.x == 0) partial[vb] = s;
    if constexpr (PC) {
        const double s2 = block_sum_f64(acc2, red);
        if (threadIdx.x == 0) pc.partial2[vb] = s2;
    }
}

// Table-free form of the same gather (Mesh::gs_struct): a point's copies
// follow from its position in the element and the element's records.
struct StructMap {
    const ElemRec *rec;         // [E][nrec]
    const uint32_t *pos_tab;    // [p3] (pos_entry)
    int p3, nrec;               // P^3, 6 + edge_slots(N)
    uint32_t magic;             // element of local index l: (l * magic) >> shift
    int shift;
};
constexpr int kMaxPosTab = kMaxP * kMaxP * kMaxP;

__host__ __device__ __forceinline__ int64_t struct_elem(const StructMap &sm, int64_t l) {
    return (int64_t)(((uint64_t)l * sm.magic) >> sm.shift);
}

// The record point l (element e, position entry pe) needs: its face's or
// its edge slot's (face 0's for an interior point, which uses none).
// Loaded first: the address of the value the point gathers depends on it.
__host__ __device__ __forceinline__ ElemRec struct_record(const StructMap &sm, int64_t e,
                                                          uint32_t pe) {
    return sm.rec[e * sm.nrec + (pe >> 12)];
}

// Where point l finds the value it loads besides its own w, as an index
// into wg = [w | the edge-group sums] (the sums sit right after the n local
// values): a face point the copy on the neighbour's face (its own index
// when it has none), a shared edge or corner node n + its group's rank, any
// other point its own index; and its code byte.  Every path gives an index
// inside wg.
struct StructSrc {
    int32_t idx;      // n + the number of edge groups stays below 2^31 (host check)
    uint8_t code;
    bool edge;
};
__host__ __device__ __forceinline__ StructSrc struct_source(const StructMap &sm, int64_t n,
                                                            int64_t l, uint32_t pe,
                                                            const ElemRec &rc) {
    const int kind = (int)(pe & 3);
    const int a = (int)((pe >> 2) & 31), b = (int)((pe >> 7) & 31);
    const uint8_t code = (uint8_t)(rc.hi & 255);
    const int32_t sa = (int32_t)((uint32_t)rc.hi << 12) >> 20;   // bits 8-19, signed
    const int32_t sb = rc.hi >> 20;                               // bits 20-31, signed
    const int32_t q = rc.lo + sa * a + sb * b;
    const bool eshared = (code & kMultMask) >= 2 && !(code & kDirichletBit);
    StructSrc s;
    const int32_t own_or_face = kind == 1 ? q : (int32_t)l;
    s.idx = (kind == 2 && eshared) ? (int32_t)n + rc.lo : own_or_face;
    s.code = kind == 0 ? (uint8_t)1 : code;
    s.edge = kind == 2;
    return s;
}
// mask(QQ^T w)_l from the loaded value: a face pair adds its partner (the
// sum a + b == b + a of the gather-scatter), a shared edge or corner node
// takes its group's sum (the gather-scatter's ascending order), points with
// m = 1 keep their own value, Dirichlet points get 0.
template <typename T>
__host__ __device__ __forceinline__ T struct_sum(T own, uint8_t code, bool edge, T src) {
    const bool shared = (code & kMultMask) >= 2;
    const T pair_sum = own + src;
    T v = edge ? (shared ? src : own) : (code == kPairCode ? pair_sum : own);
    return (code & kDirichletBit) ? T(0) : v;
}

// update_gather_body with the table-free gather: the same per-thread packs,
// the same values and the same sums, so bitwise the same results.  n is a
// multiple of 4 (P^3 is), and the 4 points of a pack lie in one element.
// wg: w followed by the edge-group sums.  Load order: the element records
// first (pinned there by a compiler fence, so none is moved into a branch),
// then r and w, then the gathered values, whose addresses need only
// the records (loads complete in issue order, so the gathers wait for the
// records, not for r and w).
template <typename T, bool PC = false>
__device__ __forceinline__ void update_struct_body(int64_t n, T *__restrict__ r,
                                                   const T *__restrict__ wg,
                                                   const StructMap &sm, CgState *st,
                                                   double *partial, int64_t vb, int64_t vgrid,
                                                   PcArgs<T> pc = PcArgs<T>{},
                                                   int packs = kVecThreads) {
    // the state's loads go out with the block's set-up; a stopped state
    // returns before the first store to global memory (uniform)
    const int stopped = st->stop;
    const T a = (T)st->alpha;
    __shared__ double cw[kVecThreads];
    __shared__ double red[16];
    __shared__ __align__(16) uint32_t pos[kMaxPosTab];
    for (int q = threadIdx.x; q < sm.p3; q += blockDim.x) pos[q] = sm.pos_tab[q];
    weights_lds(cw);
    if (stopped) return;
    double acc = 0.0, acc2 = 0.0;
    const int64_t n4 = n >> 2;
    // threads past the block's packs have none (then n is a multiple of 4)
    const int64_t stride = vgrid * packs;
    const int64_t tid = (int)threadIdx.x < packs ? xcd_block(vb, vgrid) * packs + threadIdx.x : n4;
    constexpr int K = kUpdStructPacks;
    for (int64_t q = tid; q < n4; q += K * stride) {
        int64_t qq[K];
        bool live[K];
#pragma unroll
        for (int h = 0; h < K; ++h) {
            live[h] = q + h * stride < n4;
            qq[h] = live[h] ? q + h * stride : q;
        }
        uint32_t pv[K][4];
        ElemRec rc[K][4];
#pragma unroll
        for (int h = 0; h < K; ++h) {
            const int64_t l0 = 4 * qq[h];
            const int64_t e = struct_elem(sm, l0);
            // 16-byte entries (P^3 and l0 are multiples of 4): one ds_read_b128
            const uint4 pe = reinterpret_cast<const uint4 *>(pos)[(l0 - e * sm.p3) >> 2];
            pv[h][0] = pe.x, pv[h][1] = pe.y, pv[h][2] = pe.z, pv[h][3] = pe.w;
#pragma unroll
            for (int t = 0; t < 4; ++t) rc[h][t] = struct_record(sm, e, pv[h][t]);
        }
        __asm__ volatile("" ::: "memory");
        Pack4<T> rv[K], wv[K];
#pragma unroll
        for (int h = 0; h < K; ++h) {
            rv[h] = reinterpret_cast<const Pack4<T> *>(r)[qq[h]];
            wv[h] = reinterpret_cast<const Pack4<T> *>(wg)[qq[h]];
        }
        int32_t ix[K][4];
        uint8_t cd[K][4];
        bool ed[K][4];
#pragma unroll
        for (int h = 0; h < K; ++h)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const StructSrc ss = struct_source(sm, n, 4 * qq[h] + t, pv[h][t], rc[h][t]);
                ix[h][t] = ss.idx;
                cd[h][t] = ss.code;
                ed[h][t] = ss.edge;
            }
        T src[K][4];
#pragma unroll
        for (int h = 0; h < K; ++h)
#pragma unroll
            for (int t = 0; t < 4; ++t) src[h][t] = wg[ix[h][t]];
        // a pack past the end (!live) repeats the first: it stores the same
        // values and adds exactly 0 to the sums
#pragma unroll
        for (int h = 0; h < K; ++h) {
            Pack4<T> mi{}, zv{};
            if constexpr (PC) mi = reinterpret_cast<const Pack4<T> *>(pc.minv)[qq[h]];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const T wg = struct_sum<T>(wv[h].v[t], cd[h][t], ed[h][t], src[h][t]);
                rv[h].v[t] -= a * wg;
                const double rd = (double)rv[h].v[t];
                if constexpr (PC) {
                    zv.v[t] = mi.v[t] * rv[h].v[t];
                    acc += live[h] ? rd * (double)zv.v[t] * cw[cd[h][t]] : 0.0;
                    acc2 += live[h] ? rd * rd * cw[cd[h][t]] : 0.0;
                } else {
                    acc += live[h] ? rd * rd * cw[cd[h][t]] : 0.0;
                }
            }
            reinterpret_cast<Pack4<T> *>(r)[qq[h]] = rv[h];
            if constexpr (PC) reinterpret_cast<Pack4<T> *>(pc.z)[qq[h]] = zv;
        }
    }
    const double s = block_sum_f64(acc, red);
    if (threadIdx.x == 0) partial[vb] = s;
    if constexpr (PC) {
        const double s2 = block_sum_f64(acc2, red);
        if (threadIdx.x == 0) pc.partial2[vb] = s2;
    }
}

// alpha_i = rho_{i-1} / <p, w, c> on the step the operator left; false: the
// update does not run (stopped before, or CG broke down).
__device__ __forceinline__ bool alpha_step(CgStep &h, double pw) {
    if (h.stop) return false;
    h.alpha = h.rho / pw;
    h.pw = pw;
    const bool ok = pw > 0.0 && isfinite(h.alpha);
    h.x_lag = h.rho_pending = ok ? 1 : 0;
    h.stop = ok ? 0 : 3;
    return ok;
}
// hist_alpha, hist_len: the state's, read by the caller with its other loads
__device__ __forceinline__ void store_alpha_step(CgState *st, const CgStep &h, bool was_stopped,
                                                 double *hist_alpha, int hist_len) {
    store_step(st, h);
    if (!was_stopped && hist_alpha && h.iter + 1 < hist_len) hist_alpha[h.iter + 1] = h.alpha;
}
// The alpha block (256 threads) of a three-launch iteration: the same sum in
// the same order as the update of a two-launch one.
__device__ __forceinline__ void alpha_block_body(CgState *st, const CgStep *step,
                                                 const double *part_ax, int n_ax) {
    __shared__ double red[16];
    CgStep h = *step;
    const bool stopped = h.stop != 0;
    double *const hist_alpha = st->hist_alpha;
    const int hist_len = st->hist_len;
    const double pw = sum_partials_all(part_ax, n_ax, kVecThreads, red);
    alpha_step(h, pw);
    if (threadIdx.x == 0) store_alpha_step(st, h, stopped, hist_alpha, hist_len);
}

// ---------------------------------------------------------------------------
// The update of a two-launch iteration (DirectArgs): alpha from the
// operator's partials, the edge-node groups' sums, the gather, r and the
// partials of rho, in one launch.
//
// Bound by latency: a block takes one step of 256 packs, so what counts is
// the number of dependent rounds of loads.  They are laid out by hand: (1)
// the tables (edge lists; the packs' gather sources, or positions), the
// operator's partials, r and w; (2) the edge copies and the gathered values
// (table-free: the element records first, one round more); alpha is summed
// while (2) flies.  FP32 CG, N = 7, 210 elements: four launches 15.3 us an
// iteration, two 12.3.
// ---------------------------------------------------------------------------

// Edge slots of the elements a block step of 256 packs touches: at most
// 1024 at every order (N = 1: 128 elements of 8 slots).
constexpr int kMaxStepSlots = 1024;
// Slots a thread of 256 loads ahead: 1 where a step's elements have at most
// 256 (N = 5, 7, 9, 10, 11), else 2 (the rest of N = 1 and 2 is looped over).
__host__ __device__ constexpr int direct_tasks(int N) {
    return N == 5 || N == 7 || N >= 9 ? 1 : 2;
}

// The positions (in the operator's edge array) of one slot's copies, and
// their values: a missing copy reads position 0, one line for the whole wave
// (and is not added).
// Every load is unconditional: under a condition the compiler waits for it
// where the paths join.
template <typename T>
struct SlotCopies {
    int4 lo, hi;
    T v[8];
    __device__ __forceinline__ void load_list(const DirectArgs<T> &d, int64_t g, int64_t corner) {
        lo = d.elist[g];
        hi = d.elist_hi[corner < 0 ? 0 : corner];
        if (corner < 0) hi = make_int4(-1, -1, -1, -1);
    }
    __device__ __forceinline__ void load_values(const DirectArgs<T> &d) {
        v[0] = d.wedge[lo.x < 0 ? 0 : lo.x];
        v[1] = d.wedge[lo.y < 0 ? 0 : lo.y];
        v[2] = d.wedge[lo.z < 0 ? 0 : lo.z];
        v[3] = d.wedge[lo.w < 0 ? 0 : lo.w];
        v[4] = d.wedge[hi.x < 0 ? 0 : hi.x];
        v[5] = d.wedge[hi.y < 0 ? 0 : hi.y];
        v[6] = d.wedge[hi.z < 0 ? 0 : hi.z];
        v[7] = d.wedge[hi.w < 0 ? 0 : hi.w];
    }
    // the group's sum in ascending local index
    __device__ __forceinline__ T sum(const DirectArgs<T> &d) const {
        T s = v[0];
        s = lo.y >= 0 ? s + v[1] : s;
        s = lo.z >= 0 ? s + v[2] : s;
        s = lo.w >= 0 ? s + v[3] : s;
        s = hi.x >= 0 ? s + v[4] : s;
        s = hi.y >= 0 ? s + v[5] : s;
        s = hi.z >= 0 ? s + v[6] : s;
        s = hi.w >= 0 ? s + v[7] : s;
        if (d.egen && lo.x == -2) {            // more copies than the lists hold
            const int32_t *ix = d.egen + lo.y;
            s = d.wedge[ix[0]];
            for (int t = 1; t < lo.z; ++t) s += d.wedge[ix[t]];
        }
        return s;
    }
};
__host__ __device__ __forceinline__ int corner_of_slot_fast(int P, int s) {
    const int c = (s >= P) + (s >= 2 * P) + (s >= 3 * P);
    return s < 4 * P && s - c * P < 2 ? 2 * c + (s - c * P) : -1;
}

__device__ __forceinline__ void load_fence() { __asm__ volatile("" ::: "memory"); }

// Virtual block vb of vgrid.  STRUCT: the table-free gather (sm), else the
// per-point table (mcode, gm).  TASKS: edge slots a thread loads ahead
// (direct_tasks of the order).  st: the state this update completes, written
// by block 0; dir.st_in: the state the operator left.
template <typename T, bool PC, bool STRUCT, int TASKS>
__device__ __forceinline__ void update_direct_body(int64_t n, T *__restrict__ r,
                                                   const T *__restrict__ w,
                                                   const uint8_t *__restrict__ mcode,
                                                   const GatherMap &gm, const StructMap &sm,
                                                   CgState *st, double *partial, int64_t vb,
                                                   int64_t vgrid, const PcArgs<T> &pc,
                                                   const DirectArgs<T> &dir) {
    __shared__ double cw[kVecThreads];
    __shared__ double red[16], red_pw[4];   // two: no barrier lies between their uses
    __shared__ T es[kMaxStepSlots];
    const int P = dir.N + 1, MS = edge_slots(dir.N);
    const int64_t n4 = n >> 2;
    const int64_t stride = vgrid * dir.packs;
    const int t0 = (int)threadIdx.x;
    const int64_t qb = xcd_block(vb, vgrid) * dir.packs;        // the block's first pack
    double acc = 0.0, acc2 = 0.0;
    T a = T(0);
    CgStep h = *dir.st_in;
    const bool stopped = h.stop != 0;
    double *const hist_alpha = st->hist_alpha;
    const int hist_len = st->hist_len;
    // the weights' table (read after the first barrier)
    {
        const int m = t0 & kMultMask;
        cw[t0] = m ? 1.0 / (double)m : 0.0;
    }
    // a block's threads step together; packs past the end repeat the last
    // one, store nothing and add nothing
    bool first = true;
    for (int64_t q0 = qb; first || q0 < n4; q0 += stride) {
        const int64_t qend = q0 + dir.packs < n4 ? q0 + dir.packs : n4;
        const bool live = q0 + t0 < qend;
        const int64_t q = live ? q0 + t0 : (q0 < n4 ? qend : n4) - 1;
        // ---- round 1 -------------------------------------------------------
        const int64_t l0 = 4 * (q0 < n4 ? q0 : n4 - 1);
        const int64_t lend = l0 + 4 * dir.packs < n ? l0 + 4 * dir.packs : n;
        const int64_t e0 = (int64_t)(((uint64_t)l0 * dir.p3_magic) >> dir.p3_shift);
        const int nel = (int)((int64_t)(((uint64_t)(lend - 1) * dir.p3_magic) >> dir.p3_shift) -
                              e0) + 1;
        const int nslots = nel * MS;
        const int64_t g0 = e0 * MS;
        auto slot_corner = [&](int k) -> int64_t {
            const int el = (int)(((uint32_t)k * dir.ms_magic) >> 20);
            const int c = corner_of_slot_fast(P, k - el * MS);
            return c < 0 ? -1 : 8 * (e0 + el) + c;
        };
        SlotCopies<T> sc[TASKS];
#pragma unroll
        for (int u = 0; u < TASKS; ++u) {
            // threads without a slot load the last one's
            const int k = t0 + u * kVecThreads < nslots ? t0 + u * kVecThreads : nslots - 1;
            sc[u].load_list(dir, g0 + k, slot_corner(k));
        }
        int64_t e = 0;
        uint4 pe = make_uint4(0, 0, 0, 0);
        int4 g4 = make_int4(0, 0, 0, 0);
        Code4 mv{};
        if constexpr (STRUCT) {
            e = struct_elem(sm, 4 * q);
            pe = reinterpret_cast<const uint4 *>(sm.pos_tab)[(4 * q - e * sm.p3) >> 2];
        } else {
            g4 = reinterpret_cast<const int4 *>(gm.gsrc)[q];
            mv = reinterpret_cast<const Code4 *>(mcode)[q];
        }
        Pack4<T> rv = reinterpret_cast<const Pack4<T> *>(r)[q];
        const Pack4<T> wv = reinterpret_cast<const Pack4<T> *>(w)[q];
        Pack4<T> mi{}, zv{};
        if constexpr (PC) mi = reinterpret_cast<const Pack4<T> *>(pc.minv)[q];
        load_fence();
        // past convergence block 0 passes the state on (behind the loads of
        // round 1: asked alone, a live block would wait for the state first)
        if (stopped) {                                         // uniform
            if (vb == 0 && t0 == 0) store_step(st, h);
            return;
        }
        // ---- round 2 -------------------------------------------------------
#pragma unroll
        for (int u = 0; u < TASKS; ++u) sc[u].load_values(dir);
        uint32_t pv[4];
        ElemRec rc[4];
        int32_t lk[4];
        uint8_t cd[4];
        bool ed[4];
        T src[4];
        if constexpr (STRUCT) {
            pv[0] = pe.x, pv[1] = pe.y, pv[2] = pe.z, pv[3] = pe.w;
#pragma unroll
            for (int t = 0; t < 4; ++t) rc[t] = struct_record(sm, e, pv[t]);
        } else {
            lk[0] = g4.x, lk[1] = g4.y, lk[2] = g4.z, lk[3] = g4.w;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                cd[t] = mv.v[t];
                ed[t] = is_group_code(cd[t]);
                src[t] = w[ed[t] ? (int32_t)(4 * q + t) : lk[t]];
            }
        }
        load_fence();
        if (first) {
            // <p, w, c>: the sum of sum_partials_all, its loads behind (2)'s
            constexpr int kBatch = 8;
            double v = 0.0;
            for (int k0 = 0; k0 < dir.n_ax; k0 += kBatch * kVecThreads) {
                double x[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int k = k0 + u * kVecThreads + t0;
                    x[u] = dir.part_ax[k < dir.n_ax ? k : dir.n_ax - 1];
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u)
                    v += k0 + u * kVecThreads + t0 < dir.n_ax ? x[u] : 0.0;
            }
            v = wave_sum_f64(v);
            if ((t0 & 63) == 0) red_pw[t0 >> 6] = v;
        }
        // ---- the gathered values of the table-free form, the group sums ------
        if constexpr (STRUCT) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const StructSrc ss = struct_source(sm, n, 4 * q + t, pv[t], rc[t]);
                cd[t] = ss.code;
                ed[t] = ss.edge;
                src[t] = w[ss.edge ? (int32_t)(4 * q + t) : ss.idx];
            }
        }
#pragma unroll
        for (int u = 0; u < TASKS; ++u) {
            const T v = sc[u].sum(dir);
            if (t0 + u * kVecThreads < nslots) es[t0 + u * kVecThreads] = v;
        }
        for (int k = t0 + TASKS * kVecThreads; k < nslots; k += kVecThreads) {
            SlotCopies<T> c;
            c.load_list(dir, g0 + k, slot_corner(k));
            c.load_values(dir);
            es[k] = c.sum(dir);
        }
        lds_barrier();
        if (first) {
            first = false;
            // alpha_i = rho_{i-1} / <p, w, c>; block 0 writes the state
            double pw = 0.0;
            for (int u = 0; u < kVecThreads / 64; ++u) pw += red_pw[u];
            const bool ok = alpha_step(h, pw);
            a = (T)h.alpha;
            if (vb == 0 && t0 == 0) store_alpha_step(st, h, stopped, hist_alpha, hist_len);
            if (!ok) return;                                  // uniform
        }
        // ---- r, and its weighted square --------------------------------------
        const T *ese = es;
        if constexpr (STRUCT) ese = es + (int)(e * MS - g0) - 6;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            // every lane reads LDS: other lanes at the first slot
            T wg;
            if constexpr (STRUCT) {
                const T ev = *(ed[t] ? ese + (pv[t] >> 12) : es);
                wg = struct_sum<T>(wv.v[t], cd[t], ed[t], ed[t] ? ev : src[t]);
            } else {
                const T ev = es[ed[t] ? (int)(lk[t] - g0) : 0];
                wg = copies_sum<T>(wv.v[t], cd[t], ed[t] ? ev : src[t]);
            }
            rv.v[t] -= a * wg;
            const double rd = (double)rv.v[t];
            if constexpr (PC) {
                zv.v[t] = mi.v[t] * rv.v[t];
                acc += live ? rd * (double)zv.v[t] * cw[cd[t]] : 0.0;
                acc2 += live ? rd * rd * cw[cd[t]] : 0.0;
            } else {
                acc += live ? rd * rd * cw[cd[t]] : 0.0;
            }
        }
        if (live) {
            reinterpret_cast<Pack4<T> *>(r)[q] = rv;
            if constexpr (PC) reinterpret_cast<Pack4<T> *>(pc.z)[q] = zv;
        }
        if (q0 + stride < n4) lds_barrier();                   // the next step rewrites es
    }
    // the last n mod 4 points (even orders)
    if constexpr (!STRUCT) {
        for (int64_t l = 4 * n4 + qb + t0; l < n; l += stride) {
            const uint8_t c = mcode[l];
            const int32_t lk = gm.gsrc[l];
            T src;
            if (is_group_code(c)) {
                const int cn = corner_of_slot(dir.N, lk % MS);
                SlotCopies<T> sl;
                sl.load_list(dir, lk, cn < 0 ? -1 : 8 * (int64_t)(lk / MS) + cn);
                sl.load_values(dir);
                src = sl.sum(dir);
            } else {
                src = w[lk];
            }
            const T rn = r[l] - a * copies_sum<T>(w[l], c, src);
            r[l] = rn;
            if constexpr (PC) {
                const T zn = pc.minv[l] * rn;
                pc.z[l] = zn;
                acc += (double)rn * (double)zn * cw[c];
                acc2 += (double)rn * (double)rn * cw[c];
            } else {
                acc += (double)rn * (double)rn * cw[c];
            }
        }
    }
    const double s = block_sum_f64(acc, red);
    if (t0 == 0) partial[vb] = s;
    if constexpr (PC) {
        const double s2 = block_sum_f64(acc2, red);
        if (t0 == 0) pc.partial2[vb] = s2;
    }
}

// Closes a run of two-launch iterations: one block applies the rho step the
// next operator launch would (same sums in the same order).
__device__ __forceinline__ void close_rho_body(CgState *st, const double *partial,
                                               const double *partial2, int cnt, int nthr) {
    __shared__ double red[16];
    if (st->stop || !st->rho_pending) return;    // uniform
    const double rho = sum_partials_all(partial, cnt, nthr, red);
    const double rr = partial2 ? sum_partials_all(partial2, cnt, nthr, red) : rho;
    if (threadIdx.x == 0) {
        CgStep h = load_step(st);
        rho_step(h, rho, rr, st->thresh, st->max_iter, st->fixed);
        if (st->hist_rho && h.iter < st->hist_len) st->hist_rho[h.iter] = rr;
        store_step(st, h);
    }
}

// rho_i = sum of the update partials; beta_i = rho_i / rho_{i-1}; the
// iteration count, the history and the stopping test (Algorithm 1, last
// two steps).  One block.
// partial2 (may be null): the partials of <r, r, c> when rho is the
// preconditioned <r, z, c>; the stopping test and the history use <r, r, c>.
__device__ __forceinline__ void finalize_rho_body(CgState *st, const double *partial, int cnt,
                                                  const double *partial2 = nullptr) {
    // the state is read with the partials (one round of loads instead of
    // three); a stopped state sums them and stores nothing
    const int stopped = st->stop;
    const double rho_prev = st->rho;
    const int it = st->iter + 1;
    const int fixed = st->fixed, max_iter = st->max_iter, hist_len = st->hist_len;
    const double thresh = st->thresh;
    double *const hist_rho = st->hist_rho;
    __shared__ double red[16];
    const double rho = sum_partials(partial, cnt, red);
    const double rr = partial2 ? sum_partials(partial2, cnt, red) : rho;
    if (stopped) return;
    if (threadIdx.x == 0) {
        const double beta = rho / rho_prev;
        st->beta = beta;
        st->rho = rho;
        st->rr = rr;
        st->x_lag = 1;
        st->iter = it;
        if (hist_rho && it < hist_len) hist_rho[it] = rr;
        if (!isfinite(rho) || !isfinite(rr)) st->stop = 3;
        else if (!fixed && rr <= thresh) st->stop = 1;
        else if (it >= max_iter) st->stop = 2;
    }
}

// alpha_i = rho_{i-1} / <p, w, c>, the inner product being the sum of the
// operator kernel's partials (see the CgFused mode of the local operator).
// One block.
__device__ __forceinline__ void finalize_alpha_body(CgState *st, const double *part_ax,
                                                    int64_t n_ax) {
    if (st->stop) return;
    __shared__ double red[16];
    const double pw = sum_partials(part_ax, n_ax, red);
    if (threadIdx.x == 0) {
        const double alpha = st->rho / pw;
        st->pw = pw;
        st->alpha = alpha;
        st->x_lag = 0;     // the operator launch before this one applied it
        if (!(pw > 0.0) || !isfinite(alpha)) st->stop = 3;
        const int i = st->iter + 1;
        if (st->hist_alpha && i < st->hist_len) st->hist_alpha[i] = alpha;
    }
}

}  // namespace vecb
}  // namespace sem
