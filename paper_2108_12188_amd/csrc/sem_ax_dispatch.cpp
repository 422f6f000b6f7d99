// sem_ax_dispatch.cpp -- order dispatch and launch shapes of the local operator.
#include "sem_internal.h"

#include <atomic>
#include <cstdlib>

namespace sem {

#define SEM_DECL_ORDER(N)                                                                       \
    void ax_order_##N##_f32(bool, AxMode, const AxArgs<float> &, const double *, const double *, \
                            int64_t, hipStream_t);                                              \
    void ax_order_##N##_f64(bool, AxMode, const AxArgs<double> &, const double *,               \
                            const double *, int64_t, hipStream_t);
SEM_DECL_ORDER(1)
SEM_DECL_ORDER(2)
SEM_DECL_ORDER(3)
SEM_DECL_ORDER(4)
SEM_DECL_ORDER(5)
SEM_DECL_ORDER(6)
SEM_DECL_ORDER(7)
SEM_DECL_ORDER(8)
SEM_DECL_ORDER(9)
SEM_DECL_ORDER(10)
SEM_DECL_ORDER(11)
#undef SEM_DECL_ORDER

#define SEM_DECL_BATCH(N)                                                                      \
    void ax_batch_order_##N##_f32(bool, bool, bool, bool, const AxArgs<float> *, const int2 *, \
                                  int64_t, int, const double *, const double *, hipStream_t);
SEM_DECL_BATCH(1)
SEM_DECL_BATCH(2)
SEM_DECL_BATCH(3)
SEM_DECL_BATCH(4)
SEM_DECL_BATCH(5)
SEM_DECL_BATCH(6)
SEM_DECL_BATCH(7)
SEM_DECL_BATCH(8)
SEM_DECL_BATCH(9)
SEM_DECL_BATCH(10)
SEM_DECL_BATCH(11)
#undef SEM_DECL_BATCH

using FnB = void (*)(bool, bool, bool, bool, const AxArgs<float> *, const int2 *, int64_t, int,
                     const double *, const double *, hipStream_t);
static const FnB kFnB[kMaxOrder + 1] = {
    nullptr,           ax_batch_order_1_f32, ax_batch_order_2_f32, ax_batch_order_3_f32,
    ax_batch_order_4_f32, ax_batch_order_5_f32, ax_batch_order_6_f32, ax_batch_order_7_f32,
    ax_batch_order_8_f32, ax_batch_order_9_f32, ax_batch_order_10_f32, ax_batch_order_11_f32};

using Fn32 = void (*)(bool, AxMode, const AxArgs<float> &, const double *, const double *,
                      int64_t, hipStream_t);
using Fn64 = void (*)(bool, AxMode, const AxArgs<double> &, const double *, const double *,
                      int64_t, hipStream_t);

// The CG-fused operator writes one FP64 partial per block; its grid is
// capped so that the partial sum stays short (tiles are then strided).
#ifndef SEM_AX_FUSED_MAX_BLOCKS
#define SEM_AX_FUSED_MAX_BLOCKS 2048
#endif
constexpr int64_t kAxFusedMaxBlocks = SEM_AX_FUSED_MAX_BLOCKS;
// FP64 blocks are smaller (one element at N = 7, 9, 10 and 11): at 12 M points
// twice the blocks run the FP64 iteration 0-7% faster (N = 9 on the fly 233 ->
// 217 us, N = 11 stored 349 -> 323 us); FP32 gains nothing steady from it.
constexpr int64_t kAxFusedMaxBlocks64 = 2 * kAxFusedMaxBlocks;
// the matrix-core form: blocks of one wave (N = 7; measured best of 8192,
// 16384 and 32768) and of two waves (N = 9: 1536, the blocks resident at
// once at 3 waves per SIMD and 6 blocks per CU, ahead of 3072 and 4096 at
// 10^3 ... 28^3 elements: every block walks its share of the elements
// without a partial last round)
#ifndef SEM_AX_MFMA_MAX_BLOCKS
#define SEM_AX_MFMA_MAX_BLOCKS 16384
#endif
#ifndef SEM_AX_MFMA2_MAX_BLOCKS
#define SEM_AX_MFMA2_MAX_BLOCKS 1536
#endif
constexpr int64_t kAxMfmaMaxBlocks = SEM_AX_MFMA_MAX_BLOCKS;
constexpr int64_t kAxMfma2MaxBlocks = SEM_AX_MFMA2_MAX_BLOCKS;

// the plain (stand-alone) operator: one tile per block unless capped
#ifndef SEM_AX_PLAIN_MAX_BLOCKS
#define SEM_AX_PLAIN_MAX_BLOCKS 0
#endif
constexpr int64_t kAxPlainMaxBlocks = SEM_AX_PLAIN_MAX_BLOCKS;

static int64_t ax_grid(int64_t ntiles, AxMode mode, bool fp64, bool mfma, int threads = 64) {
    const int64_t cap = mfma ? (threads == 64 ? kAxMfmaMaxBlocks : kAxMfma2MaxBlocks)
                             : (fp64 ? kAxFusedMaxBlocks64 : kAxFusedMaxBlocks);
    if (mode == AxMode::CgFused && ntiles > cap) return cap;
    if (mode != AxMode::CgFused && kAxPlainMaxBlocks > 0 && ntiles > kAxPlainMaxBlocks)
        return kAxPlainMaxBlocks;
    return ntiles;
}

static const Fn32 kFn32[kMaxOrder + 1] = {nullptr,        ax_order_1_f32, ax_order_2_f32,
                                          ax_order_3_f32, ax_order_4_f32, ax_order_5_f32,
                                          ax_order_6_f32, ax_order_7_f32, ax_order_8_f32,
                                          ax_order_9_f32, ax_order_10_f32, ax_order_11_f32};
static const Fn64 kFn64[kMaxOrder + 1] = {nullptr,        ax_order_1_f64, ax_order_2_f64,
                                          ax_order_3_f64, ax_order_4_f64, ax_order_5_f64,
                                          ax_order_6_f64, ax_order_7_f64, ax_order_8_f64,
                                          ax_order_9_f64, ax_order_10_f64, ax_order_11_f64};

// Default elements per block, at most 512 threads and 64 KiB of values in LDS: a
// multiple of 64 lanes filled as tightly as possible with (i, j) columns,
// except where one element per block measured faster because its barriers
// hold back fewer waves (3 M points, plain operator on the fly: FP64 N = 9
// 39.6 us with three elements, 29.6 with one; FP32 N = 11 32.2 us with two,
// 21.3 with one; FP64 N = 7, whose elements are one wave each, 24.1 / 22.9).
// FP32 N = 1 on the fly takes 32, two waves (us per iteration with 64 and 32:
// 1.6 M points 37.1, 34.9, 3.4 M 59.2, 58.5, 8 M 129.2, 123.2; stored factors 52.5,
// 51.4, 96.6, 96.8, 208.9, 211.1).
// The autotuner (sem_ax_shape_set) overrides them per order, precision
// and geometric-factor form.
static const int kEpb32[kMaxOrder + 1] = {0, 64, 28, 16, 5, 7, 5, 4, 3, 1, 1, 1};
static const int kEpb64[kMaxOrder + 1] = {0, 64, 28, 16, 5, 7, 5, 1, 3, 1, 1, 1};

// The plain operator where another number than the CG-fused one's measured
// faster (us at 1.6, 3.4 and 8 M points): N = 2 on the fly, FP64 28 elements 14.1,
// 25.5, 53.4, 7 (one wave) 12.8, 22.7, 47.2, FP32 8.8, 14.7, 29.7 and 9.0, 14.7, 29.6;
// FP64 with stored factors, N = 3 16 elements 15.3, 31.6, 94.5, 20 15.2, 30.7, 91.2;
// N = 6 5 elements 19.8, 36.0, 95.9, 1 19.7, 34.1, 94.3 (the fused one keeps 5: 8 M
// points 219 us an iteration, with 1 229).
static int plain_epb(int N, bool fp64, bool otf) {
    if (otf) return N == 2 ? 7 : 0;
    return !fp64 ? 0 : N == 3 ? 20 : N == 6 ? 1 : 0;
}

// Process-wide tile shapes set by the autotuner (0: built-in default),
// indexed [on-the-fly][fp64][N], and a generation counter that tells cached
// graphs and batch tables that a shape changed.
static std::atomic<int> g_epb[2][2][kMaxOrder + 1];
static std::atomic<int> g_engine[2][2][kMaxOrder + 1];
static std::atomic<int> g_shape_gen{0};

int ax_shape_generation() { return g_shape_gen.load(); }

static std::atomic<int64_t> g_cache_bytes{kInfinityCacheBytes};

bool cg_streams_vectors(int64_t footprint) { return footprint > g_cache_bytes.load(); }

void cache_bytes_set(int64_t bytes) {
    g_cache_bytes.store(bytes > 0 ? bytes : kInfinityCacheBytes);
    g_shape_gen.fetch_add(1);
}

void ax_shape_set(int N, bool fp64, bool otf, int epb) {
    g_epb[otf ? 1 : 0][fp64 ? 1 : 0][N].store(epb > 0 ? epb : 0);
    g_shape_gen.fetch_add(1);
}

bool ax_mfma_available(int N, bool fp64) { return (N == 7 || N == 9) && !fp64; }

void ax_engine_set(int N, bool fp64, bool otf, int engine) {
    g_engine[otf ? 1 : 0][fp64 ? 1 : 0][N].store(engine);
    g_shape_gen.fetch_add(1);
}

AxShape ax_shape(int N, bool fp64, bool otf, int epb_override) {
    const int P = N + 1, P2 = P * P, P3 = P2 * P;
    const size_t tsz = fp64 ? 8 : 4;
    const int engine = g_engine[otf ? 1 : 0][fp64 ? 1 : 0][N].load();
    // built-in choice: the matrix cores wherever they measured faster than
    // the best VALU tile.  us per CG iteration at 0.9 to 1 / 3 (N = 9: 2.7) / 8 M
    // points, matrix cores and VALU with one and two elements per block: N = 7
    // on the fly 19.9 38.1 71.5, 23.0 40.7 83.5, 22.1 36.7 73.3; stored factors
    // 21.0 44.7 95.2, 23.2 48.5 99.5, 23.5 44.3 96.0; N = 9 on the fly 24.6 41.0
    // 79.1, 24.9 44.4 92.1, 24.9 45.6 86.7; stored 28.8 52.0 120.4, 28.8 51.4
    // 107.2, 29.0 54.1 110.0: there the VALU with one element
    const bool mfma = engine == kAxEngineMfma ||
                      (engine == kAxEngineDefault && !(N == 9 && !otf));
    if (mfma && ax_mfma_available(N, fp64)) {
        // one element per block (one wave at N = 7, two at N = 9): the
        // operator tiles (two unpadded at N = 7, three of slices of 106
        // floats at N = 9) and the staging of r, p, x and the vertices
        AxShape s;
        s.epb = 1;
        s.threads = N == 9 ? 128 : 64;
        s.lds = N == 9 ? 4 * (3 * (size_t)P * 106 + 3 * (size_t)P3 + 32)
                       : 4 * (5 * (size_t)P3);
        s.mfma = true;
        return s;
    }
    int epb = epb_override > 0 ? epb_override : g_epb[otf ? 1 : 0][fp64 ? 1 : 0][N].load();
    if (epb <= 0) epb = fp64 ? kEpb64[N] : N == 1 && otf ? 32 : kEpb32[N];
    // clamp to the kernel limits: 512 threads and 64 KiB of element values in
    // LDS (two tiles; FP32 CG-fused tiles of odd N also stage the next tile's
    // r, p and vertices).  The padding of the tiles comes on top: at most 72 KiB
    // in all (FP64 N = 7, eight elements), of 160 per CU, so that it takes no
    // shape away (N = 9 with four elements) and two blocks still share a CU.
    const bool staged = !fp64 && P3 % 4 == 0;
    auto lds = [&](int q, int tile) {
        return 2 * tsz * (size_t)q * tile + (staged ? 8 * (size_t)q * P3 + 96 * (size_t)q : 0);
    };
    while (epb > 1 && (((epb * P2 + 63) / 64) * 64 > 512 || lds(epb, P3) > 65536)) --epb;
    AxShape s;
    s.epb = epb;
    s.threads = ((epb * P2 + 63) / 64) * 64;
    s.lds = lds(epb, ax_tile_stride(P));
    s.mfma = false;
    return s;
}

// The shape of a launch: the caller's, else the autotuner's, else the default.
static AxShape launch_shape(int N, bool fp64, bool otf, AxMode mode, int epb) {
    if (mode != AxMode::CgFused && epb <= 0 && g_epb[otf ? 1 : 0][fp64 ? 1 : 0][N].load() <= 0)
        epb = plain_epb(N, fp64, otf);
    return ax_shape(N, fp64, otf, epb);
}

template <>
void launch_ax<float>(const Mesh &m, bool otf, AxMode mode, AxArgs<float> a, hipStream_t s) {
    const AxShape sh = launch_shape(m.N, false, otf, mode, a.epb);
    a.epb = sh.epb;
    a.mfma = sh.mfma ? 1 : 0;
    a.E = m.E;
    a.D = m.b32.D;
    a.Dt = m.b32.Dt;
    a.xi = m.b32.xi;
    a.wq = m.b32.w;
    a.vert = m.vert32;
    a.edge = m.edge32;
    if (!otf) a.G = m.G32;
    const int64_t ntiles = (m.E + sh.epb - 1) / sh.epb;
    kFn32[m.N](otf, mode, a, m.h_xi.data(), m.h_w.data(),
               ax_grid(ntiles, mode, false, sh.mfma, sh.threads), s);
    check_hip(hipGetLastError(), "ax kernel launch (fp32)");
}

template <>
void launch_ax<double>(const Mesh &m, bool otf, AxMode mode, AxArgs<double> a, hipStream_t s) {
    const AxShape sh = launch_shape(m.N, true, otf, mode, a.epb);
    a.epb = sh.epb;
    a.mfma = 0;
    a.E = m.E;
    a.D = m.b64.D;
    a.Dt = m.b64.Dt;
    a.xi = m.b64.xi;
    a.wq = m.b64.w;
    a.vert = m.vert64;
    a.edge = nullptr;
    if (!otf) a.G = m.G64;
    const int64_t ntiles = (m.E + sh.epb - 1) / sh.epb;
    kFn64[m.N](otf, mode, a, m.h_xi.data(), m.h_w.data(),
               ax_grid(ntiles, mode, true, false), s);
    check_hip(hipGetLastError(), "ax kernel launch (fp64)");
}

void ax_batch_desc(const Mesh &m, bool otf, AxArgs<float> &a) {
    const AxShape sh = ax_shape(m.N, false, otf, 0);
    a.epb = sh.epb;
    a.mfma = sh.mfma ? 1 : 0;
    a.E = m.E;
    a.D = m.b32.D;
    a.Dt = m.b32.Dt;
    a.xi = m.b32.xi;
    a.wq = m.b32.w;
    a.vert = m.vert32;
    a.edge = m.edge32;
    a.G = otf ? nullptr : m.G32;
    a.vgrid = ax_grid((m.E + sh.epb - 1) / sh.epb, AxMode::CgFused, false, sh.mfma, sh.threads);
}

void launch_ax_batch(int N, bool otf, bool mfma, bool stream, bool rho, const AxArgs<float> *descs,
                     const int2 *blk, int64_t nblk, int epb, const double *xi, const double *w,
                     hipStream_t s) {
    if (nblk <= 0) return;
    kFnB[N](otf, mfma, stream, rho, descs, blk, nblk, epb, xi, w, s);
    check_hip(hipGetLastError(), "batched ax kernel launch");
}

int ax_threads(int N, bool fp64, bool otf) { return ax_shape(N, fp64, otf, 0).threads; }

int64_t cg_footprint(const Mesh &m, int tsz, bool table_free) {
    const int64_t es = edge_slots(m.N);
    int64_t b = 4 * tsz * m.n;                                          // r, p, x, w
    if (table_free) b += m.E * (6 + es) * 8 + tsz * m.n_egroups;       // records, edge sums
    else if (m.gs_in_update) b += 4 * m.n + tsz * m.n_groups_multi;    // table, group sums
    if (m.gsum_wedge || table_free) b += m.E * es * tsz;                // edge copy
    if (m.direct) b += m.E * (es + 8) * 16;                             // edge lists
    // vertices (the matrix-core operator at N = 7 reads the element edge
    // vectors instead), point codes
    b += (m.edge32 && tsz == 4 ? m.E * 36 * 4 : m.E * 24 * tsz) + m.n;
    return b;
}

int64_t ax_blocks(const Mesh &m, bool fp64, bool otf, int epb_override) {
    const AxShape sh = ax_shape(m.N, fp64, otf, epb_override);
    return ax_grid((m.E + sh.epb - 1) / sh.epb, AxMode::CgFused, fp64, sh.mfma, sh.threads);
}

}  // namespace sem
