// sem_internal.h -- shared host/device definitions of the SEM library.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/sem.h"

namespace sem {

constexpr int kMaxOrder = 11;
// Per-point code: multiplicity m (copies of the global point) in the low 7
// bits, the Dirichlet flag in bit 7.  The inner-product weight is 1/m.
constexpr int kMaxMultiplicity = 127;
constexpr uint8_t kDirichletBit = 0x80;
constexpr uint8_t kMultMask = 0x7F;
constexpr int kMaxP = kMaxOrder + 1;
// Schedules of a CG iteration on a conforming mesh (see DirectArgs): up to
// direct_max_points(N) local points two launches, up to kInlineMaxPoints (FP64:
// half of it; FP32 without matrix cores: three quarters) three, beyond it four.
// On the fly, us per iteration with four launches and with the schedule taken
// here: FP32 N = 7 0.11 M points 15.3 / 12.3, 0.88 M 21.8 / 18.9 (two), 2.2 M
// 33.6 / 32.9, 3.0 M 38.6 / 37.3, 3.9 M 44.9 / 43.8 (three); N = 9 1.1 M 30.1 /
// 28.4, 2.2 M 40.8 / 35.9, 3.8 M 52.4 / 46.2; FP64 N = 9 0.5 M 29.8 / 26.4, N = 8
// 2 M 54.9 / 51.5, N = 9 2.0 M 57.0 / 57.5 (4.1 M 91.8 / 94.6).
// VALU orders win less as the mesh grows, the partials being formed once per
// tile: N = 5 1.1 M 27.6 / 26.6, 2.0 M 35.0 / 34.7, 2.7 M 42.4 / 42.9, 3.5 M 47.4 /
// 48.2, 3.9 M 50.1 / 50.7, stored factors 2.2 M 43.5 / 41.9, 3.5 M 59.3 / 60.0;
// N = 6 3.2 M 47.4 / 48.4; N = 8 3.0 M 45.6 / 44.9, 3.6 M 50.2 / 50.9.
// FP32 N = 7 keeps four launches between 2^20 and 2^21 points, where steps of
// its update that divide evenly leave 600 to 950 blocks, too few to hide
// their loads (1.2 M 25.1 / 27.1, 1.5 M 26.4 / 27.8, 1.84 M 29.2 / 29.8, 1.97 M 30.1 /
// 30.1, 2.1 M with 1024 blocks 30.0 / 29.2).  The rule knows the order, not the
// engine, which can be set after the mesh is made.  N = 3 in FP32 and N = 1 in
// FP64, whose steps hold many small tiles, keep four beyond 2^20 points (N = 3
// 1.3 M 29.6 / 30.3, 2.8 M 46.4 / 49.1; N = 1 2.0 M 57.0 / 59.1).
// With a preconditioner every block sums twice the partials: three launches
// stop paying at 2^21 points at N = 5 (2.0 M 42.7 / 42.5, 2.9 M 53.3 / 55.5) and do
// not begin to at N = 7 (2.1 M 35.9 / 35.8, 2.5 M 41.7 / 42.5, 3.7 M 52.5 / 53.9); at
// the other orders they pay as far as without (N = 9 3.6 M 57.8 / 52.7).
// Two launches form a group's sum once per copy, in every block that touches
// it, so the limit falls where most of an element is edge and corner nodes
// (all of it at N = 1, half at N = 3).  FP32 on the fly, us per iteration with
// two / three launches: N = 1 0.15 M points 15.4 / 15.5, 0.29 M 19.1 / 17.0, 0.89 M
// 33.1 / 26.5 (four 27.4); N = 2 0.15 M 15.3 / 15.4, 0.29 M 18.4 / 17.2, 0.89 M 28.6 /
// 27.4; N = 3 0.39 M 17.4 / 17.9, 0.54 M 22.2 / 21.3, 1.0 M 27.8 / 26.2 (four 27.3);
// N = 4 1.0 M 24.6 / 25.9; N = 5 1.0 M 25.7 / 26.3, 1.3 M 28.5 / 28.5, 1.9 M 35.8 / 33.5;
// N = 7 0.96 M 20.0 / 23.2, 1.2 M 25.3 / 24.8 (four), 1.97 M 33.6 / 30.3; N = 8
// 0.97 M 24.0 / 26.1, 1.26 M 28.6 / 29.8, 1.48 M 30.2 / 28.9; N = 9 1.0 M 24.2 / 25.8,
// 1.2 M 27.4 / 28.8, 1.6 M 32.5 / 31.8.  FP64: N = 1 0.15 M 17.1 / 16.7, 0.89 M 41.5 /
// 33.6 (four 36.1), N = 3 0.39 M 20.7 / 22.4, 0.54 M 26.0 / 25.3, N = 5 0.89 M 31.8 /
// 33.0, 1.0 M 35.3 / 34.1, N = 9 1.0 M 33.2 / 34.6, 1.6 M 52.6 / 52.0.
constexpr int64_t kDirectMaxPoints = int64_t(1) << 20;
constexpr int64_t direct_max_points(int N) {
    return N < 4 ? int64_t(1) << (16 + N) : kDirectMaxPoints;
}
constexpr int64_t kInlineMaxPoints = int64_t(1) << 22;
constexpr bool mfma_order(int N) { return N == 7 || N == 9; }
inline bool takes_inline_scalars(int N, int64_t n, bool fp64, bool pc) {
    if (n <= kDirectMaxPoints) return true;
    if (N == (fp64 ? 1 : 3)) return false;
    if (fp64) return n <= kInlineMaxPoints / 2;
    if (pc && (N == 5 || N == 7)) return N == 5 && n <= kInlineMaxPoints / 2;
    if (!mfma_order(N)) return n <= kInlineMaxPoints / 4 * 3;
    return n <= kInlineMaxPoints && (N != 7 || n >= kInlineMaxPoints / 2);
}
// Most blocks of the update there, in equal steps: every operator block sums
// their partials (N = 8 1.6 M: 781 blocks 29.7, 1562 31.0; the Jacobi iterations
// of N = 8 1.6 M: 50 in 1733 us, with a cap of 1600 blocks 1837).  A block of
// the matrix-core operator reads 1024 of them in one round of loads, and more
// in a second one that waits for the first: FP32 N = 7 2.2 M points 1088 blocks
// 35.1 us, 726 32.9; 3.5 M 1143 blocks 43.7, 857 41.5; N = 9 3.6 M 1172 46.3,
// 879 45.7.
constexpr int kInlineVecBlocks = 1280;
constexpr int kInlineVecBlocksMfma = 1024;
constexpr int inline_update_blocks(int vec_blocks, int N, bool fp64) {
    const int cap = mfma_order(N) && !fp64 ? kInlineVecBlocksMfma : kInlineVecBlocks;
    const int steps = (vec_blocks + cap - 1) / cap;
    return (vec_blocks + steps - 1) / steps;
}
// local points from which a mesh takes the table-free gather by default
// (below it, where a CG iteration is mostly launch latency, the table form
// measured up to 8% faster; from it on the table-free form is as fast or
// faster, alone and in batches)
constexpr int64_t kTableFreeMinPoints = int64_t(1) << 19;

// Edge and corner nodes of an element's P^3 block (on two or three of its
// faces): 12 N - 4 of them, numbered column by column (i, j on the border
// of the face square): every border column starts at its base with its
// k = 0 node, then k = N; the 4 corner columns (bases 0, P, 2P, 3P) follow
// with k = 1 .. N-1, the other border columns (bases 4P + 2s) have no more.
// -1 for other nodes.
__host__ __device__ inline int edge_slots(int N) { return 12 * N - 4; }
__host__ __device__ inline int edge_column_base(int N, int i, int j) {
    const int P = N + 1;
    const bool bi = i == 0 || i == N, bj = j == 0 || j == N;
    if (bi && bj) return ((i == N) + 2 * (j == N)) * P;
    if (!(bi || bj)) return -1;
    int s;
    if (j == 0) s = i - 1;
    else if (j == N) s = (P - 2) + i - 1;
    else if (i == 0) s = 2 * (P - 2) + j - 1;
    else s = 3 * (P - 2) + j - 1;
    return 4 * P + 2 * s;
}
__host__ __device__ inline int edge_slot(int N, int i, int j, int k) {
    const int cb = edge_column_base(N, i, j);
    if (cb < 0) return -1;
    if (k == 0 || k == N) return cb + (k == N);
    const bool corner = (i == 0 || i == N) && (j == 0 || j == N);
    return corner ? cb + 1 + k : -1;
}
// Number (0..7) of the element corner at an edge slot, -1 for other slots.
__host__ __device__ inline int corner_of_slot(int N, int s) {
    const int P = N + 1, c = s / P, k = s - c * P;
    return (c < 4 && k < 2) ? 2 * c + k : -1;
}

// Distance of two elements' tiles in the local operator's LDS, in values
// (see the tile layout in sem_ax_order.hip).
constexpr int ax_tile_stride(int P) {
    return P == 2 ? 12 : P == 4 ? 80 : P == 6 ? 228 : P == 8 ? 576 : P == 10 ? 1060
         : P == 12 ? 1740 : P * P * P;
}

// ---------------------------------------------------------------------------
// Errors
// ---------------------------------------------------------------------------
void set_error(const std::string &msg);
[[noreturn]] void fail(sem_status code, const std::string &msg);
void check_hip(hipError_t e, const char *what);

#define SEM_HIP(call) ::sem::check_hip((call), #call)

// ---------------------------------------------------------------------------
// Device-resident CG scalars of one solve (Algorithm 1: rho, alpha, beta).
// Written only by the one-block finalize kernels; read by every block of
// the kernels that follow in stream order.
// ---------------------------------------------------------------------------
struct CgState {
    // what changes from iteration to iteration
    double rho;        // rho_{i-1}: <r, r, c> of the current residual (<r, z, c>
                       // with a preconditioner)
    double rr;         // <r, r, c> of the current residual
    double alpha;      // alpha_i
    double beta;       // beta_{i-1} used by the next p-update
    double pw;         // <p, w, c> of the current iteration
    int iter;          // completed iterations
    int stop;          // 0 running, 1 converged, 2 cap reached, 3 breakdown
    int x_lag;         // 1: x still lacks alpha_i p_i of the last completed
                       // update (single-mesh solves apply it in the next
                       // operator launch, or in the closing flush)
    int rho_pending;   // 1: the partials of the last update hold the next rho,
                       // not summed yet (two-launch iterations, see DirectArgs)
    // fixed during a solve
    double rho0;       // <r0, r0, c>
    double thresh;     // stop when rr <= thresh (= tol^2 rho_0)
    int max_iter;      // iteration cap
    int fixed;         // 1: no convergence test
    int hist_len;      // capacity of the history arrays
    int pad_;
    double *hist_rho;  // device history (may be null)
    double *hist_alpha;
};
// The part that the two copies of a two-launch iteration pass back and forth.
struct CgStep {
    double rho, rr, alpha, beta, pw;
    int iter, stop, x_lag, rho_pending;
};

// ---------------------------------------------------------------------------
// Mesh handle
// ---------------------------------------------------------------------------
template <typename T>
struct Basis {
    T *D = nullptr;    // [P][P]  D_ij = l_j'(xi_i)
    T *Dt = nullptr;   // [P][P]  transpose
    T *xi = nullptr;   // [P]
    T *w = nullptr;    // [P]
};

struct Workspace;      // CG vectors of one precision (sem_cg.cpp)

// Gather-scatter groups by size class (see sem_gs.hip).
constexpr int kMaxGsClasses = 32;
struct GsClasses {
    int ncls;
    int M[kMaxGsClasses];          // copies per group in this class
    int64_t ng[kMaxGsClasses];     // groups in this class
    int64_t zo[kMaxGsClasses];     // first word of the class in gs_zero
    int64_t io[kMaxGsClasses];     // offset of the class in gs_idx
    int64_t blk0[kMaxGsClasses];   // first block of the class in a gs launch
    // gather-scatter launches only (null: identity): DEVICE int32 [blocks],
    // the class-major logical block that position b of a launch runs; the
    // blocks sorted by the first local index of their first group, so the
    // classes of one region of the mesh run together.  A permutation of all
    // blocks: only launches that cover every block may apply it (the group
    // sums over a sub-range of classes do not).
    const int32_t *lb_order = nullptr;
};
void gs_classes_finish(GsClasses &c);
int64_t gs_total_blocks(const GsClasses &c);   // logical blocks of a whole gather-scatter

// Table-free gather inside the CG update (see Mesh::gs_struct): one record
// per face and per edge slot of an element, [E][6 + edge_slots(N)], faces
// first.  Face f = 2 d + (the face lies at coordinate N along d, its normal
// direction): the copies of its face-interior points, with face coordinates
// (a, b) (the two coordinates other than d, in i, j, k order), are
// lo + sa a + sb b, where hi = code | sa << 8 | sb << 20 with sa, sb 12-bit
// two's-complement strides (0, +-1, +-P or +-P^2; every partial sum fits
// in 32 bits); a face without a partner (or a Dirichlet face) has
// sa = sb = 0 and lo inside its own element.  Edge slot s (record 6 + s): lo = the rank of its group among the
// edge groups (0 when unshared or Dirichlet), hi = code.  code: the points'
// multiplicity | Dirichlet byte.
struct alignas(8) ElemRec {
    int32_t lo, hi;
};
// Per local position of the element (P^3 entries): bits 0-1 kind (0
// interior, 1 face interior, 2 edge or corner node), bits 2-6 and 7-11 the
// face coordinates a, b, bits 12-20 the record (face f, or 6 + edge slot).
__host__ __device__ inline uint32_t pos_entry(int kind, int a, int b, int rec) {
    return (uint32_t)kind | ((uint32_t)a << 2) | ((uint32_t)b << 7) | ((uint32_t)rec << 12);
}

struct Mesh {
    int device = 0;
    int64_t E = 0;
    int N = 0, P = 0, P3 = 0;
    int64_t n = 0;            // local points
    int64_t n_glob = 0;
    int64_t n_groups = 0, n_shared = 0, n_dir = 0, n_dir1 = 0;
    GsClasses gs{};           // shared-point groups by size class

    // host copies of the basis (FP64, this library's own construction)
    std::vector<double> h_xi, h_w, h_D;

    // device arrays
    double *vert64 = nullptr;     // [E][8][3]
    float *vert32 = nullptr;      // [E][8][3]
    float *edge32 = nullptr;      // N = 7: [E][12][3] element edge vectors from vert32
    float *G32 = nullptr;         // [E][6][P3]
    double *G64 = nullptr;        // [E][6][P3]
    double *B64 = nullptr;        // [E][P3] mass w_q |J_q|
    uint8_t *mcode = nullptr;     // [n]: multiplicity | Dirichlet bit
    int32_t *gs_idx = nullptr;    // [n_shared], class-major, groups of M ascending indices
    int32_t *gs_lb_order = nullptr;   // gs.lb_order's array
    uint32_t *gs_zero = nullptr;  // bit g & 31 of word zo + (g >> 5): group g is masked
    int32_t *dir_idx = nullptr;   // [n_dir], the n_dir1 points of one copy first
    // Shared sums inside the CG update (used when every shared point lies on
    // the surface of its element's P^3 block): gsrc[l] is the other copy of
    // a pair (m = 2), the rank of a larger group among the n_groups_multi
    // groups with m > 2 (whose sums a gather-scatter variant over blocks
    // gs_blk_multi.. writes to a compact array), else l itself.
    bool gs_in_update = false;
    int64_t n_groups_multi = 0, gs_blk_multi = 0;
    int32_t *gsrc = nullptr;       // [n]
    // When every copy of a group with m > 2 is an edge or corner node of its
    // element (edge_slot), the CG operator also writes those nodes' values
    // to a compact [E][edge_slots(N)] array and the group sums read it:
    // wedge_idx lists, for the groups with m > 2 in gs_idx's layout from
    // offset wedge_io0, the copies' positions e * edge_slots(N) + slot.
    bool gsum_wedge = false;
    int64_t wedge_io0 = 0;
    int32_t *wedge_idx = nullptr;
    // Table-free form of the same gather (odd N, conforming meshes, unless
    // SEM_MESH_GATHER_TABLE): the update derives every point's copies from
    // its position in the element (pos_tab) and the element's face and edge
    // records (ElemRec) instead of loading gsrc and mcode.  The sums of the
    // n_egroups edge and corner groups of two or more copies (ecls /
    // ewedge_idx: positions in the compact edge array) follow w in class
    // order.  Division of a local index by P^3: (l * p3_magic) >> p3_shift
    // (checked on the host for every l < n).  gs_struct: its tables are
    // present (batched and served solves use it then); gs_struct_solo: a
    // single-mesh solve uses it too (from kTableFreeMinPoints points on, or
    // when forced), else the per-point table gsrc, which is then present.
    // The two forms give bitwise identical results.
    bool gs_struct = false;
    bool gs_struct_solo = false;
    ElemRec *erec = nullptr;       // [E][6 + edge_slots(N)]
    uint32_t *pos_tab = nullptr;   // [P3]
    GsClasses ecls{};
    int64_t n_egroups = 0;
    int32_t *ewedge_idx = nullptr;
    uint32_t p3_magic = 0;
    int p3_shift = 0;
    // Two-launch CG iterations (n <= direct_max_points(N), every group of more
    // than two copies made of edge and corner nodes): the update sums those
    // groups itself from the operator's compact edge array.  elist[e * MS +
    // s] (MS = edge_slots(N)): the positions in that array of the copies of
    // the node at edge slot s of element e, ascending, -1 past the last; the
    // fifth to eighth copy of a corner node in elist_hi[8 e + corner] (see
    // corner_of_slot).  More copies than that: {-2, offset into egen, count,
    // 0}.  gsrc_direct is gsrc with e * MS + s for the points of groups of
    // more than two copies.
    // two or three launches, [preconditioned], per precision
    bool inline32[2] = {false, false}, inline64[2] = {false, false};
    bool inline_scalars(bool fp64, bool pc) const { return fp64 ? inline64[pc] : inline32[pc]; }
    bool direct = false;
    int4 *elist = nullptr;         // [E][MS]
    int4 *elist_hi = nullptr;      // [E][8], behind elist in its allocation
    int32_t *egen = nullptr;
    int32_t *gsrc_direct = nullptr;   // [n]
    // Jacobi preconditioner (built on first use): 1 / diag(A) on the free
    // points, 0 on the Dirichlet points, local form
    double *minv64 = nullptr;
    float *minv32 = nullptr;
    Basis<float> b32;
    Basis<double> b64;
    void *basis_blob = nullptr;
    double *scratch = nullptr;    // reduction partials / small scalars
    size_t scratch_len = 0;       // in doubles
    CgState *state = nullptr;     // device CG state for sem_dot / solves
    size_t device_bytes = 0;

    Workspace *ws32 = nullptr;
    Workspace *ws64 = nullptr;
};

Mesh *as_mesh(sem_mesh_t m);

// Relative tolerance of one inner FP32 solve of the mixed-precision
// refinement when the outer relative residual is rel and the target is tol:
// the reduction still needed, with a factor 10 to spare, but never tighter
// than the configured inner tolerance (nor looser than 1/2).  The last
// outer step then solves only as far as the target requires.
inline double refine_inner_tol(double inner_tol, double tol, double rel) {
    double t = rel > 0.0 ? 0.1 * tol / rel : inner_tol;
    if (t < inner_tol) t = inner_tol;
    if (t > 0.5) t = 0.5;
    return t;
}

// Host tables of a mesh's scatter map (sem_tables.cpp; no device calls).
struct HostTables {
    int64_t n_glob = 0, n_groups = 0, n_shared = 0, n_dir = 0, n_dir1 = 0;
    GsClasses gs{};
    std::vector<uint8_t> mcode;     // [n]
    std::vector<int32_t> gs_idx;    // class-major ascending member lists
    std::vector<int32_t> gs_lb_order;  // see GsClasses::lb_order
    std::vector<uint32_t> gs_zero;  // see Mesh::gs_zero
    std::vector<int32_t> dir_idx;   // Dirichlet local points
    bool gs_in_update = false;      // every shared point on its element's surface
    int64_t n_groups_multi = 0;     // groups with more than two copies
    int64_t gs_blk_multi = 0;       // their first gather-scatter block
    bool gsum_wedge = false;        // every copy of those groups an edge or corner node
    int64_t wedge_io0 = 0;          // gs_idx offset of the first such group
    std::vector<int32_t> wedge_idx; // copies' positions in the compact edge array
    std::vector<int32_t> gsrc;      // [n] (only when gs_in_update), see Mesh::gsrc
    bool gs_struct = false;         // the table-free form applies, see Mesh::gs_struct
    std::vector<ElemRec> erec;
    std::vector<uint32_t> pos_tab;
    GsClasses ecls{};
    int64_t n_egroups = 0;
    std::vector<int32_t> ewedge_idx;
    uint32_t p3_magic = 0;
    int p3_shift = 0;
    // two-launch iterations, see Mesh::direct (build_direct_tables)
    bool direct = false;
    std::vector<int4> elist, elist_hi;
    std::vector<int32_t> egen;
    std::vector<int32_t> gsrc_direct;   // gsrc with the edge slots of larger groups
};
// Fills the tables of the two-launch iteration where it applies; points: also
// the per-point table, which a mesh with the table-free gather need not have;
// keep_gsrc: t.gsrc stays valid beside it.
void build_direct_tables(int64_t E, int N, HostTables &t, bool points = true,
                         bool keep_gsrc = true);
// Validates glob_id / dirichlet (fail() on error) and fills t.
void build_tables(int64_t E, int N, const int64_t *gid, const uint8_t *dir, HostTables &t);

// ---------------------------------------------------------------------------
// Host basis construction (sem_basis.cpp)
// ---------------------------------------------------------------------------
void gll_points(int N, std::vector<double> &xi, std::vector<double> &w);
void derivative_matrix(const std::vector<double> &xi, std::vector<double> &D);

// ---------------------------------------------------------------------------
// Kernel launchers
// ---------------------------------------------------------------------------
enum class AxMode { Plain = 0, CgFused = 1 };

template <typename T>
struct AxArgs {
    int64_t E;
    int epb;                    // elements per block
    const T *u;                 // Plain: input u. CgFused: residual r
    T *p;                       // CgFused: search direction, updated in place
    T *w;                       // output
    const T *G;                 // precomputed factors [E][6][P3]
    const T *vert;              // vertices [E][8][3] (on-the-fly form)
    const T *edge;              // FP32, N = 7, may be null: edge vectors [E][12][3]
                                // (the matrix-core on-the-fly form reads these)
    const T *D;                 // [P][P]
    const T *Dt;                // [P][P]
    const T *xi;                // [P]
    const T *wq;                // [P]
    CgState *st;                // CgFused: beta, stop flag
    double *partial;            // CgFused: one FP64 partial of sum p w per block
    int64_t vgrid;              // batched launches: this problem's own grid size
    T *wedge;                   // CgFused, may be null: w of the edge and corner
                                // nodes, [E][edge_slots(N)]
    T *x;                       // CgFused, may be null: solution; when st->x_lag,
                                // x += alpha p_old (previous iteration's step)
    int mfma;                   // host side: launch the matrix-core form (FP32,
                                // N = 7; one element per wave-sized block)
    int stream;                 // CgFused FP32: p and x accesses non-temporal
                                // (cg_streams_vectors of the iteration's footprint)
    // Two- and three-launch iterations (null / 0: the state is final when this runs):
    // every block sums the last update's rho partials itself and block 0
    // writes the new state to st_out, which nothing else of this launch reads.
    CgStep *st_out;
    const double *rho_part;     // partials of <r, r, c>, or of <r, z, c>
    const double *rr_part;      // preconditioned: partials of <r, r, c>
    int n_rho;
};

// Two- and three-launch CG iterations.  The four-launch form spends a launch
// on the one-block sum of rho and a dependent launch on the group sums (and
// alpha).  With three launches the operator's blocks each sum the rho
// partials of the last update; with two the update's blocks also each sum the
// operator's partials to alpha, and the edge-node groups they need; the state passes from the solve's CgState through the operator
// to a CgStep beside it and through the update back, each launch reading one
// copy while its block 0 writes the other.
constexpr int kMaxAxThreads = 512;      // largest operator block
template <typename T>
struct DirectArgs {
    const CgStep *st_in;        // the step the operator left
    const double *part_ax;      // the operator's partials of <p, w, c>
    int n_ax;
    const T *wedge;             // the operator's compact edge array
    const int4 *elist, *elist_hi;
    const int32_t *egen;
    int N;
    int packs;                  // packs of 4 points per block step (step_packs)
    uint32_t p3_magic;          // l / P^3 = (l * p3_magic) >> p3_shift for l < 2^31
    int p3_shift;
    uint32_t ms_magic;          // k / MS = (k * ms_magic) >> 20 for k < 1024
};

// Packs of 4 points that a block of 256 threads takes per step on a mesh of
// two-launch iterations: as many whole elements as fit (216 at N = 5, 250 at
// N = 9, 256 at N = 1, 3 and 7), so that a step forms the edge sums of its own
// elements only; 256 where an element is no whole number of packs or more than
// 256.  On the fly, us per iteration with 256 and with this: N = 9 FP32 0.12 M
// points 14.2 / 13.6, 1.0 M 23.0 / 22.4, FP64 1.0 M 35.0 / 32.2; N = 5 FP32
// 0.11 M 14.1 / 13.5, 0.59 M 19.0 / 18.4.
constexpr int step_packs(int N) {
    const int p3 = (N + 1) * (N + 1) * (N + 1);
    return p3 % 4 == 0 && p3 / 4 <= 256 ? 256 / (p3 / 4) * (p3 / 4) : 256;
}

// step: the CgStep beside a workspace's state
template <typename T>
DirectArgs<T> direct_args(const Mesh &m, const CgStep *step, const T *wedge,
                          const double *part_ax, int n_ax) {
    // l * (magic P^3 - 2^shift) < 2^31 * 2^lg <= 2^shift, and the same for MS <= 128
    int lg = 0;
    while ((1 << lg) < m.P3) ++lg;
    const int shift = 31 + lg;
    return {step, part_ax, n_ax, wedge, m.elist, m.elist_hi, m.egen, m.N, step_packs(m.N),
            (uint32_t)(((uint64_t)1 << shift) / (uint64_t)m.P3 + 1), shift,
            (1u << 20) / (uint32_t)edge_slots(m.N) + 1};
}

// Jacobi preconditioning in the CG update (preconditioned CG, Sec. 3.2;
// Algorithm 1 is its unpreconditioned case): z = minv r is written, and the block partials of
// <r, z, c> (partial) and <r, r, c> (partial2) are reduced.
template <typename T>
struct PcArgs {
    const T *minv;      // null: no preconditioner
    T *z;
    double *partial2;
};

// Launch configuration chosen for an order (threads, elements per block,
// dynamic LDS bytes).
struct AxShape {
    int epb;
    int threads;
    size_t lds;
    bool mfma;                  // matrix-core form (epb 1, one wave per block)
};
AxShape ax_shape(int N, bool fp64, bool otf, int epb_override);
void ax_shape_set(int N, bool fp64, bool otf, int epb);
// Contraction engine per order, precision and G form: 0 default, 1 VALU FMA,
// 2 matrix cores (FP32, N = 7 only).
constexpr int kAxEngineDefault = 0, kAxEngineValu = 1, kAxEngineMfma = 2;
bool ax_mfma_available(int N, bool fp64);
void ax_engine_set(int N, bool fp64, bool otf, int engine);
int ax_shape_generation();
// threads of a block of the CG-fused operator
int ax_threads(int N, bool fp64, bool otf);

// Fills the basis / geometry pointers and the shape from the mesh; the
// caller sets u, p, w, mcode, st, partial (and epb to force a shape).
template <typename T>
void launch_ax(const Mesh &m, bool otf, AxMode mode, AxArgs<T> a, hipStream_t s);
int64_t ax_blocks(const Mesh &m, bool fp64, bool otf, int epb_override);
// Bytes a CG iteration of mesh m with tsz-byte vectors keeps touching: r,
// p, x, w, the gather records (table_free) or table, the operator's edge
// copy, vertices and codes.
int64_t cg_footprint(const Mesh &m, int tsz, bool table_free);

// The CG-fused operator reads and writes p and x non-temporally when the
// iteration (of one mesh, or of a whole batch) exceeds the 256 MB Infinity
// Cache, so that the cache keeps what the rest of the iteration reads again
// (in FP64 only with G on the fly: the precomputed FP64 factors, read with
// plain loads, fill the cache either way).
constexpr int64_t kInfinityCacheBytes = int64_t(256) << 20;
bool cg_streams_vectors(int64_t footprint);
// The cache size assumed by cg_streams_vectors (0: kInfinityCacheBytes);
// changing it invalidates captured graphs and batch tables like a new tile
// shape does.
void cache_bytes_set(int64_t bytes);

// Fills `a` (basis, geometry, epb, vgrid) for a batched FP32 launch of mesh m.
void ax_batch_desc(const Mesh &m, bool otf, AxArgs<float> &a);
// One FP32 CG-fused operator launch over many problems of order N:
// blk[b] = (descriptor index, virtual block).
// stream: p and x non-temporal (cg_streams_vectors of the batch's footprint)
// rho: every problem's rho is formed first (AxArgs::st_out set in all of them)
void launch_ax_batch(int N, bool otf, bool mfma, bool stream, bool rho, const AxArgs<float> *descs,
                     const int2 *blk, int64_t nblk, int epb, const double *xi, const double *w,
                     hipStream_t s);

// gather-scatter / mask / vector kernels (sem_gs.hip, sem_vec.hip)
template <typename T>
void launch_gs(const Mesh &m, T *w, hipStream_t s);
template <typename T>
void launch_mask(const Mesh &m, T *w, hipStream_t s);
// w <- mask(QQ^T w), one launch
template <typename T>
void launch_gs_mask(const Mesh &m, T *w, hipStream_t s);
// b = mask(QQ^T (B f)), one launch; b must not overlap f
template <typename T>
void launch_rhs(const Mesh &m, const double *f, T *b, hipStream_t s);
// CG step after the fused operator: gather-scatter, then alpha from the
// operator kernel's partials of <p, w, c>
template <typename T>
void launch_gs_cg(const Mesh &m, T *w, CgState *st, const double *ax_partial, int n_ax_partial,
                  hipStream_t s);
// The same for the gather in the update: gsum[k] = sum of the copies of the
// k-th group with m > 2 (ascending local index; read from wedge, the
// operator's compact copy of the edge and corner nodes, when m.gsum_wedge,
// else from w; neither is modified), and alpha.
// step (may be null): a three-launch iteration, alpha goes from step to st.
template <typename T>
void launch_group_sums_cg(const Mesh &m, const T *w, const T *wedge, T *gsum, CgState *st,
                          const CgStep *step, const double *ax_partial, int n_ax_partial,
                          hipStream_t s);
// The same for the table-free gather (needs m.gs_struct): gsum[k] = sum of
// the copies of the k-th edge or corner group of two or more copies
// (ascending local index, read from wedge, the operator's compact edge
// array), then alpha.
template <typename T>
void launch_edge_sums_cg(const Mesh &m, const T *wedge, T *gsum, CgState *st,
                         const CgStep *step, const double *ax_partial, int n_ax_partial,
                         hipStream_t s);
int gs_cg_blocks(const Mesh &m);
int64_t gs_logical_blocks(const Mesh &m);

// Algorithm 1 vector kernels (sem_vec.hip).  Reductions write one FP64
// partial per block (`partial`, at least vec_blocks(n) entries) and a
// one-block finalize kernel sums them in index order.
int vec_blocks(int64_t n);
// blocks (and partials) of the CG update of a mesh; pc: preconditioned
int update_blocks(const Mesh &m, bool fp64, bool pc);
// r -= alpha mask(w); rho = <r, r, c>; then beta, convergence, history (x is
// advanced by the next operator launch or launch_x_flush)
template <typename T>
void launch_update(const Mesh &m, T *r, const T *w, CgState *st, double *partial,
                   hipStream_t s, PcArgs<T> pc = PcArgs<T>{});
// x += alpha p when st->x_lag (the step of the last completed update)
template <typename T>
void launch_x_flush(const Mesh &m, T *x, const T *p, const CgState *st, hipStream_t s);
// The same with w read as QQ^T w, w holding the operator's masked local
// output and gsum the group sums of launch_group_sums_cg: pairs are summed
// inside the update (needs m.gs_in_update).
template <typename T>
void launch_update_gather(const Mesh &m, T *r, const T *w, const T *gsum, CgState *st,
                          double *partial, hipStream_t s, PcArgs<T> pc = PcArgs<T>{});
// The same with the table-free gather (needs m.gs_struct): wg holds w
// (n values) followed by the edge-group sums of launch_edge_sums_cg;
// bitwise the results of launch_update_gather.
template <typename T>
void launch_update_struct(const Mesh &m, T *r, const T *wg, CgState *st, double *partial,
                          hipStream_t s, PcArgs<T> pc = PcArgs<T>{});
// The same two forms leave rho to the next operator launch when
// m.inline_scalars().  In a two-launch iteration (m.direct): step -> st.
template <typename T>
void launch_update_direct(const Mesh &m, bool table_free, T *r, const T *w, const T *wedge,
                          CgState *st, const CgStep *step, const double *part_ax, int n_ax, double *partial,
                          hipStream_t s, PcArgs<T> pc = PcArgs<T>{});
// Ends a run of two-launch iterations: the pending rho, as the next operator
// launch (nthr threads a block) would form it.
void launch_close_rho(CgState *st, const double *partial, const double *partial2, int cnt,
                      int nthr, hipStream_t s);
// The state into pinned host memory by a kernel, then *host_seq = seq: the host
// learns of it without a copy command or an event in the stream, either of
// which holds the stream for about 10 us.
void launch_publish_state(const CgState *st, CgState *host, uint64_t *host_seq, uint64_t seq,
                          hipStream_t s);
// r = b - w (w may be null: r = b); p = 0; rho_0 = <r, r, c>; initial state.
// With pc.minv: z = minv r, rho = <r, z, c>, and the threshold and the
// reported residual use <r, r, c>.
template <typename T>
void launch_cg_init(const Mesh &m, const T *b, const T *w, T *r, T *p, CgState *st,
                    double *partial, hipStream_t s, PcArgs<T> pc = PcArgs<T>{});
// Jacobi: minv = 1/d on free points, 0 on Dirichlet points (both precisions)
void launch_jacobi_invert(const Mesh &m, const double *d, double *minv64, float *minv32,
                          hipStream_t s);
// d_l = (A_L)_{ll} of every local point from the geometry (FP64, unassembled)
void launch_diag_local(const Mesh &m, double *d, hipStream_t s);
// *out = <a, b, c>
template <typename T>
void launch_dot(const Mesh &m, const T *a, const T *b, double *out, double *partial,
                hipStream_t s);
// The same weighted inner product with its block partials in a file-scope
// device array of the library (no device allocation; sem_dot_noalloc).
template <typename T>
void launch_dot_noalloc(const Mesh &m, const T *a, const T *b, double *out, hipStream_t s);
// r = b - w and *out = <r, r, c>  (FP64 outer residual of the refinement)
void launch_residual64(const Mesh &m, const double *b, const double *w, double *r, double *out,
                       double *partial, hipStream_t s);
// alpha = rho / (sum of both partial sets)
void launch_finalize_alpha(CgState *st, const double *part_ax, int64_t n_ax, hipStream_t s);
// dst = (float)(src / sqrt(*nrm2))
void launch_scale_to_f32(int64_t n, const double *src, const double *nrm2, float *dst,
                         hipStream_t s);
// x += sqrt(*nrm2) * (double)d
void launch_axpy_from_f32(int64_t n, double *x, const double *nrm2, const float *d,
                          hipStream_t s);
// elementwise helpers
template <typename Ts, typename Td>
void launch_convert(int64_t n, const Ts *src, Td *dst, hipStream_t s);
void launch_mul64(int64_t n, const double *a, const double *b, double *out, hipStream_t s);

// FP64 geometry setup (sem_geom.hip)
int64_t launch_geometry(Mesh &m, hipStream_t s);
void launch_coords(const Mesh &m, double *xyz, hipStream_t s);
template <typename T>
void launch_rhs_mass(const Mesh &m, const double *f, T *b, hipStream_t s);

}  // namespace sem
