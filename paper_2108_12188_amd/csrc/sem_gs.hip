// sem_gs.hip -- gather-scatter QQ^T and the Dirichlet mask.
//
// Gather-scatter (Sec. 3.1, Sec. 4.3): every global point held by m > 1
// local copies forms a group; the copies' values are summed in ascending
// local index and the sum is written back to every copy.  Groups are stored
// by size class (all groups of one class have the same m), so a block only
// ever sees one m: no divergence across lanes, and the index list needs no
// offsets array.  Inside a class, groups are in ascending order of their
// first local index, which keeps neighbouring lanes on neighbouring faces.
#include "sem_gs_body.h"
#include "sem_internal.h"
#include "sem_vec_body.h"

namespace sem {
namespace {

using namespace gsb;

// Physical block b runs logical block lb: the blocks that land on one XCD
// (b mod 8) take one contiguous range of the group list, i.e. one region
// of the mesh, so the neighbouring copies they touch share that XCD's L2.
__device__ __forceinline__ int64_t logical_block(int64_t b, int64_t nb_phys) {
    const int64_t per = nb_phys / kXcds;
    return (b % kXcds) * per + b / kXcds;
}

// Logical blocks lb0 .. lb0 + nb_logical - 1.  st (may be null): a stopped
// CG state makes the whole grid exit at once.  With part_ax, the grid has
// one more block, which forms alpha from the operator's partials (Algorithm
// 1; it needs none of this kernel's results).
template <typename T>
__global__ void __launch_bounds__(kGsThreads)
gs_kernel(const GsClasses cls, int64_t lb0, int64_t nb_logical, const int32_t *__restrict__ idx,
          T *__restrict__ w, CgState *st, const double *part_ax, int64_t n_ax) {
    if (st && st->stop) return;
    int64_t nb = gridDim.x;
    if (part_ax) {
        if (blockIdx.x == gridDim.x - 1) {
            vecb::finalize_alpha_body(st, part_ax, n_ax);
            return;
        }
        --nb;
    }
    const int64_t b = logical_block(blockIdx.x, nb);
    if (b < nb_logical) gs_logical_block(cls, lb0 + b, idx, InPlace<T>{w});
}

// Group sums of the classes with M >= mmin: logical blocks lb0 .. lb0 +
// nb_logical - 1 of the class list's block numbering; the last block forms
// alpha from the operator's partials (three-launch iterations: step -> st).
template <typename T>
__global__ void __launch_bounds__(kGsThreads)
group_sums_kernel(const GsClasses cls, int64_t lb0, int64_t nb_logical,
                  const int32_t *__restrict__ idx, int64_t io0, const T *__restrict__ src,
                  T *__restrict__ out, CgState *st, const CgStep *step, const double *part_ax,
                  int64_t n_ax, int mmin) {
    if (blockIdx.x == gridDim.x - 1) {
        if (step) vecb::alpha_block_body(st, step, part_ax, (int)n_ax);
        else vecb::finalize_alpha_body(st, part_ax, n_ax);
        return;
    }
    // three-launch iterations: st is being written by the alpha block
    if (step ? step->stop : st->stop) return;
    const int64_t b = logical_block(blockIdx.x, gridDim.x - 1);
    if (b < nb_logical) gs_sums_logical_block<T>(cls, lb0 + b, idx, io0, src, out, mmin);
}

constexpr int kPointsPerThread = 4;
constexpr int64_t kPointsPerBlock = (int64_t)kGsThreads * kPointsPerThread;

// w <- mask(QQ^T w): the first nb_gs blocks take the groups and write zeros
// to the masked ones, the others zero the Dirichlet points of one copy.
// Bound by memory (the strided faces touch almost every line of w).  Calls of
// the gather-scatter with the mask as a pass of its own, in one launch, and
// without a mask: FP64 N = 7 2.1 M points 15.0, 11.7, 11.8 us, 16.8 M 71.0,
// 67.0, 66.7; FP32 12.5, 9.7, 9.8 and 43.1, 40.1, 39.9.  With the masked groups
// last in their class (no bits) the plain pass lost 2 to 7% to its locality;
// with the flag read from a group's first point, or the loads of masked groups
// left out, the launch took longer than the two passes at 6 to 17 M points.
template <typename T>
__global__ void __launch_bounds__(kGsThreads)
gs_mask_kernel(const GsClasses cls, int64_t nb_gs, int64_t nb_logical,
               const int32_t *__restrict__ idx, const InPlaceMasked<T> a,
               const int32_t *__restrict__ dir1, int64_t n_dir1) {
    if (blockIdx.x < nb_gs) {
        const int64_t b = logical_block(blockIdx.x, nb_gs);
        if (b < nb_logical) gs_logical_block(cls, b, idx, a);
        return;
    }
    const int64_t t0 = (blockIdx.x - nb_gs) * kPointsPerBlock + threadIdx.x;
#pragma unroll
    for (int u = 0; u < kPointsPerThread; ++u) {
        const int64_t t = t0 + (int64_t)u * kGsThreads;
        if (t < n_dir1) a.w[dir1[t]] = T(0);
    }
}

// b = mask(QQ^T (B f)) in one launch: the first nb_gs blocks take the shared
// points by groups, the others the points of one copy in order; every point
// is written once and f is only read, so no block waits for another.
template <typename T>
__global__ void __launch_bounds__(kGsThreads)
rhs_kernel(const GsClasses cls, int64_t nb_gs, int64_t nb_logical,
           const int32_t *__restrict__ idx, const MassSource<T> a,
           const uint8_t *__restrict__ mcode, int64_t n) {
    if (blockIdx.x < nb_gs) {
        const int64_t b = logical_block(blockIdx.x, nb_gs);
        if (b < nb_logical) gs_logical_block(cls, b, idx, a);
        return;
    }
    const int64_t l0 = (blockIdx.x - nb_gs) * kPointsPerBlock + threadIdx.x;
    uint8_t code[kPointsPerThread];
    double v[kPointsPerThread];
#pragma unroll
    for (int u = 0; u < kPointsPerThread; ++u) {
        const int64_t l = l0 + (int64_t)u * kGsThreads;
        code[u] = l < n ? mcode[l] : 0;
        v[u] = l < n ? a.B[l] * a.f[l] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kPointsPerThread; ++u) {
        if ((code[u] & kMultMask) != 1) continue;
        a.b[l0 + (int64_t)u * kGsThreads] = (code[u] & kDirichletBit) ? T(0) : (T)v[u];
    }
}

template <typename T>
__global__ void mask_kernel(const int32_t *__restrict__ dir, int64_t n_dir, T *__restrict__ w) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n_dir) w[dir[t]] = T(0);
}

}  // namespace

int64_t gs_logical_blocks(const Mesh &m) { return gs_total_blocks(m.gs); }

namespace {
// physical grid: a logical block count rounded up to a multiple of the XCD count
int gs_phys_blocks(int64_t b) { return (int)(b > 0 ? ((b + kXcds - 1) / kXcds) * kXcds : 1); }
}  // namespace

int gs_cg_blocks(const Mesh &m) { return gs_phys_blocks(gs_logical_blocks(m)); }

template <typename T>
void launch_gs(const Mesh &m, T *w, hipStream_t s) {
    if (m.n_groups == 0) return;
    const int nb = gs_cg_blocks(m);
    hipLaunchKernelGGL((gs_kernel<T>), dim3(nb), dim3(kGsThreads), 0, s, m.gs, (int64_t)0,
                       gs_logical_blocks(m), m.gs_idx, w, (CgState *)nullptr,
                       (const double *)nullptr, (int64_t)0);
    check_hip(hipGetLastError(), "gs kernel launch");
}

template <typename T>
void launch_mask(const Mesh &m, T *w, hipStream_t s) {
    if (m.n_dir == 0) return;
    const int64_t nb = (m.n_dir + 255) / 256;
    hipLaunchKernelGGL((mask_kernel<T>), dim3((unsigned)nb), dim3(256), 0, s, m.dir_idx, m.n_dir, w);
    check_hip(hipGetLastError(), "mask kernel launch");
}

template <typename T>
void launch_gs_mask(const Mesh &m, T *w, hipStream_t s) {
    const int64_t nlb = gs_logical_blocks(m);
    const int64_t nb = m.n_groups ? gs_phys_blocks(nlb) : 0;
    const int64_t total = nb + (m.n_dir1 + kPointsPerBlock - 1) / kPointsPerBlock;
    if (total == 0) return;
    hipLaunchKernelGGL((gs_mask_kernel<T>), dim3((unsigned)total), dim3(kGsThreads), 0, s, m.gs,
                       nb, nlb, m.gs_idx, (InPlaceMasked<T>{{w}, m.gs_zero}), m.dir_idx, m.n_dir1);
    check_hip(hipGetLastError(), "gs kernel launch");
}

template <typename T>
void launch_rhs(const Mesh &m, const double *f, T *b, hipStream_t s) {
    const int64_t nlb = gs_logical_blocks(m);
    const int64_t nb = m.n_groups ? gs_phys_blocks(nlb) : 0;
    const int64_t total = nb + (m.n + kPointsPerBlock - 1) / kPointsPerBlock;
    hipLaunchKernelGGL((rhs_kernel<T>), dim3((unsigned)total), dim3(kGsThreads), 0, s, m.gs, nb,
                       nlb, m.gs_idx, (MassSource<T>{m.B64, f, b, m.gs_zero}), m.mcode, m.n);
    check_hip(hipGetLastError(), "rhs kernel launch");
}

template <typename T>
void launch_gs_cg(const Mesh &m, T *w, CgState *st, const double *ax_partial, int n_ax_partial,
                  hipStream_t s) {
    const int64_t nlb = gs_logical_blocks(m);
    if (nlb > 0) {
        hipLaunchKernelGGL((gs_kernel<T>), dim3(gs_phys_blocks(nlb) + 1), dim3(kGsThreads), 0, s,
                           m.gs, (int64_t)0, nlb, m.gs_idx, w, st, ax_partial,
                           (int64_t)n_ax_partial);
        check_hip(hipGetLastError(), "gs/cg kernel launch");
    } else {
        launch_finalize_alpha(st, ax_partial, n_ax_partial, s);
    }
}

template <typename T>
void launch_group_sums_cg(const Mesh &m, const T *w, const T *wedge, T *gsum, CgState *st,
                          const CgStep *step, const double *ax_partial, int n_ax_partial, hipStream_t s) {
    const int64_t nlb = gs_logical_blocks(m) - m.gs_blk_multi;
    if (nlb > 0) {
        const bool compact = m.gsum_wedge;
        hipLaunchKernelGGL((group_sums_kernel<T>), dim3(gs_phys_blocks(nlb) + 1),
                           dim3(kGsThreads), 0, s, m.gs, m.gs_blk_multi, nlb,
                           compact ? m.wedge_idx : m.gs_idx, compact ? m.wedge_io0 : (int64_t)0,
                           compact ? wedge : w, gsum, st, step, ax_partial, (int64_t)n_ax_partial, 3);
        check_hip(hipGetLastError(), "group sums kernel launch");
    } else if (step) {
        hipLaunchKernelGGL((group_sums_kernel<T>), dim3(1), dim3(kGsThreads), 0, s, m.gs,
                           (int64_t)0, (int64_t)0, (const int32_t *)nullptr, (int64_t)0,
                           (const T *)nullptr, gsum, st, step, ax_partial,
                           (int64_t)n_ax_partial, 0);
        check_hip(hipGetLastError(), "alpha kernel launch");
    } else {
        launch_finalize_alpha(st, ax_partial, n_ax_partial, s);
    }
}

template <typename T>
void launch_edge_sums_cg(const Mesh &m, const T *wedge, T *gsum, CgState *st,
                         const CgStep *step, const double *ax_partial, int n_ax_partial, hipStream_t s) {
    const int64_t nlb = gs_total_blocks(m.ecls);
    if (nlb > 0) {
        hipLaunchKernelGGL((group_sums_kernel<T>), dim3(gs_phys_blocks(nlb) + 1),
                           dim3(kGsThreads), 0, s, m.ecls, (int64_t)0, nlb, m.ewedge_idx,
                           (int64_t)0, wedge, gsum, st, step, ax_partial, (int64_t)n_ax_partial, 2);
        check_hip(hipGetLastError(), "edge sums kernel launch");
    } else if (step) {
        hipLaunchKernelGGL((group_sums_kernel<T>), dim3(1), dim3(kGsThreads), 0, s, m.gs,
                           (int64_t)0, (int64_t)0, (const int32_t *)nullptr, (int64_t)0,
                           (const T *)nullptr, gsum, st, step, ax_partial,
                           (int64_t)n_ax_partial, 0);
        check_hip(hipGetLastError(), "alpha kernel launch");
    } else {
        launch_finalize_alpha(st, ax_partial, n_ax_partial, s);
    }
}

template void launch_gs<float>(const Mesh &, float *, hipStream_t);
template void launch_gs<double>(const Mesh &, double *, hipStream_t);
template void launch_gs_mask<float>(const Mesh &, float *, hipStream_t);
template void launch_gs_mask<double>(const Mesh &, double *, hipStream_t);
template void launch_rhs<float>(const Mesh &, const double *, float *, hipStream_t);
template void launch_rhs<double>(const Mesh &, const double *, double *, hipStream_t);
template void launch_mask<float>(const Mesh &, float *, hipStream_t);
template void launch_mask<double>(const Mesh &, double *, hipStream_t);
template void launch_gs_cg<float>(const Mesh &, float *, CgState *, const double *, int,
                                  hipStream_t);
template void launch_gs_cg<double>(const Mesh &, double *, CgState *, const double *, int,
                                   hipStream_t);
template void launch_edge_sums_cg<float>(const Mesh &, const float *, float *, CgState *,
                                         const CgStep *,
                                         const double *, int, hipStream_t);
template void launch_edge_sums_cg<double>(const Mesh &, const double *, double *, CgState *,
                                         const CgStep *,
                                          const double *, int, hipStream_t);
template void launch_group_sums_cg<float>(const Mesh &, const float *, const float *, float *,
                                          CgState *, const CgStep *, const double *, int,
                                          hipStream_t);
template void launch_group_sums_cg<double>(const Mesh &, const double *, const double *,
                                           double *, CgState *, const CgStep *,
                                           const double *, int, hipStream_t);

}  // namespace sem
