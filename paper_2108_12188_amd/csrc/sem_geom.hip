// sem_geom.hip -- FP64 setup of the geometric factors, mass and coordinates.
//
// Elements are trilinear images of the reference cube (Sec. 5.1: "linearly
// deformed").  At GLL point (xi_i, xi_j, xi_k) the columns of the Jacobian
// are x_xi, x_eta, x_gamma; with the cofactor rows r0 = x_eta x x_gamma,
// r1 = x_gamma x x_xi, r2 = x_xi x x_eta and |J| = x_xi . r0, the inverse
// Jacobian rows are r_a / |J|, so the symmetric factors of Eq. 4 are
//   G_ab = w_q |J| (J^-1 J^-T)_ab = (w_q / |J|) r_a . r_b,
// stored as (G11, G12, G13, G22, G23, G33), and the diagonal mass is
// B_q = w_q |J|.
#include <type_traits>

#include "sem_geom_body.h"
#include "sem_internal.h"

namespace sem {
namespace {

struct GeomArgs {
    int64_t E;
    int P;
    const double *vert;
    const double *xi;
    const double *w;
    double *G64;
    float *G32;
    double *B64;
    unsigned long long *bad;   // smallest element index with |J| <= 0
};

__device__ __forceinline__ void corner(const double *v, int c, double out[3]) {
    out[0] = v[3 * c];
    out[1] = v[3 * c + 1];
    out[2] = v[3 * c + 2];
}

// Jacobian columns of the trilinear map at reference point (x, y, z).
__device__ void jac_columns(const double *v, double x, double y, double z, double Jx[3],
                            double Jy[3], double Jz[3]) {
    const double fx[2] = {0.5 * (1 - x), 0.5 * (1 + x)};
    const double fy[2] = {0.5 * (1 - y), 0.5 * (1 + y)};
    const double fz[2] = {0.5 * (1 - z), 0.5 * (1 + z)};
    const double dx[2] = {-0.5, 0.5};
    for (int d = 0; d < 3; ++d) {
        Jx[d] = Jy[d] = Jz[d] = 0.0;
    }
    for (int c = 0; c < 2; ++c)
        for (int b = 0; b < 2; ++b)
            for (int a = 0; a < 2; ++a) {
                double p[3];
                corner(v, a + 2 * b + 4 * c, p);
                const double sx = dx[a] * fy[b] * fz[c];
                const double sy = fx[a] * dx[b] * fz[c];
                const double sz = fx[a] * fy[b] * dx[c];
                for (int d = 0; d < 3; ++d) {
                    Jx[d] += sx * p[d];
                    Jy[d] += sy * p[d];
                    Jz[d] += sz * p[d];
                }
            }
}

__device__ __forceinline__ void cross3(const double a[3], const double b[3], double o[3]) {
    o[0] = a[1] * b[2] - a[2] * b[1];
    o[1] = a[2] * b[0] - a[0] * b[2];
    o[2] = a[0] * b[1] - a[1] * b[0];
}
__device__ __forceinline__ double dotv(const double a[3], const double b[3]) {
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// The six factors (G11, G12, G13, G22, G23, G33) at GLL point (i, j, k)
// of the element with vertices v; returns |J| (weights w, points xi).
__device__ double gfactors(const double *v, const double *xi, const double *w, int i, int j,
                           int k, double G[6], double *wq_out = nullptr) {
    double Jx[3], Jy[3], Jz[3];
    jac_columns(v, xi[i], xi[j], xi[k], Jx, Jy, Jz);
    double r0[3], r1[3], r2[3];
    cross3(Jy, Jz, r0);
    cross3(Jz, Jx, r1);
    cross3(Jx, Jy, r2);
    const double det = dotv(Jx, r0);
    const double wq = w[i] * w[j] * w[k];
    const double s = wq / det;
    G[0] = s * dotv(r0, r0);
    G[1] = s * dotv(r0, r1);
    G[2] = s * dotv(r0, r2);
    G[3] = s * dotv(r1, r1);
    G[4] = s * dotv(r1, r2);
    G[5] = s * dotv(r2, r2);
    if (wq_out) *wq_out = wq;
    return det;
}

__global__ void geometry_kernel(GeomArgs g) {
    const int P = g.P, P2 = P * P, P3 = P2 * P;
    const int64_t n = g.E * P3;
    const int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= n) return;
    const int64_t e = l / P3;
    const int q = (int)(l - e * P3);
    const int i = q % P, j = (q / P) % P, k = q / P2;
    double G[6], wq = 0.0;
    const double det = gfactors(g.vert + 24 * e, g.xi, g.w, i, j, k, G, &wq);
    if (!(det > 0.0)) atomicMin(g.bad, (unsigned long long)e);
    const int64_t gb = e * 6 * P3 + q;
    if (g.G64)
        for (int c = 0; c < 6; ++c) g.G64[gb + (int64_t)c * P3] = G[c];
    if (g.G32)
        for (int c = 0; c < 6; ++c) g.G32[gb + (int64_t)c * P3] = (float)G[c];
    g.B64[l] = wq * det;
}

// Pencils along k: thread (slot, i, j) of a block holds the P points of its
// line in element blockIdx.x * epb + slot, so the waves store whole rows and
// the point's indices come from one division by a constant per line.
template <int P>
struct Pencils {
    static constexpr int kP2 = P * P, kP3 = kP2 * P;
    static constexpr int kEpb = kP2 >= 256 ? 1 : 256 / kP2;
    static constexpr int kThreads = ((kEpb * kP2 + 63) / 64) * 64;
    static unsigned blocks(int64_t E) { return (unsigned)((E + kEpb - 1) / kEpb); }
};

// Diagonal of the element operator A_L = sum_{a,b} D_a^T G_ab D_b (Eq. 4)
// at local point q = (i, j, k): the unit vector e_q has derivative
// D[l][i] along the i-line through q (likewise j, k), so the diagonal
// blocks contribute sum_l D[l][i]^2 G11(l, j, k) (and the j-, k-lines),
// and the mixed blocks, whose lines meet only at q, 2 D[i][i] D[j][j] G12(q)
// and so on.  The factors come from the vertices (FP64), so the result
// does not depend on which G form the mesh stores.
//
// Bound by FP64 arithmetic: a point's factors (one divide) cost more than its
// 3 P line terms, so each point's are formed once, from the column polynomials
// that the operator uses; G11 and G22 go through LDS, where the lines along i
// and j read them (rows padded to an odd stride), G33 stays in the line's own
// thread.  N = 7, 2.1 M points: 220 us with the factors formed anew for each
// line term, 19 once per point from the eight vertices, 15.7 so.
template <int P>
__global__ void __launch_bounds__(Pencils<P>::kThreads)
diag_local_kernel(int64_t E, const double *__restrict__ vert, const double *__restrict__ xi,
                  const double *__restrict__ w, const double *__restrict__ D,
                  double *__restrict__ diag) {
    using L = Pencils<P>;
    constexpr int kRowS = P | 1, kSlice = P * kRowS;
    __shared__ double g11[L::kEpb][P][kSlice], g22[L::kEpb][P][kSlice];
    const int slot = threadIdx.x / L::kP2, ij = threadIdx.x - slot * L::kP2;
    const int j = ij / P, i = ij - j * P;
    const int64_t e = (int64_t)blockIdx.x * L::kEpb + slot;
    const bool act = slot < L::kEpb && e < E;
    double g33[P], s[P];
    if (act) {
        const double di = D[i * P + i], dj = D[j * P + j];
        const ColumnGeom<double> cg =
            column_geom<double>(vert + 24 * e, xi[i], xi[j], w[i] * w[j]);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const double z = xi[k];
            const Vec3<double> r0 = axpy3(z, cg.R01, cg.R00), r1 = axpy3(z, cg.R11, cg.R10);
            const Vec3<double> r2 = axpy3(z, axpy3(z, cg.R22, cg.R21), cg.R20);
            const double f = cg.wij * w[k] / (cg.d0 + z * (cg.d1 + z * cg.d2));
            g11[slot][k][j * kRowS + i] = f * dot3(r0, r0);
            g22[slot][k][j * kRowS + i] = f * dot3(r1, r1);
            g33[k] = f * dot3(r2, r2);
            const double dk = D[k * P + k];
            s[k] = 2.0 * di * dj * (f * dot3(r0, r1)) + 2.0 * di * dk * (f * dot3(r0, r2)) +
                   2.0 * dj * dk * (f * dot3(r1, r2));
        }
    }
    __syncthreads();
    if (!act) return;
    double d2i[P], d2j[P];
#pragma unroll
    for (int t = 0; t < P; ++t) {
        d2i[t] = D[t * P + i] * D[t * P + i];
        d2j[t] = D[t * P + j] * D[t * P + j];
    }
    double *out = diag + e * L::kP3 + ij;
#pragma unroll
    for (int k = 0; k < P; ++k) {
        double v = 0.0;
#pragma unroll
        for (int t = 0; t < P; ++t) {
            v += d2i[t] * g11[slot][k][j * kRowS + t];
            v += d2j[t] * g22[slot][k][t * kRowS + i];
            v += D[t * P + k] * D[t * P + k] * g33[t];
        }
        out[k * L::kP2] = v + s[k];
    }
}

// Bound by its stores (24 bytes a point); a line's thread reads the element's
// vertices once.  N = 7, 2.1 M points: 10.2 us, 4.9 TB/s; 21 us with a thread
// per point, each reading the vertices and dividing by P.
template <int P>
__global__ void __launch_bounds__(Pencils<P>::kThreads)
coords_kernel(int64_t E, const double *__restrict__ vert, const double *__restrict__ xi,
              double *__restrict__ xyz) {
    using L = Pencils<P>;
    const int slot = threadIdx.x / L::kP2, ij = threadIdx.x - slot * L::kP2;
    const int j = ij / P, i = ij - j * P;
    const int64_t e = (int64_t)blockIdx.x * L::kEpb + slot;
    if (slot >= L::kEpb || e >= E) return;
    const double x = xi[i], y = xi[j];
    const double fx[2] = {0.5 * (1 - x), 0.5 * (1 + x)};
    const double fy[2] = {0.5 * (1 - y), 0.5 * (1 + y)};
    double v[24];
#pragma unroll
    for (int c = 0; c < 24; ++c) v[c] = vert[24 * e + c];
    double *out = xyz + e * L::kP3 + ij;
    const int64_t n = E * L::kP3;
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const double z = xi[k];
        const double fz[2] = {0.5 * (1 - z), 0.5 * (1 + z)};
        double s[3] = {0, 0, 0};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const double f = fx[c & 1] * fy[(c >> 1) & 1] * fz[c >> 2];
            for (int d = 0; d < 3; ++d) s[d] += f * v[3 * c + d];
        }
        for (int d = 0; d < 3; ++d) out[(int64_t)d * n + k * L::kP2] = s[d];
    }
}

// launch(std::integral_constant<int, P>) for the mesh's order
template <typename F>
void with_points(int P, const F &launch) {
    switch (P) {
        case 2: launch(std::integral_constant<int, 2>()); break;
        case 3: launch(std::integral_constant<int, 3>()); break;
        case 4: launch(std::integral_constant<int, 4>()); break;
        case 5: launch(std::integral_constant<int, 5>()); break;
        case 6: launch(std::integral_constant<int, 6>()); break;
        case 7: launch(std::integral_constant<int, 7>()); break;
        case 8: launch(std::integral_constant<int, 8>()); break;
        case 9: launch(std::integral_constant<int, 9>()); break;
        case 10: launch(std::integral_constant<int, 10>()); break;
        case 11: launch(std::integral_constant<int, 11>()); break;
        case 12: launch(std::integral_constant<int, 12>()); break;
        default: fail(SEM_EUNSUPPORTED, "order not built");
    }
}
static_assert(kMaxP == 12, "with_points lists every order");

}  // namespace

int64_t launch_geometry(Mesh &m, hipStream_t s) {
    unsigned long long *bad = nullptr;
    SEM_HIP(hipMalloc(&bad, sizeof(unsigned long long)));
    SEM_HIP(hipMemsetAsync(bad, 0xFF, sizeof(unsigned long long), s));
    GeomArgs g{m.E, m.P, m.vert64, m.b64.xi, m.b64.w, m.G64, m.G32, m.B64, bad};
    const int64_t nb = (m.n + 255) / 256;
    hipLaunchKernelGGL(geometry_kernel, dim3((unsigned)nb), dim3(256), 0, s, g);
    hipError_t le = hipGetLastError();
    unsigned long long res = 0;
    hipError_t ce = hipMemcpyAsync(&res, bad, sizeof res, hipMemcpyDeviceToHost, s);
    hipError_t se = hipStreamSynchronize(s);
    (void)hipFree(bad);
    check_hip(le, "geometry kernel launch");
    check_hip(ce, "geometry result copy");
    check_hip(se, "geometry kernel");
    return res == ~0ull ? -1 : (int64_t)res;
}

void launch_diag_local(const Mesh &m, double *d, hipStream_t s) {
    with_points(m.P, [&](auto p) {
        constexpr int P = decltype(p)::value;
        hipLaunchKernelGGL((diag_local_kernel<P>), dim3(Pencils<P>::blocks(m.E)),
                           dim3(Pencils<P>::kThreads), 0, s, m.E, m.vert64, m.b64.xi, m.b64.w,
                           m.b64.D, d);
    });
    check_hip(hipGetLastError(), "diagonal kernel launch");
}

void launch_coords(const Mesh &m, double *xyz, hipStream_t s) {
    with_points(m.P, [&](auto p) {
        constexpr int P = decltype(p)::value;
        hipLaunchKernelGGL((coords_kernel<P>), dim3(Pencils<P>::blocks(m.E)),
                           dim3(Pencils<P>::kThreads), 0, s, m.E, m.vert64, m.b64.xi, xyz);
    });
    check_hip(hipGetLastError(), "coords kernel launch");
}

}  // namespace sem
