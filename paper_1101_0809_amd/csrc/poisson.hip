// poisson.hip -- electrostatic initial field (Section 4.3): the discrete
// Poisson equation of Eq. poiphi for the cell-centred potential,
//   sum_a (-Phi_{c-e_a} + 2 Phi_c - Phi_{c+e_a}) / d_a^2 = 4 pi rho_c,
// on the periodic grid, then E from Eq. egradphidis,
//   E^x at face i = (Phi_{i-1} - Phi_i) / dx  (and y, z alike),
// so that div_h E = 4 pi rho cell by cell.  The operator is symmetric and
// positive definite on grid functions of zero mean; the right side has its
// mean removed (a uniform background) and conjugate gradients run on that
// subspace.  Scalars (alpha, beta, residual norms) stay on the device: each
// iteration is two launches with no host round trip; the host reads the
// residual every kCheck iterations to stop.
//
// What bounds an iteration on the usual grids is launches, not bytes (64^3:
// ten planes of 2 MB, cache resident).  The reductions are therefore finished
// by their readers -- every workgroup sums the previous kernel's partials
// itself, in the one fixed order, instead of waiting for a one-workgroup
// kernel -- and the new search direction is formed where the stencil reads it.
// Six launches became two: 32 -> 14 us per iteration at 64^3 (the check of the
// residual included), 68 -> 42 us at 128^3.
#include <algorithm>
#include <cmath>

#include "pic_internal.h"

namespace pic {
namespace {

constexpr int kThreads = 256;
constexpr int kBlocks = 1024;  // reduction workgroups
constexpr int kCheck = 16;

// device scalars: [0], [1] r.r of even and odd iterations  [2] target r.r
// [4] b.b  [5] sum rho  [6] r.r for the host

// Sum of v over the workgroup, in a fixed order (a binary tree: across the
// waves in LDS, then inside the first wave), returned to every thread.
__device__ __forceinline__ double block_sum(double v, double* sh)
{
    const int t = threadIdx.x;
    __syncthreads();  // sh may still be read from an earlier sum
    sh[t] = v;
    __syncthreads();
    if (t < 64) {
        static_assert(kThreads == 256, "two levels across the waves");
        v = (sh[t] + sh[t + 128]) + (sh[t + 64] + sh[t + 192]);
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) v += __shfl_down(v, w, 64);
        if (t == 0) sh[0] = v;
    }
    __syncthreads();
    return sh[0];
}

// Sum of nb partials, in the same fixed order in every workgroup.
__device__ __forceinline__ double sum_partials(const double* __restrict__ part, int nb, double* sh)
{
    double v = 0.0;
    for (int b = threadIdx.x; b < nb; b += kThreads) v += part[b];
    return block_sum(v, sh);
}

// A cell (fewer than 2^32 of them) and its six periodic neighbours: the cell,
// x - 1, x + 1, y - 1, y + 1, z - 1, z + 1.
struct Star {
    uint32_t q[7];
};

__device__ __forceinline__ Star star_of(const GridK& g, uint32_t p)
{
    const uint32_t nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const uint32_t row = p / nx, i = p - row * nx, k = row / ny, j = row - k * ny;
    const uint32_t sz = nx * ny;
    Star s;
    s.q[0] = p;
    s.q[1] = i == 0 ? p + (nx - 1) : p - 1;
    s.q[2] = i == nx - 1 ? p - (nx - 1) : p + 1;
    s.q[3] = j == 0 ? p + (ny - 1) * nx : p - nx;
    s.q[4] = j == ny - 1 ? p - (ny - 1) * nx : p + nx;
    s.q[5] = k == 0 ? p + (nz - 1) * sz : p - sz;
    s.q[6] = k == nz - 1 ? p - (nz - 1) * sz : p + sz;
    return s;
}

// -Laplacian_h x at a cell, x[] as in Star
__device__ __forceinline__ double neg_lap(const GridK& g, const double (&x)[7])
{
    const double c = x[0];
    double r = (2.0 * c - x[1] - x[2]) * g.inv_h[0] * g.inv_h[0] + (2.0 * c - x[3] - x[4]) * g.inv_h[1] * g.inv_h[1];
    if (g.n[2] > 1) r += (2.0 * c - x[5] - x[6]) * g.inv_h[2] * g.inv_h[2];
    return r;
}

__global__ __launch_bounds__(kThreads) void k_sum(const double* __restrict__ x, int64_t n, double* __restrict__ part)
{
    __shared__ double sh[kThreads];
    double v = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < n; p += (int64_t)gridDim.x * kThreads) v += x[p];
    const double t = block_sum(v, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// out[slot] = sum of the nb partials (fixed order: deterministic)
__global__ __launch_bounds__(kThreads) void k_finish(const double* __restrict__ part, int nb, double* __restrict__ s,
                                                     int slot)
{
    __shared__ double sh[kThreads];
    const double t = sum_partials(part, nb, sh);
    if (threadIdx.x == 0) s[slot] = t;
}

// b = 4 pi (rho - mean); r = b, phi = 0; partial b.b
__global__ __launch_bounds__(kThreads) void k_cg_init(int64_t n, const double* __restrict__ rho,
                                                      const double* __restrict__ s, double* __restrict__ phi,
                                                      double* __restrict__ r, double* __restrict__ part)
{
    __shared__ double sh[kThreads];
    const double mean = s[5] / (double)n;
    double v = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < n; p += (int64_t)gridDim.x * kThreads) {
        const double b = 4.0 * kPi * (rho[p] - mean);
        r[p] = b;
        phi[p] = 0.0;
        v += b * b;
    }
    const double t = block_sum(v, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// Iteration it, first half: r.r (of the partials part_r that k_cg_init or
// k_cg_update left) into s[it & 1]; the search direction p = r + beta p_old,
// beta = r.r / old r.r (it > 0; p is left as it is once the iterate is frozen,
// and is r itself at it = 0); Ap = A p; partial p.Ap into part_p.  A cell's p
// is written once; its neighbours form theirs again from r and p_old.
__global__ __launch_bounds__(kThreads) void k_cg_apply(GridK g, int it, int nb, double* __restrict__ s,
                                                       const double* __restrict__ part_r,
                                                       const double* __restrict__ r, const double* __restrict__ p_old,
                                                       double* __restrict__ p_new, double* __restrict__ ap,
                                                       double* __restrict__ part_p)
{
    __shared__ double sh[kThreads];
    // the first cell's values load while the partials are summed, and each
    // next cell's while its predecessor is computed
    const uint32_t n = (uint32_t)g.ncell, step = gridDim.x * kThreads;
    uint32_t c = blockIdx.x * kThreads + threadIdx.x;
    double rv[7], pv[7];
    auto load = [&](uint32_t q) {
        const Star st = star_of(g, q);
#pragma unroll
        for (int k = 0; k < 7; ++k) rv[k] = r[st.q[k]];
#pragma unroll
        for (int k = 0; k < 7; ++k) pv[k] = p_old[st.q[k]];
    };
    if (c < n) load(c);
    const double rr = sum_partials(part_r, nb, sh);
    if (blockIdx.x == 0 && threadIdx.x == 0) s[it & 1] = rr;
    const double rr_old = s[(it & 1) ^ 1];
    const bool first = it == 0, frozen = !first && !(rr_old > s[2]);
    const double beta = first || frozen ? 0.0 : rr / rr_old;
    double v = 0.0;
    while (c < n) {
        double p[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) p[k] = first ? rv[k] : (frozen ? pv[k] : rv[k] + beta * pv[k]);
        const uint32_t at = c;
        c = n - c > step ? c + step : n;
        if (c < n) load(c);
        const double a = neg_lap(g, p);
        p_new[at] = p[0];
        ap[at] = a;
        v += p[0] * a;
    }
    const double t = block_sum(v, sh);
    if (threadIdx.x == 0) part_p[blockIdx.x] = t;
}

// Iteration it, second half: alpha = r.r / p.Ap; phi += alpha p; r -= alpha
// Ap; partial new r.r.  Once r.r has reached the target the iterate is frozen
// (alpha = 0): the host checks every kCheck iterations, and iterations past
// the rounding floor of this singular (periodic) system make p.Ap a rounding
// residue, alpha arbitrary and the residual grow again.
__global__ __launch_bounds__(kThreads) void k_cg_update(int64_t n, int it, int nb, const double* __restrict__ s,
                                                        const double* __restrict__ part_p,
                                                        const double* __restrict__ pp, const double* __restrict__ ap,
                                                        double* __restrict__ phi, double* __restrict__ r,
                                                        double* __restrict__ part_r)
{
    __shared__ double sh[kThreads];
    const int64_t step = (int64_t)gridDim.x * kThreads;
    int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    double x[4];
    auto load = [&](int64_t q) {
        x[0] = phi[q];
        x[1] = pp[q];
        x[2] = r[q];
        x[3] = ap[q];
    };
    if (c < n) load(c);
    const double pap = sum_partials(part_p, nb, sh), rr = s[it & 1];
    const double alpha = rr > s[2] && pap > 0.0 ? rr / pap : 0.0;
    double v = 0.0;
    while (c < n) {
        const double f = x[0] + alpha * x[1];
        const double rn = x[2] - alpha * x[3];
        const int64_t at = c;
        c += step;
        if (c < n) load(c);
        phi[at] = f;
        r[at] = rn;
        v += rn * rn;
    }
    const double t = block_sum(v, sh);
    if (threadIdx.x == 0) part_r[blockIdx.x] = t;
}

// s[dst] = f s[src]
__global__ void k_scale(double* s, int dst, int src, double f)
{
    if (threadIdx.x == 0) s[dst] = f * s[src];
}

// E from the potential (Eq. egradphidis)
__global__ __launch_bounds__(kThreads) void k_e_of_phi(GridK g, const double* __restrict__ phi, double* __restrict__ E)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= g.ncell) return;
    const int64_t N = g.ncell;
    const int64_t row = p / g.n[0];
    const int i = (int)(p - row * g.n[0]);
    const int k = (int)(row / g.n[1]);
    const int j = (int)(row - (int64_t)k * g.n[1]);
    const int64_t sy = g.n[0], sz = (int64_t)g.n[0] * g.n[1];
    const int64_t im = i == 0 ? p + (g.n[0] - 1) : p - 1;
    const int64_t jm = j == 0 ? p + (int64_t)(g.n[1] - 1) * sy : p - sy;
    const int64_t km = k == 0 ? p + (int64_t)(g.n[2] - 1) * sz : p - sz;
    const double c = phi[p];
    E[p] = (phi[im] - c) * g.inv_h[0];
    E[N + p] = (phi[jm] - c) * g.inv_h[1];
    E[2 * N + p] = g.n[2] > 1 ? (phi[km] - c) * g.inv_h[2] : 0.0;
}

__global__ __launch_bounds__(kThreads) void k_add_const(double* __restrict__ x, int64_t n, const double* __restrict__ s,
                                                        double scale)
{
    const double v = scale * s[5] / (double)n;
    for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < n; p += (int64_t)gridDim.x * kThreads) x[p] += v;
}

unsigned grid_for(int64_t n) { return (unsigned)std::min<int64_t>(kBlocks, (n + kThreads - 1) / kThreads); }

}  // namespace

hipError_t solve_poisson(Ctx& c, double* rho, bool neutralize, double tol, int64_t max_iter, int64_t* iters,
                         double* rel_residual, hipStream_t s)
{
    const int64_t n = c.k.ncell;
    // scratch: phi and the two search directions in bn, r and Ap in the
    // adjoint planes; partials and scalars in the reduction buffer
    double* phi = c.bn;
    double* p[2] = {c.bn + n, c.bn + 2 * n};
    double* r = c.adj;
    double* ap = c.adj + n;
    double* part = c.red;
    double* part_p = c.red + kBlocks;
    double* sc = c.red + 2 * kBlocks;
    const unsigned gb = grid_for(n);
    const int nb = (int)gb;
    hipLaunchKernelGGL(k_sum, dim3(gb), dim3(kThreads), 0, s, rho, n, part);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kThreads), 0, s, part, nb, sc, 5);
    if (neutralize)  // the uniform background: minus the mean charge density
        hipLaunchKernelGGL(k_add_const, dim3(gb), dim3(kThreads), 0, s, c.rho_bg, n, sc, -1.0);
    hipLaunchKernelGGL(k_cg_init, dim3(gb), dim3(kThreads), 0, s, n, rho, sc, phi, r, part);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kThreads), 0, s, part, nb, sc, 4);
    hipLaunchKernelGGL(k_scale, dim3(1), dim3(64), 0, s, sc, 2, 4, tol * tol);  // target r.r
    double host[7] = {0, 0, 0, 0, 0, 0, 0};
    hipError_t e = hipMemcpyAsync(host, sc, sizeof(host), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    const double bb = host[4];
    int64_t it = 0;
    double rr = bb;
    const double target = tol * tol * bb;
    while (bb > 0.0 && rr > target && it < max_iter) {
        for (int q = 0; q < kCheck && it < max_iter; ++q, ++it) {
            hipLaunchKernelGGL(k_cg_apply, dim3(gb), dim3(kThreads), 0, s, c.k, (int)it, nb, sc, part, r, p[it & 1],
                               p[(it & 1) ^ 1], ap, part_p);
            hipLaunchKernelGGL(k_cg_update, dim3(gb), dim3(kThreads), 0, s, n, (int)it, nb, sc, part_p,
                               p[(it & 1) ^ 1], ap, phi, r, part);
        }
        hipLaunchKernelGGL(k_finish, dim3(1), dim3(kThreads), 0, s, part, nb, sc, 6);  // r.r for the host
        e = hipMemcpyAsync(host, sc, sizeof(host), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        rr = host[6];
    }
    hipLaunchKernelGGL(k_e_of_phi, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, c.k, phi,
                       c.fields);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    *iters = it;
    *rel_residual = bb > 0.0 ? std::sqrt(rr / bb) : 0.0;
    return hipSuccess;
}

}  // namespace pic
