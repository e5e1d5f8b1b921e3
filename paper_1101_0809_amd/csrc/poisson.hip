// poisson.hip -- electrostatic initial field (Section 4.3): the discrete
// Poisson equation of Eq. poiphi for the cell-centred potential,
//   sum_a (-Phi_{c-e_a} + 2 Phi_c - Phi_{c+e_a}) / d_a^2 = 4 pi rho_c,
// on the periodic grid, then E from Eq. egradphidis,
//   E^x at face i = (Phi_{i-1} - Phi_i) / dx  (and y, z alike),
// so that div_h E = 4 pi rho cell by cell.  The operator is symmetric and
// positive definite on grid functions of zero mean; the right side has its
// mean removed (a uniform background) and conjugate gradients run on that
// subspace.  Scalars (alpha, beta, residual norms) stay on the device.  Grids
// of up to 524288 cells take all iterations in one launch (k_cg_run); on others
// each iteration is two launches with no host round trip, and the host reads
// the residual every kCheck iterations to stop.
//
// What bounds an iteration on the usual grids is launches, not bytes (64^3:
// ten planes of 2 MB, cache resident).  The reductions are therefore finished
// by their readers -- every workgroup sums the previous kernel's partials
// itself, in the one fixed order, instead of waiting for a one-workgroup
// kernel -- and the new search direction is formed where the stencil reads it.
// Six launches became two: 32 -> 14 us per iteration at 64^3 (the check of the
// residual included), 68 -> 42 us at 128^3.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>

#include "pic_internal.h"

namespace pic {
namespace {

constexpr int kThreads = 256;
constexpr int kBlocks = 1024;  // reduction workgroups
constexpr int kCheck = 16;

// device scalars: [0], [1] r.r of even and odd iterations  [2] target r.r
// [4] b.b  [5] sum rho  [6] r.r for the host  [7] r.r before it (k_cg_run)
// [8], [9] status of k_cg_run  [16] .. its slots

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

// ---------------------------------------------------------------------------
// The iterations in one launch, for grids whose state fits the registers of
// one workgroup per CU.  A workgroup keeps kRunThreads x CPT consecutive cells:
// r (also in LDS, for neighbours among them, and in memory, for the other
// workgroups), phi, and p of each cell and of its six neighbours, which is
// formed again from the neighbours' r as in k_cg_apply, so that r is all that
// is exchanged.  In place of the two kernel boundaries of an iteration the
// workgroups exchange their partial sums: each stores its own in a slot and
// reads everybody's, which is at once the reduction (in the same order
// everywhere) and the barrier.  Slots and r go past the XCDs' L2s: stored and
// loaded by atomics of agent scope, each wave's stores of r having ended before
// its workgroup's slot is written.  Bound by those round trips (three or four of
// about a microsecond per exchange).  A solve at 24^3, 64^3 and 80^3, and at
// 128^2 and 512^2: 1.17, 3.77, 6.17, 3.77, 21.0 -> 0.51, 2.07, 3.60, 1.22, 10.0
// ms.  Larger grids (128^3: 42 us an iteration in two launches) would spill, and
// wait less for launches.
// ---------------------------------------------------------------------------
constexpr int kRunThreads = 1024, kRunCells = 2;  // cells per thread at most (4 spill)
constexpr int kRunIters = 2048;                  // iterations of a launch at most
// Reads of a slot (a microsecond each) before giving up: what a wait in vain costs
// is then no more than the solve in separate launches that follows it (64^3: 4 ms).
constexpr int kRunPolls = 1 << 12;
constexpr unsigned long long kEmpty = 0xfff8dead00000001ull;  // a slot not written yet (a NaN no sum yields)

// status[0]: iterations done; status[1]: nonzero if a workgroup gave up.
__global__ void k_run_prepare(unsigned long long* slots, int n, unsigned long long* status)
{
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t < n) slots[t] = kEmpty;
    if (t < 2) status[t] = 0;
}

__device__ __forceinline__ void store_agent(unsigned long long* p, unsigned long long v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double load_agent(const double* p)
{
    return __longlong_as_double((long long)__hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT));
}

// v of the lane that the DPP control CTRL names, 0.0 where there is none or the
// row (of 16 lanes) is not in ROWS.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double v)
{
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
    return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}

// Sum over the wave, in lane 63 (four row shifts and two row broadcasts, which
// need no LDS: the sums are on the path between the workgroups).
__device__ __forceinline__ double wave_sum63(double v)
{
    v += dpp_or_zero<0x111, 0xf>(v);  // row_shr:1
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// Iterations it0 .. it1 - 1, fewer once r.r has reached the target s[2].  s[6]:
// r.r before and after.  polls: reads of a slot before giving up.
template <int CPT>
__global__ __launch_bounds__(kRunThreads) void k_cg_run(GridK g, int it0, int it1, int polls, double* __restrict__ s,
                                                        unsigned long long* slots, unsigned long long* status,
                                                        double* r, double* __restrict__ phi, double* __restrict__ p)
{
    constexpr int NT = kRunThreads, NW = NT / 64, K = NT * CPT;
    static_assert(kCus <= NT && kCus % 64 == 0, "a thread per slot");
    __shared__ double lr[K], mine[NW], all[NW];
    __shared__ int gave_up;
    const int t = threadIdx.x, wv = t >> 6;
    const int W = gridDim.x;
    const uint32_t n = (uint32_t)g.ncell, base = blockIdx.x * K;
    if (t == 0) gave_up = 0;
    // Publish the workgroup's sum of v for epoch e, after the stores of all of
    // its waves; clear the slot of epoch e + 2 (that of e - 2, which everybody
    // has read: everybody has published e - 1).
    auto publish = [&](double v, int e) {
        v = wave_sum63(v);
        if ((t & 63) == 63) mine[wv] = v;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (t == 0) {
            double sum = 0.0;
            for (int w = 0; w < NW; ++w) sum += mine[w];
            store_agent(slots + (e & 3) * kCus + blockIdx.x,
                        sum != sum ? 0x7ff8000000000000ull : (unsigned long long)__double_as_longlong(sum));
            store_agent(slots + ((e + 2) & 3) * kCus + blockIdx.x, kEmpty);
        }
    };
    // Sum of everybody's sums of epoch e; false if one did not come.
    auto collect = [&](int e, double& sum) -> bool {
        double v = 0.0;
        if (t < W) {
            const double* slot = (const double*)slots + (e & 3) * kCus + t;
            unsigned long long b = kEmpty;
            for (int q = 0; q < polls && b == kEmpty; ++q)
                b = (unsigned long long)__double_as_longlong(load_agent(slot));
            if (b == kEmpty) gave_up = 1;
            v = __longlong_as_double((long long)b);
        }
        if (t < kCus) {
            v = wave_sum63(v);
            if ((t & 63) == 63) all[wv] = v;
        }
        __syncthreads();
        sum = 0.0;
        for (int w = 0; w < kCus / 64; ++w) sum += all[w];
        return !gave_up;
    };

    double rv[CPT], f[CPT], pv[CPT][7];
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
        const uint32_t c = base + t + u * NT;
        rv[u] = f[u] = 0.0;
        for (int k = 0; k < 7; ++k) pv[u][k] = 0.0;
        if (c < n) {
            rv[u] = r[c];
            f[u] = phi[c];
            if (it0 > 0) {
                const Star st = star_of(g, c);
#pragma unroll
                for (int k = 0; k < 7; ++k) pv[u][k] = p[st.q[k]];
            }
        }
        lr[t + u * NT] = rv[u];
    }
    __syncthreads();
    const double target = s[2];
    double rr = s[6], rr_old = s[7];
    int it = it0, e = 0;
    bool good = true;
    while (rr > target && it < it1) {
        const double beta = it == 0 ? 0.0 : rr / rr_old;
        double ap[CPT], v = 0.0;
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            const uint32_t c = base + t + u * NT;
            ap[u] = 0.0;
            if (c >= n) continue;
            const Star st = star_of(g, c);
            double x[7];
            x[0] = rv[u];
#pragma unroll
            for (int k = 1; k < 7; ++k)
                x[k] = st.q[k] - base < (uint32_t)K ? lr[st.q[k] - base] : load_agent(r + st.q[k]);
#pragma unroll
            for (int k = 0; k < 7; ++k) pv[u][k] = it == 0 ? x[k] : x[k] + beta * pv[u][k];
            ap[u] = neg_lap(g, pv[u]);
            v += pv[u][0] * ap[u];
        }
        publish(v, e);
        double pap;
        good = collect(e++, pap);
        if (!good) break;
        const double alpha = pap > 0.0 ? rr / pap : 0.0;
        v = 0.0;
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            const uint32_t c = base + t + u * NT;
            f[u] += alpha * pv[u][0];
            rv[u] -= alpha * ap[u];
            v += rv[u] * rv[u];
            if (c < n) store_agent((unsigned long long*)r + c, (unsigned long long)__double_as_longlong(rv[u]));
            lr[t + u * NT] = rv[u];
        }
        publish(v, e);
        rr_old = rr;
        good = collect(e++, rr);
        if (!good) break;
        ++it;
    }
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
        const uint32_t c = base + t + u * NT;
        if (c < n) {
            phi[c] = f[u];
            p[c] = pv[u][0];
        }
    }
    if (t == 0 && !good) atomicExch(&status[1], 1ull);
    if (t == 0 && blockIdx.x == 0) {
        s[6] = rr;
        s[7] = rr_old;
        status[0] = (unsigned long long)it;
    }
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

// The one-launch form of a device is one solve's at a time: of two, each could
// hold half of the CUs and wait for the other.  The solve that finds it taken
// (from another thread) runs in separate launches.
class RunTurn {
  public:
    RunTurn()
    {
        static std::atomic<bool> taken[kDevices];
        int dev = -1;
        if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kDevices && !taken[dev].exchange(true))
            flag_ = &taken[dev];
    }
    ~RunTurn()
    {
        if (flag_) flag_->store(false);
    }
    RunTurn(const RunTurn&) = delete;
    RunTurn& operator=(const RunTurn&) = delete;
    bool mine() const { return flag_ != nullptr; }

  private:
    static constexpr int kDevices = 64;
    std::atomic<bool>* flag_ = nullptr;
};

// Workgroups of the one-launch form that the current device runs at once.
int resident_workgroups(const void* kernel)
{
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, kRunThreads, 0) != hipSuccess)
        return 0;
    return std::min(kCus, cus * per);
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
    const unsigned long long* status = (const unsigned long long*)(sc + 8);
    double host[10] = {0};
    hipError_t e = hipMemcpyAsync(host, sc, sizeof(host), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    const double bb = host[4];
    int64_t it = 0;
    double rr = bb;
    const double target = tol * tol * bb;
    // In one launch: one workgroup per CU at most, all of which have to be
    // running at once, so the device has to hold them (one that shows fewer CUs
    // would lose the wait in every solve).  If one is kept waiting too long (by
    // another process or stream on the GPU) all give up, and the solve starts
    // again in separate launches; so it does if a launch made no iteration.
    c.poisson_form = 1;
    const RunTurn turn;
    const int cells = (int)((n + (int64_t)kCus * kRunThreads - 1) / ((int64_t)kCus * kRunThreads));
    const int cpt = cells <= 1 ? 1 : kRunCells;
    auto* run = cpt == 1 ? k_cg_run<1> : k_cg_run<kRunCells>;
    const int64_t wgs = (n + kRunThreads * cpt - 1) / (kRunThreads * cpt);
    const PoissonLimits& lim = c.poisson_limits;
    const int polls = lim.polls < 0 ? kRunPolls : lim.polls;
    const int iters_max = lim.iterations < 0 ? kRunIters : lim.iterations;
    const int held = lim.workgroups < 0 ? resident_workgroups((const void*)run) : std::min(kCus, lim.workgroups);
    if (turn.mine() && bb > 0.0 && rr > target && it < max_iter && wgs <= held) {
        c.poisson_form = 2;
        unsigned long long* slots = (unsigned long long*)(sc + 16);
        const dim3 grid((unsigned)wgs);
        hipLaunchKernelGGL(k_scale, dim3(1), dim3(64), 0, s, sc, 6, 4, 1.0);
        while (rr > target && it < max_iter) {
            hipLaunchKernelGGL(k_run_prepare, dim3(4 * kCus / kThreads), dim3(kThreads), 0, s, slots, 4 * kCus,
                               (unsigned long long*)status);
            const int last = (int)std::min<int64_t>(max_iter, it + iters_max);
            hipLaunchKernelGGL(run, grid, dim3(kRunThreads), 0, s, c.k, (int)it, last, polls, sc, slots,
                               (unsigned long long*)status, r, phi, p[0]);
            e = hipGetLastError();  // a launch that was refused leaves the status as it was prepared
            if (e == hipSuccess) e = hipMemcpyAsync(host, sc, sizeof(host), hipMemcpyDeviceToHost, s);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            if (e != hipSuccess) return e;
            unsigned long long st[2];
            std::memcpy(st, host + 8, sizeof(st));
            if (st[1] || (int64_t)st[0] <= it) {
                c.poisson_form = 3;
                it = 0;
                rr = bb;
                hipLaunchKernelGGL(k_cg_init, dim3(gb), dim3(kThreads), 0, s, n, rho, sc, phi, r, part);
                break;
            }
            it = (int64_t)st[0];
            rr = host[6];
        }
        // counted in whole checks, as by the launches below
        if (!(rr > target)) it = std::min(max_iter, (it + kCheck - 1) / kCheck * kCheck);
    }
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
