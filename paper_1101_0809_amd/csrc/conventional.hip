// conventional.hip -- the particle step with the "conventional" uniform-order
// field interpolation of Eq. wrong1, the comparison of Section 5 (Fig. 2):
// gather with the mean of adjacent order-1 1/2 cell factors on a component's
// node axes, then the push (Appendix, Eq. p2), the position advance (Eq.
// coordscheme) and the order-1 1/2 charge-conserving current (Eq. current).
// FP64; the charge density and the current of given moves are those of the
// order-1 1/2 scheme.
//
// 2D3V: one workgroup per tile stages E^n, B^n (cells T0-1-M .. T0+T+1+M)
// and accumulates the current (T0-2-M .. T0+T+1+M) in LDS.  3D: the two
// regions do not fit in LDS together with a drift margin, so a first pass
// gathers, pushes and moves with the fields staged (margin 1, 105 KB), keeping
// the start position in the species' spare particle copy and the cell shifts
// in its id array, and a second pass deposits the current (margin 2, 98 KB):
// particles that stay in their cell first (54 contributions), then the
// others (144).
#include <type_traits>

#include "tile_io.h"

namespace pic {
namespace {

__device__ __forceinline__ void add_global(double* p, double v) { unsafeAtomicAdd(p, v); }

constexpr int kCvT2 = kTile2, kCvM2 = 2, kCvNT2 = 256;

__global__ __launch_bounds__(kCvNT2) void k_step_conv2(GridK g, StepArgs a, const double* __restrict__ fields,
                                                     const double* __restrict__ bfield, double* __restrict__ Jg)
{
    constexpr int T = kCvT2, M = kCvM2, NT = kCvNT2;
    constexpr int LF = T + 3 + 2 * M, NF = LF * LF;  // cells T0-1-M .. T0+T+1+M
    constexpr int LJ = T + 4 + 2 * M, NJ = LJ * LJ;  // cells T0-2-M .. T0+T+1+M
    __shared__ double sf[6 * NF];
    __shared__ double sj[3 * NJ];
    const int tile = xcd_tile(blockIdx.x, g.ntiles);
    const int T0[2] = {(tile % g.nt[0]) * T, (tile / g.nt[0]) * T};
    const int64_t N = g.ncell;
    const int nx = g.n[0], ny = g.n[1];
    for (int e = threadIdx.x; e < 6 * NF; e += NT) {
        const int comp = e / NF, r = e - comp * NF;
        const int64_t cell = (int64_t)wrapi(T0[1] - 1 - M + r / LF, ny) * nx + wrapi(T0[0] - 1 - M + r % LF, nx);
        sf[e] = comp < 3 ? fields[comp * N + cell] : bfield[(comp - 3) * N + cell];
    }
    for (int e = threadIdx.x; e < 3 * NJ; e += NT) sj[e] = 0.0;
    __syncthreads();
    const double c = g.c, c2 = c * c;
    const double qmdt2 = 0.5 * a.qm * g.dt;
    const int64_t begin = a.tile_start[tile], end = a.tile_start[tile + 1];
    for (int64_t p = begin + threadIdx.x; p < end; p += NT) {
        int i0[3];
        double d0[3];
        PosIO<double, 2>::load(a, p, i0, d0);
        double w[3];
        for (int ax = 0; ax < 3; ++ax) w[ax] = ((const double*)a.mom[ax])[p];
        const double qp = a.q * ((const double*)a.weight)[p];
        AxisC<double> ax0[3];
        for (int ax = 0; ax < 3; ++ax) ax0[ax] = form_factor_conv<double>(d0[ax]);
        const int rel[2] = {tile_rel(i0[0], T0[0], nx, T, M), tile_rel(i0[1], T0[1], ny, T, M)};
        const bool inside = rel[0] >= -M && rel[0] <= T - 1 + M && rel[1] >= -M && rel[1] <= T - 1 + M;
        double E[3], B[3];
        if (inside) {
            const int fb = (rel[0] + 1 + M) + (rel[1] + 1 + M) * LF;
            auto F = [&](int comp, int oa, int ob, int) -> double { return sf[comp * NF + fb + oa + ob * LF]; };
            gather2_conv<double>(ax0, F, E, B);
        } else {
            auto F = [&](int comp, int oa, int ob, int) -> double {
                const int64_t cell = (int64_t)wrapi(i0[1] + ob, ny) * nx + wrapi(i0[0] + oa, nx);
                return comp < 3 ? fields[comp * N + cell] : bfield[(comp - 3) * N + cell];
            };
            gather2_conv<double>(ax0, F, E, B);
        }
        for (int ax = 0; ax < 3; ++ax) B[ax] += g.bext[ax];
        push<double>(qmdt2, c2, E, B, w);
        for (int ax = 0; ax < 3; ++ax) ((double*)a.mom[ax])[p] = w[ax];
        const double inv = 1.0 / ::sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2] + c2);
        double disp[3], d1[3];
        for (int ax = 0; ax < 3; ++ax) disp[ax] = w[ax] * inv * g.cfl[ax];
        int delta[3] = {0, 0, 0};
        PosIO<double, 2>::move(a, p, g, i0, d0, disp, d1, delta, true);
        double dm[3][4], dp[3][4], jfac[3];
        int s[2];
        for (int ax = 0; ax < 2; ++ax) {
            double s1[3];
            cell_weights<double>(d1[ax], s1);
            window<double>(ax0[ax].s, s1, delta[ax], dm[ax], dp[ax]);
            s[ax] = (delta[ax] < 0 ? -1 : 0) - 1;
        }
        for (int ax = 0; ax < 3; ++ax) jfac[ax] = g.jscale[ax] * qp;
        const double jz = qp * (0.25 * g.inv_vol) * c * w[2] * inv;
        if (inside) {
            const int jb = (rel[0] + s[0] + 2 + M) + (rel[1] + s[1] + 2 + M) * LJ;
            auto S = [&](int comp, int ix, int iy, int, double v) { atomicAdd(&sj[comp * NJ + jb + ix + iy * LJ], v); };
            deposit2<double>(dm, dp, jfac, jz, S);
        } else {
            auto S = [&](int comp, int ix, int iy, int, double v) {
                const int64_t cell = (int64_t)wrapi(i0[1] + s[1] + iy, ny) * nx + wrapi(i0[0] + s[0] + ix, nx);
                add_global(&Jg[comp * N + cell], v);
            };
            deposit2<double>(dm, dp, jfac, jz, S);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 3 * NJ; e += NT) {
        const double v = sj[e];
        if (v == 0.0) continue;
        const int comp = e / NJ, r = e - comp * NJ;
        const int64_t cell = (int64_t)wrapi(T0[1] - 2 - M + r / LJ, ny) * nx + wrapi(T0[0] - 2 - M + r % LJ, nx);
        add_global(&Jg[comp * N + cell], v);
    }
}

constexpr int kCvM3a = 1, kCvM3b = 2;
constexpr int kCvNTa = 512, kCvUa = 4;  // pass 1: threads, slots per thread ordered at a time
constexpr int kCvNTb = 768, kCvUb = 2;  // pass 2
// From kCvFull particles in a workgroup's share on, pass 2 has four waves per
// SIMD (128 VGPRs, no spills): 64^3 x 8 278 -> 268 us a step, 89 x 30 x 88 x 4
// (1780 a tile) 199 -> 188, but 64^3 x 2 (1024) 118.2 -> 118.9.
constexpr int kCvNTbFull = 1024, kCvFull = 1400;
constexpr int64_t kCvFixed = 800;       // staging and flush, in particles (tile_split)
// Field region: 13 cells per axis in rows of 14 and planes of 182 + 2 doubles,
// modulo 16 those of the sort's lane classes; current region: 16 cells in rows of
// 18 and planes of 288 + 8.  The rows give every z layer of a tile's cells each
// class as often: a dense tile's chunk holds one or two layers, and where a class
// runs out its rows are incomplete.  20 steps of 64^3 x 32, w_th = 0.02: 26.1 ms
// with rows of 13 and 17 (24.4 in storage order), 19.3 like this; x 2: 2.31, 2.30.
constexpr int kCvRowF = 14, kCvPlaneF = 13 * 14 + 2;
constexpr int kCvRowJ = 18, kCvPlaneJ = 16 * 18 + 8;
static_assert(even_layers(kCvRowF) && even_layers(kCvRowJ), "a layer holds every class as often");

// Pass 1's word on a particle's move: bits 2 ax .. 2 ax + 1 the cell shift plus
// one, bit 6 no shift on any axis, bit 7 the particle within the current
// region's margin of the tile, bits 8 .. 11 the class of its window's first
// cell there.
constexpr int kCvStill = 64, kCvInside = 128;

// Pass 1 (252 LDS reads per particle) takes the particles in class rows
// (order_rows) of their cell, pass 2 (54 or 144 LDS atomics) in those of their
// window: LDS bank conflicts were 36 and 18% of the CU-busy cycles in storage
// order.  82 and 58 -> 56 and 50 us at 64^3 x 2 per cell; 20 steps of 64^3 x 6
// per cell with the energies 6.25 -> 4.55 ms, hot (w_th = 0.2) 13.3 -> 7.5 ms.
// All fields of a tile in flight at once: 20 steps of 64^3 x 2 2830 -> 2655 us.
__global__ __launch_bounds__(kCvNTa) void k_push_conv3(GridK g, StepArgs a, PartArrays spare,
                                                     const double* __restrict__ fields,
                                                     const double* __restrict__ bfield, int split)
{
    constexpr int T = kTile3, M = kCvM3a, NT = kCvNTa;
    constexpr int LF = T + 3 + 2 * M;  // cells T0-1-M .. T0+T+1+M
    constexpr int ROW = kCvRowF, PLANE = kCvPlaneF, NF = LF * PLANE;
    constexpr int MB = kCvM3b;
    static_assert(ROW >= LF && PLANE >= LF * ROW, "rows and planes hold the region");
    __shared__ double sf[6 * NF];
    __shared__ ClassRows<NT, kCvUa> rows;
    __shared__ unsigned int n_fallback;
    const int unit = xcd_tile(blockIdx.x, g.ntiles * split);
    const int tile = unit / split;
    const int T0[3] = {(tile % g.nt[0]) * T, ((tile / g.nt[0]) % g.nt[1]) * T, (tile / (g.nt[0] * g.nt[1])) * T};
    const int64_t N = g.ncell;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    int64_t begin = a.tile_start[tile], end = a.tile_start[tile + 1];
    tile_share(unit - tile * split, split, begin, end);
    if (begin >= end) return;
    {
        const bool small = nx < LF || ny < LF || nz < LF;
        const Columns<LF, LF, ROW> cols(g, T0[0] - 1 - M, T0[1] - 1 - M, small);
        stage_planes<6 * LF, NT, kAllPlanes<6 * LF, NT>, double>(
            cols,
            [&](int t) {
                const int comp = t / LF;
                return (comp < 3 ? fields + comp * N : bfield + (comp - 3) * N) +
                       plane_offset(g, T0[2] - 1 - M + t - comp * LF, small);
            },
            [&](int t) { return sf + t * PLANE; });
    }
    if (threadIdx.x == 0) n_fallback = 0;
    const double c2 = g.c * g.c;
    const double qmdt2 = 0.5 * a.qm * g.dt;

    auto place = [&](const int i0[3], int rel[3]) -> bool {  // true inside the field region
        bool inside = true;
        for (int ax = 0; ax < 3; ++ax) {
            rel[ax] = tile_rel_long(i0[ax], T0[ax], g.n[ax], T, M);
            inside = inside && rel[ax] >= -M && rel[ax] <= T - 1 + M;
        }
        return inside;
    };
    auto advance = [&](int64_t p, auto on_tile) {
        constexpr bool kTileFields = decltype(on_tile)::value;
        int i0[3], rel[3];
        double d0[3], w[3];
        PosIO<double, 3>::load(a, p, i0, d0);
        for (int ax = 0; ax < 3; ++ax) w[ax] = ((const double*)a.mom[ax])[p];
        AxisC<double> ax0[3];
        for (int ax = 0; ax < 3; ++ax) ax0[ax] = form_factor_conv<double>(d0[ax]);
        place(i0, rel);
        double E[3], B[3];
        if (kTileFields) {
            const int fb = (rel[0] + 1 + M) + (rel[1] + 1 + M) * ROW + (rel[2] + 1 + M) * PLANE;
            auto F = [&](int comp, int oa, int ob, int oc) -> double {
                return sf[comp * NF + fb + oa + ob * ROW + oc * PLANE];
            };
            gather3_conv<double>(ax0, F, E, B);
        } else {
            auto F = [&](int comp, int oa, int ob, int oc) -> double {
                const int64_t cell =
                    ((int64_t)wrapi(i0[2] + oc, nz) * ny + wrapi(i0[1] + ob, ny)) * nx + wrapi(i0[0] + oa, nx);
                return comp < 3 ? fields[comp * N + cell] : bfield[(comp - 3) * N + cell];
            };
            gather3_conv<double>(ax0, F, E, B);
        }
        for (int ax = 0; ax < 3; ++ax) B[ax] += g.bext[ax];
        push<double>(qmdt2, c2, E, B, w);
        for (int ax = 0; ax < 3; ++ax) ((double*)a.mom[ax])[p] = w[ax];
        const double inv = 1.0 / ::sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2] + c2);
        double disp[3], d1[3];
        for (int ax = 0; ax < 3; ++ax) disp[ax] = w[ax] * inv * g.cfl[ax];
        int delta[3] = {0, 0, 0};
        PosIO<double, 3>::move(a, p, g, i0, d0, disp, d1, delta, true);
        int word = kCvStill | kCvInside, jb = 0;
        constexpr int stride[3] = {1, kCvRowJ, kCvPlaneJ};
        for (int ax = 0; ax < 3; ++ax) {
            ((double*)spare.pos[ax])[p] = (double)i0[ax] + d0[ax];
            word |= (delta[ax] + 1) << (2 * ax);
            if (delta[ax] != 0) word &= ~kCvStill;
            if (rel[ax] < -MB || rel[ax] > T - 1 + MB) word &= ~kCvInside;
            jb += (rel[ax] + (delta[ax] < 0 ? -1 : 0) + 1 + MB) * stride[ax];
        }
        spare.id[p] = (int64_t)(word | (jb & (kRowClasses - 1)) << 8);
    };

    uint32_t* out = (uint32_t*)spare.weight + 2 * begin;  // particles off the field region (4 bytes of 8 used)
    for (int64_t cb = begin; cb < end; cb += ClassRows<NT, kCvUa>::W) {
        __syncthreads();  // the fields are staged; the last chunk's order is used up
        const int m = (int)min(end - cb, (int64_t)ClassRows<NT, kCvUa>::W);
        const int nin = order_rows(rows, m, [&](int sl) -> int {
            int i0[3], rel[3];
            double d0[3];
            PosIO<double, 3>::load(a, cb + sl, i0, d0);
            if (!place(i0, rel)) {
                out[atomicAdd(&n_fallback, 1u)] = (uint32_t)(cb - begin + sl);
                return -1;
            }
            return (rel[0] + M + (rel[1] + M) * ROW + (rel[2] + M) * PLANE) & (kRowClasses - 1);
        });
        for (int q = threadIdx.x; q < nin; q += NT) advance(cb + rows.perm[q], std::true_type{});
    }
    __syncthreads();
    for (unsigned q = threadIdx.x; q < n_fallback; q += NT) advance(begin + out[q], std::false_type{});
    if (threadIdx.x == 0 && a.counters) {
        atomicAdd(&a.counters[1], (unsigned long long)n_fallback);
        atomicAdd(&a.counters[2], (unsigned long long)(end - begin));
    }
}

// Pass 2: the particles that stay in their cell, then those that cross within
// the region, then those outside it (a wave runs one form at a time).
template <int NT>
__global__ __launch_bounds__(NT) void k_deposit_conv3(GridK g, StepArgs a, PartArrays spare,
                                                        double* __restrict__ Jg, int split)
{
    constexpr int T = kTile3, M = kCvM3b;
    constexpr int LJ = T + 4 + 2 * M;  // cells T0-2-M .. T0+T+1+M
    constexpr int ROW = kCvRowJ, PLANE = kCvPlaneJ, NJ = LJ * PLANE;
    __shared__ double sj[3 * NJ];
    __shared__ ClassRows<NT, kCvUb> rows;
    __shared__ unsigned int n_cross, n_out;
    const int unit = xcd_tile(blockIdx.x, g.ntiles * split);
    const int tile = unit / split;
    const int T0[3] = {(tile % g.nt[0]) * T, ((tile / g.nt[0]) % g.nt[1]) * T, (tile / (g.nt[0] * g.nt[1])) * T};
    const int64_t N = g.ncell;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    int64_t begin = a.tile_start[tile], end = a.tile_start[tile + 1];
    tile_share(unit - tile * split, split, begin, end);
    if (begin >= end) return;
    for (int e = threadIdx.x; e < 3 * NJ; e += NT) sj[e] = 0.0;
    if (threadIdx.x == 0) n_cross = n_out = 0;
    auto deposit = [&](int64_t p, auto form) {  // 0: still, 1: crossing, 2: outside
        constexpr int kForm = decltype(form)::value;
        const int64_t code = spare.id[p];
        int i0[3], rel[3], s[3];
        double dm[3][4], dp[3][4], s0[3][3], s1[3][3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const double x0 = ((const double*)spare.pos[ax])[p];
            const double x1 = ((const double*)a.pos[ax])[p];
            const double f0 = floor(x0);
            i0[ax] = (int)f0;
            const int delta = kForm == 0 ? 0 : (int)((code >> (2 * ax)) & 3) - 1;
            cell_weights<double>(x0 - f0, s0[ax]);
            cell_weights<double>(x1 - floor(x1), s1[ax]);
            if (kForm != 0) {
                // in registers first: a select between neighbouring weights
                // would become a load at a run-time index from scratch memory
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    asm("" : "+v"(s0[ax][k]));
                    asm("" : "+v"(s1[ax][k]));
                }
                window<double>(s0[ax], s1[ax], delta, dm[ax], dp[ax]);
            }
            s[ax] = (delta < 0 ? -1 : 0) - 1;
            rel[ax] = tile_rel_long(i0[ax], T0[ax], g.n[ax], T, M);
        }
        const double qp = a.q * ((const double*)a.weight)[p];
        double jfac[3];
        for (int ax = 0; ax < 3; ++ax) jfac[ax] = g.jscale[ax] * qp;
        if (kForm < 2) {
            const int jb = (rel[0] + s[0] + 2 + M) + (rel[1] + s[1] + 2 + M) * ROW + (rel[2] + s[2] + 2 + M) * PLANE;
            auto S = [&](int comp, int ix, int iy, int iz, double v) {
                atomicAdd(&sj[comp * NJ + jb + ix + iy * ROW + iz * PLANE], v);
            };
            if (kForm == 0) deposit3_still<double>(s0, s1, jfac, S);
            else deposit3<double>(dm, dp, jfac, S);
        } else {
            int xi[4], yj[4];
            int64_t zk[4];
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                xi[o] = wrapi(i0[0] + s[0] + o, nx);
                yj[o] = wrapi(i0[1] + s[1] + o, ny) * nx;
                zk[o] = (int64_t)wrapi(i0[2] + s[2] + o, nz) * ny * nx;
            }
            auto S = [&](int comp, int ix, int iy, int iz, double v) {
                add_global(&Jg[comp * N + zk[iz] + yj[iy] + xi[ix]], v);
            };
            deposit3<double>(dm, dp, jfac, S);
        }
    };
    auto in_rows = [&](auto form) {
        constexpr int want = decltype(form)::value == 0 ? kCvStill | kCvInside : kCvInside;
        for (int64_t cb = begin; cb < end; cb += ClassRows<NT, kCvUb>::W) {
            __syncthreads();  // the region is clear; the last chunk's order is used up
            const int m = (int)min(end - cb, (int64_t)ClassRows<NT, kCvUb>::W);
            const int n = order_rows(rows, m, [&](int sl) -> int {
                const int word = (int)spare.id[cb + sl];
                if (want & kCvStill) {
                    if (!(word & kCvInside)) n_out = 1;
                    else if (!(word & kCvStill)) n_cross = 1;
                }
                return (word & (kCvStill | kCvInside)) == want ? (word >> 8) & (kRowClasses - 1) : -1;
            });
            for (int q = threadIdx.x; q < n; q += NT) deposit(cb + rows.perm[q], form);
        }
        __syncthreads();
    };
    in_rows(std::integral_constant<int, 0>{});
    if (n_cross) in_rows(std::integral_constant<int, 1>{});
    if (n_out)
        for (int64_t p = begin + threadIdx.x; p < end; p += NT)
            if (!((int)spare.id[p] & kCvInside)) deposit(p, std::integral_constant<int, 2>{});
    const bool small = nx < LJ || ny < LJ || nz < LJ;
    const Columns<LJ, LJ, ROW> cols(g, T0[0] - 2 - M, T0[1] - 2 - M, small);
    flush_planes<3 * LJ, NT>(
        cols, [&](int t) { return sj + t * PLANE; },
        [&](int t) {
            const int comp = t / LJ;
            return Jg + comp * N + plane_offset(g, T0[2] - 2 - M + t - comp * LJ, small);
        });
}

}  // namespace

hipError_t launch_particle_step_conv(Ctx& c, Species& sp, hipStream_t s)
{
    if (sp.n == 0) return hipSuccess;
    StepArgs a{};
    for (int ax = 0; ax < 3; ++ax) {
        a.pos[ax] = sp.cur.pos[ax];
        a.mom[ax] = sp.cur.mom[ax];
    }
    a.weight = sp.cur.weight;
    a.tile_start = sp.tile_start;
    a.q = sp.d.q;
    a.qm = sp.d.q / sp.d.m;
    a.counters = c.counters;
    double* J = c.fields + 6 * c.k.ncell;
    if (c.k.dims == 3) {
        const int split = tile_split(c.k.ntiles, sp.n, kCvFixed);
        const dim3 grid((unsigned)(c.k.ntiles * split));
        hipLaunchKernelGGL(k_push_conv3, grid, dim3(kCvNTa), 0, s, c.k, a, sp.alt, c.fields, c.bn, split);
        if (sp.n / c.k.ntiles / split >= kCvFull)
            hipLaunchKernelGGL(k_deposit_conv3<kCvNTbFull>, grid, dim3(kCvNTbFull), 0, s, c.k, a, sp.alt, J, split);
        else
            hipLaunchKernelGGL(k_deposit_conv3<kCvNTb>, grid, dim3(kCvNTb), 0, s, c.k, a, sp.alt, J, split);
    } else {
        hipLaunchKernelGGL(k_step_conv2, dim3(c.k.ntiles), dim3(kCvNT2), 0, s, c.k, a, c.fields, c.bn, J);
    }
    return hipGetLastError();
}

}  // namespace pic
