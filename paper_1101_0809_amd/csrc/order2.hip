// order2.hip -- the particle step with the alternating form factor of order
// 2 1/2 (Section 4.5): gather of E with alpha (Eq. alphax) and of B^n with
// beta (Eq. betax) at quadratic node and cubic cell factors, the push
// (Appendix, Eq. p2), the position advance (Eq. coordscheme) and the
// charge-conserving current (Eq. current, one-quarter form) on a 5-cell
// window per axis; plus the order-2 1/2 charge density (Eq. rho) and the
// current of given moves.  FP64.
//
// One workgroup per cell tile (the tiles of the cell sort).  It stages E^n and
// B^n over the cells the tile's particles can read (offsets -2 .. +2 around
// each particle cell, plus a margin M for drift since the sort) and
// accumulates the current over the cells their windows can reach (-3 .. +3,
// plus M) in LDS, added to the grid once at the end; in 3D the two regions
// are handled by two passes.  A particle further than M cells from its tile
// reads and adds in global memory instead.
#include <algorithm>
#include <type_traits>

#include "tile_io.h"

namespace pic {
namespace {

__device__ __forceinline__ void add_global(double* p, double v) { unsafeAtomicAdd(p, v); }

// window5 with both weight sets in registers first: a select between two
// entries of one array (the window shifted one cell or not) would otherwise
// become one load at a run-time index, which keeps the array in scratch
// memory.
__device__ __forceinline__ void window5_reg(const double (&s0)[4], const double (&s1)[4], int shift, double dm[5],
                                            double dp[5])
{
    double a[4], b[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        a[k] = s0[k];
        b[k] = s1[k];
        asm("" : "+v"(a[k]));
        asm("" : "+v"(b[k]));
    }
    window5<double>(a, b, shift, dm, dp);
}

// The single pass, used in 2D3V (its two regions fit in LDS with margin 2).
constexpr int kO2M2 = 2, kO2NT2 = 256;

template <int D>
__global__ __launch_bounds__(kO2NT2) void k_step_o2(GridK g, StepArgs a, const double* __restrict__ fields,
                                                    const double* __restrict__ bfield, double* __restrict__ Jg)
{
    static_assert(D == 2, "the 3D order-2 1/2 step runs in two passes");
    constexpr int T = kTile2, M = kO2M2, NT = kO2NT2;
    constexpr int LF = T + 4 + 2 * M;  // field region: cells T0-2-M .. T0+T+1+M
    constexpr int LJ = T + 6 + 2 * M;  // current region: cells T0-3-M .. T0+T+2+M
    constexpr int NF = D == 3 ? LF * LF * LF : LF * LF;
    constexpr int NJ = D == 3 ? LJ * LJ * LJ : LJ * LJ;
    __shared__ double sf[6 * NF];
    __shared__ double sj[3 * NJ];
    __shared__ unsigned int n_fallback;

    const int tile = xcd_tile(blockIdx.x, g.ntiles);
    const int T0[3] = {(tile % g.nt[0]) * T, ((tile / g.nt[0]) % g.nt[1]) * T,
                       D == 3 ? (tile / (g.nt[0] * g.nt[1])) * T : 0};
    const int64_t N = g.ncell;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];

    for (int e = threadIdx.x; e < 6 * NF; e += NT) {
        const int comp = e / NF, r = e - comp * NF;
        const int gx = wrapi(T0[0] - 2 - M + r % LF, nx);
        const int gy = wrapi(T0[1] - 2 - M + (r / LF) % LF, ny);
        const int gz = D == 3 ? wrapi(T0[2] - 2 - M + r / (LF * LF), nz) : 0;
        const int64_t cell = ((int64_t)gz * ny + gy) * nx + gx;
        sf[e] = comp < 3 ? fields[comp * N + cell] : bfield[(comp - 3) * N + cell];
    }
    for (int e = threadIdx.x; e < 3 * NJ; e += NT) sj[e] = 0.0;
    if (threadIdx.x == 0) n_fallback = 0;
    __syncthreads();

    const double c = g.c, c2 = c * c;
    const double qmdt2 = 0.5 * a.qm * g.dt;
    const int64_t begin = a.tile_start[tile], end = a.tile_start[tile + 1];
    unsigned int my_fallback = 0;
    for (int64_t p = begin + threadIdx.x; p < end; p += NT) {
        int i0[3];
        double d0[3];
        PosIO<double, D>::load(a, p, i0, d0);
        double w[3];
        for (int ax = 0; ax < 3; ++ax) w[ax] = ((const double*)a.mom[ax])[p];
        const double qp = a.q * ((const double*)a.weight)[p];
        Axis2<double> ax0[3];
        for (int ax = 0; ax < 3; ++ax) ax0[ax] = form_factor2<double>(ax < D ? d0[ax] : 0.0);

        int rel[3] = {0, 0, 0};
        bool inside = true;
        for (int ax = 0; ax < D; ++ax) {
            const int r = tile_rel(i0[ax], T0[ax], g.n[ax], T, M);
            rel[ax] = r;
            inside = inside && r >= -M && r <= T - 1 + M;
        }
        my_fallback += inside ? 0 : 1;

        double E[3], B[3];
        if (inside) {
            const int fb = (rel[0] + 2 + M) + (rel[1] + 2 + M) * LF + (D == 3 ? (rel[2] + 2 + M) * LF * LF : 0);
            auto F = [&](int comp, int oa, int ob, int oc) -> double {
                return sf[comp * NF + fb + oa + ob * LF + (D == 3 ? oc * LF * LF : 0)];
            };
            if (D == 3) gather3_o2<double>(ax0, F, E, B);
            else gather2_o2<double>(ax0, F, E, B);
        } else {
            auto F = [&](int comp, int oa, int ob, int oc) -> double {
                const int64_t cell = ((int64_t)(D == 3 ? wrapi(i0[2] + oc, nz) : 0) * ny + wrapi(i0[1] + ob, ny)) * nx +
                                     wrapi(i0[0] + oa, nx);
                return comp < 3 ? fields[comp * N + cell] : bfield[(comp - 3) * N + cell];
            };
            if (D == 3) gather3_o2<double>(ax0, F, E, B);
            else gather2_o2<double>(ax0, F, E, B);
        }
        for (int ax = 0; ax < 3; ++ax) B[ax] += g.bext[ax];

        push<double>(qmdt2, c2, E, B, w);
        for (int ax = 0; ax < 3; ++ax) ((double*)a.mom[ax])[p] = w[ax];
        const double inv = 1.0 / ::sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2] + c2);
        double disp[3];
        for (int ax = 0; ax < 3; ++ax) disp[ax] = w[ax] * inv * g.cfl[ax];
        double d1[3];
        int delta[3] = {0, 0, 0};
        PosIO<double, D>::move(a, p, g, i0, d0, disp, d1, delta, true);

        // window per axis: start i0 + h0, end (i0 + delta) + h1
        double dm[3][5], dp[3][5];
        int s[3] = {0, 0, 0};
        for (int ax = 0; ax < D; ++ax) {
            const Axis2<double> e1 = form_factor2<double>(d1[ax]);
            const int shift = delta[ax] + e1.h - ax0[ax].h;
            window5_reg(ax0[ax].s, e1.s, shift, dm[ax], dp[ax]);
            s[ax] = ax0[ax].h + (shift < 0 ? shift : 0) - 2;  // window start, from the particle cell
        }
        double jfac[3];
        for (int ax = 0; ax < 3; ++ax) jfac[ax] = g.jscale[ax] * qp;
        const double jz = D == 2 ? qp * (0.25 * g.inv_vol) * c * w[2] * inv : 0.0;
        if (inside) {
            const int jb = (rel[0] + s[0] + 3 + M) + (rel[1] + s[1] + 3 + M) * LJ +
                           (D == 3 ? (rel[2] + s[2] + 3 + M) * LJ * LJ : 0);
            auto S = [&](int comp, int ix, int iy, int iz, double v) {
                atomicAdd(&sj[comp * NJ + jb + ix + iy * LJ + (D == 3 ? iz * LJ * LJ : 0)], v);
            };
            if (D == 3) deposit3_o2<double>(dm, dp, jfac, S);
            else deposit2_o2<double>(dm, dp, jfac, jz, S);
        } else {
            auto S = [&](int comp, int ix, int iy, int iz, double v) {
                const int64_t cell =
                    ((int64_t)(D == 3 ? wrapi(i0[2] + s[2] + iz, nz) : 0) * ny + wrapi(i0[1] + s[1] + iy, ny)) * nx +
                    wrapi(i0[0] + s[0] + ix, nx);
                add_global(&Jg[comp * N + cell], v);
            };
            if (D == 3) deposit3_o2<double>(dm, dp, jfac, S);
            else deposit2_o2<double>(dm, dp, jfac, jz, S);
        }
    }
    if (my_fallback) atomicAdd(&n_fallback, my_fallback);
    __syncthreads();
    for (int e = threadIdx.x; e < 3 * NJ; e += NT) {
        const double v = sj[e];
        if (v == 0.0) continue;
        const int comp = e / NJ, r = e - comp * NJ;
        const int gx = wrapi(T0[0] - 3 - M + r % LJ, nx);
        const int gy = wrapi(T0[1] - 3 - M + (r / LJ) % LJ, ny);
        const int gz = D == 3 ? wrapi(T0[2] - 3 - M + r / (LJ * LJ), nz) : 0;
        add_global(&Jg[comp * N + ((int64_t)gz * ny + gy) * nx + gx], v);
    }
    if (threadIdx.x == 0 && a.counters) {
        atomicAdd(&a.counters[1], (unsigned long long)n_fallback);
        atomicAdd(&a.counters[2], (unsigned long long)(end - begin));
    }
}

// 3D in two passes, each staging one region with a wider drift margin than
// the single pass could afford (its two regions at margin 0 fill the LDS).
// Pass 1: gather, push and move with E^n, B^n over cells T0-3 .. T0+T+2 (132
// KB); the start position goes to the spare particle copy (idle between
// sorts) and a word on the move (MoveWord) to its id array.  Pass 2: the
// current over cells T0-5 .. T0+T+4 (140 KB).  Both are bound by the LDS (252
// reads, 144 or 300 atomics per particle), so both take the particles in
// class rows (order_rows) of the stencil's first point: the sort's own class
// order does not serve them, since the stencil starts at int(x + 1/2).  LDS
// bank conflicts fell from 33 and 19% of the CU-busy cycles to 7 and 5%, the
// passes from 86 and 98 to 76 and 76 us at 64^3 x 2 per cell (half of it the
// staging and flush of 1024 particles' tiles), and 20 steps of 64^3 x 6 from
// 11.6 to 7.0 ms with the energies.  Pass 1 has two waves per SIMD to hide
// its latencies: 768 threads spill 43 registers and gain nothing.  All fields
// of a tile in flight at once: 20 steps of 64^3 x 2 3530 -> 3300 us.
constexpr int kO2M3a = 1, kO2M3b = 2;
constexpr int kO2NTa = 512, kO2Ua = 4;  // pass 1 (200 VGPRs): threads, slots per thread ordered at a time
constexpr int kO2NTb = 768, kO2Ub = 2;  // pass 2 (134 VGPRs)
// From kO2Full particles in a workgroup's share on, pass 2 has four waves per
// SIMD (128 VGPRs, two spilled): 64^3 x 8 401 -> 389 us a step, 89 x 30 x 88 x 4
// (1780 a tile) 289 -> 277, but 40 x 36 x 30 x 3 (648 a share) 69.6 -> 70.0.
constexpr int kO2NTbFull = 1024, kO2Full = 1400;
constexpr int64_t kO2Fixed = 800;  // staging and flush, in particles (tile_split)

// Pass 1's word on a particle's move: bits 2 ax .. 2 ax + 1 the cell shift plus
// one, bit 6 int(x + 1/2) unchanged on every axis, bit 7 the particle within
// the current region's margin of the tile, bits 8 .. 11 the class of its
// window's first cell there.
constexpr int kMvStill = 64, kMvInside = 128;

__global__ __launch_bounds__(kO2NTa) void k_push_o2_3d(GridK g, StepArgs a, PartArrays spare,
                                                       const double* __restrict__ fields,
                                                       const double* __restrict__ bfield, int split)
{
    constexpr int T = kTile3, M = kO2M3a, NT = kO2NTa;
    constexpr int LF = T + 4 + 2 * M, NF = LF * LF * LF;
    constexpr int MB = kO2M3b, LJ = T + 6 + 2 * MB;
    static_assert(even_layers(LF) && even_layers(LJ), "a layer holds every class as often");
    __shared__ double sf[6 * NF];
    __shared__ ClassRows<NT, kO2Ua> rows;
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
        const Columns<LF, LF, LF> cols(g, T0[0] - 2 - M, T0[1] - 2 - M, small);
        stage_planes<6 * LF, NT, kAllPlanes<6 * LF, NT>, double>(
            cols,
            [&](int t) {
                const int comp = t / LF;
                return (comp < 3 ? fields + comp * N : bfield + (comp - 3) * N) +
                       plane_offset(g, T0[2] - 2 - M + t - comp * LF, small);
            },
            [&](int t) { return sf + t * (LF * LF); });
    }
    if (threadIdx.x == 0) n_fallback = 0;
    const double c2 = g.c * g.c;
    const double qmdt2 = 0.5 * a.qm * g.dt;

    // Cell relative to the tile; true inside the field region.
    auto place = [&](const int i0[3], int rel[3]) -> bool {
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
        Axis2<double> ax0[3];
        for (int ax = 0; ax < 3; ++ax) ax0[ax] = form_factor2<double>(d0[ax]);
        place(i0, rel);
        double E[3], B[3];
        if (kTileFields) {
            const int fb = (rel[0] + 2 + M) + (rel[1] + 2 + M) * LF + (rel[2] + 2 + M) * LF * LF;
            auto F = [&](int comp, int oa, int ob, int oc) -> double {
                return sf[comp * NF + fb + oa + ob * LF + oc * LF * LF];
            };
            gather3_o2<double>(ax0, F, E, B);
        } else {
            auto F = [&](int comp, int oa, int ob, int oc) -> double {
                const int64_t cell =
                    ((int64_t)wrapi(i0[2] + oc, nz) * ny + wrapi(i0[1] + ob, ny)) * nx + wrapi(i0[0] + oa, nx);
                return comp < 3 ? fields[comp * N + cell] : bfield[(comp - 3) * N + cell];
            };
            gather3_o2<double>(ax0, F, E, B);
        }
        for (int ax = 0; ax < 3; ++ax) B[ax] += g.bext[ax];
        push<double>(qmdt2, c2, E, B, w);
        for (int ax = 0; ax < 3; ++ax) ((double*)a.mom[ax])[p] = w[ax];
        const double inv = 1.0 / ::sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2] + c2);
        double disp[3], d1[3];
        for (int ax = 0; ax < 3; ++ax) disp[ax] = w[ax] * inv * g.cfl[ax];
        int delta[3] = {0, 0, 0};
        PosIO<double, 3>::move(a, p, g, i0, d0, disp, d1, delta, true);
        int word = kMvStill | kMvInside, jb = 0;
        constexpr int stride[3] = {1, LJ, LJ * LJ};
        for (int ax = 0; ax < 3; ++ax) {
            ((double*)spare.pos[ax])[p] = (double)i0[ax] + d0[ax];
            const int shift = delta[ax] + (d1[ax] >= 0.5 ? 1 : 0) - ax0[ax].h;
            word |= (delta[ax] + 1) << (2 * ax);
            if (shift != 0) word &= ~kMvStill;
            if (rel[ax] < -MB || rel[ax] > T - 1 + MB) word &= ~kMvInside;
            jb += (rel[ax] + ax0[ax].h + (shift < 0 ? shift : 0) + 1 + MB) * stride[ax];
        }
        spare.id[p] = (int64_t)(word | (jb & (kRowClasses - 1)) << 8);
    };

    uint32_t* out = (uint32_t*)spare.weight + 2 * begin;  // particles off the field region (4 bytes of 8 used)
    for (int64_t cb = begin; cb < end; cb += ClassRows<NT, kO2Ua>::W) {
        __syncthreads();  // the fields are staged; the last chunk's order is used up
        const int m = (int)min(end - cb, (int64_t)ClassRows<NT, kO2Ua>::W);
        const int nin = order_rows(rows, m, [&](int sl) -> int {
            int i0[3], rel[3];
            double d0[3];
            PosIO<double, 3>::load(a, cb + sl, i0, d0);
            if (!place(i0, rel)) {
                out[atomicAdd(&n_fallback, 1u)] = (uint32_t)(cb - begin + sl);
                return -1;
            }
            const int h[3] = {d0[0] >= 0.5 ? 1 : 0, d0[1] >= 0.5 ? 1 : 0, d0[2] >= 0.5 ? 1 : 0};
            return ((rel[0] + M + h[0]) + (rel[1] + M + h[1]) * LF + (rel[2] + M + h[2]) * LF * LF) & (kRowClasses - 1);
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

// One particle's windows for the current pass: start position from the spare
// copy, end position and cell shifts from pass 1.
struct O2Move {
    int i0[3], rel[3], s[3];
};

__device__ __forceinline__ void o2_windows(const GridK& g, const StepArgs& a, const PartArrays& spare, int64_t p,
                                           const int T0[3], double (&dm)[3][5], double (&dp)[3][5], O2Move& mv)
{
    const int64_t code = spare.id[p];
    for (int ax = 0; ax < 3; ++ax) {
        const double x0 = ((const double*)spare.pos[ax])[p];
        const double x1 = ((const double*)a.pos[ax])[p];
        const double f0 = floor(x0), f1 = floor(x1);
        mv.i0[ax] = (int)f0;
        const int delta = (int)((code >> (2 * ax)) & 3) - 1;
        const Axis2<double> e0 = form_factor2<double>(x0 - f0);
        const Axis2<double> e1 = form_factor2<double>(x1 - f1);
        const int shift = delta + e1.h - e0.h;
        window5_reg(e0.s, e1.s, shift, dm[ax], dp[ax]);
        mv.s[ax] = e0.h + (shift < 0 ? shift : 0) - 2;
        mv.rel[ax] = tile_rel_long(mv.i0[ax], T0[ax], g.n[ax], kTile3, kO2M3b);
    }
}

// Pass 2.  First the particles whose int(x + 1/2) stays put on every axis (most
// of them at thermal speeds; 144 contributions), then the others within the
// region (300), then those outside it, so that a wave does not run two forms
// for a few lanes.
template <int NT>
__global__ __launch_bounds__(NT) void k_deposit_o2_3d(GridK g, StepArgs a, PartArrays spare,
                                                          double* __restrict__ Jg, int split)
{
    constexpr int T = kTile3, M = kO2M3b;
    constexpr int LJ = T + 6 + 2 * M, NJ = LJ * LJ * LJ;
    __shared__ double sj[3 * NJ];
    __shared__ ClassRows<NT, kO2Ub> rows;
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
        double dm[3][5], dp[3][5];
        O2Move mv;
        o2_windows(g, a, spare, p, T0, dm, dp, mv);
        const double qp = a.q * ((const double*)a.weight)[p];
        double jfac[3];
        for (int ax = 0; ax < 3; ++ax) jfac[ax] = g.jscale[ax] * qp;
        if (kForm < 2) {
            const int jb = (mv.rel[0] + mv.s[0] + 3 + M) + (mv.rel[1] + mv.s[1] + 3 + M) * LJ +
                           (mv.rel[2] + mv.s[2] + 3 + M) * LJ * LJ;
            auto S = [&](int comp, int ix, int iy, int iz, double v) {
                atomicAdd(&sj[comp * NJ + jb + ix + iy * LJ + iz * LJ * LJ], v);
            };
            if (kForm == 0) deposit3_o2_still<double>(dm, dp, jfac, S);
            else deposit3_o2<double>(dm, dp, jfac, S);
        } else {
            int xi[5], yj[5];
            int64_t zk[5];
#pragma unroll
            for (int o = 0; o < 5; ++o) {
                xi[o] = wrapi(mv.i0[0] + mv.s[0] + o, nx);
                yj[o] = wrapi(mv.i0[1] + mv.s[1] + o, ny) * nx;
                zk[o] = (int64_t)wrapi(mv.i0[2] + mv.s[2] + o, nz) * ny * nx;
            }
            auto S = [&](int comp, int ix, int iy, int iz, double v) {
                add_global(&Jg[comp * N + zk[iz] + yj[iy] + xi[ix]], v);
            };
            deposit3_o2<double>(dm, dp, jfac, S);
        }
    };
    auto in_rows = [&](auto form) {
        constexpr int want = decltype(form)::value == 0 ? kMvStill | kMvInside : kMvInside;
        for (int64_t cb = begin; cb < end; cb += ClassRows<NT, kO2Ub>::W) {
            __syncthreads();  // the region is clear; the last chunk's order is used up
            const int m = (int)min(end - cb, (int64_t)ClassRows<NT, kO2Ub>::W);
            const int n = order_rows(rows, m, [&](int sl) -> int {
                const int word = (int)spare.id[cb + sl];
                if (want & kMvStill) {
                    if (!(word & kMvInside)) n_out = 1;
                    else if (!(word & kMvStill)) n_cross = 1;
                }
                return (word & (kMvStill | kMvInside)) == want ? (word >> 8) & (kRowClasses - 1) : -1;
            });
            for (int q = threadIdx.x; q < n; q += NT) deposit(cb + rows.perm[q], form);
        }
        __syncthreads();
    };
    in_rows(std::integral_constant<int, 0>{});
    if (n_cross) in_rows(std::integral_constant<int, 1>{});
    if (n_out)
        for (int64_t p = begin + threadIdx.x; p < end; p += NT)
            if (!((int)spare.id[p] & kMvInside)) deposit(p, std::integral_constant<int, 2>{});
    const bool small = nx < LJ || ny < LJ || nz < LJ;
    const Columns<LJ, LJ, LJ> cols(g, T0[0] - 3 - M, T0[1] - 3 - M, small);
    flush_planes<3 * LJ, NT>(
        cols, [&](int t) { return sj + t * (LJ * LJ); },
        [&](int t) {
            const int comp = t / LJ;
            return Jg + comp * N + plane_offset(g, T0[2] - 3 - M + t - comp * LJ, small);
        });
}

// Current of given moves x0 -> x1 (positions in cell units, x1 not wrapped),
// one thread per move, global atomics.
template <int D>
__global__ __launch_bounds__(256) void k_deposit_pairs_o2(GridK g, const double* __restrict__ x0,
                                                          const double* __restrict__ x1,
                                                          const double* __restrict__ charge, int64_t n,
                                                          double* __restrict__ J)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    int i0[3] = {0, 0, 0}, s[3] = {0, 0, 0};
    double dm[3][5], dp[3][5];
    for (int ax = 0; ax < D; ++ax) {
        const double a0 = x0[ax * n + p], a1 = x1[ax * n + p];
        const double f0 = floor(a0), f1 = floor(a1);
        const Axis2<double> e0 = form_factor2<double>(a0 - f0);
        const Axis2<double> e1 = form_factor2<double>(a1 - f1);
        i0[ax] = (int)f0;
        const int shift = ((int)f1 + e1.h) - ((int)f0 + e0.h);
        window5_reg(e0.s, e1.s, shift, dm[ax], dp[ax]);
        s[ax] = e0.h + (shift < 0 ? shift : 0) - 2;
    }
    const double q = charge[p];
    double jfac[3];
    for (int ax = 0; ax < 3; ++ax) jfac[ax] = g.jscale[ax] * q;
    // 2D3V: J^z from the z displacement, (q/V) (z1 - z0) dz/dt / 4
    const double jz = D == 2 ? q * 0.25 * g.inv_vol * (x1[2 * n + p] - x0[2 * n + p]) / g.inv_h[2] / g.dt : 0.0;
    const int64_t N = g.ncell;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    auto S = [&](int comp, int ix, int iy, int iz, double v) {
        const int64_t cell = ((int64_t)(D == 3 ? wrapi(i0[2] + s[2] + iz, nz) : 0) * ny + wrapi(i0[1] + s[1] + iy, ny)) *
                                 nx +
                             wrapi(i0[0] + s[0] + ix, nx);
        add_global(&J[comp * N + cell], v);
    };
    if (D == 3) deposit3_o2<double>(dm, dp, jfac, S);
    else deposit2_o2<double>(dm, dp, jfac, jz, S);
}

// Charge density (Eq. rho) at order 2 1/2: cubic cell factors on 4 cells per
// axis, added into rho (charge per unit volume).  Positions x[ax][p], weights
// weight[p].
struct Rows3 {
    const double* x[3];
};

// The same for a cell-sorted species, `split` workgroups per tile: particles
// within M cells of their tile accumulate into an LDS density tile (cells T0-2-M ..
// T0+T+1+M), added to the grid once; the rest go straight to global memory.
// 64 global atomics per particle took 944 us of an energy sample at 64^3 x 2;
// the tile takes 40.  On few tiles one workgroup each was the slower form (13 x 14
// x 15 x 4, 8 tiles: an energy sample 94 us with global atomics, 138 with a
// workgroup per tile, 69 with shares of kRhoShare particles).
constexpr int kRhoShare = 64;

template <int D, int T, int M, int NT>
__global__ __launch_bounds__(NT) void k_rho_o2_tiled(GridK g, Rows3 pos, const double* __restrict__ weight,
                                                     const int64_t* __restrict__ ts, int split, double q,
                                                     double* __restrict__ rho)
{
    constexpr int L = T + 4 + 2 * M, LZ = D == 3 ? L : 1, NL = L * L * LZ;
    __shared__ double sr[NL];
    const int unit = xcd_tile(blockIdx.x, g.ntiles * split), tile = unit / split;
    const int T0[3] = {(tile % g.nt[0]) * T, ((tile / g.nt[0]) % g.nt[1]) * T,
                       D == 3 ? (tile / (g.nt[0] * g.nt[1])) * T : 0};
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    int64_t begin = ts[tile], end = ts[tile + 1];
    tile_share(unit - tile * split, split, begin, end);
    if (begin >= end) return;
    for (int e = threadIdx.x; e < NL; e += NT) sr[e] = 0.0;
    __syncthreads();
    for (int64_t p = begin + threadIdx.x; p < end; p += NT) {
        int i0[3] = {0, 0, 0}, rel[3] = {0, 0, 0};
        Axis2<double> w[3];
        bool inside = true;
        for (int ax = 0; ax < 3; ++ax) {
            double d = 0.0;
            if (ax < D) {
                const double x = pos.x[ax][p];
                const double f = floor(x);
                i0[ax] = (int)f;
                d = x - f;
                rel[ax] = tile_rel(i0[ax], T0[ax], g.n[ax], T, M);
                inside = inside && rel[ax] >= -M && rel[ax] <= T - 1 + M;
            }
            w[ax] = form_factor2<double>(d);
        }
        const double qv = q * weight[p] * g.inv_vol;
        // first point of the window in the LDS tile
        const int lb = rel[0] + w[0].h + M + L * (rel[1] + w[1].h + M + (D == 3 ? L * (rel[2] + w[2].h + M) : 0));
#pragma unroll
        for (int c = 0; c < (D == 3 ? 4 : 1); ++c) {
            const double wz = D == 3 ? w[2].s[c] : 1.0;
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const double v = qv * wz * w[1].s[b] * w[0].s[a];
                    if (inside) {
                        atomicAdd(&sr[lb + a + L * (b + L * c)], v);
                    } else {
                        const int64_t kz = D == 3 ? (int64_t)wrapi(i0[2] + w[2].h - 2 + c, nz) * ny : 0;
                        const int64_t jy = (kz + wrapi(i0[1] + w[1].h - 2 + b, ny)) * nx;
                        add_global(&rho[jy + wrapi(i0[0] + w[0].h - 2 + a, nx)], v);
                    }
                }
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NL; e += NT) {
        const double v = sr[e];
        if (v == 0.0) continue;
        const int lx = e % L, ly = (e / L) % L, lz = e / (L * L);
        const int gx = wrapi(T0[0] - 2 - M + lx, nx), gy = wrapi(T0[1] - 2 - M + ly, ny);
        const int gz = D == 3 ? wrapi(T0[2] - 2 - M + lz, nz) : 0;
        add_global(&rho[((int64_t)gz * ny + gy) * nx + gx], v);
    }
}

template <int D>
__global__ __launch_bounds__(256) void k_rho_o2(GridK g, Rows3 pos, const double* __restrict__ weight, int64_t n,
                                                double q, double* __restrict__ rho)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    int i0[3] = {0, 0, 0};
    Axis2<double> w[3];
    for (int ax = 0; ax < 3; ++ax) {
        double d = 0.0;
        if (ax < D) {
            const double x = pos.x[ax][p];
            const double f = floor(x);
            i0[ax] = (int)f;
            d = x - f;
        }
        w[ax] = form_factor2<double>(d);
    }
    const double qv = q * weight[p] * g.inv_vol;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    for (int c = 0; c < (D == 3 ? 4 : 1); ++c) {
        const double wz = D == 3 ? w[2].s[c] : 1.0;
        const int64_t kz = D == 3 ? (int64_t)wrapi(i0[2] + w[2].h - 2 + c, nz) * ny : 0;
        for (int b = 0; b < 4; ++b) {
            const int64_t jy = (kz + wrapi(i0[1] + w[1].h - 2 + b, ny)) * nx;
            for (int a = 0; a < 4; ++a)
                add_global(&rho[jy + wrapi(i0[0] + w[0].h - 2 + a, nx)], qv * wz * w[1].s[b] * w[0].s[a]);
        }
    }
}

unsigned blocks256(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_particle_step_o2(Ctx& c, Species& sp, hipStream_t s)
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
        const int split = tile_split(c.k.ntiles, sp.n, kO2Fixed);
        const dim3 grid((unsigned)(c.k.ntiles * split));
        hipLaunchKernelGGL(k_push_o2_3d, grid, dim3(kO2NTa), 0, s, c.k, a, sp.alt, c.fields, c.bn, split);
        if (sp.n / c.k.ntiles / split >= kO2Full)
            hipLaunchKernelGGL(k_deposit_o2_3d<kO2NTbFull>, grid, dim3(kO2NTbFull), 0, s, c.k, a, sp.alt, J, split);
        else
            hipLaunchKernelGGL(k_deposit_o2_3d<kO2NTb>, grid, dim3(kO2NTb), 0, s, c.k, a, sp.alt, J, split);
    } else
        hipLaunchKernelGGL(k_step_o2<2>, dim3(c.k.ntiles), dim3(kO2NT2), 0, s, c.k, a, c.fields, c.bn, J);
    return hipGetLastError();
}

hipError_t launch_deposit_only_o2(const Ctx& c, const double* x0, const double* x1, const double* charge,
                                  int64_t n, double* J, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    if (c.k.dims == 3)
        hipLaunchKernelGGL(k_deposit_pairs_o2<3>, dim3(blocks256(n)), dim3(256), 0, s, c.k, x0, x1, charge, n, J);
    else
        hipLaunchKernelGGL(k_deposit_pairs_o2<2>, dim3(blocks256(n)), dim3(256), 0, s, c.k, x0, x1, charge, n, J);
    return hipGetLastError();
}

hipError_t launch_rho_o2(const Ctx& c, const double* const x[3], const double* weight, int64_t n, double q,
                         double* rho, hipStream_t s, const int64_t* tile_start)
{
    if (n == 0) return hipSuccess;
    Rows3 pos{{x[0], x[1], x[2]}};
    // shares of kRhoShare particles, up to two workgroups per CU in all
    const int64_t avg = n / c.k.ntiles;
    const int split = (int)std::max<int64_t>(1, std::min(2 * kCus / c.k.ntiles, (int)(avg / kRhoShare)));
    const dim3 grid((unsigned)(c.k.ntiles * split));
    if (tile_start && c.k.dims == 3)
        hipLaunchKernelGGL((k_rho_o2_tiled<3, kTile3, 2, 256>), grid, dim3(256), 0, s, c.k, pos, weight, tile_start,
                           split, q, rho);
    else if (tile_start)
        hipLaunchKernelGGL((k_rho_o2_tiled<2, kTile2, 2, 256>), grid, dim3(256), 0, s, c.k, pos, weight, tile_start,
                           split, q, rho);
    else if (c.k.dims == 3)
        hipLaunchKernelGGL(k_rho_o2<3>, dim3(blocks256(n)), dim3(256), 0, s, c.k, pos, weight, n, q, rho);
    else
        hipLaunchKernelGGL(k_rho_o2<2>, dim3(blocks256(n)), dim3(256), 0, s, c.k, pos, weight, n, q, rho);
    return hipGetLastError();
}

}  // namespace pic
