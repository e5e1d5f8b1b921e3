// tile_io.h -- moves between the grid and a tile's LDS regions in 3D, and the
// order in which a workgroup takes a tile's particles so that their LDS
// accesses do not conflict.
#pragma once

#include "pic_math.h"

namespace pic {
namespace {

// The x, y columns of a tile region, dealt to the lanes of every wave: the
// lane's c-th column is at grid offset off[c] within a z plane and at lds[c]
// within a plane of the region (off < 0: no such column).  Packed, or
// (ALIGNED, rows of up to 16 columns) with 16 lanes to a row, so that no row is
// split over two accesses.  A region's planes then go
// wave by wave with a scalar base address each, so that an element costs its
// load and its store and no index arithmetic (decoding and wrapping every
// element took 6 of the 12 us in which a tile of 14^3 cells x 6 was staged).
template <int LX, int LY, int ROW, bool ALIGNED = false>
struct Columns {
    static_assert(!ALIGNED || LX <= 16, "a row fits 16 lanes");
    static constexpr int LANES = ALIGNED ? 16 : LX;  // lanes of a row
    static constexpr int CH = (LANES * LY + 63) / 64;
    int off[CH], lds[CH];
    __device__ __forceinline__ Columns(const GridK& g, int fx, int fy, bool small, int tid = (int)threadIdx.x)
    {
        auto wr = [&](int v, int n) { return small ? wrapi(v, n) : wrap1(v, n); };
        const int lane = tid & 63;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int e = lane + 64 * c, ly = e / LANES, lx = e - ly * LANES;
            lds[c] = lx + ly * ROW;
            off[c] = lx < LX && ly < LY ? wr(fy + ly, g.n[1]) * g.n[0] + wr(fx + lx, g.n[0]) : -1;
        }
    }
};

__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

// Grid offset of z plane gz (in [-n, 2n), or anywhere if the axis is short).
__device__ __forceinline__ int64_t plane_offset(const GridK& g, int gz, bool small)
{
    return (int64_t)(small ? wrapi(gz, g.n[2]) : wrap1(gz, g.n[2])) * g.n[1] * g.n[0];
}

// Planes of a wave when NT threads move NP of them.
template <int NP, int NT>
constexpr int kAllPlanes = (NP * 64 + NT - 1) / NT;

// Planes 0 .. NP - 1 of a region into LDS by all NT threads: src(t) is plane
// t's grid plane, dst(t) its place in LDS.  SK planes' loads of a wave are in
// flight before their values are stored: all of them (kAllPlanes) where the
// registers are free, since the fields, new in every step, come from beyond
// the L2.  The conventional push (78 planes of 13^2, 8 waves) in one batch
// against five: 70 -> 62 us for two rounds of tiles.
template <int NP, int NT, int SK, class R, class Cols, class Src, class Dst>
__device__ __forceinline__ void stage_planes(const Cols& cols, Src src, Dst dst)
{
    constexpr int NW = NT / 64, CH = Cols::CH;
    for (int t0 = wave_index(); t0 < NP; t0 += NW * SK) {
        double v[SK][CH];
#pragma unroll
        for (int k = 0; k < SK; ++k) {
            const int t = t0 + k * NW;
            if (t < NP) {
                const double* s = src(t);
#pragma unroll
                for (int c = 0; c < CH; ++c)
                    if (cols.off[c] >= 0) v[k][c] = s[cols.off[c]];
            }
        }
#pragma unroll
        for (int k = 0; k < SK; ++k) {
            const int t = t0 + k * NW;
            if (t < NP) {
                R* o = dst(t);
#pragma unroll
                for (int c = 0; c < CH; ++c)
                    if (cols.off[c] >= 0) o[cols.lds[c]] = (R)v[k][c];
            }
        }
    }
}

// Adds the non-zero entries of planes 0 .. NP - 1 of an LDS region, src(t), to
// the grid planes dst(t) with global atomics, by all NT threads; CLEAR: and
// clears them.
template <int NP, int NT, bool CLEAR = false, class Cols, class Src, class Dst>
__device__ __forceinline__ void flush_planes(const Cols& cols, Src src, Dst dst)
{
    for (int t = wave_index(); t < NP; t += NT / 64) {
        double* s = src(t);
        double* o = dst(t);
#pragma unroll
        for (int c = 0; c < Cols::CH; ++c)
            if (cols.off[c] >= 0) {
                const double v = s[cols.lds[c]];
                if (v != 0.0) {
                    unsafeAtomicAdd(o + cols.off[c], v);
                    if (CLEAR) s[cols.lds[c]] = 0.0;
                }
            }
    }
}

// The 3D field tile (Tile3): E^n and B^n on the tile plus its margins and the
// stencil, in stored planes.  The components that are node-centred in z (E^z,
// B^x, B^y) never read the first plane and store planes 1..11 only.
__host__ __device__ constexpr int fplane0(int comp)  // first stored plane of a field component
{
    return comp < 2 ? 12 * comp : (comp < 5 ? 24 + 11 * (comp - 2) : 57);
}
__host__ __device__ constexpr int fnodez(int comp) { return comp >= 2 && comp <= 4 ? 1 : 0; }
constexpr int kFieldPlanes3 = 69;  // 12 + 12 + 11 + 11 + 11 + 12

// Stored plane t of the field tile: its component, and its z position.
__device__ __forceinline__ int field_plane3(int t, int& lz)
{
    const int comp = t < 12 ? 0 : (t < 24 ? 1 : (t < 35 ? 2 : (t < 46 ? 3 : (t < 57 ? 4 : 5))));
    lz = t - fplane0(comp) + fnodez(comp);
    return comp;
}

// ---------------------------------------------------------------------------
// Class rows of a workgroup: an order of up to NT * U particles in which any C
// consecutive ones are of distinct lane classes as far as the class counts
// allow.  A particle's class is its LDS base index modulo C (16 lanes of 8-byte
// values per LDS pass, 32 of 4-byte ones): the same stencil offset of distinct
// classes lies in distinct banks, and without this order a pass over random
// cells takes about three times as long.  Row r holds the rank-r particle of every
// class that has one; ranks follow the storage order (a wave owns a contiguous
// block and a prefix over the waves orders the blocks), so a row's particles
// are also near each other in memory.
// ---------------------------------------------------------------------------
constexpr int kRowClasses = 16;

// Whether every z layer of a 3D tile's cells, kept in rows of `row`, holds each
// class as often.
constexpr bool even_layers(int row)
{
    int n[kRowClasses] = {};
    for (int c = 0; c < kTile3 * kTile3; ++c) ++n[(c % kTile3 + c / kTile3 * row) % kRowClasses];
    for (int k = 0; k < kRowClasses; ++k)
        if (n[k] != kTile3 * kTile3 / kRowClasses) return false;
    return true;
}

template <int NT, int U, int C = kRowClasses>
struct ClassRows {
    static constexpr int W = NT * U, NW = NT / 64;
    unsigned cnt[NW][C];  // per wave: particles of each class; then their first rank
    unsigned tot[C];
    uint16_t perm[W];               // position -> slot
};

// Orders the slots 0 .. m - 1 (m <= W): cls(slot) is the slot's class, or -1
// to leave it out.  Returns the number of slots placed; perm is valid until
// the next call.  Called by the whole workgroup; the caller puts a barrier
// between the last use of perm and the next call.
template <int NT, int U, int C, class Cls>
__device__ __forceinline__ int order_rows(ClassRows<NT, U, C>& s, int m, Cls cls)
{
    static_assert(ClassRows<NT, U, C>::W <= 65536 && C <= 64, "16-bit slots, a lane per class");
    const int t = threadIdx.x, wv = t >> 6, lane = t & 63;
    if (lane < C) s.cnt[wv][lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    int cl[U];
    unsigned rk[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int sl = (wv * U + u) * 64 + lane;
        cl[u] = sl < m ? cls(sl) : -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (cl[u] >= 0) rk[u] = atomicAdd(&s.cnt[wv][cl[u]], 1u);
    __syncthreads();
    if (t < C) {
        unsigned run = 0;
        for (int w = 0; w < NT / 64; ++w) {
            const unsigned x = s.cnt[w][t];
            s.cnt[w][t] = run;
            run += x;
        }
        s.tot[t] = run;
    }
    __syncthreads();
    unsigned tot[C], all = 0;
#pragma unroll
    for (int k = 0; k < C; ++k) {
        tot[k] = s.tot[k];
        all += tot[k];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (cl[u] >= 0) {
            // the rows before this one, then the smaller classes of this row
            const unsigned r = rk[u] + s.cnt[wv][cl[u]];
            unsigned pos = 0;
#pragma unroll
            for (int k = 0; k < C; ++k) pos += min(tot[k], r + (k < cl[u] ? 1u : 0u));
            s.perm[pos] = (uint16_t)((wv * U + u) * 64 + lane);
        }
    __syncthreads();
    return (int)all;
}

// This workgroup's share [begin, end) of a tile's slots, one of `split` equal
// shares in multiples of 64.
__device__ __forceinline__ void tile_share(int part, int split, int64_t& begin, int64_t& end)
{
    if (split == 1) return;
    const int64_t len = ((end - begin + split - 1) / split + 63) / 64 * 64;
    begin += part * len;
    end = min(begin + len, end);
}

}  // namespace
}  // namespace pic
