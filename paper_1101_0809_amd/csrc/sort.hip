// sort.hip -- periodic counting sort of a species by cell, in tile-major cell
// order, so that the particles of one tile (the unit of work of the particle
// kernel) are contiguous.  Inside a tile the order serves the particle
// kernel's LDS banks:
//   3D: the cells are grouped by lane class (see cell_class3) and slot s of
//       the tile's range holds a particle of class s mod C wherever the class
//       counts allow (round g of the tile = one particle of each class); the
//       particles left over by the fuller classes fill the empty places;
//   2D: rank-interleaved -- the particle of rank 0 of every cell, then those
//       of rank 1, and so on, so that consecutive lanes work in distinct cells.
// Histogram with atomics (the returned slot is the particle's rank in its
// cell), the tiles' sums, a per-tile pass turning the counts into offsets and
// those into final slots, the inverse map (which particle fills each slot), and
// one gather of the particle arrays into the spare copy, which becomes
// current.  Not part of the paper's method; it only fixes
// the memory order.
#include "pic_internal.h"

namespace pic {
namespace {

constexpr int kSortThreads = 256;

__device__ __forceinline__ void unpack(uint32_t c, int i[3])
{
    i[0] = (int)(c & 2047u);
    i[1] = (int)((c >> 11) & 2047u);
    i[2] = (int)(c >> 22);
}

// Tile-local keys of the T^3 cells of a 3D tile (T = kTile3), x fastest:
// class-major, class k owning keys k * T^3 / C .. (k + 1) * T^3 / C - 1, a
// class's cells in (lz, ly) order.  Each row (ly, lz) holds at most one cell of
// a class (T < C consecutive x offsets).  A table in constant memory: a tile's
// workgroup that counted the rows itself took 5 of the 29 us of a 64^3 x 8
// histogram.
template <class R>
struct ClassMajor {
    static constexpr int T = kTile3, C = lane_classes<R>();
    static_assert(T < C && (T * T * T) % C == 0, "one cell of a class per row, equal classes");
    uint16_t key[T * T * T];
    constexpr ClassMajor() : key()
    {
        int next[C] = {};
        for (int c = 0; c < T * T * T; ++c) {
            const int cls = cell_class3<R>(c % T, c / T % T, c / (T * T));
            key[c] = (uint16_t)(cls * (T * T * T / C) + next[cls]++);
        }
    }
};
template <class R>
__constant__ const ClassMajor<R> kClassMajor{};

// Sort key of particle p.  lut (3D): the class-major keys.
template <class R, int D, int T>
__device__ __forceinline__ uint32_t key_of(const GridK& g, const PartArrays& a, int64_t p,
                                           const uint16_t* lut)
{
    int i[3] = {0, 0, 0};
    if (sizeof(R) == 4) {
        unpack(a.cell[p], i);
    } else {
        for (int ax = 0; ax < D; ++ax) i[ax] = (int)floor(((const double*)a.pos[ax])[p]);
    }
    for (int ax = 0; ax < 3; ++ax)  // positions are in [0, N); clamp so keys stay in range
        i[ax] = i[ax] < 0 ? 0 : (i[ax] >= g.n[ax] ? g.n[ax] - 1 : i[ax]);
    const int tx = i[0] / T, ty = i[1] / T, tz = D == 3 ? i[2] / T : 0;
    const uint32_t tile = ((uint32_t)tz * g.nt[1] + ty) * g.nt[0] + tx;
    const uint32_t lx = i[0] - tx * T, ly = i[1] - ty * T, lz = D == 3 ? i[2] - tz * T : 0;
    uint32_t local = ly * T + lx;
    if (D == 3) local = lut[(lz * T + ly) * T + lx];
    return tile * (uint32_t)(D == 3 ? T * T * T : T * T) + local;
}

__global__ void k_zero_u32(uint32_t* p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kSortThreads + threadIdx.x;
    if (i < n) p[i] = 0;
}

template <class R, int D, int T>
__global__ __launch_bounds__(kSortThreads) void k_histogram(GridK g, PartArrays a, int64_t n,
                                                            uint32_t* __restrict__ key,
                                                            uint32_t* __restrict__ rank,
                                                            uint32_t* __restrict__ hist)
{
    const int64_t p = (int64_t)blockIdx.x * kSortThreads + threadIdx.x;
    if (p >= n) return;
    const uint32_t k = key_of<R, D, T>(g, a, p, D == 3 ? kClassMajor<R>.key : nullptr);
    key[p] = k;
    rank[p] = atomicAdd(&hist[k], 1u);
}

// Histogram of a species that is still grouped by the tiles of its previous
// sort (particles move at most one cell per step): one workgroup per old tile
// range.  Each of its waves takes a contiguous block of the range and counts
// the particles still in that tile per cell in its own LDS counters (a
// wave's atomics rank its lanes in lane order, so the ranks follow the
// storage order), a prefix over the waves orders the blocks, and each cell's
// rank range in the global histogram is reserved with one atomic.  The ranks
// of a cell's particles therefore keep their old order: a particle that did
// not move keeps its place, and the final gather stays a near copy.  A
// particle now in another tile takes its rank from a global atomic directly.
// Ranks stay unique per cell.  A lane keeps the cells and ranks of up to H
// particles in registers until the prefix is known; of a fuller tile they go
// through memory, which takes twice the bytes.  Bound by those: 216 -> 132 us
// for 16.8 million particles in half of 128^3 (a tile without particles leaves
// at once), 29 -> 24 us for 64^3 x 8.  Rounds past a wave's block are left out (of a
// tile of 256 particles they cost a fifth), and 64 VGPRs keep two workgroups to a
// CU: a sort of 2^26 particles on 8192^2 cells 5.25 -> 4.62 ms, on 1024 x 512 x 1024
// 17.7 -> 15.5.
constexpr uint32_t kLocalRank = 1u << 31;

template <class R, int D, int T>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8)))
void k_histogram_tiled(GridK g, PartArrays a, const int64_t* __restrict__ ts, uint32_t* __restrict__ key,
                       uint32_t* __restrict__ rank, uint32_t* __restrict__ hist)
{
    constexpr int TPD = D == 3 ? T * T * T : T * T;
    constexpr int NTH = 1024, NW = NTH / 64, U = 8;  // threads, waves, slots of a lane in flight
    constexpr int H = 32, kGone = -1;                // slots a lane can hold; one that left the tile
    __shared__ uint32_t cnt[NW][TPD];                // per wave, then per wave's first rank
    __shared__ uint16_t lut[D == 3 ? TPD : 1];       // the class-major keys
    const int t = blockIdx.x;
    const int wv = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    const int64_t b = ts[t], e = ts[t + 1];
    if (b >= e) return;
    const uint32_t k0 = (uint32_t)t * TPD;
    for (int c = threadIdx.x; c < NW * TPD; c += NTH) (&cnt[0][0])[c] = 0;
    for (int c = threadIdx.x; c < TPD; c += NTH)
        if (D == 3) lut[c] = kClassMajor<R>.key[c];
    __syncthreads();
    // wave w: slots [b + w L, b + (w + 1) L)
    const int64_t L = (e - b + NW - 1) / NW;
    const int64_t wb = b + wv * L, we = min(e, wb + L);
    const bool held = L <= H * 64;
    int32_t hold[H];  // cell | rank << 9
    auto count = [&](int64_t p0, int32_t* out) {  // slots p0, p0 + 64, ...
        uint32_t k[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (p0 + u * 64 < we) k[u] = key_of<R, D, T>(g, a, p0 + u * 64, lut);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = p0 + u * 64;
            if (p >= we) continue;
            const uint32_t kl = k[u] - k0;
            const bool stays = kl < (uint32_t)TPD;
            const uint32_t r = stays ? atomicAdd(&cnt[wv][kl], 1u) : atomicAdd(&hist[k[u]], 1u);
            key[p] = k[u];
            if (out) out[u] = stays ? (int32_t)(kl | r << 9) : kGone;
            if (!out || !stays) rank[p] = stays ? kLocalRank | r : r;
        }
    };
    if (held) {
#pragma unroll
        for (int h = 0; h < H / U; ++h)
            if (wb + h * U * 64 < we) count(wb + lane + h * U * 64, hold + h * U);
    } else {
        for (int64_t p0 = wb + lane; p0 < we; p0 += U * 64) count(p0, nullptr);
    }
    __syncthreads();
    // per cell: the waves' first ranks, then the reservation of the whole range
    for (int c = threadIdx.x; c < TPD; c += NTH) {
        uint32_t run = 0;
        for (int w = 0; w < NW; ++w) {
            const uint32_t m = cnt[w][c];
            cnt[w][c] = run;
            run += m;
        }
        const uint32_t base = run ? atomicAdd(&hist[k0 + c], run) : 0u;
        for (int w = 0; w < NW; ++w) cnt[w][c] += base;
    }
    __syncthreads();
    if (held) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            if (h % U == 0 && wb + h * 64 >= we) return;
            const int64_t p = wb + lane + h * 64;
            if (p < we && hold[h] != kGone) rank[p] = cnt[wv][hold[h] & (TPD - 1)] + ((uint32_t)hold[h] >> 9);
        }
        return;
    }
    for (int64_t p = wb + lane; p < we; p += 64) {
        const uint32_t rp = rank[p];
        if (rp & kLocalRank) rank[p] = cnt[wv][key[p] - k0] + (rp & ~kLocalRank);
    }
}

// Particles per tile, a wave to a tile, and per group of kTileGroup tiles (a
// workgroup): tsum[t] = particles of the group's tiles before t, gsum[group].
constexpr int kTileGroup = 16;

template <int TPD>
__global__ __launch_bounds__(64 * kTileGroup) void k_tile_sums(const uint32_t* __restrict__ cnt, int ntiles,
                                                               uint32_t* __restrict__ tsum,
                                                               uint32_t* __restrict__ gsum)
{
    __shared__ uint32_t sum[kTileGroup];
    const int wv = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    const int t = (int)blockIdx.x * kTileGroup + wv;
    uint32_t v = 0;
    if (t < ntiles)
        for (int c = lane; c < TPD; c += 64) v += cnt[(int64_t)t * TPD + c];
    for (int off = 32; off > 0; off >>= 1) v += (uint32_t)__shfl_xor((int)v, off, 64);
    if (lane == 0) sum[wv] = v;
    __syncthreads();
    if ((int)threadIdx.x < kTileGroup) {
        uint32_t run = 0;
        for (int w = 0; w < (int)threadIdx.x; ++w) run += sum[w];
        const int tt = (int)blockIdx.x * kTileGroup + (int)threadIdx.x;
        if (tt < ntiles) tsum[tt] = run;
        if ((int)threadIdx.x == kTileGroup - 1) gsum[blockIdx.x] = run + sum[kTileGroup - 1];
    }
}

// From kScanGroups groups on, one workgroup turns gsum into the particles before
// each group: added up by every tile they cost reads as the square of the tiles.
// A sort of 2^26 particles on 8192^2 cells (16384 groups): 5.69 ms with the tiles
// adding, 5.25 like this; on 1024 x 512 x 1024 (65536) 25.7 and 17.7; of 2^22 on
// 2048^2 (1024) 0.336 and 0.337.
constexpr int kScanGroups = 1024;

__global__ __launch_bounds__(1024) void k_group_scan(uint32_t* __restrict__ gsum, int groups)
{
    constexpr int NW = 16, U = 4;
    __shared__ uint32_t wsum[NW];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    uint32_t carry = 0;
    for (int g0 = t * U; g0 - t * U < groups; g0 += 1024 * U) {
        uint32_t v[U], sum = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u] = g0 + u < groups ? gsum[g0 + u] : 0u;
            sum += v[u];
        }
        uint32_t incl = sum;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t x = (uint32_t)__shfl_up((int)incl, off, 64);
            if (lane >= off) incl += x;
        }
        if (lane == 63) wsum[wv] = incl;
        __syncthreads();
        uint32_t run = carry + incl - sum;
        for (int w = 0; w < NW; ++w) {
            run += w < wv ? wsum[w] : 0u;
            carry += wsum[w];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (g0 + u < groups) gsum[g0 + u] = run;
            run += v[u];
        }
        __syncthreads();
    }
}

// The exclusive scan of the counts of tile t's TPD cells, one per thread of its
// workgroup: replaces the thread's count in offs by its cell's first
// cell-sorted position, which is returned; start: the tile's, cnt: the count,
// nt: the tile's particles.  Every workgroup adds up the groups before its own
// (unless they are scanned, see above): that saves two launches and a pass over
// the keys.  With it and one gather in place of 8 a sort has 6 launches in place
// of 14: 175 -> 145 us for 64^3 x 8, 75 -> 45 us for 290,000 particles.
template <int TPD>
__device__ __forceinline__ uint32_t tile_offsets(uint32_t* __restrict__ offs, const uint32_t* __restrict__ tsum,
                                                 const uint32_t* __restrict__ gsum, bool scanned, int t,
                                                 uint32_t& start, uint32_t& cnt, uint32_t& nt)
{
    constexpr int NW = TPD / 64;
    __shared__ uint32_t before[NW], own[NW];
    const int c = threadIdx.x, lane = c & 63, wv = c >> 6;
    cnt = offs[(int64_t)t * TPD + c];
    uint32_t pre = 0;
    if (scanned) pre = c == 0 ? gsum[t / kTileGroup] : 0u;
    else
        for (int q = c; q < t / kTileGroup; q += TPD) pre += gsum[q];
    for (int off = 32; off > 0; off >>= 1) pre += (uint32_t)__shfl_xor((int)pre, off, 64);
    uint32_t incl = cnt;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t x = (uint32_t)__shfl_up((int)incl, off, 64);
        if (lane >= off) incl += x;
    }
    if (lane == 0) before[wv] = pre;
    if (lane == 63) own[wv] = incl;
    __syncthreads();
    start = tsum[t];
    nt = 0;
    uint32_t waves = 0;
    for (int w = 0; w < NW; ++w) {
        start += before[w];
        waves += w < wv ? own[w] : 0u;
        nt += own[w];
    }
    const uint32_t cb = start + waves + incl - cnt;
    offs[(int64_t)t * TPD + c] = cb;
    return cb;
}

// Final slot of every particle of one tile in the rank-interleaved order,
// written per cell-sorted position: dest[cb + r] for the particle of rank r of
// the cell starting at cb.  Rank level r holds the cells with more than r
// particles, in the tile's cell order, contiguously after level r - 1.  One workgroup per
// tile, one thread per cell; only 4-byte writes.
template <int TPD>
__global__ __launch_bounds__(TPD) void k_dest(uint32_t* __restrict__ offs, const uint32_t* __restrict__ tsum,
                                              const uint32_t* __restrict__ gsum, bool scanned, int64_t n,
                                              uint32_t* __restrict__ dest, int64_t* __restrict__ ts)
{
    constexpr int NW = TPD / 64;
    __shared__ uint32_t wsum[NW];
    __shared__ uint32_t wmax[NW];
    const int c = threadIdx.x;
    const int lane = c & 63, wv = c >> 6;
    uint32_t base, cnt, nt;
    const int64_t cb = tile_offsets<TPD>(offs, tsum, gsum, scanned, blockIdx.x, base, cnt, nt);
    if (c == 0) ts[blockIdx.x] = base;  // the tile table of the new order
    if (c == 0 && blockIdx.x == gridDim.x - 1) ts[gridDim.x] = n;
    uint32_t m = cnt;
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
    if (lane == 0) wmax[wv] = m;
    __syncthreads();
    uint32_t maxcnt = 0;
    for (int w = 0; w < NW; ++w) maxcnt = max(maxcnt, wmax[w]);
    int64_t level_base = base;
    for (uint32_t r = 0; r < maxcnt; ++r) {
        const bool flag = cnt > r;
        const unsigned long long mask = __ballot(flag);
        const uint32_t below = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
        if (lane == 0) wsum[wv] = (uint32_t)__popcll(mask);
        __syncthreads();
        uint32_t pre = 0, tot = 0;
        for (int w = 0; w < NW; ++w) {
            pre += w < wv ? wsum[w] : 0u;
            tot += wsum[w];
        }
        if (flag) dest[cb + r] = (uint32_t)(level_base + pre + below);
        level_base += tot;
        __syncthreads();
    }
}

// 3D: the class-round order.  With n_t particles in the tile, slot s belongs to
// column s mod C, row s / C; column k has rows_k = ceil((n_t - k) / C) rows.
// The particle of class k and index g within its class (cells of the class in
// key order, then rank) takes row g of column k if g < rows_k; the others
// (classes with more particles than rows), in (class, g) order, fill the empty
// rows of the poorer columns in (column, row) order.  The two counts agree:
// both classes and columns sum to n_t.  This kernel turns the counts into
// offsets and writes the slots of those others, per cell-sorted position as in
// k_dest; k_final_src finds the slot of a particle within its rows by itself
// (its class is its key's).  With all slots written here, 4 bytes at the cells'
// strides, the pass took 109 us for 16.8 million particles (now 72) and 15 for
// 2.1 million (now 10).
template <int C>
__global__ __launch_bounds__(kTile3 * kTile3 * kTile3) void k_dest3(uint32_t* __restrict__ offs,
                                                                     const uint32_t* __restrict__ tsum,
                                                                     const uint32_t* __restrict__ gsum,
                                                                     bool scanned, int64_t n,
                                                                     uint32_t* __restrict__ dest,
                                                                     int64_t* __restrict__ ts)
{
    constexpr int TPD = kTile3 * kTile3 * kTile3;
    constexpr int CPC = TPD / C;  // cells per class
    __shared__ uint32_t ccnt[C], cbase[C], rows[C], hpre[C + 1], lpre[C + 1];
    const int c = threadIdx.x;
    uint32_t tb, cnt, nt;
    const uint32_t cb = tile_offsets<TPD>(offs, tsum, gsum, scanned, blockIdx.x, tb, cnt, nt);
    if (c == 0) ts[blockIdx.x] = tb;  // the tile table of the new order
    if (c == 0 && blockIdx.x == gridDim.x - 1) ts[gridDim.x] = n;
    if (nt == 0) return;
    if (c % CPC == 0) cbase[c / CPC] = cb - tb;
    __syncthreads();
    if (c < C) {
        ccnt[c] = (c + 1 < C ? cbase[c + 1] : nt) - cbase[c];
        rows[c] = nt > (uint32_t)c ? (nt - c + C - 1) / C : 0u;
    }
    __syncthreads();
    if (c == 0) {
        hpre[0] = 0;
        lpre[0] = 0;
        for (int k = 0; k < C; ++k) {
            hpre[k + 1] = hpre[k] + (rows[k] > ccnt[k] ? rows[k] - ccnt[k] : 0u);
            lpre[k + 1] = lpre[k] + (ccnt[k] > rows[k] ? ccnt[k] - rows[k] : 0u);
        }
    }
    __syncthreads();
    const int cls = c / CPC;
    const uint32_t g0 = cb - tb - cbase[cls];
    for (uint32_t r = g0 < rows[cls] ? rows[cls] - g0 : 0u; r < cnt; ++r) {
        const uint32_t k = lpre[cls] + (g0 + r - rows[cls]);
        int lam = 0;
        while (lam < C - 1 && hpre[lam + 1] <= k) ++lam;
        dest[(int64_t)cb + r] = tb + (ccnt[lam] + (k - hpre[lam])) * C + lam;
    }
}

// This workgroup's place in a run of consecutive blocks per XCD: workgroup
// ids are dealt round-robin to the 8 XCDs, so XCD x takes blocks
// [x * per, (x + 1) * per) (one more for the first nb % 8 XCDs), and the
// blocks an XCD runs at a time touch neighbouring memory.
__device__ __forceinline__ int xcd_block()
{
    const int nb = gridDim.x;
    const int per = nb / kXcds, rem = nb % kXcds;
    const int x = blockIdx.x % kXcds, local = blockIdx.x / kXcds;
    return x < rem ? x * (per + 1) + local : rem * (per + 1) + (x - rem) * per + local;
}

// Which particle fills each final slot: the inverse of the final-slot map, by
// one 4-byte scatter, so that the move writes every slot once, in order.
// Each XCD takes a contiguous run of particles: a tile's particles scatter
// into the same few tile ranges of src, whose lines are then written whole
// in one XCD's L2 rather than in pieces by all of them.
// CPC: cells per class of a 3D tile (0 in 2D, where dest holds every slot), C
// classes; the tile table ts is that of the new order.
template <int C, int CPC>
__global__ __launch_bounds__(kSortThreads) void k_final_src(int64_t n, const uint32_t* __restrict__ key,
                                                            const uint32_t* __restrict__ rank,
                                                            const uint32_t* __restrict__ offs,
                                                            const uint32_t* __restrict__ dest,
                                                            const int64_t* __restrict__ ts,
                                                            uint32_t* __restrict__ src)
{
    const int blk = xcd_block();
    const int64_t p = (int64_t)blk * kSortThreads + threadIdx.x;
    if (p >= n) return;
    const uint32_t k = key[p], pos = offs[k] + rank[p];
    if (CPC > 0) {
        const uint32_t tile = k / (C * CPC), cls = k / CPC % C;
        const uint32_t tb = (uint32_t)ts[tile], nt = (uint32_t)ts[tile + 1] - tb;
        const uint32_t gi = pos - offs[k - k % CPC];
        const uint32_t rows = nt > cls ? (nt - cls + C - 1) / C : 0u;
        if (gi < rows) {
            src[tb + gi * C + cls] = (uint32_t)p;
            return;
        }
    }
    src[dest[pos]] = (uint32_t)p;
}

// Move the particle arrays: slot q of the spare copy takes particle src[q].
// Writes are coalesced; reads are local, since a particle's new slot is
// mostly in or near the tile range it came from.  Each XCD takes a
// contiguous run of slots, so a tile's reads gather in one XCD's L2.  The
// arrays are rows of the grid (0..2 positions, 3..5 momenta, 6 weight, 7 id,
// 8 the FP32 cell), so that one is moved after the other: the source lines that
// the tiles in flight on an XCD touch then fit its L2, where all arrays at once
// would not.  (A launch per array ran dry between them: 8 of 4 to 12 us for up
// to 2 million particles.)  gridDim.x is a multiple of the XCDs, which makes a
// block's XCD the same in every row.  A thread moves kGatherU particles, all
// their loads in flight before the stores.
constexpr int kGatherU = 4;

template <class V>
__device__ __forceinline__ void gather_array(const void* from, void* to, int64_t q0, int64_t n,
                                             const uint32_t* __restrict__ src)
{
    const V* __restrict__ in = (const V*)from;
    V* __restrict__ out = (V*)to;
    int64_t p[kGatherU];
#pragma unroll
    for (int u = 0; u < kGatherU; ++u) {
        const int64_t q = q0 + u * kSortThreads;
        p[u] = q < n ? (int64_t)src[q] : -1;
    }
    V v[kGatherU];
#pragma unroll
    for (int u = 0; u < kGatherU; ++u)
        if (p[u] >= 0) v[u] = in[p[u]];
#pragma unroll
    for (int u = 0; u < kGatherU; ++u)
        if (p[u] >= 0) out[q0 + u * kSortThreads] = v[u];
}

template <class R>
__global__ __launch_bounds__(kSortThreads) void k_gather_final(PartArrays from, PartArrays to, int64_t n,
                                                               const uint32_t* __restrict__ src)
{
    const int64_t q0 = (int64_t)xcd_block() * kSortThreads * kGatherU + threadIdx.x;
    switch (blockIdx.y) {
        case 0: return gather_array<R>(from.pos[0], to.pos[0], q0, n, src);
        case 1: return gather_array<R>(from.pos[1], to.pos[1], q0, n, src);
        case 2: return gather_array<R>(from.pos[2], to.pos[2], q0, n, src);
        case 3: return gather_array<R>(from.mom[0], to.mom[0], q0, n, src);
        case 4: return gather_array<R>(from.mom[1], to.mom[1], q0, n, src);
        case 5: return gather_array<R>(from.mom[2], to.mom[2], q0, n, src);
        case 6: return gather_array<R>(from.weight, to.weight, q0, n, src);
        case 7: return gather_array<int64_t>(from.id, to.id, q0, n, src);
        default: return gather_array<uint32_t>(from.cell, to.cell, q0, n, src);
    }
}

unsigned nblk(int64_t n) { return (unsigned)((n + kSortThreads - 1) / kSortThreads); }

template <class R, int D, int T>
hipError_t sort_impl(Ctx& c, Species& sp, hipStream_t s)
{
    const int64_t n = sp.n;
    constexpr int TPD = D == 3 ? T * T * T : T * T;
    const unsigned groups = (unsigned)((c.k.ntiles + kTileGroup - 1) / kTileGroup);
    uint32_t* tsum = (uint32_t*)c.rho_m;  // idle between the calls that fill it; at least a double per cell
    uint32_t* gsum = tsum + c.k.ntiles;
    hipLaunchKernelGGL(k_zero_u32, dim3(nblk(c.nkeys)), dim3(kSortThreads), 0, s, c.hist, (int64_t)c.nkeys);
    if (n > 0 && sp.sorted)  // still grouped by the tiles of the previous sort
        hipLaunchKernelGGL((k_histogram_tiled<R, D, T>), dim3(c.k.ntiles), dim3(1024), 0, s, c.k,
                           sp.cur, sp.tile_start, sp.key, sp.rank, c.hist);
    else if (n > 0)
        hipLaunchKernelGGL((k_histogram<R, D, T>), dim3(nblk(n)), dim3(kSortThreads), 0, s, c.k,
                           sp.cur, n, sp.key, sp.rank, c.hist);
    hipLaunchKernelGGL((k_tile_sums<TPD>), dim3(groups), dim3(64 * kTileGroup), 0, s, c.hist, c.k.ntiles, tsum, gsum);
    const bool scanned = groups >= kScanGroups;
    if (scanned) hipLaunchKernelGGL(k_group_scan, dim3(1), dim3(1024), 0, s, gsum, (int)groups);
    if (D == 3)
        hipLaunchKernelGGL((k_dest3<lane_classes<R>()>), dim3(c.k.ntiles), dim3(TPD), 0, s, c.hist, tsum, gsum,
                           scanned, n, sp.dest, sp.tile_start);
    else
        hipLaunchKernelGGL((k_dest<TPD>), dim3(c.k.ntiles), dim3(TPD), 0, s, c.hist, tsum, gsum, scanned, n, sp.dest,
                           sp.tile_start);
    if (n > 0) {
        // the inverse of the final slots, and one gather into the spare copy,
        // which becomes current
        constexpr int C = D == 3 ? lane_classes<R>() : 1;
        hipLaunchKernelGGL((k_final_src<C, D == 3 ? TPD / C : 0>), dim3(nblk(n)), dim3(kSortThreads), 0, s, n, sp.key,
                           sp.rank, c.hist, sp.dest, sp.tile_start, sp.src);
        const unsigned blocks = (nblk((n + kGatherU - 1) / kGatherU) + kXcds - 1) / kXcds * kXcds;
        hipLaunchKernelGGL((k_gather_final<R>), dim3(blocks, sizeof(R) == 4 ? 9 : 8), dim3(kSortThreads), 0, s,
                           sp.cur, sp.alt, n, sp.src);
        const PartArrays t = sp.cur;
        sp.cur = sp.alt;
        sp.alt = t;
        sp.swapped ^= 1;
    }
    sp.sorted = true;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_sort(Ctx& c, Species& sp, hipStream_t s)
{
    if (c.g.precision == PIC_FP64)
        return c.k.dims == 3 ? sort_impl<double, 3, kTile3>(c, sp, s) : sort_impl<double, 2, kTile2>(c, sp, s);
    return c.k.dims == 3 ? sort_impl<float, 3, kTile3>(c, sp, s) : sort_impl<float, 2, kTile2>(c, sp, s);
}

}  // namespace pic
