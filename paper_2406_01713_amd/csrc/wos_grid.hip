// wos_grid.hip -- builds the cell lists that the walks look obstacles up in
// (see kGridMin in wos_params.hpp).
//
// Every list must hold each obstacle that can attain the distance to the
// boundary at a point the walk maps to the cell.  The cell is taken enlarged
// (pad), so it holds every such point; an obstacle whose distance from it
// exceeds, by the margin, the largest outer distance in it or some obstacle's
// largest distance over it is never the nearest there, and one whose distance
// exceeds a threshold range's end by the margin is never nearer than a walker
// with a threshold in the range.  The margin (2^-16 of the geometry's size)
// is far above the rounding of the distances here and in the walks.
//
// One kernel.  A block takes a tile of up to 64 cells and keeps the obstacles
// that can matter somewhere in it (about 120 of 2048 in 7-D, ten times that in
// the middle of the box), each of its waves those that can matter in its 16
// cells.  Four lanes share a cell, each taking every fourth of these obstacles:
// the cell's limit, the number of entries per level, then the entries.
// Bound by the four lanes' turns through the obstacles of the cells in the middle
// and by vector arithmetic: 0.46 ms for 2048 spheres in 7-D, 0.29 in 6-D, 0.05 in
// 2-D, 0.03 to 0.07 for 256.  (A counting and a filling kernel with a lane per
// cell, every lane of a wave going through the same obstacles one by one and a
// wave's entries reserved on one counter: 1.48, 1.54, 0.08 and 0.06 to 0.23 ms,
// of which the few tiles in the middle, with some 1500 obstacles each, and up to
// 0.1 ms the counter.)  The host makes the clusters meanwhile (0.2 ms for 256
// spheres, 1.7 for 2048).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "wos_launch.hpp"
#include "wos_walk.hpp"

namespace wos {

namespace {

struct CellBox {
    float mid[kMaxDim], half[kMaxDim];
};

// Cells per axis of a block's tile (64 cells) and of a wave's part of it (16).
constexpr int kCellsPerWave = 16;
constexpr int kSlices = kWave / kCellsPerWave;  // lanes that share a cell
template <int K>
constexpr int tile_side(int i)
{
    constexpr int side[9][8] = {{},
                                {64},
                                {8, 8},
                                {4, 4, 4},
                                {4, 4, 2, 2},
                                {4, 2, 2, 2, 2},
                                {2, 2, 2, 2, 2, 2},
                                {2, 2, 2, 2, 2, 2, 1},
                                {2, 2, 2, 2, 2, 2, 1, 1}};
    return side[K][i];
}
template <int K>
constexpr int wave_side(int i)
{
    constexpr int side[9][8] = {{},
                                {16},
                                {4, 4},
                                {4, 2, 2},
                                {2, 2, 2, 2},
                                {2, 2, 2, 2, 1},
                                {2, 2, 2, 2, 1, 1},
                                {2, 2, 2, 2, 1, 1, 1},
                                {2, 2, 2, 2, 1, 1, 1, 1}};
    return side[K][i];
}
template <int K>
constexpr bool sides_fit()
{
    int cells = 1, waves = 1;
    for (int i = 0; i < K; ++i) {
        if (tile_side<K>(i) % wave_side<K>(i) != 0) return false;
        cells *= wave_side<K>(i);
        waves *= tile_side<K>(i) / wave_side<K>(i);
    }
    return cells == kCellsPerWave && waves == kBlock / kWave;
}

// Index of the lane's cell (cells: none), its box and those around the wave's
// and the block's cells; some: the wave has a cell.
template <int K>
__device__ __forceinline__ uint32_t place(const GridBuild& g, CellBox& cell, CellBox& wave, CellBox& tile, bool& some)
{
    static_assert(sides_fit<K>(), "a tile is four waves' parts of 16 cells");
    uint32_t blk = blockIdx.x, wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t loc = threadIdx.x % kCellsPerWave, c = 0, mul = 1;
    bool in = true;
    some = true;
#pragma unroll
    for (int i = K - 1; i >= 0; --i) {
        const uint32_t ts = tile_side<K>(i), ws = wave_side<K>(i), last = g.n[i] - 1, nb = last / ts + 1;
        const uint32_t t0 = (blk % nb) * ts, t1 = min(t0 + ts, g.n[i]);
        const uint32_t w0 = t0 + (wv % (ts / ws)) * ws, j = w0 + loc % ws;
        blk /= nb;
        wv /= ts / ws;
        loc /= ws;
        in = in && j <= last;
        some = some && w0 <= last;
        const uint32_t jj = min(j, last), a = min(w0, last), z = min(w0 + ws, g.n[i]);
        c += jj * mul;
        mul *= g.n[i];
        cell.mid[i] = g.lo[i] + ((float)jj + 0.5f) * g.h;
        cell.half[i] = 0.5f * g.h + g.pad[i];
        wave.mid[i] = g.lo[i] + 0.5f * (float)(a + z) * g.h;
        wave.half[i] = 0.5f * (float)(z - a) * g.h + g.pad[i];
        tile.mid[i] = g.lo[i] + 0.5f * (float)(t0 + t1) * g.h;
        tile.half[i] = 0.5f * (float)(t1 - t0) * g.h + g.pad[i];
    }
    return in ? c : g.cells;
}
template <int K>
unsigned tile_count(const GridBuild& g)
{
    unsigned n = 1;
    for (int i = 0; i < K; ++i) n *= (g.n[i] - 1) / tile_side<K>(i) + 1;
    return n;
}

// Squared distance from the cell to a box obstacle or to a sphere's centre, and
// the largest one over the cell (an upper bound).
template <int K, bool BOX>
__device__ __forceinline__ float near2(const CellBox& b, cptr<float> r, int d)
{
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const float t = fmaxf(fabsf(r[i] - b.mid[i]) - (BOX ? b.half[i] + r[d + i] : b.half[i]), 0.0f);
        s = fmaf(t, t, s);
    }
    return s;
}

template <int K, bool BOX>
__device__ __forceinline__ float far_dist(const CellBox& b, cptr<float> r, int d)
{
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        float t = fabsf(r[i] - b.mid[i]) + b.half[i];
        if (BOX) t = fmaxf(t - r[d + i], 0.0f);
        s = fmaf(t, t, s);
    }
    return Math<float>::sqrt(s) - (BOX ? 0.0f : r[d]);
}

// Largest distance to the outer boundary over the cell (an upper bound).
template <int K>
__device__ __forceinline__ float outer_max(const GridBuild& g, const CellBox& b)
{
    if (g.outer_kind == 0) {
        float m = __builtin_huge_valf();
#pragma unroll
        for (int i = 0; i < K; ++i)
            m = fminf(m, fminf(fminf(b.mid[i] + b.half[i] - g.olo[i], g.ohi[i] - (b.mid[i] - b.half[i])),
                               0.5f * (g.ohi[i] - g.olo[i])));
        return m;
    }
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const float t = fmaxf(fabsf(b.mid[i] - g.oc[i]) - b.half[i], 0.0f);
        s = fmaf(t, t, s);
    }
    return g.orad - Math<float>::sqrt(s);
}

// Whether an obstacle at squared distance s (radius rad, 0 for a box) is within
// lim of the cell.
__device__ __forceinline__ bool within(float s, float rad, float lim)
{
    const float t = lim + rad;
    return t >= 0.0f && s <= t * t;
}

// Level of a listed obstacle: 0..3; 4 for one past lim.
__device__ __forceinline__ int level_of(const GridBuild& g, float s, float rad, float lim)
{
    if (!within(s, rad, lim)) return 4;
    const float nd = (Math<float>::sqrt(s) - rad) - g.margin;
    return nd <= g.lev[0] ? 0 : nd <= g.lev[1] ? 1 : nd <= g.lev[2] ? 2 : 3;
}

__device__ __forceinline__ int lanes_before(uint64_t v)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(v >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)v, 0u));
}
__device__ __forceinline__ float wave_min(float v)
{
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) v = fminf(v, __shfl_xor(v, off, kWave));
    return v;
}

// A set of row indices: n in ids, or (null) 0 to n - 1.
struct Rows {
    const uint32_t* ids;
    int n;
    __device__ __forceinline__ int at(int k) const { return ids ? (int)ids[k] : k; }
};

// The block's obstacles: those of all m within the tile's limit.  What is left
// out is never in a cell's list and never sets a cell's limit: an obstacle is no
// nearer to a cell, and no less far from it, than to the tile around it, and a
// cell's limit is at most the tile's (the two margins cover the one in the
// cell's limit and rounding).  More than kCandMax: all.
constexpr int kCandMax = 3072;
template <int K, bool BOX>
__device__ __forceinline__ Rows block_rows(const GridBuild& g, const CellBox& b, int d, cptr<float> rows, int m,
                                           uint32_t* cand)
{
    constexpr int NW = kBlock / kWave;
    __shared__ float red[NW];
    __shared__ int cnt[NW];
    const int S = BOX ? box_stride(d) : sph_stride(d);
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    float lim = outer_max<K>(g, b);
    for (int j = threadIdx.x; j < m; j += kBlock) lim = fminf(lim, far_dist<K, BOX>(b, rows + (int64_t)j * S, d));
    lim = wave_min(lim);
    if (lane == 0) red[wv] = lim;
    __syncthreads();
    for (int w = 0; w < NW; ++w) lim = fminf(lim, red[w]);
    lim += 2.0f * g.margin;
    int n = 0;
    for (int j0 = 0; j0 < m; j0 += kBlock) {  // block-uniform
        const int j = j0 + (int)threadIdx.x;
        cptr<float> r = rows + (int64_t)(j < m ? j : 0) * S;
        const bool keep = j < m && within(near2<K, BOX>(b, r, d), BOX ? 0.0f : r[d], lim);
        const uint64_t v = __builtin_amdgcn_ballot_w64(keep);
        if (lane == 0) cnt[wv] = __popcll(v);
        __syncthreads();
        int at = n + lanes_before(v);
        for (int w = 0; w < NW; ++w) {
            at += w < wv ? cnt[w] : 0;
            n += cnt[w];
        }
        if (keep && at < kCandMax) cand[at] = (uint32_t)j;
        __syncthreads();
    }
    return n <= kCandMax ? Rows{cand, n} : Rows{nullptr, m};
}

// The wave's, likewise, out of the block's.  More than kMineMax: the block's.
constexpr int kMineMax = 1024;
template <int K, bool BOX>
__device__ __forceinline__ Rows wave_rows(const GridBuild& g, const CellBox& b, int d, cptr<float> rows, Rows from,
                                          uint32_t* mine)
{
    const int S = BOX ? box_stride(d) : sph_stride(d);
    const int lane = threadIdx.x & (kWave - 1);
    float lim = outer_max<K>(g, b);
    for (int k = lane; k < from.n; k += kWave)
        lim = fminf(lim, far_dist<K, BOX>(b, rows + (int64_t)from.at(k) * S, d));
    lim = wave_min(lim) + 2.0f * g.margin;
    int n = 0;
    for (int k0 = 0; k0 < from.n; k0 += kWave) {  // wave-uniform
        const int k = k0 + lane, j = from.at(k < from.n ? k : 0);
        cptr<float> r = rows + (int64_t)j * S;
        const bool keep = k < from.n && within(near2<K, BOX>(b, r, d), BOX ? 0.0f : r[d], lim);
        const uint64_t v = __builtin_amdgcn_ballot_w64(keep);
        const int at = n + lanes_before(v);
        if (keep && at < kMineMax) mine[at] = (uint32_t)j;
        n += __popcll(v);
    }
    wave_lds_fence();
    return n <= kMineMax ? Rows{mine, n} : from;
}

// The list is made of up to kParts parts of `cap` entries, each with a counter of
// its own in which the waves reserve their entries: some 12 ns each on one
// counter, 0.2 ms for a table of 16384 waves; 256 waves per part leave 3 us.  A
// wave's part is a hash of its number, so parts fill alike.
constexpr unsigned kParts = 64;
constexpr unsigned kToldStride = 32;  // words from counter to counter: a cache line
constexpr unsigned kToldWords = kParts * kToldStride + 1;

// Headers and lists of all cells.  told receives each part's number of entries
// and, last, whether some cell holds too many; a wave whose entries end past its
// part writes none (the caller then starts again with room for all).
template <int K, bool BOX>
__global__ void __launch_bounds__(kBlock)
grid_build_kernel(GridBuild g, int d, const float* rows_, int m, GridCell* __restrict__ cells,
                  uint32_t* __restrict__ list, uint32_t cap, unsigned parts, unsigned* __restrict__ told)
{
    __shared__ uint32_t cand[kCandMax];
    __shared__ uint32_t mine[kBlock / kWave][kMineMax];
    const int lane = threadIdx.x & (kWave - 1), slice = lane / kCellsPerWave;
    CellBox b, wave, tile;
    bool some;
    const uint32_t c = place<K>(g, b, wave, tile, some);
    const bool valid = c < g.cells;
    cptr<float> rows = to_const(rows_);
    const int S = BOX ? box_stride(d) : sph_stride(d);
    const Rows all = block_rows<K, BOX>(g, tile, d, rows, m, cand);
    if (!some) return;  // wave-uniform; no barrier follows
    const Rows own = wave_rows<K, BOX>(g, wave, d, rows, all, mine[threadIdx.x / kWave]);
    auto each = [&](auto f) {
#pragma unroll 4
        for (int k = slice; k < own.n; k += kSlices) {
            const int j = own.at(k);
            f(j, rows + (int64_t)j * S);
        }
    };
    auto level = [&](cptr<float> r, float lim) {
        return level_of(g, near2<K, BOX>(b, r, d), BOX ? 0.0f : r[d], lim);
    };

    // the cell's limit, over its lanes; lanes without a cell list nothing
    float lim = outer_max<K>(g, b);
    each([&](int, cptr<float> r) { lim = fminf(lim, far_dist<K, BOX>(b, r, d)); });
#pragma unroll
    for (int off = kCellsPerWave; off < kWave; off *= 2) lim = fminf(lim, __shfl_xor(lim, off, kWave));
    lim = valid ? lim + g.margin : -__builtin_huge_valf();

    uint32_t n[4] = {0, 0, 0, 0};  // this lane's entries per level
    each([&](int, cptr<float> r) {
        const int l = level(r, lim);
#pragma unroll
        for (int i = 0; i < 4; ++i) n[i] += l == i ? 1u : 0u;
    });
    // a level's entries follow the (rounded-up) ranges before it, slice by slice
    uint32_t stored = 0, counts = 0, pos[4], fill[4], end[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t total = 0, before = 0;
#pragma unroll
        for (int s = 0; s < kSlices; ++s) {
            const uint32_t v = (uint32_t)__shfl((int)n[i], s * kCellsPerWave + lane % kCellsPerWave, kWave);
            total += v;
            before += s < slice ? v : 0u;
        }
        pos[i] = stored + before;
        fill[i] = stored + total;
        const uint32_t code = grid_encode(fill[i]);
        if (code > 255u) told[kToldWords - 1] = 1u;
        counts |= (code < 255u ? code : 255u) << (8 * i);
        stored = end[i] = grid_decode(code < 255u ? code : 255u);
    }
    // the wave's place in the list: the cells' one after another
    const uint32_t mine_n = slice == 0 ? stored : 0u;
    const uint32_t incl = wave_incl_scan(mine_n);
    const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    const unsigned number = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    const unsigned part = __builtin_amdgcn_readfirstlane((number * 0x9E3779B1u) >> 16) % parts;
    uint32_t base = 0;
    if (lane == 0 && sum > 0) base = atomicAdd(told + part * kToldStride, sum);
    base = __builtin_amdgcn_readfirstlane(base);
    const uint32_t off = part * cap + base + (uint32_t)__shfl((int)(incl - mine_n), lane % kCellsPerWave, kWave);
    if (valid && slice == 0) {
        cells[c].off = off;
        cells[c].counts = counts;
    }
    if (sum == 0 || base > cap || sum > cap - base) return;

    // the entries; an obstacle's level comes from the same values as above, so
    // it finds the place counted for it
    uint32_t first = 0;
    each([&](int j, cptr<float> r) {
        const int l = level(r, lim);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (l == i && pos[i] < end[i]) {
                if (pos[i] == 0) first = (uint32_t)j;
                list[off + pos[i]++] = (uint32_t)j;
            }
    });
    // rounded-up counts: repeat the cell's first entry
#pragma unroll
    for (int o = kCellsPerWave; o < kWave; o *= 2) first |= (uint32_t)__shfl_xor((int)first, o, kWave);
    if (slice == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            for (uint32_t k = fill[i]; k < end[i]; ++k) list[off + k] = first;
    }
}

// Entries to make room for before they are counted: uniform scenes hold 1 to 1.6
// per cell up to 256 obstacles and, growing with their number, 1.3, 2.6, 5, 8 and
// 10 in 2- to 6-D and above for 2048 spheres, up to 14 for boxes.
template <int K, bool BOX>
double entries_guess(uint32_t cells, int m)
{
    constexpr double per[9] = {0, 6000, 6000, 1000, 400, 220, 170, 170, 170};
    return cells * (1.35 + m / (BOX && K > 5 ? 130.0 : per[K]));
}

// Enqueues a build on the default stream, the table's size first guessed and,
// once a build has counted, as the job says.
template <int K, bool BOX>
hipError_t start_k(const GridBuild& g, int d, const float* rows, int m, GridJob& job)
{
    const unsigned grid = tile_count<K>(g);
    if (!job.parts) {
        job.parts = 1;
        while (job.parts < kParts && grid * (kBlock / kWave) / job.parts > 256) job.parts *= 2;
        job.cap = (uint32_t)(std::min<double>(entries_guess<K, BOX>(g.cells, m), kGridEntriesMax) / job.parts);
    }
    // [headers | told | list] in one allocation
    hipError_t e = hipMalloc(&job.hd, (size_t)g.cells * sizeof(GridCell) + kToldWords * sizeof(unsigned) +
                                          (size_t)job.parts * job.cap * sizeof(uint32_t));
    if (e != hipSuccess) {
        job.hd = nullptr;
        return e;
    }
    unsigned* told = reinterpret_cast<unsigned*>(job.hd + g.cells);
    e = launch_fill_u32(told, kToldWords, 0u, nullptr);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((grid_build_kernel<K, BOX>), dim3(grid), dim3(kBlock), 0, nullptr, g, d, rows, m, job.hd,
                       told + kToldWords, job.cap, job.parts, told);
    return hipGetLastError();
}

}  // namespace

hipError_t grid_start(const GridBuild& g, int d, bool box, const float* rows, int64_t m, GridJob& job)
{
    if (m < 1 || m > INT32_MAX || g.cells < 1) return hipSuccess;
#define WOS_GRID_CASE(K) \
    case K: return box ? start_k<K, true>(g, d, rows, (int)m, job) : start_k<K, false>(g, d, rows, (int)m, job);
    switch (g.k) {
        WOS_GRID_CASE(1)
        WOS_GRID_CASE(2)
        WOS_GRID_CASE(3)
        WOS_GRID_CASE(4)
        WOS_GRID_CASE(5)
        WOS_GRID_CASE(6)
        WOS_GRID_CASE(7)
        WOS_GRID_CASE(8)
    default: return hipErrorInvalidValue;
    }
#undef WOS_GRID_CASE
}

hipError_t grid_finish(const GridBuild& g, int d, bool box, const float* rows, int64_t m, GridJob& job,
                       GridCell** cells, uint32_t** list)
{
    *cells = nullptr;
    *list = nullptr;
    while (job.hd) {
        unsigned* d_told = reinterpret_cast<unsigned*>(job.hd + g.cells);
        unsigned told[kToldWords];
        const hipError_t e = hipMemcpy(told, d_told, sizeof(told), hipMemcpyDeviceToHost);
        uint32_t most = 0;
        uint64_t total = 0;
        for (unsigned i = 0; e == hipSuccess && i < job.parts; ++i) {
            most = std::max(most, told[i * kToldStride]);
            total += told[i * kToldStride];
        }
        const bool overfull = e == hipSuccess && told[kToldWords - 1] != 0;
        // obstacles in a corner of the box need far less room than was guessed: from
        // 16 MB on that is worth a second build
        const bool loose = most < job.cap / 2 && (uint64_t)job.parts * (job.cap - most) > (4u << 20);
        if (e == hipSuccess && !overfull && most <= job.cap && !loose) {
            *cells = job.hd;
            *list = d_told + kToldWords;
            job.hd = nullptr;
            return hipSuccess;
        }
        (void)hipFree(job.hd);
        job.hd = nullptr;
        if (e != hipSuccess || overfull || total > kGridEntriesMax) return e;
        // a second time, with room for what there is
        if ((uint64_t)job.parts * most > kGridEntriesMax) {
            job.parts = 1;
            most = (uint32_t)total;
        }
        job.cap = std::max(most, 1u);
        const hipError_t again = grid_start(g, d, box, rows, m, job);
        if (again != hipSuccess) {
            (void)hipFree(job.hd);
            job.hd = nullptr;
            return again;
        }
    }
    return hipSuccess;
}

}  // namespace wos
