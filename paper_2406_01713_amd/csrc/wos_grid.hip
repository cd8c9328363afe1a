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
// Each block first keeps the obstacles that can matter anywhere in the box
// around its tile of up to 256 cells, then each lane
// builds its cell's list from those.  Bound by vector arithmetic: without the
// first pass every cell tests every obstacle three times (2.8e5 cells, 7-D:
// 0.34 ms for 256 spheres, 2.8 ms for 2048).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "wos_launch.hpp"
#include "wos_walk.hpp"

namespace wos {

namespace {

struct CellBox {
    float lo[kMaxDim], hi[kMaxDim];
};

// Cells per axis of a block's tile: at most kBlock cells, near-cubic, so the
// box around them is small.
template <int K>
constexpr int tile_side(int i)
{
    constexpr int side[9][8] = {{},
                                {256},
                                {16, 16},
                                {6, 6, 7},
                                {4, 4, 4, 4},
                                {3, 3, 3, 3, 3},
                                {3, 3, 3, 2, 2, 2},
                                {3, 3, 2, 2, 2, 2, 1},
                                {2, 2, 2, 2, 2, 2, 2, 2}};
    return side[K][i];
}
template <int K>
constexpr int tile_cells()
{
    int n = 1;
    for (int i = 0; i < K; ++i) n *= tile_side<K>(i);
    return n;
}

// Index of the thread's cell (cells: none), the cell's box and the box around
// the block's tile.
template <int K>
__device__ __forceinline__ uint32_t tile_cell(const GridBuild& g, CellBox& cell, CellBox& tile)
{
    uint32_t blk = blockIdx.x, loc = threadIdx.x, c = 0, mul = 1;
    bool in = threadIdx.x < (unsigned)tile_cells<K>();
#pragma unroll
    for (int i = K - 1; i >= 0; --i) {
        const uint32_t s = tile_side<K>(i), nb = (g.n[i] + s - 1) / s;
        const uint32_t t0 = (blk % nb) * s, j = t0 + loc % s;
        const uint32_t t1 = min(t0 + s, g.n[i]);
        blk /= nb;
        loc /= s;
        in = in && j < g.n[i];
        const uint32_t jj = min(j, g.n[i] - 1);
        c += jj * mul;
        mul *= g.n[i];
        cell.lo[i] = g.lo[i] + (float)jj * g.h - g.pad[i];
        cell.hi[i] = g.lo[i] + ((float)jj + 1.0f) * g.h + g.pad[i];
        tile.lo[i] = g.lo[i] + (float)t0 * g.h - g.pad[i];
        tile.hi[i] = g.lo[i] + (float)t1 * g.h + g.pad[i];
    }
    return in ? c : g.cells;
}
template <int K>
unsigned tile_count(const GridBuild& g)
{
    unsigned n = 1;
    for (int i = 0; i < K; ++i) n *= (g.n[i] + tile_side<K>(i) - 1) / tile_side<K>(i);
    return n;
}

// Distance from the cell to the obstacle, and the largest distance to it over
// the cell (an upper bound inside it).
template <int K, bool BOX>
__device__ __forceinline__ float near_dist(const CellBox& b, cptr<float> r, int d)
{
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const float w = BOX ? r[d + i] : 0.0f;
        const float t = fmaxf(fmaxf(b.lo[i] - (r[i] + w), (r[i] - w) - b.hi[i]), 0.0f);
        s = fmaf(t, t, s);
    }
    return sqrtf(s) - (BOX ? 0.0f : r[d]);
}

template <int K, bool BOX>
__device__ __forceinline__ float far_dist(const CellBox& b, cptr<float> r, int d)
{
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        float t = fmaxf(fabsf(b.lo[i] - r[i]), fabsf(b.hi[i] - r[i]));
        if (BOX) t = fmaxf(t - r[d + i], 0.0f);
        s = fmaf(t, t, s);
    }
    return sqrtf(s) - (BOX ? 0.0f : r[d]);
}

// Largest distance to the outer boundary over the cell (an upper bound).
template <int K>
__device__ __forceinline__ float outer_max(const GridBuild& g, const CellBox& b)
{
    if (g.outer_kind == 0) {
        float m = __builtin_huge_valf();
#pragma unroll
        for (int i = 0; i < K; ++i)
            m = fminf(m, fminf(fminf(b.hi[i] - g.olo[i], g.ohi[i] - b.lo[i]), 0.5f * (g.ohi[i] - g.olo[i])));
        return m;
    }
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const float t = fmaxf(fmaxf(b.lo[i] - g.oc[i], g.oc[i] - b.hi[i]), 0.0f);
        s = fmaf(t, t, s);
    }
    return g.orad - sqrtf(s);
}

// Obstacle level in a cell: 0..3 for a listed obstacle, 4 for none.
__device__ __forceinline__ int level_of(const GridBuild& g, float nd, float lim)
{
    if (!(nd <= lim)) return 4;
    nd -= g.margin;
    return nd <= g.lev[0] ? 0 : nd <= g.lev[1] ? 1 : nd <= g.lev[2] ? 2 : 3;
}

// Obstacles (row indices, ascending) that can matter in one of the block's
// cells: nearer to the box b around them than the limit of that box.  What is
// left out is never in a cell's list and never sets a cell's limit, since a
// cell's limit is at most the box's and an obstacle is no nearer to, and no
// less far from, a cell than the box around it.  More than kCandMax: all (-1).
constexpr int kCandMax = 3072;
template <int K, bool BOX>
__device__ __forceinline__ int block_candidates(const GridBuild& g, const CellBox& b, int d, cptr<float> rows, int m,
                                                uint32_t* cand)
{
    constexpr int NW = kBlock / kWave;
    __shared__ float red[NW];
    __shared__ int cnt[NW];
    const int S = BOX ? box_stride(d) : sph_stride(d);
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    float lim = outer_max<K>(g, b);
    for (int j = threadIdx.x; j < m; j += kBlock) lim = fminf(lim, far_dist<K, BOX>(b, rows + (int64_t)j * S, d));
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) lim = fminf(lim, __shfl_xor(lim, off, kWave));
    if (lane == 0) red[wv] = lim;
    __syncthreads();
    for (int w = 0; w < NW; ++w) lim = fminf(lim, red[w]);
    lim += 2.0f * g.margin;  // a cell's limit includes one margin
    int n = 0;
    for (int j0 = 0; j0 < m; j0 += kBlock) {  // block-uniform
        const int j = j0 + (int)threadIdx.x;
        const bool keep = j < m && near_dist<K, BOX>(b, rows + (int64_t)(j < m ? j : 0) * S, d) <= lim;
        const uint64_t v = __builtin_amdgcn_ballot_w64(keep);
        if (lane == 0) cnt[wv] = __popcll(v);
        __syncthreads();
        int at = n;
        for (int w = 0; w < NW; ++w) {
            at += w < wv ? cnt[w] : 0;
            n += cnt[w];
        }
        at += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(v >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)v, 0u));
        if (keep && at < kCandMax) cand[at] = (uint32_t)j;
        __syncthreads();
    }
    return n <= kCandMax ? n : -1;
}

// Pass 1: each cell's limit, header counts and place in the list.
template <int K, bool BOX>
__global__ void __launch_bounds__(kBlock)
grid_count_kernel(GridBuild g, int d, const float* rows_, int m, float* __restrict__ lims,
                  GridCell* __restrict__ cells, unsigned* __restrict__ total, unsigned* __restrict__ overfull)
{
    __shared__ uint32_t cand[kCandMax];
    CellBox b, tile;
    const uint32_t c = tile_cell<K>(g, b, tile);
    const bool valid = c < g.cells;
    cptr<float> rows = to_const(rows_);
    const int S = BOX ? box_stride(d) : sph_stride(d);
    const int nc = block_candidates<K, BOX>(g, tile, d, rows, m, cand);
    const int mm = nc < 0 ? m : nc;
    auto row_of = [&](int i) { return nc < 0 ? i : (int)__builtin_amdgcn_readfirstlane(cand[i]); };
    float lim = outer_max<K>(g, b);
    for (int i = 0; i < mm; ++i) lim = fminf(lim, far_dist<K, BOX>(b, rows + (int64_t)row_of(i) * S, d));
    lim += g.margin;
    uint32_t n[4] = {0, 0, 0, 0};
    for (int j = 0; j < mm; ++j) {
        const int l = level_of(g, near_dist<K, BOX>(b, rows + (int64_t)row_of(j) * S, d), lim);
#pragma unroll
        for (int i = 0; i < 4; ++i) n[i] += (l <= i) ? 1u : 0u;
    }
    uint32_t stored = 0, counts = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // a range's entries follow the (rounded-up) ranges before it
        const uint32_t code = grid_encode(stored + n[i] - (i > 0 ? n[i > 0 ? i - 1 : 0] : 0u));
        if (code > 255u) *overfull = 1u;
        counts |= (code < 255u ? code : 255u) << (8 * i);
        stored = grid_decode(code < 255u ? code : 255u);
    }
    stored = valid ? stored : 0u;
    const uint32_t incl = wave_incl_scan(stored);
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    uint32_t base = 0;
    if ((threadIdx.x & (kWave - 1)) == 0 && all > 0) base = atomicAdd(total, all);
    base = __builtin_amdgcn_readfirstlane(base);
    if (valid) {
        cells[c].off = base + incl - stored;
        cells[c].counts = counts;
        lims[c] = lim;
    }
}

// Pass 2: the entries, by level, in row order within a level.
template <int K, bool BOX>
__global__ void __launch_bounds__(kBlock)
grid_fill_kernel(GridBuild g, int d, const float* rows_, int m, const float* __restrict__ lims,
                 const GridCell* __restrict__ cells, uint32_t* __restrict__ list)
{
    __shared__ uint32_t cand[kCandMax];
    cptr<float> rows = to_const(rows_);
    const int S = BOX ? box_stride(d) : sph_stride(d);
    CellBox b, tile;
    const uint32_t c = tile_cell<K>(g, b, tile);
    const int nc = block_candidates<K, BOX>(g, tile, d, rows, m, cand);  // every thread takes part
    const int mm = nc < 0 ? m : nc;
    auto row_of = [&](int i) { return nc < 0 ? i : (int)__builtin_amdgcn_readfirstlane(cand[i]); };
    if (c >= g.cells) return;
    const GridCell h = cells[c];
    uint32_t pos[4], end[4], at = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        pos[i] = at;
        at = end[i] = grid_decode((h.counts >> (8 * i)) & 0xFFu);
    }
    if (at == 0) return;
    const float lim = lims[c];
    for (int i0 = 0; i0 < mm; ++i0) {
        const int j = row_of(i0);
        const int l = level_of(g, near_dist<K, BOX>(b, rows + (int64_t)j * S, d), lim);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (l == i && pos[i] < end[i]) list[h.off + pos[i]++] = (uint32_t)j;
    }
    // rounded-up counts: repeat the cell's first entry
    const uint32_t first = list[h.off];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        for (; pos[i] < end[i]; ++pos[i]) list[h.off + pos[i]] = first;
}

template <int K, bool BOX>
hipError_t build_k(const GridBuild& g, int d, const float* rows, int m, GridCell** cells, uint32_t** list)
{
    const unsigned grid = tile_count<K>(g);
    unsigned told[2] = {0, 0};  // entries, whether some cell holds too many
    // [headers | limits | told], kept together: a second allocation and its
    // release cost more than the limits' megabyte
    GridCell* hd = nullptr;
    uint32_t* entries = nullptr;
    hipError_t e = hipMalloc(&hd, (size_t)g.cells * (sizeof(GridCell) + sizeof(float)) + sizeof(told));
    float* lims = reinterpret_cast<float*>(hd + g.cells);
    unsigned* d_told = reinterpret_cast<unsigned*>(lims + g.cells);
    if (e == hipSuccess) e = launch_fill_u32(d_told, 2, 0u, nullptr);
    if (e == hipSuccess) {
        hipLaunchKernelGGL((grid_count_kernel<K, BOX>), dim3(grid), dim3(kBlock), 0, nullptr, g, d, rows, m, lims, hd,
                           d_told, d_told + 1);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpy(told, d_told, sizeof(told), hipMemcpyDeviceToHost);
    const unsigned total = told[0];
    const bool fits = total <= kGridEntriesMax && told[1] == 0;
    if (e == hipSuccess && fits) e = hipMalloc(&entries, std::max<size_t>(total, 1) * sizeof(uint32_t));
    if (e == hipSuccess && fits) {
        hipLaunchKernelGGL((grid_fill_kernel<K, BOX>), dim3(grid), dim3(kBlock), 0, nullptr, g, d, rows, m, lims, hd,
                           entries);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    }
    if (e == hipSuccess && fits) {
        *cells = hd;
        *list = entries;
    } else {
        (void)hipFree(hd);
        (void)hipFree(entries);
    }
    return e;
}

}  // namespace

hipError_t build_grid(const GridBuild& g, int d, bool box, const float* rows, int64_t m, GridCell** cells,
                      uint32_t** list)
{
    *cells = nullptr;
    *list = nullptr;
    if (m < 1 || m > INT32_MAX || g.cells < 1) return hipSuccess;
#define WOS_GRID_CASE(K)                                                              \
    case K:                                                                           \
        return box ? build_k<K, true>(g, d, rows, (int)m, cells, list) : build_k<K, false>(g, d, rows, (int)m, cells, list);
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

}  // namespace wos
