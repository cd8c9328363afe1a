// wos_plain.hip -- plain walk kernel: one walk per lane, one wave per (query,
// 64-walk chunk); the wave runs until its longest walk ends (forward, or
// forward + backward sums when BWD: the backward pass regenerates the same
// walks from their Philox counters).  Compiled once per precision
// (WOS_PLAIN_T = float or double).
#include <hip/hip_runtime.h>

#include "wos_launch.hpp"
#include "wos_walk.hpp"

namespace wos {

namespace {

// ------------------------------------------------------------------------
// Plain kernel.  FP32: at least 4 waves per SIMD (at most 128 registers per
// lane) where that needs no scratch memory (d <= 6, and d = 7 without a
// point source), else at least 3 (168 registers); left free, the allocator
// may take a few more and fall a wave lower.
// ------------------------------------------------------------------------
template <typename T, int D, bool SRC>
constexpr int plain_waves()
{
    return sizeof(T) != 4 ? 1 : (D < 7 || (D == 7 && !SRC)) ? 4 : 3;
}

template <typename T, int D, bool BWD, bool SRC, bool LISTS>
__global__ void __launch_bounds__(kBlock, (plain_waves<T, D, SRC>()))
plain_kernel(const EnvP<T>* penv, const T* __restrict__ queries, int64_t n_units, int32_t chunks,
             int64_t n_walks, int64_t w_base, uint32_t q_base, const uint64_t* __restrict__ key_add,
             double* __restrict__ partials, double* __restrict__ records)
{
    __shared__ uint32_t pair_lds[kBlock / kWave][kPairLds];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t unit = (int64_t)blockIdx.x * (kBlock / kWave) + wv;
    if (unit >= n_units) return;
    const int64_t q = unit / chunks;
    const int64_t wi = (unit - q * chunks) * kWave + lane;
    const cenv<T> p = (cenv<T>)penv;
    uint32_t k0 = p->key0, k1 = p->key1;
    apply_key_add(k0, k1, key_add);

    T xq[D];
    cptr<T> qrow = to_const(queries) + q * D;
#pragma unroll
    for (int i = 0; i < D; ++i) xq[i] = qrow[i];

    const bool active = wi < n_walks;
    Walker<T, D> s;
    walker_start<T, D, D>(s, xq, (uint32_t)(w_base + wi));
    WalkEnd<T> e;
    e.u = e.gs = e.S = e.goal_w = T(0);
    e.ex = 0;
    e.steps = 0;
    e.status = kTruncated;
    e.cls = kOuter;
    WorkCount wc(pair_lds[wv]);
    const UnitStart<T> st = unit_start<T, D, D>(p, xq, wc);
    // every lane steps until the wave's last walk ends (a finished lane runs
    // along idle), so the obstacle scans and the work tally stay wave-uniform
    bool done = !active;
    while (__builtin_amdgcn_ballot_w64(!done) != 0) {
        WalkEnd<T> ek;
        const bool fin = walker_step<T, D, BWD, LISTS, D, SRC>(p, s, q_base + (uint32_t)q, k0, k1, ek, wc, !done, st);
        if (fin && !done) {
            e = ek;
            done = true;
        }
    }

    double a[nacc(D)];
#pragma unroll
    for (int i = 0; i < nacc(D); ++i) a[i] = 0.0;
    if (active) accumulate<T, D, D, SRC>(a, e, s.v0, p, xq);
    add_work(a, 7 + 2 * D, wc);
    wave_store<nacc(D)>(a, partials + unit * nacc(D));

    if (records != nullptr && active) {
        double* r = records + wi * (D + 7);
        const double sc = walk_scale(e);
        r[0] = (double)e.u * sc;
#pragma unroll
        for (int i = 0; i < D; ++i) r[1 + i] = walk_grad<T, D, D, SRC>(e, s.v0, p, xq, i, sc);
        r[D + 1] = (double)e.S;
        r[D + 2] = (double)e.goal_w * sc;
        r[D + 3] = (double)e.steps;
        r[D + 4] = (double)e.status;
        r[D + 5] = (double)e.cls;
        r[D + 6] = walk_dsigma<T, SRC>(e, sc);
    }
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

template <typename T, int D, bool BWD, bool SRC>
static void plain_go(bool lists, unsigned grid, const EnvP<T>* p, const T* queries, int64_t units, int32_t chunks,
                     int64_t n_walks, int64_t w_base, uint32_t q_base, const uint64_t* key_add, double* partials,
                     double* records, hipStream_t st)
{
    if (lists)
        hipLaunchKernelGGL((plain_kernel<T, D, BWD, SRC, true>), dim3(grid), dim3(kBlock), 0, st, p, queries, units,
                           chunks, n_walks, w_base, q_base, key_add, partials, records);
    else
        hipLaunchKernelGGL((plain_kernel<T, D, BWD, SRC, false>), dim3(grid), dim3(kBlock), 0, st, p, queries, units,
                           chunks, n_walks, w_base, q_base, key_add, partials, records);
}

template <typename T, int D>
static hipError_t plain_d(bool bwd, bool src, bool lists, const EnvP<T>* p, const T* queries, int64_t n_q,
                          int64_t n_walks, int64_t w_base, uint32_t q_base, const uint64_t* key_add, double* partials,
                          double* records, hipStream_t st)
{
    const int32_t chunks = (int32_t)((n_walks + kWave - 1) / kWave);
    const int64_t units = n_q * chunks;
    if (units == 0) return hipSuccess;
    const unsigned grid = blocks_for(units, kBlock / kWave);
    auto* go = bwd ? (src ? plain_go<T, D, true, true> : plain_go<T, D, true, false>)
                   : (src ? plain_go<T, D, false, true> : plain_go<T, D, false, false>);
    go(lists, grid, p, queries, units, chunks, n_walks, w_base, q_base, key_add, partials, records, st);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_plain(int d, bool bwd, bool src, bool lists, const EnvP<T>* p, const T* queries, int64_t n_q,
                        int64_t n_walks, int64_t w_base, uint32_t q_base, const uint64_t* key_add,
                        double* partials, double* records, hipStream_t st)
{
    switch (d) {
    case 2: return plain_d<T, 2>(bwd, src, lists, p, queries, n_q, n_walks, w_base, q_base, key_add, partials, records, st);
    case 3: return plain_d<T, 3>(bwd, src, lists, p, queries, n_q, n_walks, w_base, q_base, key_add, partials, records, st);
    case 4: return plain_d<T, 4>(bwd, src, lists, p, queries, n_q, n_walks, w_base, q_base, key_add, partials, records, st);
    case 5: return plain_d<T, 5>(bwd, src, lists, p, queries, n_q, n_walks, w_base, q_base, key_add, partials, records, st);
    case 6: return plain_d<T, 6>(bwd, src, lists, p, queries, n_q, n_walks, w_base, q_base, key_add, partials, records, st);
    case 7: return plain_d<T, 7>(bwd, src, lists, p, queries, n_q, n_walks, w_base, q_base, key_add, partials, records, st);
    case 8: return plain_d<T, 8>(bwd, src, lists, p, queries, n_q, n_walks, w_base, q_base, key_add, partials, records, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_plain<WOS_PLAIN_T>(int, bool, bool, bool, const EnvP<WOS_PLAIN_T>*, const WOS_PLAIN_T*, int64_t,
                                              int64_t, int64_t, uint32_t, const uint64_t*, double*, double*,
                                              hipStream_t);

}  // namespace wos
