// wos_plain.hip -- plain walk kernel: one wave per (query, range of walks) of
// one environment, in FP32 or FP64, lanes refilled within the range (forward,
// or forward + backward sums when BWD: the backward pass regenerates the same
// walks from their Philox counters).  Compiled once per precision
// (WOS_PLAIN_T = float or double) and half of the dimensions
// (WOS_PLAIN_LOW = 1: 2 to 5, 0: 6 to 8).
#include <hip/hip_runtime.h>

#include "wos_launch.hpp"
#include "wos_walk.hpp"

namespace wos {

namespace {

// One wave per block: a wave's LDS and registers go to the next unit as soon
// as it ends (blocks of 4 waves wait for their slowest: 6-D forward set 5.72
// against 5.44 ms).
constexpr int kPlainBlock = kWave;

// FP32: at least 4 waves per SIMD (at most 128 registers per lane) where that
// needs no scratch memory (d <= 6, and d = 7 without a point source), else at
// least 3 (168 registers); left free, the allocator may take a few more and
// fall a wave lower.  (Bounds of 5, 6 or 8 for d <= 5 change nothing: those
// kernels need few registers as they are.)
template <typename T, int D, bool SRC>
constexpr int plain_waves()
{
    return sizeof(T) != 4 ? 1 : (D < 7 || (D == 7 && !SRC)) ? 4 : 3;
}
constexpr int kLdsWaves = 4;  // waves per SIMD the record queue leaves room for

template <typename T, int D, bool BWD, bool SRC, bool LISTS>
__global__ void __launch_bounds__(kPlainBlock, (plain_waves<T, D, SRC>()))
plain_kernel(const EnvP<T>* penv, const T* __restrict__ queries, int64_t n_units, int32_t chunks, int32_t wpu, int lanes,
             int64_t n_walks, int64_t w_base, uint32_t q_base, double* __restrict__ partials,
             double* __restrict__ records)
{
    extern __shared__ __align__(16) unsigned char lds_all[];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const WaveLds<T, SRC, LISTS, true> lds(lds_all + wv * wave_lds<T, SRC, LISTS, true>(D, kLdsWaves), D, kLdsWaves);
    const int64_t unit = (int64_t)blockIdx.x * (kPlainBlock / kWave) + wv;
    if (unit >= n_units) return;
    const int64_t q = unit / chunks;
    const int64_t w0 = (unit - q * chunks) * wpu;
    const cenv<T> p = (cenv<T>)penv;
    const int32_t n = (int32_t)(n_walks - w0 < wpu ? n_walks - w0 : wpu);
    run_unit<T, D, D, BWD, SRC, LISTS, true>(p, to_const(queries) + q * D, q_base + (uint32_t)q,
                                             (uint32_t)(w_base + w0), n, lanes, p->key0, p->key1, lds,
                                             partials + unit * nacc(D), records ? records + w0 * (D + 7) : nullptr);
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

template <typename T, int D, bool BWD, bool SRC, bool LISTS>
static void plain_go(unsigned grid, const EnvP<T>* p, const T* queries, int64_t units, int32_t chunks, int32_t wpu, int lanes,
                     int64_t n_walks, int64_t w_base, uint32_t q_base, double* partials, double* records,
                     hipStream_t st)
{
    const size_t lds = (kPlainBlock / kWave) * wave_lds<T, SRC, LISTS, true>(D, kLdsWaves);
    hipLaunchKernelGGL((plain_kernel<T, D, BWD, SRC, LISTS>), dim3(grid), dim3(kPlainBlock), lds, st, p, queries, units,
                       chunks, wpu, lanes, n_walks, w_base, q_base, partials, records);
}

template <typename T, int D>
hipError_t launch_plain_d(bool bwd, bool src, bool lists, const EnvP<T>* p, const T* queries, int64_t n_q,
                          int64_t n_walks, int32_t wpu, int lanes, int64_t w_base, uint32_t q_base, double* partials,
                          double* records, hipStream_t st)
{
    const int32_t chunks = (int32_t)((n_walks + wpu - 1) / wpu);
    const int64_t units = n_q * chunks;
    if (units == 0) return hipSuccess;
    auto* go = bwd ? (src ? (lists ? plain_go<T, D, true, true, true> : plain_go<T, D, true, true, false>)
                          : (lists ? plain_go<T, D, true, false, true> : plain_go<T, D, true, false, false>))
                   : (src ? (lists ? plain_go<T, D, false, true, true> : plain_go<T, D, false, true, false>)
                          : (lists ? plain_go<T, D, false, false, true> : plain_go<T, D, false, false, false>));
    go(blocks_for(units, kPlainBlock / kWave), p, queries, units, chunks, wpu, lanes, n_walks, w_base, q_base, partials, records, st);
    return hipGetLastError();
}

#define WOS_PLAIN_INST(D)                                                                                             \
    template hipError_t launch_plain_d<WOS_PLAIN_T, D>(bool, bool, bool, const EnvP<WOS_PLAIN_T>*, const WOS_PLAIN_T*, \
                                                       int64_t, int64_t, int32_t, int, int64_t, uint32_t, double*, double*, \
                                                       hipStream_t);
#if WOS_PLAIN_LOW
WOS_PLAIN_INST(2)
WOS_PLAIN_INST(3)
WOS_PLAIN_INST(4)
WOS_PLAIN_INST(5)
#else
WOS_PLAIN_INST(6)
WOS_PLAIN_INST(7)
WOS_PLAIN_INST(8)
#endif

}  // namespace wos
