// wos_persistent.hip -- persistent_kernel: ragged batch of environments in one
// launch: resident waves pull work units (env, query, walk range) from a
// device counter, and a lane whose walk ends starts the unit's next walk at
// once (lane refill), so a wave is not held by its longest walk.  Compiled
// without and with point-source terms (WOS_PERSISTENT_SRC = 0, 1), and with
// steps that scan clusters or read cell lists (WOS_PERSISTENT_LISTS = 0, 1;
// the latter also for batches of at most 5 dimensions, WOS_PERSISTENT_MAXD).
#include <hip/hip_runtime.h>

#include "wos_launch.hpp"
#include "wos_walk.hpp"

namespace wos {

namespace {

// ------------------------------------------------------------------------
// Persistent ragged-batch kernel (FP32).
// ------------------------------------------------------------------------
typedef __attribute__((address_space(4))) const BatchEnv CBatch;

// Waves per SIMD.  4 (at most 128 registers per lane, 10 KB of LDS) where
// dimensions up to 8 share the kernel: 3 (6 %) and 5 (spills) measured slower.
// Batches of at most 5 dimensions have a kernel of their own, which needs
// fewer registers and waits more (their walkers meet obstacles on most steps,
// two dependent loads each): at 5 waves 64.1, 68.7, 71.1 and 60.0e9
// walk-steps/s in 2 to 5 dimensions (256 spheres), 58.4, 62.2, 68.0, 57.2 at 4,
// 63.3, 66.6, 73.8, 55.9 at 6; in the shared kernel 3-D ran at 55.3.  With the
// point-source terms 5 waves are 4 % slower than 4 (spills).
template <bool SRC, int MAXD>
constexpr int kWaves = (MAXD > 5 || SRC) ? 4 : 5;

// Launch shape: 1, 2 or 4 waves per block (the dynamic LDS holds a slice per
// wave, sized by the batch's largest dimension).
template <bool BWD, bool SRC, bool LISTS, int MAXD>
__global__ void __launch_bounds__(4 * kWave, (kWaves<SRC, MAXD>))
persistent_kernel(const EnvP<float>* envs, const BatchEnv* benv, int n_benv, int max_d,
                  const float* __restrict__ queries, int64_t total_units,
                  uint32_t key0, uint32_t key1, const uint64_t* __restrict__ key_add,
                  unsigned* counter, double* __restrict__ partials)
{
    extern __shared__ __align__(16) unsigned char lds_all[];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const WaveLds<float, SRC, LISTS, false> lds(lds_all + wv * wave_lds<float, SRC, LISTS, false>(max_d, kWaves<SRC, MAXD>), max_d,
                                                  kWaves<SRC, MAXD>);
    uint32_t k0 = key0, k1 = key1;
    apply_key_add(k0, k1, key_add);
    CBatch* B = (CBatch*)benv;
    const unsigned one = ((threadIdx.x & (kWave - 1)) == 0) ? 1u : 0u;
    // A wave takes at most total_units units, so the loop is bounded even if
    // the counter were wrong.  Every lane issues the atomic (lane 0 adds 1,
    // the others 0): no lane-dependent branch around it, so the loop stays
    // wave-uniform; lane 0's old value is the unit index.
    for (int64_t taken = 0; taken < total_units; ++taken) {
        const unsigned u = __builtin_amdgcn_readfirstlane(atomicAdd(counter, one));
        if ((int64_t)u >= total_units) break;
        // last env whose first unit is <= u (empty envs share the next offset)
        int lo = 0, hi = n_benv - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (B[mid].unit_off <= (int64_t)u) lo = mid;
            else hi = mid - 1;
        }
        CBatch& be = B[lo];
        const cenv<float> p = (cenv<float>)(envs + be.slot);
        const int64_t local = (int64_t)u - be.unit_off;
        const int64_t ql = local / be.splits;
        const int64_t w_begin = (local - ql * be.splits) * (int64_t)be.wps;
        const int64_t w_end = (w_begin + be.wps < be.n_walks) ? w_begin + be.wps : be.n_walks;
        // walks of the unit counted from w_begin in 32 bits (a unit holds at
        // most wps < 2^31 walks); walk ids are taken modulo 2^32
        const int32_t n = (int32_t)(w_end - w_begin);
        cptr<float> qrow = to_const(queries) + (be.q_off + ql) * be.q_stride;
        double* out = partials + (int64_t)u * kNAccBatch;
#define WOS_UNIT(D)                                                                                               \
    case D:                                                                                                       \
        if constexpr (D <= MAXD)                                                                                  \
            run_unit<float, D, kMaxDim, BWD, SRC, LISTS, false>(p, qrow, (uint32_t)ql, (uint32_t)w_begin, n,       \
                                                                be.lanes, k0, k1, lds, out, nullptr);              \
        break;
        switch (be.d) {
            WOS_UNIT(2)
            WOS_UNIT(3)
            WOS_UNIT(4)
            WOS_UNIT(5)
            WOS_UNIT(6)
            WOS_UNIT(7)
            WOS_UNIT(8)
        }
#undef WOS_UNIT
    }
}

}  // namespace

template <bool BWD, bool SRC, bool LISTS, int MAXD>
static hipError_t persistent_go(int grid, int block, const EnvP<float>* envs, const BatchEnv* benv, int n_benv, int max_d,
                                const float* queries, int64_t total_units, uint32_t key0, uint32_t key1,
                                const uint64_t* key_add, unsigned* counter, double* partials, hipStream_t st)
{
    const size_t lds = (block / kWave) * wave_lds<float, SRC, LISTS, false>(max_d, kWaves<SRC, MAXD>);
    hipLaunchKernelGGL((persistent_kernel<BWD, SRC, LISTS, MAXD>), dim3(grid), dim3(block), lds, st, envs, benv, n_benv,
                       max_d, queries, total_units, key0, key1, key_add, counter, partials);
    return hipGetLastError();
}

template <bool SRC, bool LISTS, int MAXD>
hipError_t launch_persistent_variant(bool bwd, int grid, int block, const EnvP<float>* envs, const BatchEnv* benv,
                                     int n_benv, int max_d, const float* queries, int64_t total_units, uint32_t key0,
                                     uint32_t key1, const uint64_t* key_add, unsigned* counter, double* partials,
                                     hipStream_t st)
{
    if (block != kWave && block != 2 * kWave && block != 4 * kWave) return hipErrorInvalidValue;
    return bwd ? persistent_go<true, SRC, LISTS, MAXD>(grid, block, envs, benv, n_benv, max_d, queries, total_units, key0, key1, key_add, counter, partials, st)
               : persistent_go<false, SRC, LISTS, MAXD>(grid, block, envs, benv, n_benv, max_d, queries, total_units, key0, key1, key_add, counter, partials, st);
}

template <bool SRC, bool LISTS, int MAXD>
int persistent_blocks_per_cu(bool bwd, int max_d, int block)
{
    int per_cu = 0;
    const size_t lds = (block / kWave) * wave_lds<float, SRC, LISTS, false>(max_d, kWaves<SRC, MAXD>);
    const hipError_t e =
        bwd ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, persistent_kernel<true, SRC, LISTS, MAXD>, block, lds)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, persistent_kernel<false, SRC, LISTS, MAXD>, block, lds);
    return (e == hipSuccess && per_cu > 0) ? per_cu : 1;
}

template hipError_t launch_persistent_variant<(WOS_PERSISTENT_SRC != 0), (WOS_PERSISTENT_LISTS != 0), WOS_PERSISTENT_MAXD>(
    bool, int, int, const EnvP<float>*, const BatchEnv*, int, int, const float*, int64_t, uint32_t, uint32_t,
    const uint64_t*, unsigned*, double*, hipStream_t);
template int persistent_blocks_per_cu<(WOS_PERSISTENT_SRC != 0), (WOS_PERSISTENT_LISTS != 0), WOS_PERSISTENT_MAXD>(bool, int, int);

}  // namespace wos
