// wos_persistent.hip -- persistent_kernel: ragged batch of environments in one
// launch: resident waves pull work units (env, query, walk range) from a
// device counter, and a lane whose walk ends starts the unit's next walk at
// once (lane refill), so a wave is not held by its longest walk.  Compiled
// without and with point-source terms (WOS_PERSISTENT_SRC = 0, 1), and with
// steps that scan clusters or read cell lists (WOS_PERSISTENT_LISTS = 0, 1).
#include <hip/hip_runtime.h>

#include "wos_launch.hpp"
#include "wos_walk.hpp"

namespace wos {

namespace {

// ------------------------------------------------------------------------
// Persistent ragged-batch kernel (FP32).
// ------------------------------------------------------------------------
typedef __attribute__((address_space(4))) const BatchEnv CBatch;

// One walk step of an env of dimension d on the shared 8-wide walker state.
template <bool BWD, bool SRC, bool LISTS>
__device__ __forceinline__ bool step_any_d(int d, cenv<float> p, Walker<float, kMaxDim>& s, uint32_t q,
                                           uint32_t k0, uint32_t k1, WalkEnd<float>& e, WorkCount& wc,
                                           bool live, const UnitStart<float>& st)
{
    switch (d) {
    case 2: return walker_step<float, 2, BWD, LISTS, kMaxDim, SRC>(p, s, q, k0, k1, e, wc, live, st);
    case 3: return walker_step<float, 3, BWD, LISTS, kMaxDim, SRC>(p, s, q, k0, k1, e, wc, live, st);
    case 4: return walker_step<float, 4, BWD, LISTS, kMaxDim, SRC>(p, s, q, k0, k1, e, wc, live, st);
    case 5: return walker_step<float, 5, BWD, LISTS, kMaxDim, SRC>(p, s, q, k0, k1, e, wc, live, st);
    case 6: return walker_step<float, 6, BWD, LISTS, kMaxDim, SRC>(p, s, q, k0, k1, e, wc, live, st);
    case 7: return walker_step<float, 7, BWD, LISTS, kMaxDim, SRC>(p, s, q, k0, k1, e, wc, live, st);
    default: return walker_step<float, 8, BWD, LISTS, kMaxDim, SRC>(p, s, q, k0, k1, e, wc, live, st);
    }
}

__device__ __forceinline__ UnitStart<float> start_any_d(int d, cenv<float> p, const float (&xq)[kMaxDim], WorkCount& wc)
{
    switch (d) {
    case 2: return unit_start<float, 2, kMaxDim>(p, xq, wc);
    case 3: return unit_start<float, 3, kMaxDim>(p, xq, wc);
    case 4: return unit_start<float, 4, kMaxDim>(p, xq, wc);
    case 5: return unit_start<float, 5, kMaxDim>(p, xq, wc);
    case 6: return unit_start<float, 6, kMaxDim>(p, xq, wc);
    case 7: return unit_start<float, 7, kMaxDim>(p, xq, wc);
    default: return unit_start<float, 8, kMaxDim>(p, xq, wc);
    }
}

// Gradient sums and sums of squares of a work unit (2 x kMaxDim doubles per
// lane) live in LDS: they change only when a walk ends, and keeping them out
// of registers leaves the walk loop without register spills.  Layout per
// wave: [entry][lane], so a wave's accesses to one entry are contiguous.
constexpr int kLdsAcc = 2 * kMaxDim;

// One work unit: walks [w_begin, w_end) of one query, with lane refill.  The
// walker state is 8 wide for every d, so the dimension only selects the step
// code.  Accumulators other than the gradient ones stay in registers.
template <bool BWD, bool SRC, bool LISTS>
__device__ __forceinline__ void run_unit(cenv<float> p, CBatch& be, int64_t local, const float* queries,
                                         uint32_t k0, uint32_t k1, double* lds, uint32_t* pairs, double* out)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int d = be.d;
    const int64_t n_walks = be.n_walks;
    const int64_t ql = local / be.splits;
    const int64_t sp = local - ql * be.splits;
    const int64_t w_begin = sp * (int64_t)be.wps;
    const int64_t w_end = (w_begin + be.wps < n_walks) ? w_begin + be.wps : n_walks;
    // walks of the unit counted from w_begin in 32 bits (a unit holds at
    // most wps < 2^31 walks); walk ids are taken modulo 2^32 as before
    const int32_t n_unit = (int32_t)(w_end - w_begin);
    const uint32_t id0 = (uint32_t)w_begin;

    float xq[kMaxDim];
    cptr<float> qrow = to_const(queries) + (be.q_off + ql) * be.q_stride;
#pragma unroll
    for (int i = 0; i < kMaxDim; ++i) xq[i] = (i < d) ? qrow[i < d ? i : 0] : 0.0f;

    // registers: [0] u, [1] u^2, then steps, truncated, degenerate, u S,
    // goal weight, sphere and box distances and cluster boxes (the nacc
    // layout without the gradient entries; the last three from the wave's
    // work tally)
    constexpr int NR = kNAccBatch - kLdsAcc;
    double a[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) a[i] = 0.0;
    double* g = lds + lane;
#pragma unroll
    for (int i = 0; i < kLdsAcc; ++i) g[i * kWave] = 0.0;

    // lanes [0, be.lanes) carry walks; the rest (with more than one lane per
    // walker) only take part in the member scans of the pair rounds
    const int lanes = be.lanes;
    Walker<float, kMaxDim> s;
    bool active = lane < lanes && lane < n_unit;
    walker_start<float, kMaxDim, kMaxDim>(s, xq, id0 + (uint32_t)lane);
    int32_t base = lanes;
    const uint32_t qi = (uint32_t)ql;
    WorkCount wc(pairs);
    const UnitStart<float> st = start_any_d(d, p, xq, wc);

    while (__builtin_amdgcn_ballot_w64(active) != 0) {
        WalkEnd<float> e;
        // idle lanes (the unit has no walks left for them) step along
        bool fin = step_any_d<BWD, SRC, LISTS>(d, p, s, qi, k0, k1, e, wc, active, st);
        fin = fin && active;
        {
            if (fin) {
                const double sc = walk_scale(e);
                const double u = (double)e.u * sc;
                a[0] += u;
                a[1] += u * u;
                a[2] += (double)e.steps;
                a[3] += (e.status == kTruncated) ? 1.0 : 0.0;
                a[4] += (e.status == kDegenerate) ? 1.0 : 0.0;
                a[5] += walk_dsigma<float, SRC>(e, sc);
                a[6] += (double)e.goal_w * sc;
                // static indices (unrolled, guarded by d) keep the walker in
                // registers; a runtime loop bound would index it dynamically
                // and move it to scratch memory
#pragma unroll
                for (int i = 0; i < kMaxDim; ++i) {
                    if (i < d) {
                        const double gi = walk_grad<float, kMaxDim, kMaxDim, SRC>(e, s.v0, p, xq, i, sc);
                        g[i * kWave] += gi;
                        g[(kMaxDim + i) * kWave] += gi * gi;
                    }
                }
            }
        }
        // lane refill: finished lanes take the unit's next walks in lane order
        const uint64_t m = __builtin_amdgcn_ballot_w64(fin);
        if (m) {
            if (fin) {
                const uint32_t rank =
                    __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                const int32_t wn = base + (int32_t)rank;
                if (wn < n_unit) {
                    walker_start<float, kMaxDim, kMaxDim>(s, xq, id0 + (uint32_t)wn);
                } else {
                    active = false;
                }
            }
            base += __popcll(m);
        }
    }
    add_work(a, 7, wc);
    // back to the nacc(kMaxDim) layout for the partial row
    double row[kNAccBatch];
    row[0] = a[0];
    row[1] = a[1];
#pragma unroll
    for (int i = 0; i < kLdsAcc; ++i) row[2 + i] = g[i * kWave];
#pragma unroll
    for (int i = 2; i < NR; ++i) row[kLdsAcc + i] = a[i];
    wave_store<kNAccBatch>(row, out);
}

// LDS of a wave: the gradient accumulators, then the pair-scan slice.
constexpr size_t kWaveLds = kLdsAcc * kWave * sizeof(double) + kPairLds * sizeof(uint32_t);

// Launch shape: 1, 2 or 4 waves per block (the dynamic LDS holds a kWaveLds
// slice per wave) and at least 4 resident waves per SIMD in every shape (the
// second launch bound: at most 128 registers per lane).  4 waves per SIMD
// measured faster than 3 (6 %) or 5 (18 %, spills).
template <bool BWD, bool SRC, bool LISTS>
__global__ void __launch_bounds__(4 * kWave, 4)
persistent_kernel(const EnvP<float>* envs, const BatchEnv* benv, int n_benv,
                  const float* __restrict__ queries, int64_t total_units,
                  uint32_t key0, uint32_t key1, const uint64_t* __restrict__ key_add,
                  unsigned* counter, double* __restrict__ partials)
{
    extern __shared__ __align__(16) unsigned char wave_lds[];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    double* lds = reinterpret_cast<double*>(wave_lds + wv * kWaveLds);
    uint32_t* pairs = reinterpret_cast<uint32_t*>(lds + kLdsAcc * kWave);
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
        run_unit<BWD, SRC, LISTS>(p, be, (int64_t)u - be.unit_off, queries, k0, k1, lds, pairs,
                           partials + (int64_t)u * kNAccBatch);
    }
}

}  // namespace

template <bool BWD, bool SRC, bool LISTS>
static hipError_t persistent_go(int grid, int block, const EnvP<float>* envs, const BatchEnv* benv, int n_benv,
                                const float* queries, int64_t total_units, uint32_t key0, uint32_t key1,
                                const uint64_t* key_add, unsigned* counter, double* partials, hipStream_t st)
{
    hipLaunchKernelGGL((persistent_kernel<BWD, SRC, LISTS>), dim3(grid), dim3(block), (block / kWave) * kWaveLds, st, envs,
                       benv, n_benv, queries, total_units, key0, key1, key_add, counter, partials);
    return hipGetLastError();
}

template <bool SRC, bool LISTS>
hipError_t launch_persistent_variant(bool bwd, int grid, int block, const EnvP<float>* envs, const BatchEnv* benv,
                                     int n_benv, const float* queries, int64_t total_units, uint32_t key0,
                                     uint32_t key1, const uint64_t* key_add, unsigned* counter, double* partials,
                                     hipStream_t st)
{
    if (block != kWave && block != 2 * kWave && block != 4 * kWave) return hipErrorInvalidValue;
    return bwd ? persistent_go<true, SRC, LISTS>(grid, block, envs, benv, n_benv, queries, total_units, key0, key1, key_add, counter, partials, st)
               : persistent_go<false, SRC, LISTS>(grid, block, envs, benv, n_benv, queries, total_units, key0, key1, key_add, counter, partials, st);
}

template <bool SRC, bool LISTS>
int persistent_blocks_per_cu(bool bwd, int block)
{
    int per_cu = 0;
    const size_t lds = (block / kWave) * kWaveLds;
    const hipError_t e =
        bwd ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, persistent_kernel<true, SRC, LISTS>, block, lds)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, persistent_kernel<false, SRC, LISTS>, block, lds);
    return (e == hipSuccess && per_cu > 0) ? per_cu : 1;
}

template hipError_t launch_persistent_variant<(WOS_PERSISTENT_SRC != 0), (WOS_PERSISTENT_LISTS != 0)>(
    bool, int, int, const EnvP<float>*, const BatchEnv*, int, const float*, int64_t, uint32_t, uint32_t,
    const uint64_t*, unsigned*, double*, hipStream_t);
template int persistent_blocks_per_cu<(WOS_PERSISTENT_SRC != 0), (WOS_PERSISTENT_LISTS != 0)>(bool, int);

}  // namespace wos
