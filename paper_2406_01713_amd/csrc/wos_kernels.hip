// wos_kernels.hip -- kernels around the walks for gfx950 (CDNA4, wave64), and
// the dispatch of the persistent walk kernel's variants.
//
//   finalize_*         per-query means, standard errors and backward products
//                      from per-wave partial sums, in a fixed order
//   plan_update        one gradient-ascent step of the planning loop
//
// The walk kernels are in wos_plain.hip and wos_persistent.hip, all walk
// arithmetic in wos_device.hpp; the estimator is Sec. IV-A of
// the paper (screened WoS, first-sphere gradient), the step rule Sec. VII.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "wos_launch.hpp"
#include "wos_walk.hpp"

namespace wos {

namespace {

__device__ __forceinline__ double se_of(double s, double s2, double n)
{
    if (n < 2.0) return 0.0;
    const double m = s / n;
    const double var = (s2 - n * m * m) / (n - 1.0);
    return var > 0.0 ? ::sqrt(var / n) : 0.0;
}

// A query's outputs from its sums a (nacc(D) layout) over n_walks walks.
template <typename T, int D, bool BWD>
__device__ __forceinline__ void write_query(const double (&a)[nacc(D)], int64_t q, int64_t n_walks,
                                            T* __restrict__ out_u, T* __restrict__ out_grad,
                                            double* __restrict__ out_stats, const T* __restrict__ ubar,
                                            T* __restrict__ out_dx, double* __restrict__ out_dq,
                                            double* __restrict__ out_jac, double* __restrict__ prod)
{
    const double n = (double)n_walks;
    out_u[q] = (T)(a[0] / n);
    if (out_grad) {
#pragma unroll
        for (int i = 0; i < D; ++i) out_grad[q * D + i] = (T)(a[2 + i] / n);
    }
    if (out_stats) {
        double* st = out_stats + q * (D + 4);
        st[0] = se_of(a[0], a[1], n);
#pragma unroll
        for (int i = 0; i < D; ++i) st[1 + i] = se_of(a[2 + i], a[2 + D + i], n);
        st[D + 1] = a[2 + 2 * D] / n;
        st[D + 2] = a[3 + 2 * D];
        st[D + 3] = a[4 + 2 * D];
    }
    if (BWD && out_jac) {
        double* j = out_jac + q * (D + 2);
#pragma unroll
        for (int i = 0; i < D; ++i) j[i] = a[2 + i] / n;
        j[D] = a[5 + 2 * D] / n;
        j[D + 1] = a[6 + 2 * D] / n;
    }
    if (BWD && ubar) {
        const double ub = (double)ubar[q];
        const double dqs = a[5 + 2 * D] / n, dqg = a[6 + 2 * D] / n;
        if (out_dq) {
            out_dq[2 * q] = dqs;
            out_dq[2 * q + 1] = dqg;
        }
        prod[2 * q] = ub * dqs;
        prod[2 * q + 1] = ub * dqg;
#pragma unroll
        for (int i = 0; i < D; ++i) out_dx[q * D + i] = (T)(ub * (a[2 + i] / n));
    }
}

// One block per query: thread t sums chunks t, t + kBlock, ... in order, then a
// butterfly over each wave and the waves in index order, so the result does
// not depend on timing.
template <typename T, int D, bool BWD>
__global__ void __launch_bounds__(kBlock)
finalize_plain(const double* __restrict__ partials, int64_t n_q, int32_t chunks, int64_t n_walks,
               T* __restrict__ out_u, T* __restrict__ out_grad, double* __restrict__ out_stats,
               const T* __restrict__ ubar, T* __restrict__ out_dx, double* __restrict__ out_dq,
               double* __restrict__ out_jac, double* __restrict__ prod)
{
    const int64_t q = blockIdx.x;
    if (q >= n_q) return;
    constexpr int NA = nacc(D);
    constexpr int NW = kBlock / kWave;
    __shared__ double wsum[NW][NA];
    double a[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) a[i] = 0.0;
    const double* row = partials + q * chunks * NA;
    for (int c = threadIdx.x; c < chunks; c += kBlock) {
#pragma unroll
        for (int i = 0; i < NA; ++i) a[i] += row[(int64_t)c * NA + i];
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) a[i] = wave_sum(a[i]);
    const int wv = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
#pragma unroll
        for (int i = 0; i < NA; ++i) wsum[wv][i] = a[i];
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        a[i] = wsum[0][i];
        for (int w = 1; w < NW; ++w) a[i] += wsum[w][i];
    }
    write_query<T, D, BWD>(a, q, n_walks, out_u, out_grad, out_stats, ubar, out_dx, out_dq, out_jac, prod);
}

// Few chunks per query: one thread sums them in order.  (A block per query
// whose sums are one row each spends 256 threads and their wave sums on it:
// 16384 queries of one chunk in 2-D 124 us, a seventh of the whole call.)
constexpr int kFewChunks = 8;
template <typename T, int D, bool BWD>
__global__ void __launch_bounds__(kWave)
finalize_few(const double* __restrict__ partials, int64_t n_q, int32_t chunks, int64_t n_walks,
             T* __restrict__ out_u, T* __restrict__ out_grad, double* __restrict__ out_stats,
             const T* __restrict__ ubar, T* __restrict__ out_dx, double* __restrict__ out_dq,
             double* __restrict__ out_jac, double* __restrict__ prod)
{
    const int64_t q = (int64_t)blockIdx.x * kWave + threadIdx.x;
    if (q >= n_q) return;
    constexpr int NA = nacc(D);
    double a[NA];
    const double* row = partials + q * chunks * NA;
#pragma unroll
    for (int i = 0; i < NA; ++i) a[i] = row[i];
    for (int c = 1; c < chunks; ++c) {
#pragma unroll
        for (int i = 0; i < NA; ++i) a[i] += row[(int64_t)c * NA + i];
    }
    write_query<T, D, BWD>(a, q, n_walks, out_u, out_grad, out_stats, ubar, out_dx, out_dq, out_jac, prod);
}

// Fixed-order block reduction (deterministic run to run).
__global__ void __launch_bounds__(kBlock)
reduce_pairs(const double* __restrict__ prod, int64_t n, double* out0, double* out1)
{
    __shared__ double s0[kBlock], s1[kBlock];
    double a = 0.0, b = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += kBlock) {
        a += prod[2 * i];
        b += prod[2 * i + 1];
    }
    s0[threadIdx.x] = a;
    s1[threadIdx.x] = b;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            s0[threadIdx.x] += s0[threadIdx.x + w];
            s1[threadIdx.x] += s1[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *out0 = s0[0];
        *out1 = s1[0];
    }
}

template <bool BWD>
__global__ void __launch_bounds__(kBlock)
finalize_batch(const BatchEnv* __restrict__ benv, const double* __restrict__ partials,
               const float* __restrict__ ubar, float* __restrict__ out_u,
               float* __restrict__ out_grad, int grad_stride, double* __restrict__ out_stats,
               float* __restrict__ out_dx, double* __restrict__ out_dsigma,
               double* __restrict__ out_dg, float* __restrict__ out_dir, unsigned* counter)
{
    __shared__ double s0[kBlock], s1[kBlock];
    const BatchEnv be = benv[blockIdx.x];
    const int d = be.d;
    const double n = (double)be.n_walks;
    double bs = 0.0, bg = 0.0;
    // a thread per query, or, with 64 or more walk ranges per query (one
    // planning start with 1e5 walks has about 800), a wave per query whose
    // lanes stride over the ranges and are then summed across the wave
    const bool by_wave = be.splits >= kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int q0 = by_wave ? (int)(threadIdx.x / kWave) : (int)threadIdx.x;
    const int dq = by_wave ? kBlock / kWave : kBlock;
    for (int ql = q0; ql < be.n_q; ql += dq) {  // wave-uniform when by_wave
        double a[kNAccBatch];
#pragma unroll
        for (int i = 0; i < kNAccBatch; ++i) a[i] = 0.0;
        const double* row = partials + (be.unit_off + (int64_t)ql * be.splits) * kNAccBatch;
        if (by_wave) {
            for (int c = lane; c < be.splits; c += kWave)
#pragma unroll
                for (int i = 0; i < kNAccBatch; ++i) a[i] += row[c * kNAccBatch + i];
#pragma unroll
            for (int i = 0; i < kNAccBatch; ++i) a[i] = wave_sum(a[i]);
            if (lane != 0) continue;
        } else {
            for (int c = 0; c < be.splits; ++c)
#pragma unroll
                for (int i = 0; i < kNAccBatch; ++i) a[i] += row[c * kNAccBatch + i];
        }
        const int64_t qg = be.q_off + ql;
        out_u[qg] = (float)(a[0] / n);
        // partial rows use the 8-wide layout of nacc(kMaxDim)
        constexpr int M = kMaxDim;
        if (out_grad)
#pragma unroll
            for (int i = 0; i < M; ++i) out_grad[qg * grad_stride + i] = (i < d) ? (float)(a[2 + i] / n) : 0.0f;
        if (out_dir) {  // unit direction from the FP64 sums, scaled by the largest entry first
            double m = 0.0, g2 = 0.0;
#pragma unroll
            for (int i = 0; i < M; ++i) m = (i < d) ? ::fmax(m, ::fabs(a[2 + i])) : m;
            if (m > 0.0)
#pragma unroll
                for (int i = 0; i < M; ++i) g2 += (i < d) ? (a[2 + i] / m) * (a[2 + i] / m) : 0.0;
            const double r = (g2 > 0.0) ? 1.0 / ::sqrt(g2) : 0.0;
#pragma unroll
            for (int i = 0; i < M; ++i)
                out_dir[qg * grad_stride + i] = (i < d && m > 0.0) ? (float)((a[2 + i] / m) * r) : 0.0f;
        }
        if (out_stats) {
            double* st = out_stats + qg * kBatchStats;
            st[0] = se_of(a[0], a[1], n);
#pragma unroll
            for (int i = 0; i < M; ++i) st[1 + i] = (i < d) ? se_of(a[2 + i], a[2 + M + i], n) : 0.0;
            st[M + 1] = a[2 + 2 * M] / n;
            st[M + 2] = a[3 + 2 * M];
            st[M + 3] = a[4 + 2 * M];
            st[M + 4] = a[7 + 2 * M] / n;                    // sphere distances per walk
            st[M + 5] = a[8 + 2 * M] / n;                    // box distances per walk
            st[M + 6] = (a[2 + 2 * M] / n) * (double)be.n_cl;  // cluster bounds per walk
            st[M + 7] = a[9 + 2 * M] / n;                    // cluster boxes per walk
        }
        if (BWD) {
            const double ub = (double)ubar[qg];
            bs += ub * (a[5 + 2 * M] / n);
            bg += ub * (a[6 + 2 * M] / n);
#pragma unroll
            for (int i = 0; i < kMaxDim; ++i)
                out_dx[qg * kBatchStride + i] = (i < d) ? (float)(ub * (a[2 + i] / n)) : 0.0f;
        }
    }
    if (BWD) {
        s0[threadIdx.x] = bs;
        s1[threadIdx.x] = bg;
        __syncthreads();
        for (int w = kBlock / 2; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) {
                s0[threadIdx.x] += s0[threadIdx.x + w];
                s1[threadIdx.x] += s1[threadIdx.x + w];
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            out_dsigma[be.slot] = s0[0];
            out_dg[be.slot] = s1[0];
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *counter = 0u;  // ready for the next launch
}

// ------------------------------------------------------------------------
// Planning update (Sec. III gradient ascent, Sec. VII step rule).
// ------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(kBlock)
plan_update(const EnvP<float>* penv, float* __restrict__ x, int64_t n, const float* __restrict__ dir,
            int grad_stride, float s_ub, double* __restrict__ path_len, int32_t* __restrict__ stalls,
            int32_t* __restrict__ status, uint64_t* step)
{
    __shared__ uint32_t pair_lds[kBlock / kWave][kPairLds];
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const cenv<float> p = (cenv<float>)penv;
    // every lane evaluates the distance (the matrix-core cluster test needs
    // the whole wave); lanes past n use start 0 (or the origin) and write nothing
    const bool valid = s < n;
    const int64_t si = valid ? s : 0;
    float xs[D];
#pragma unroll
    for (int i = 0; i < D; ++i) xs[i] = (n > 0) ? x[si * D + i] : 0.0f;
    WorkCount wc(pair_lds[__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)]);
    const Near<float> near = distance<float, D, false>(p, xs, wc, valid, Math<float>::inf());
    const float R = near.R();
    if (valid) {
        float dz2 = 0.0f;
        if (p->has_src) {
#pragma unroll
            for (int i = 0; i < D; ++i) dz2 = Math<float>::fma(xs[i] - p->src_z[i], xs[i] - p->src_z[i], dz2);
        }
        if (R < p->eps) {
            status[s] = (near.cls() == kGoal) ? 1 : 2;
        } else if (p->has_src && dz2 < s_ub * s_ub) {
            status[s] = 1;  // a point-source goal is reached within one nominal step
        } else {
            status[s] = 0;
            float g[D];
            float g2 = 0.0f;
#pragma unroll
            for (int i = 0; i < D; ++i) {
                g[i] = dir[s * grad_stride + i];
                g2 = Math<float>::fma(g[i], g[i], g2);
            }
            if (g2 == 0.0f) {
                stalls[s] += 1;
            } else {
                const float h = Math<float>::min(s_ub, 0.5f * R);
                const float f = h / ::sqrtf(g2);
#pragma unroll
                for (int i = 0; i < D; ++i) x[s * D + i] = Math<float>::fma(f, g[i], xs[i]);
                path_len[s] += (double)h;
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *step += 1;
}

// ------------------------------------------------------------------------
// Varadhan read-out (Sec. III, eq. transformation_varadhan): w = -sqrt(t) ln u,
// t = 1 / sigma, grad w = -sqrt(t) grad u / u; u <= 0 (no signal) gives
// w = +inf and grad w = 0.  One thread per query.
// ------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(kBlock)
varadhan_kernel(const T* __restrict__ u, const T* __restrict__ grad, int64_t n, int d, int stride,
                T sqrt_t, T* __restrict__ w, T* __restrict__ grad_w)
{
    const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= n) return;
    const T uq = u[q];
    const bool ok = uq > T(0);
    w[q] = ok ? -sqrt_t * ::log(uq) : Math<T>::inf();
    if (grad_w) {
        const T f = ok ? -sqrt_t / uq : T(0);
        for (int i = 0; i < d; ++i) grad_w[q * stride + i] = f * grad[q * stride + i];
    }
}

__global__ void fill_u32(unsigned* p, int64_t n, unsigned v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void fill_f64(double* p, int64_t n, double v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

// ------------------------------------------------------------------------
// Launchers.
// ------------------------------------------------------------------------
template <typename T, int D>
static hipError_t fin_d(bool bwd, const double* partials, int64_t n_q, int32_t chunks, int64_t n_walks,
                        T* out_u, T* out_grad, double* out_stats, const T* ubar, T* out_dx,
                        double* out_dq, double* out_jac, double* prod, hipStream_t st)
{
    if (n_q == 0) return hipSuccess;
    auto* go = chunks <= kFewChunks ? (bwd ? finalize_few<T, D, true> : finalize_few<T, D, false>)
                                    : (bwd ? finalize_plain<T, D, true> : finalize_plain<T, D, false>);
    const unsigned grid = chunks <= kFewChunks ? blocks_for(n_q, kWave) : (unsigned)n_q;
    hipLaunchKernelGGL(go, dim3(grid), dim3(chunks <= kFewChunks ? kWave : kBlock), 0, st, partials, n_q, chunks,
                       n_walks, out_u, out_grad, out_stats, ubar, out_dx, out_dq, out_jac, prod);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_finalize_plain(int d, bool bwd, const double* partials, int64_t n_q, int32_t chunks,
                                 int64_t n_walks, T* out_u, T* out_grad, double* out_stats,
                                 const T* ubar, T* out_dx, double* out_dq, double* out_jac,
                                 double* prod, hipStream_t st)
{
    switch (d) {
    case 2: return fin_d<T, 2>(bwd, partials, n_q, chunks, n_walks, out_u, out_grad, out_stats, ubar, out_dx, out_dq, out_jac, prod, st);
    case 3: return fin_d<T, 3>(bwd, partials, n_q, chunks, n_walks, out_u, out_grad, out_stats, ubar, out_dx, out_dq, out_jac, prod, st);
    case 4: return fin_d<T, 4>(bwd, partials, n_q, chunks, n_walks, out_u, out_grad, out_stats, ubar, out_dx, out_dq, out_jac, prod, st);
    case 5: return fin_d<T, 5>(bwd, partials, n_q, chunks, n_walks, out_u, out_grad, out_stats, ubar, out_dx, out_dq, out_jac, prod, st);
    case 6: return fin_d<T, 6>(bwd, partials, n_q, chunks, n_walks, out_u, out_grad, out_stats, ubar, out_dx, out_dq, out_jac, prod, st);
    case 7: return fin_d<T, 7>(bwd, partials, n_q, chunks, n_walks, out_u, out_grad, out_stats, ubar, out_dx, out_dq, out_jac, prod, st);
    case 8: return fin_d<T, 8>(bwd, partials, n_q, chunks, n_walks, out_u, out_grad, out_stats, ubar, out_dx, out_dq, out_jac, prod, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_finalize_plain<float>(int, bool, const double*, int64_t, int32_t, int64_t, float*,
                                                 float*, double*, const float*, float*, double*, double*, double*,
                                                 hipStream_t);
template hipError_t launch_finalize_plain<double>(int, bool, const double*, int64_t, int32_t, int64_t,
                                                  double*, double*, double*, const double*, double*,
                                                  double*, double*, double*, hipStream_t);

hipError_t launch_reduce_pairs(const double* prod, int64_t n, double* out0, double* out1, hipStream_t st)
{
    hipLaunchKernelGGL(reduce_pairs, dim3(1), dim3(kBlock), 0, st, prod, n, out0, out1);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_plain(int d, bool bwd, bool src, bool lists, const EnvP<T>* p, const T* queries, int64_t n_q,
                        int64_t n_walks, int32_t wpu, int lanes, int64_t w_base, uint32_t q_base, double* partials,
                        double* records, hipStream_t st)
{
#define WOS_PLAIN_CASE(D) \
    case D: return launch_plain_d<T, D>(bwd, src, lists, p, queries, n_q, n_walks, wpu, lanes, w_base, q_base, partials, records, st);
    switch (d) {
        WOS_PLAIN_CASE(2)
        WOS_PLAIN_CASE(3)
        WOS_PLAIN_CASE(4)
        WOS_PLAIN_CASE(5)
        WOS_PLAIN_CASE(6)
        WOS_PLAIN_CASE(7)
        WOS_PLAIN_CASE(8)
    default: return hipErrorInvalidValue;
    }
#undef WOS_PLAIN_CASE
}
template hipError_t launch_plain<float>(int, bool, bool, bool, const EnvP<float>*, const float*, int64_t, int64_t,
                                        int32_t, int, int64_t, uint32_t, double*, double*, hipStream_t);
template hipError_t launch_plain<double>(int, bool, bool, bool, const EnvP<double>*, const double*, int64_t, int64_t,
                                         int32_t, int, int64_t, uint32_t, double*, double*, hipStream_t);

// f(SRC, LISTS, MAXD) as constants: the variant for a batch's features (the
// kernel for at most 5 dimensions reads lists only).
template <typename F>
static auto persistent_variant(bool src, bool lists, int max_d, F f)
{
    using std::integral_constant;
    using Y = std::true_type;
    using N = std::false_type;
    using Any = integral_constant<int, kMaxDim>;
    using Low = integral_constant<int, 5>;
    if (!lists) return src ? f(Y{}, N{}, Any{}) : f(N{}, N{}, Any{});
    if (max_d > Low::value) return src ? f(Y{}, Y{}, Any{}) : f(N{}, Y{}, Any{});
    return src ? f(Y{}, Y{}, Low{}) : f(N{}, Y{}, Low{});
}

hipError_t launch_persistent(bool bwd, bool src, bool lists, int grid, int block, const EnvP<float>* envs,
                             const BatchEnv* benv, int n_benv, int max_d, const float* queries, int64_t total_units,
                             uint32_t key0, uint32_t key1, const uint64_t* key_add, unsigned* counter,
                             double* partials, hipStream_t st)
{
    if (total_units == 0) return hipSuccess;
    return persistent_variant(src, lists, max_d, [&](auto s, auto l, auto m) {
        return launch_persistent_variant<s.value, l.value, m.value>(bwd, grid, block, envs, benv, n_benv, max_d,
                                                                    queries, total_units, key0, key1, key_add, counter,
                                                                    partials, st);
    });
}

int persistent_resident_blocks(bool bwd, bool src, bool lists, int max_d, int block)
{
    const int per_cu = persistent_variant(src, lists, max_d, [&](auto s, auto l, auto m) {
        return persistent_blocks_per_cu<s.value, l.value, m.value>(bwd, max_d, block);
    });
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return per_cu;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 1;
    return per_cu * cus;
}

hipError_t launch_finalize_batch(bool bwd, const BatchEnv* benv, int n_benv, const double* partials,
                                 const float* ubar, float* out_u, float* out_grad,
                                 int grad_stride, double* out_stats, float* out_dx, double* out_dsigma,
                                 double* out_dg, float* out_dir, unsigned* counter, hipStream_t st)
{
    if (n_benv == 0) return hipSuccess;
    if (bwd)
        hipLaunchKernelGGL(finalize_batch<true>, dim3(n_benv), dim3(kBlock), 0, st, benv, partials, ubar, out_u,
                           out_grad, grad_stride, out_stats, out_dx, out_dsigma, out_dg, out_dir, counter);
    else
        hipLaunchKernelGGL(finalize_batch<false>, dim3(n_benv), dim3(kBlock), 0, st, benv, partials, ubar, out_u,
                           out_grad, grad_stride, out_stats, out_dx, out_dsigma, out_dg, out_dir, counter);
    return hipGetLastError();
}

hipError_t launch_plan_update(int d, const EnvP<float>* p, float* x, int64_t n, const float* dir,
                              int grad_stride, float s_ub, double* path_len, int32_t* stalls,
                              int32_t* status, uint64_t* step, hipStream_t st)
{
    const unsigned grid = n > 0 ? blocks_for(n, kBlock) : 1u;
#define WOS_PLAN_CASE(DD)                                                                              \
    case DD:                                                                                           \
        hipLaunchKernelGGL(plan_update<DD>, dim3(grid), dim3(kBlock), 0, st, p, x, n, dir, grad_stride,  \
                           s_ub, path_len, stalls, status, step);                                      \
        break;
    switch (d) {
        WOS_PLAN_CASE(2)
        WOS_PLAN_CASE(3)
        WOS_PLAN_CASE(4)
        WOS_PLAN_CASE(5)
        WOS_PLAN_CASE(6)
        WOS_PLAN_CASE(7)
        WOS_PLAN_CASE(8)
    default: return hipErrorInvalidValue;
    }
#undef WOS_PLAN_CASE
    return hipGetLastError();
}

template <typename T>
hipError_t launch_varadhan(const T* u, const T* grad, int64_t n, int d, int stride, double sigma, T* w,
                           T* grad_w, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const T sqrt_t = (T)(1.0 / std::sqrt(sigma));
    hipLaunchKernelGGL((varadhan_kernel<T>), dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, st, u, grad, n, d,
                       stride, sqrt_t, w, grad_w);
    return hipGetLastError();
}
template hipError_t launch_varadhan<float>(const float*, const float*, int64_t, int, int, double, float*, float*,
                                           hipStream_t);
template hipError_t launch_varadhan<double>(const double*, const double*, int64_t, int, int, double, double*,
                                            double*, hipStream_t);

hipError_t launch_fill_u32(unsigned* p, int64_t n, unsigned v, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, st, p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_f64(double* p, int64_t n, double v, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_f64, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, st, p, n, v);
    return hipGetLastError();
}

}  // namespace wos
