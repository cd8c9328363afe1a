// wos_walk.hpp -- pieces shared by the walk kernels: the launch's key, the
// contribution of a finished walk to the partial sums and their wave sums.
#pragma once
#include <cmath>

#include "wos_device.hpp"

namespace wos {

constexpr int kBlock = 256;  // 4 waves per block for the plain / finalize kernels
constexpr int kNAccBatch = nacc(kMaxDim);  // a batched partial row

__device__ __forceinline__ void apply_key_add(uint32_t& k0, uint32_t& k1, const uint64_t* key_add)
{
    if (key_add) {
        const uint64_t key = (((uint64_t)k1 << 32) | k0) + *to_const(key_add);
        k0 = (uint32_t)key;
        k1 = (uint32_t)(key >> 32);
    }
}

// Sum the accumulators of a wave and let lane 0 store them.
template <int N>
__device__ __forceinline__ void wave_store(double (&a)[N], double* out)
{
#pragma unroll
    for (int i = 0; i < N; ++i) a[i] = wave_sum(a[i]);
    if ((threadIdx.x & (kWave - 1)) == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) out[i] = a[i];
    }
}

// 2^ex: the factor between a finished walk's stored weighted terms and their
// values (the FP32 walk keeps the weight's exponent apart; FP64 does not).
template <typename T>
__device__ __forceinline__ double walk_scale(const WalkEnd<T>& e)
{
    if (sizeof(T) == 8) return 1.0;
    return ::ldexp(1.0, e.ex);
}

// One-point gradient of a finished walk: gs v0, plus gs0 (z - x_0) when a
// point source lies in the first ball (gs0 carries no weight, so no scale).
template <typename T, int D, int DA, bool SRC>
__device__ __forceinline__ double walk_grad(const WalkEnd<T>& e, const T (&v0)[DA], cenv<T> p, const T* xq, int i,
                                            double sc)
{
    const double g = (double)(e.gs * v0[i]) * sc;
    if (SRC) return g + (double)(e.gs0 * (p->src_z[i] - xq[i]));
    return g;
}

// d u_hat / d sigma of a finished walk: (W g) S, plus the source part.
template <typename T, bool SRC>
__device__ __forceinline__ double walk_dsigma(const WalkEnd<T>& e, double sc)
{
    if (SRC) return ((double)e.ubd * (double)e.S + (double)e.srcS) * sc;
    return (double)e.u * (double)e.S * sc;
}

// Contribution of one finished walk to an accumulator row laid out for DA
// coordinates (nacc(DA) entries), of which the first D are in use.
template <typename T, int D, int DA, bool SRC>
__device__ __forceinline__ void accumulate(double (&a)[nacc(DA)], const WalkEnd<T>& e, const T (&v0)[DA],
                                           cenv<T> p, const T* xq)
{
    const double sc = walk_scale(e);
    const double u = (double)e.u * sc;
    a[0] += u;
    a[1] += u * u;
#pragma unroll
    for (int i = 0; i < D; ++i) {
        const double g = walk_grad<T, D, DA, SRC>(e, v0, p, xq, i, sc);
        a[2 + i] += g;
        a[2 + DA + i] += g * g;
    }
    a[2 + 2 * DA] += (double)e.steps;
    a[3 + 2 * DA] += (e.status == kTruncated) ? 1.0 : 0.0;
    a[4 + 2 * DA] += (e.status == kDegenerate) ? 1.0 : 0.0;
    a[5 + 2 * DA] += walk_dsigma<T, SRC>(e, sc);
    a[6 + 2 * DA] += (double)e.goal_w * sc;
}

// The wave's work tally goes into lane 0's accumulators before the wave sum.
template <int N>
__device__ __forceinline__ void add_work(double (&a)[N], int at, const WorkCount& wc)
{
    if ((threadIdx.x & (kWave - 1)) == 0) {
        a[at] += (double)wc.sph;
        a[at + 1] += (double)wc.box;
        a[at + 2] += (double)wc.cbox;
    }
}

}  // namespace wos
