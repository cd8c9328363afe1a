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
__device__ __forceinline__ double walk_scale(int32_t ex)
{
    if (sizeof(T) == 8) return 1.0;
    return ::ldexp(1.0, ex);
}

// One-point gradient of a finished walk: gs v0, plus gs0 (z - x_0) when a
// point source lies in the first ball (gs0 carries no weight, so no scale).
template <typename T, int D, bool SRC>
__device__ __forceinline__ double walk_grad(const WalkEnd<T>& e, const T (&v0)[D], cenv<T> p, const T (&xq)[D], int i,
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

// ------------------------------------------------------------------------
// One work unit: walks [0, n) of one query, with lane refill: a lane whose
// walk ends starts the unit's next walk at once and makes its first step, from
// the query point's distance (UnitStart), in the same iteration.
//
// A finished walk leaves a record in the wave's LDS queue.  Records are added
// up when the queue is nearly full and at the unit's end, one per lane: the
// walk's first direction is drawn again there, so the walk loop carries
// neither it nor the FP64 sums' arithmetic.  (Adding each walk up when it
// ended cost about 80 vector instructions in every iteration in which any of
// the 64 walks did, half of them in 7-D and all in 2-D, and eight registers
// and seven selects per step for the direction.)
//
// LDS of a wave: gradient sums and their squares, [2 dim][64] doubles per
// lane; the record queue of `cap` entries (kRecReal values of T, then two or
// four words); and the scan's slice.
// ------------------------------------------------------------------------
template <bool SRC>
constexpr int kRecReal = SRC ? 7 : 4;
template <bool REC>
constexpr int kRecWord = REC ? 4 : 2;

// Scan slices: the pair scan's, or the cell lists' (cell_min).
template <bool LISTS>
constexpr int kScanLds = LISTS ? 2 * kWave : kPairLds;

// Queue entries and LDS bytes of a wave in a launch whose largest dimension
// is d, at `waves` resident waves per SIMD of a CU's 160 KB.
template <typename T, bool SRC, bool LISTS, bool REC>
constexpr int rec_cap(int d, int waves)
{
    const size_t fixed = (size_t)2 * d * kWave * sizeof(double) + kScanLds<LISTS> * sizeof(uint32_t);
    const size_t rec = kRecReal<SRC> * sizeof(T) + kRecWord<REC> * sizeof(uint32_t);
    const size_t cap = ((size_t)163840 / (4 * waves) / 64 * 64 - fixed) / rec;
    return cap > (size_t)kWave ? kWave : (int)cap;
}
template <typename T, bool SRC, bool LISTS, bool REC>
constexpr size_t wave_lds(int d, int waves)
{
    return ((size_t)2 * d * kWave * sizeof(double) + kScanLds<LISTS> * sizeof(uint32_t) +
            rec_cap<T, SRC, LISTS, REC>(d, waves) * (kRecReal<SRC> * sizeof(T) + kRecWord<REC> * sizeof(uint32_t)) +
            15) / 16 * 16;
}

// The wave's slice, laid out for dimension `dim` (the launch's largest).
template <typename T, bool SRC, bool LISTS, bool REC>
struct WaveLds {
    double* g;
    T* real;
    uint32_t* word;
    uint32_t* scan;
    int cap;
    __device__ __forceinline__ WaveLds(unsigned char* base, int dim, int waves)
        : cap(rec_cap<T, SRC, LISTS, REC>(dim, waves))
    {
        g = reinterpret_cast<double*>(base);
        real = reinterpret_cast<T*>(g + 2 * dim * kWave);
        word = reinterpret_cast<uint32_t*>(real + kRecReal<SRC> * cap);
        scan = word + kRecWord<REC> * cap;
    }
};

// The unit's sums go to `out` in the nacc(DA) layout.  id0: the first walk's
// index word; lanes: lanes that carry walks (the others only take part in
// the scans); records (REC): rows of walks, at the unit's first.
template <typename T, int D, int DA, bool BWD, bool SRC, bool LISTS, bool REC>
__device__ __forceinline__ void run_unit(cenv<T> p, cptr<T> qrow, uint32_t q, uint32_t id0, int32_t n, int lanes,
                                         uint32_t k0, uint32_t k1, const WaveLds<T, SRC, LISTS, REC>& lds,
                                         double* out, double* records)
{
    const int lane = threadIdx.x & (kWave - 1);
    constexpr bool kBound = D <= kStepBoundMaxDim;
    T xq[D];
#pragma unroll
    for (int i = 0; i < D; ++i) xq[i] = qrow[i];
    WorkCount wc(lds.scan);
    const UnitStart<T> st = unit_start<T, D>(p, xq, n, wc);

    // sums of u, u^2, u S and the goal weight; steps, truncated and degenerate
    // walks are counted for the wave
    double su = 0.0, su2 = 0.0, sS = 0.0, sg = 0.0;
    uint64_t steps = (uint64_t)n, trunc = 0, degen = 0;
    double* g = lds.g + lane;
#pragma unroll
    for (int i = 0; i < 2 * D; ++i) g[i * kWave] = 0.0;
    int qn = 0;  // records waiting

    const bool absorbed0 = st.R < p->eps, first_only = absorbed0 || p->max_steps <= 1;
    if (first_only) {  // every walk ends at the query point
        const double u = absorbed0 ? (double)st.g : 0.0;
        if (lane == 0) {
            su = u * n;
            su2 = u * u * n;
            sS = u * 0.0 * n;
            sg = (absorbed0 && st.cls == kGoal) ? (double)n : 0.0;
        }
        (absorbed0 ? degen : trunc) = (uint64_t)n;
        if (REC && records)
            for (int32_t w = lane; w < n; w += kWave) {
                double* r = records + (int64_t)w * (D + 7);
                for (int i = 0; i < D + 7; ++i) r[i] = 0.0;
                r[0] = u;
                r[D + 2] = (absorbed0 && st.cls == kGoal) ? 1.0 : 0.0;
                r[D + 3] = 1.0;
                r[D + 4] = absorbed0 ? (double)kDegenerate : (double)kTruncated;
                r[D + 5] = (double)st.cls;
                r[D + 6] = u * 0.0;
            }
    }

    Walker<T, D> s;
    bool active = !first_only && lane < lanes && lane < n;
    walker_start<T, D>(s, xq, st.R, lane);
    const T rb_abs = p->rb_abs, eps = p->eps;
    const uint32_t max_steps = p->max_steps, env = p->env_id;
    int32_t base = lanes;
    for (;;) {
        const bool any = __builtin_amdgcn_ballot_w64(active) != 0;  // wave-uniform, as everything about the queue
        bool fin = false;
        Near<T> near = {};
        uint64_t m = 0;
        if (any) {
            walker_move<T, D, BWD, SRC>(p, s, active, id0 + (uint32_t)s.w, q, env, k0, k1);
            // R(x) is a minimum of distances, each 1-Lipschitz, and the walker
            // moved R: the next R is at most 2 R, and with the margins (rb_abs
            // covers the rounding of the positions and of every component's
            // computed distance, +inf where coordinates are unbounded) at most
            // this computed bound, so it is a threshold the scans may cull
            // against (in the dimensions where it does, kStepBoundMaxDim)
            // without changing R or its component.  2 (1 + 2^-10) R
            T ub = Math<T>::inf();
            if (kBound) ub = Math<T>::fma(s.R, T(2.001953125), rb_abs);
            near = distance<T, D, LISTS>(fresh(p), s.x, wc, active, ub);
            s.R = near.R();
            const uint64_t act = __builtin_amdgcn_ballot_w64(active);
            steps += (uint64_t)__popcll(act);
            fin = active && (s.R < eps || s.k + 1 >= max_steps);
            m = __builtin_amdgcn_ballot_w64(fin);
            if (m == 0) continue;
        }
        int left = __popcll(m);
        const int rank =
            (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        int from = 0;
        for (;;) {
            const int take = left < lds.cap ? left : lds.cap;
            if (qn > 0 && (!any || qn + take > lds.cap)) {
                // add the waiting records up, one per lane
                wave_lds_fence();
                if (lane < qn) {
                    WalkEnd<T> e;
                    const T* r = lds.real + lane;
                    const uint32_t* wd = lds.word + lane;
                    e.u = r[0];
                    e.gs = r[lds.cap];
                    e.S = r[2 * lds.cap];
                    e.goal_w = r[3 * lds.cap];
                    e.gs0 = SRC ? r[(SRC ? 4 : 0) * lds.cap] : T(0);
                    e.ubd = SRC ? r[(SRC ? 5 : 0) * lds.cap] : T(0);
                    e.srcS = SRC ? r[(SRC ? 6 : 0) * lds.cap] : T(0);
                    e.ex = (int32_t)wd[0];
                    const uint32_t w = wd[lds.cap];
                    T v0[D];
                    direction<T, D>(0u, id0 + w, q, env, k0, k1, v0);
                    const double sc = walk_scale<T>(e.ex);
                    const double u = (double)e.u * sc;
                    su += u;
                    su2 += u * u;
                    sS += walk_dsigma<T, SRC>(e, sc);
                    sg += (double)e.goal_w * sc;
                    double* rec = nullptr;
                    if (REC && records) rec = records + (int64_t)w * (D + 7);
#pragma unroll
                    for (int i = 0; i < D; ++i) {
                        const double gi = walk_grad<T, D, SRC>(e, v0, p, xq, i, sc);
                        g[i * kWave] += gi;
                        g[(D + i) * kWave] += gi * gi;
                        if (REC && rec) rec[1 + i] = gi;
                    }
                    if (REC && rec) {
                        const uint32_t end = wd[(REC ? 3 : 0) * lds.cap];
                        rec[0] = u;
                        rec[D + 1] = (double)e.S;
                        rec[D + 2] = (double)e.goal_w * sc;
                        rec[D + 3] = (double)wd[(REC ? 2 : 0) * lds.cap];
                        rec[D + 4] = (double)(end & 0xFFu);
                        rec[D + 5] = (double)(end >> 8);
                        rec[D + 6] = walk_dsigma<T, SRC>(e, sc);
                    }
                }
                wave_lds_fence();
                qn = 0;
            }
            if (left == 0) break;
            if (fin && rank >= from && rank < from + take) {
                WalkEnd<T> e = {};
                const bool cut = !(s.R < eps);  // truncated: contributes nothing
                const int cls = end_cls<T, D, LISTS>(fresh(p), s.x, near);
                if (!cut) e = walker_end<T, D, LISTS, SRC>(fresh(p), s, cls, st.gfac);
                const int at = qn + rank - from;
                T* r = lds.real + at;
                uint32_t* wd = lds.word + at;
                r[0] = e.u;
                r[lds.cap] = e.gs;
                r[2 * lds.cap] = e.S;
                r[3 * lds.cap] = e.goal_w;
                if (SRC) {
                    r[(SRC ? 4 : 0) * lds.cap] = e.gs0;
                    r[(SRC ? 5 : 0) * lds.cap] = e.ubd;
                    r[(SRC ? 6 : 0) * lds.cap] = e.srcS;
                }
                wd[0] = (uint32_t)e.ex;
                wd[lds.cap] = (uint32_t)s.w;
                if (REC) {
                    wd[(REC ? 2 : 0) * lds.cap] = s.k + 1;
                    wd[(REC ? 3 : 0) * lds.cap] = (uint32_t)(cut ? kTruncated : kAbsorbed) | ((uint32_t)cls << 8);
                }
            }
            qn += take;
            from += take;
            left -= take;
        }
        if (!any) break;
        if (m) {
            trunc += (uint64_t)__popcll(__builtin_amdgcn_ballot_w64(fin && !(s.R < eps)));
            // lane refill: finished lanes take the unit's next walks in lane order
            const int32_t wn = base + rank;
            if (fin) {
                walker_start<T, D>(s, xq, st.R, wn);
                active = wn < n;
            }
            base += __popcll(m);
        }
    }
    // partial row: the first D of DA coordinates are in use
    constexpr int NA = nacc(DA);
    double row[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) row[i] = 0.0;
    row[0] = su;
    row[1] = su2;
#pragma unroll
    for (int i = 0; i < D; ++i) {
        row[2 + i] = g[i * kWave];
        row[2 + DA + i] = g[(D + i) * kWave];
    }
    row[5 + 2 * DA] = sS;
    row[6 + 2 * DA] = sg;
    if (lane == 0) {
        row[2 + 2 * DA] = (double)steps;
        row[3 + 2 * DA] = (double)trunc;
        row[4 + 2 * DA] = (double)degen;
        row[7 + 2 * DA] = (double)wc.sph;
        row[8 + 2 * DA] = (double)wc.box;
        row[9 + 2 * DA] = (double)wc.cbox;
    }
    wave_store<NA>(row, out);
}

}  // namespace wos
