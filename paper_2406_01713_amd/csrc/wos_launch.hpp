// wos_launch.hpp -- host-side launchers of the libwos kernels (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wos_params.hpp"

namespace wos {

// Whether the steps can do without the cluster scan: every kind's obstacles
// are in cell lists or few enough to be scanned.
template <typename T>
bool lists_ok(const EnvP<T>& p)
{
    return (p.sph_cells || !p.n_cl_sph) && (p.box_cells || !p.n_cl_box);
}

// Plain walk kernel: one wave per (query, range of `wpu` walks), lanes
// refilled within the range.  Writes one partial-sum row per wave, chunks =
// ceil(n_walks / wpu) rows per query.  p is a device pointer; src selects the
// variant with point-source terms, lists the one whose steps read cell lists
// or scan every obstacle (EnvP must be fit for it: lists_ok).
template <typename T>
hipError_t launch_plain(int d, bool bwd, bool src, bool lists, const EnvP<T>* p, const T* queries, int64_t n_q,
                        int64_t n_walks, int32_t wpu, int lanes, int64_t w_base, uint32_t q_base, double* partials,
                        double* records, hipStream_t st);
template <typename T, int D>
hipError_t launch_plain_d(bool bwd, bool src, bool lists, const EnvP<T>* p, const T* queries, int64_t n_q,
                          int64_t n_walks, int32_t wpu, int lanes, int64_t w_base, uint32_t q_base, double* partials,
                          double* records, hipStream_t st);

// Per-query means / standard errors (and backward products) from the plain
// kernel's partials.  With bwd: prod (Q x 2) receives grad_u[q] * (du/dsigma,
// du/dg) where ubar is given, out_jac (Q x (d + 2), optional) the unweighted
// FP64 means (grad u, du/dsigma, du/dg).
template <typename T>
hipError_t launch_finalize_plain(int d, bool bwd, const double* partials, int64_t n_q,
                                 int32_t chunks, int64_t n_walks, T* out_u, T* out_grad,
                                 double* out_stats, const T* ubar, T* out_dx, double* out_dq,
                                 double* out_jac, double* prod, hipStream_t st);

// Deterministic sum of the Q x 2 products into two scalars.
hipError_t launch_reduce_pairs(const double* prod, int64_t n, double* out0, double* out1,
                               hipStream_t st);

// Persistent ragged-batch kernel (FP32): grid of resident waves pulling work
// units from *counter; refills lanes with the next walk of the unit.  src
// selects the variant with point-source terms (any env of the batch).
hipError_t launch_persistent(bool bwd, bool src, bool lists, int grid, int block, const EnvP<float>* envs,
                             const BatchEnv* benv, int n_benv, int max_d, const float* queries,
                             int64_t total_units, uint32_t key0, uint32_t key1,
                             const uint64_t* key_add, unsigned* counter, double* partials,
                             hipStream_t st);

// The variants of the above.
template <bool SRC, bool LISTS, int MAXD>
hipError_t launch_persistent_variant(bool bwd, int grid, int block, const EnvP<float>* envs, const BatchEnv* benv,
                                     int n_benv, int max_d, const float* queries, int64_t total_units, uint32_t key0,
                                     uint32_t key1, const uint64_t* key_add, unsigned* counter, double* partials,
                                     hipStream_t st);
template <bool SRC, bool LISTS, int MAXD>
int persistent_blocks_per_cu(bool bwd, int max_d, int block);

// Resident waves of the persistent kernel for a block size (occupancy x CUs).
// max_d: the batch's largest dimension.
int persistent_resident_blocks(bool bwd, bool src, bool lists, int max_d, int block);

// Outputs of a batched launch; one block per env; also resets *counter.
// out_dir (optional, rows like out_grad) receives grad / |grad| formed from
// the FP64 sums, so it exists where the mean gradient is below FP32 range.
hipError_t launch_finalize_batch(bool bwd, const BatchEnv* benv, int n_benv,
                                 const double* partials, const float* ubar,
                                 float* out_u, float* out_grad, int grad_stride,
                                 double* out_stats, float* out_dx, double* out_dsigma,
                                 double* out_dg, float* out_dir, unsigned* counter, hipStream_t st);

// One planning update: x += min(s_ub, R/2) dir, dir the unit gradient
// direction (a zero row counts a stall); bumps *step.
hipError_t launch_plan_update(int d, const EnvP<float>* p, float* x, int64_t n, const float* dir,
                              int grad_stride, float s_ub, double* path_len, int32_t* stalls,
                              int32_t* status, uint64_t* step, hipStream_t st);

// Varadhan read-out w = -sqrt(1/sigma) ln u (and its gradient when grad and
// grad_w are given, rows of `stride` elements, first d used).
template <typename T>
hipError_t launch_varadhan(const T* u, const T* grad, int64_t n, int d, int stride, double sigma, T* w,
                           T* grad_w, hipStream_t st);

// Cell lists of one obstacle kind (see kGridMin): the geometry of the table
// and what bounds the walker's threshold in it.
struct GridBuild {
    int k = 0;                           // coordinates the obstacles depend on
    uint32_t n[kMaxDim], cells = 0;      // cells per axis (1 past k), their product
    float lo[kMaxDim], h = 0;            // first corner, edge
    float pad[kMaxDim];                  // enlargement of a cell (rounding of its coordinate)
    float margin = 0;                    // enlargement of every distance comparison
    float lev[3];                        // threshold ranges
    int outer_kind = 0;
    float olo[kMaxDim], ohi[kMaxDim], oc[kMaxDim], orad = 0;
};

// The lists of m obstacles (device FP32 rows of dimension d): grid_start
// enqueues their build on the default stream, grid_finish waits for it and hands
// over one allocation, whose start *cells receives (*list points into it).
// *cells stays null, with hipSuccess, where the lists would take more than
// kGridEntriesMax entries or one of them more than a count byte says.  A job
// started but not finished is given up by freeing its hd.
constexpr uint32_t kGridEntriesMax = 1u << 25;
struct GridJob {
    GridCell* hd = nullptr;
    unsigned parts = 0;  // of the list, `cap` entries each
    uint32_t cap = 0;
};
hipError_t grid_start(const GridBuild& g, int d, bool box, const float* rows, int64_t m, GridJob& job);
hipError_t grid_finish(const GridBuild& g, int d, bool box, const float* rows, int64_t m, GridJob& job,
                       GridCell** cells, uint32_t** list);

// Fill kernels (used instead of hipMemsetAsync so the calls are capturable).
hipError_t launch_fill_u32(unsigned* p, int64_t n, unsigned v, hipStream_t st);
hipError_t launch_fill_f64(double* p, int64_t n, double v, hipStream_t st);

}  // namespace wos
