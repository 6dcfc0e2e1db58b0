// ccm_inst_walk.hip -- the neighbour-row kernels of one embedding dimension
// (ccm_walk.h), compiled once per E = 1..10 with -DCCM_INST_E=E.
#include <algorithm>

#include "ccm_walk.h"
#include "ccm_inst.h"

#ifndef CCM_INST_E
#error "compile with -DCCM_INST_E=<embedding dimension>"
#endif

namespace ccmk {

template <int E>
hipError_t launch_order_points_e(const RowJob* jobs, int n_jobs, int max_ne, const float* emb,
                                 const int32_t* qord, float* pts, float* box, int* todo_n,
                                 hipStream_t st) {
  const unsigned runs = (unsigned)((max_ne + 63) / 64);
  k_order_points<E><<<dim3((runs + kWaves - 1) / kWaves, (unsigned)n_jobs), kBlock, 0, st>>>(
      jobs, emb, qord, pts, box, todo_n);
  return hipGetLastError();
}

template <int E>
hipError_t launch_rows_e(const RowJob* jobs, int n_jobs, int max_ne, int max_w, int per_block,
                         const float* pts, const float* box, const int32_t* qord,
                         uint64_t* rows, RowTodo* todo, int* todo_n, hipStream_t st) {
  const dim3 grid((unsigned)((max_ne + per_block - 1) / per_block), (unsigned)n_jobs);
  k_rows<E><<<grid, kBlock, row_lds_bytes(max_w), st>>>(jobs, per_block, pts, box, qord, rows,
                                                        todo, todo_n);
  // a resident grid over the rows it has left, usually none
  const unsigned rows_all = (unsigned)std::min<int64_t>(2048, (int64_t)max_ne * n_jobs);
  k_rows_repeats<E><<<rows_all, kBlock, row_lds_bytes(max_w), st>>>(jobs, todo, todo_n, pts, box,
                                                                    qord, rows);
  return hipGetLastError();
}

template <int E>
hipError_t launch_walk_e(int keys, const WalkGroup* groups, const RowJob* embs,
                         const Item* items, int n_items, int per, const uint64_t* masks,
                         const uint64_t* rows, const int32_t* qord, const float* emb,
                         const double* tgt, double* out, int excl, int query_set,
                         hipStream_t st) {
  if (keys)
    k_walk<E, true><<<(unsigned)n_items, kBlock, 0, st>>>(groups, embs, items, per, masks, rows,
                                                          qord, emb, tgt, out, excl, query_set);
  else
    k_walk<E, false><<<(unsigned)n_items, kBlock, 0, st>>>(groups, embs, items, per, masks, rows,
                                                           qord, emb, tgt, out, excl, query_set);
  return hipGetLastError();
}

template <int E>
hipError_t launch_walk_moments_e(int shared, const Realization* rzs, const WalkOut* where,
                                 const Item* items, int n_items, const double* out,
                                 const int32_t* pj, const int32_t* qord, const double* tgt,
                                 Moments* partial, int query_set, hipStream_t st) {
  if (shared)
    k_walk_moments<kSharedQ[E]><<<(unsigned)n_items, kBlock, 0, st>>>(
        rzs, where, items, out, pj, qord, tgt, partial, query_set);
  else
    k_walk_moments<DefaultQ<E>::Q><<<(unsigned)n_items, kBlock, 0, st>>>(
        rzs, where, items, out, pj, qord, tgt, partial, query_set);
  return hipGetLastError();
}

template hipError_t launch_order_points_e<CCM_INST_E>(const RowJob*, int, int, const float*,
                                                      const int32_t*, float*, float*, int*,
                                                      hipStream_t);
template hipError_t launch_rows_e<CCM_INST_E>(const RowJob*, int, int, int, int, const float*,
                                              const float*, const int32_t*, uint64_t*, RowTodo*,
                                              int*, hipStream_t);
template hipError_t launch_walk_e<CCM_INST_E>(int, const WalkGroup*, const RowJob*,
                                              const Item*, int, int,
                                              const uint64_t*, const uint64_t*, const int32_t*,
                                              const float*, const double*, double*, int, int,
                                              hipStream_t);
template hipError_t launch_walk_moments_e<CCM_INST_E>(int, const Realization*, const WalkOut*,
                                                      const Item*, int, const double*,
                                                      const int32_t*, const int32_t*,
                                                      const double*, Moments*, int,
                                                      hipStream_t);

}  // namespace ccmk
