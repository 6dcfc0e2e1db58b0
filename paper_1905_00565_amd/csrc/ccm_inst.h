// ccm_inst.h -- launchers of the kernels that are compiled once per embedding
// dimension E (or E_max).  Each is defined in ccm_inst.hip and instantiated
// in the translation unit built for that E; the dispatchers in
// ccm_kernels.hip pick one by E.  Arguments as the dispatchers of the same
// name in ccm_internal.h.
#pragma once
#include "ccm_internal.h"

namespace ccmk {

template <int E>
hipError_t launch_crossmap_e(int mode, int grid, const Realization* rzs, const Item* items,
                             int n_items, int* next, const float* emb, const float* pts,
                             const int32_t* pj, const int32_t* qord, const int32_t* start,
                             const double* tgt, Moments* partial, int query_set, int window,
                             Dump d, const int32_t* table, int table_n_e, hipStream_t st);

template <int E>
hipError_t launch_spread_e(int mode, const Realization* rzs, const Item* items, int n_items,
                           const float* emb, const float* pts, const int32_t* pj,
                           const int32_t* qord, const int32_t* start, const double* tgt,
                           double* pred, Moments* partial, int query_set, int window,
                           hipStream_t st);

template <int E>
hipError_t launch_multi_e(int mode, int grid, const Realization* rzs, const int32_t* self_of,
                          const Item* items, int n_items, int* next, const float* emb,
                          const float* pts, const int32_t* pj, const int32_t* qord,
                          const int32_t* start, const double* tt, int m_series, void* partial,
                          int query_set, int window, const int32_t* table, int table_n_e,
                          hipStream_t st);

template <int E>
hipError_t launch_nested_e(int mode, int grid, const Realization* rzs, const Item* items,
                           int n_items, int* next, const float* emb, const float* pts,
                           const int32_t* pj, const int32_t* qord, const int32_t* start,
                           const double* tgt, const int32_t* seg, Moments* partial, int window,
                           hipStream_t st);

template <int EMAX>
hipError_t launch_shared_e(int mode, int grid, const Realization* rzs, const Item* items,
                           int n_items, int* next, const float* emb, const float* pts,
                           const int32_t* pj, const int32_t* qord, const int32_t* start,
                           const double* tgt, Moments* partial, int window, hipStream_t st);

template <int E>
hipError_t launch_table_build_e(const TableJob* jobs, int n_jobs, int max_n_e, const float* emb,
                                int32_t* table, hipStream_t st);

template <int E>
hipError_t launch_order_points_e(const RowJob* jobs, int n_jobs, int max_ne, const float* emb,
                                 const int32_t* qord, float* pts, float* box, int* todo_n,
                                 hipStream_t st);

template <int E>
hipError_t launch_rows_e(const RowJob* jobs, int n_jobs, int max_ne, int max_w, int per_block,
                         const float* pts, const float* box, const int32_t* qord,
                         uint64_t* rows, RowTodo* todo, int* todo_n, hipStream_t st);

template <int E>
hipError_t launch_walk_e(int keys, const WalkGroup* groups, const RowJob* embs,
                         const Item* items, int n_items, int per, const uint64_t* masks,
                         const uint64_t* rows, const int32_t* qord, const float* emb,
                         const double* tgt, double* out, int excl, int query_set,
                         hipStream_t st);

template <int E>
hipError_t launch_walk_moments_e(int shared, const Realization* rzs, const WalkOut* where,
                                 const Item* items, int n_items, const double* out,
                                 const int32_t* pj, const int32_t* qord, const double* tgt,
                                 Moments* partial, int query_set, hipStream_t st);

template <int E>
hipError_t launch_multi_keys_e(const Realization* rzs, const int32_t* self_of,
                               const WalkOut* where, const Item* items, int n_items,
                               const double* keys, const int32_t* pj, const int32_t* qord,
                               const double* tt, int m_series, void* partial, int query_set,
                               hipStream_t st);

template <int E>
hipError_t launch_multi_group_e(const Realization* rzs, const int32_t* self_of,
                                const WalkGroup* groups, const WalkLib* libs, const Item* items,
                                int n_items, const double* keys, const int32_t* qord,
                                const double* tt, int m_series, void* partial, hipStream_t st);

}  // namespace ccmk
