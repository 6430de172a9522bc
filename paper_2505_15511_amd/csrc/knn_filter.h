// libnomad: launch of the nearest-neighbour filter (instances in knn_filter.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "knn_filter_kernel.h"

using namespace nomad_knn;

// n_blocks workgroups of `waves` wavefronts (knn_filter_waves) over the work list `blocks`.  assign.out != nullptr: one
// neighbour wanted, see k_knn_filter; otherwise cand [n_q * list_len] and tau [n_q] are filled.
hipError_t launch_knn_filter(hipStream_t st, uint32_t n_blocks, int waves, const KnnSets& P, const KnnBlock* blocks, int32_t list_len,
                             int32_t* cand, float* keys, float* tau, const KnnAssign& assign);
