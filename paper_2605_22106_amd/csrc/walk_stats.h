// Statistics of one event of arbor_walk, shared by its own launch and the
// rehydration plan's (which runs them in a second workgroup).
#pragma once

#include "arbor_internal.h"

namespace arbor {

namespace {

// three block-wide sums in one exchange; sm holds 48 values
__device__ void block_sum3(int64_t (&v)[3], int64_t *sm) {
  const int lane = lane_id(), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int q = 0; q < 3; ++q) v[q] = wave_sum(v[q]);
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < 3; ++q) sm[16 * q + w] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 3; ++q) v[q] = wave_sum(lane < nw ? sm[16 * q + lane] : (int64_t)0);
  __syncthreads();
}

// Per-event statistics of the device-side controller (arbor_walk): one
// workgroup after each allocation of a step.  transition = 1: row[0] = sum of
// the keep-counts, row[1] = tokens the rehydration of this step restores from
// the token store (Path* blocks with c_i < n_i), row[2] = tokens evicted
// (sum of c_i - k_i where k_i < c_i), row[3] = 0.  transition = 0 (the gated
// Pressure event, budget `budget`): if it fired (resident tokens >= budget),
// row[0] = the new sum, row[2] += its evictions, row[3] = 1.
__device__ __forceinline__ void walk_stats_body(const Tree &t, const int32_t *__restrict__ k,
                                                const uint8_t *__restrict__ on_path,
                                                int64_t budget, int transition, int rehydrate,
                                                int64_t *__restrict__ row, int32_t *status) {
  __shared__ int64_t sm[3 * 16];
  if (status_failed(status)) return;
  int64_t v[3] = {0, 0, 0};   // sum k, evicted, restored or resident
#pragma unroll 4
  for (int i = threadIdx.x; i < t.V; i += blockDim.x) {
    const int c = t.n_kept[i], ki = k[i], n = t.n_full[i];
    v[0] += ki;
    v[1] += ki < c ? c - ki : 0;
    v[2] += transition ? (on_path[i] && rehydrate && c < n ? n - c : 0) : c;
  }
  block_sum3(v, sm);
  if (threadIdx.x == 0) {
    if (transition) {
      row[0] = v[0];
      row[1] = v[2];
      row[2] = v[1];
      row[3] = 0;
    } else if (v[2] >= budget) {
      row[0] = v[0];
      row[2] += v[1];
      row[3] = 1;
    }
  }
}

}  // namespace

}  // namespace arbor
