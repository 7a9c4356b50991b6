// Sums of listed (row, coefficient) pairs over some columns of a bf16 matrix: the second layer of a step (k_w2_list in gather.hip,
// k_refine_w2 in batch_select.hip).
#pragma once

#include <limits.h>

#include "device_utils.h"

namespace hire {

// acc += sum of the n entries' rows, eight columns per lane: LPR lanes share a row (columns points at the lane's in row 0; rows have
// d values), the WAVES waves of a workgroup take kWave / LPR rows each per load.  `first`: this lane's first entry.  entry(t) has
// to name a readable row with coefficient 0 for n <= t < n + 2 kBatch; what is read there is not used.  A lane has two batches of FL
// rows in flight.  No request sits behind a branch, or the wait for the batch before it would be one for all that is under way,
// and the rows of a batch are requested in the order in which they are added up, in which they return.  k_w2_list for 64 tokens at
// the ~1B shape, us, with a branch around the requests / this: 20.4 / 20.0.
// SHORT: n is one batch at most, and no second one is requested.
template <int LPR, int FL, int WAVES, bool SHORT = false, typename Entry>
__device__ __forceinline__ void add_listed_rows(const uint16_t* __restrict__ columns, int d, int n, int first,
                                                Entry&& entry, float (&acc)[8]) {
  const char* base = reinterpret_cast<const char*>(columns);
  constexpr int kStride = WAVES * (kWave / LPR), kBatch = kStride * FL;
  auto request = [&](int t0, uint4 (&wv)[FL], float (&cf)[FL]) __attribute__((always_inline)) {
    const uint4* at[FL];
#pragma unroll
    for (int u = 0; u < FL; ++u) {
      const uint2 e = entry(t0 + u * kStride);
      cf[u] = __uint_as_float(e.y);
      at[u] = reinterpret_cast<const uint4*>(base + (uint64_t)e.x * (2u * (uint32_t)d));  // one multiply-add
    }
#pragma unroll
    for (int u = 0; u < FL; ++u) {
      wv[u] = *at[u];
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto add = [&](const uint4 (&wv)[FL], const float (&cf)[FL], int known) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < FL; ++u) {
      const uint32_t keep = first + u * kStride < known ? 0xFFFFFFFFu : 0u;  // (an infinite weight behind the end is no 0 * inf)
      const uint4 v = make_uint4(wv[u].x & keep, wv[u].y & keep, wv[u].z & keep, wv[u].w & keep);
      const float wf[8] = {bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y),
                           bf16_lo(v.z), bf16_hi(v.z), bf16_lo(v.w), bf16_hi(v.w)};
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[q] = fmaf(cf[u], wf[q], acc[q]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  uint4 wa[FL], wb[FL];
  float ca[FL], cb[FL];
  request(first, wa, ca);
  if constexpr (SHORT) {
    add(wa, ca, n);
    return;
  }
  request(first + kBatch, wb, cb);
  int t0 = 0;
  for (; t0 + 2 * kBatch < n; t0 += 2 * kBatch) {  // uniform
    add(wa, ca, INT_MAX);
    request(t0 + 2 * kBatch + first, wa, ca);
    add(wb, cb, INT_MAX);
    request(t0 + 3 * kBatch + first, wb, cb);
  }
  add(wa, ca, n - t0);
  if (t0 + kBatch < n) add(wb, cb, n - t0 - kBatch);
}

// The sums of the lanes of a wave that hold the same columns, in a fixed tree, to all of them.
template <int LPR>
__device__ __forceinline__ void fold_lanes(float (&acc)[8]) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
#pragma unroll
    for (int m = LPR; m < kWave; m <<= 1) acc[q] += __shfl_xor(acc[q], m);
  }
}

}  // namespace hire
