// What the kernels of the FFN step for one to eight tokens share (ffn_fast.hip, ffn_fast_tokens.hip).
#pragma once

#include "fast_select.h"
#include "kernels.h"
#include "rows_mfma.h"

namespace hire {

// State of the route at the head of every workspace, one region per token.  The histograms of the keys have to be zero
// when a step starts; the step's last kernel leaves them so and says in the first region how many regions are clean.
constexpr unsigned long long kCookie = 0x48695245464e4f00ull;  // + the number of clean regions

struct FastRegion {
  unsigned long long cookie; // of the first region
  uint32_t fallbacks[2];     // first region: selections whose k'-th key / k-th h were found without the histogram
  uint32_t bin1;             // threshold bin of the keys of the running step, 0: not known from the histogram; by the
                             // gathering kernel, with need1 the keys of that bin that are selected
  uint32_t anchor1, anchor2; // top bins of the two windows for the running step, written by the scorer kernel
  uint32_t need1;
  uint32_t zeros[8];         // stays zero: what lanes beyond the end of a key array load
  uint32_t pad[48];
  uint32_t hist1[kWin];      // slot s: scorer keys in fine bin anchor1 - s
  uint32_t hist2[kWin];      // slot s: activations in fine bin anchor2 - s
};
static_assert(offsetof(FastRegion, zeros) == 32 && offsetof(FastRegion, hist1) == 256, "region layout");
static_assert(sizeof(FastRegion) == kFastRegionBytes, "region size");

__device__ __forceinline__ int clean_regions(const FastRegion* first) {
  const unsigned long long n = first->cookie - kCookie;
  return n <= (unsigned long long)kFastTokens ? (int)n : 0;
}

constexpr int kOwnUnits = 64;  // units of a workgroup of the gathering kernels

// Sixteen bytes per lane and load, 256 chunks of a row in flight.
struct RowChunks {
  uint4 v[4];
  __device__ __forceinline__ void issue(const uint4* row, int c0, int cpr) {
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = load_streaming(&row[min(c0 + u * kWave + lane_id(), cpr - 1)]);
  }
};
}  // namespace hire
