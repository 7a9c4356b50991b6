// What the kernels of the FFN step for one to eight tokens share (ffn_fast.hip, ffn_fast_tokens.hip).
#pragma once

#include "fast_select.h"
#include "hist.h"
#include "kernels.h"
#include "rows_mfma.h"

namespace hire {

// State of the route at the head of every workspace, one region per token.  The consumers of a window histogram take
// its counts for the keys' own, so it has to be exact whenever it is used.  Two things see to that:
//  * The histograms of the keys are zero when a step that uses them starts.  The step's scorer kernel takes the cookie
//    away, leaving the number of clean regions in `clean` for the kernels that follow, and the last one, which clears the
//    histograms, gives it back: a step that ends in between (a launch that the runtime refused) leaves no cookie behind,
//    and the next step selects without histograms.
//  * The anchors bound every key and activation.  Should one lie above its anchor all the same (row-norm bounds of other
//    weights, scales that do not belong to the codes), it would be missing from the counts: whoever meets it says so in
//    `beyond1` / `beyond2`, and the selection goes by the keys alone.
// (kCookie, in hist.h: steps whose layout lies on the regions of further tokens leave it at one region)

struct FastRegion {
  unsigned long long cookie; // of the first region
  uint32_t fallbacks[2];     // first region: selections whose k'-th key / k-th h were found without the histogram
  uint32_t bin1;             // threshold bin of the keys of the running step, 0: not known from the histogram; by the
                             // gathering kernel, with need1 the keys of that bin that are selected
  uint32_t anchor1, anchor2; // top bins of the two windows for the running step, written by the scorer kernel
  uint32_t need1;
  uint32_t clean;            // first region: regions whose key histograms were zero when the running step started
  uint32_t beyond1, beyond2; // not 0: a key (an activation) of the running step lies above its anchor
  uint32_t spare;
  uint32_t zeros[8];         // stays zero: what lanes beyond the end of a key array load
  uint32_t pad[44];
  uint32_t hist1[kWin];      // slot s (steps of several tokens: at spread_slot(s)): scorer keys in fine bin anchor1 - s
  uint32_t hist2[kWin];      // ... activations in fine bin anchor2 - s
};
static_assert(offsetof(FastRegion, zeros) % 16 == 0 && offsetof(FastRegion, hist1) == 256, "region layout");
static_assert(sizeof(FastRegion) == kFastRegionBytes, "region size");

// By one thread of a step's scorer kernel, with the cookie as it was found (asked for early: a round trip to memory): if
// there is one, it is taken away.
__device__ __forceinline__ void take_cookie(FastRegion* first, unsigned long long cookie) {
  const unsigned long long n = cookie - kCookie;
  first->clean = n <= (unsigned long long)kFastTokens ? (uint32_t)n : 0u;
  first->cookie = 0ull;
}
// By a step's last kernel, which clears the key histograms of the step's B tokens.
__device__ __forceinline__ void give_cookie(FastRegion* first, int clean, int B) {
  first->cookie = kCookie + (unsigned long long)max(clean, B);
}

// Counts a key (its IEEE bits) in the window below the anchor; zeros are never counted.
template <bool SPREAD, typename K>
__device__ __forceinline__ void count_in_window(K bits, uint32_t anchor, uint32_t* hist, uint32_t* beyond) {
  const uint32_t bin = fine_bin(bits), slot = anchor - bin;
  if (bits == (K)0) return;
  if (slot < (uint32_t)kWin) atomicAdd(&hist[SPREAD ? spread_slot((int)slot) : (int)slot], 1u);
  else if (bin > anchor) *beyond = 1u;
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
