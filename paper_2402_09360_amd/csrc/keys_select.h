// Selection of the k' largest scorer keys of one token by a workgroup of sixteen waves (k_keys_select in batch_select.hip;
// gather_mfma.hip runs it beside the filter stage), and the window histogram that it shares with the selection of the
// activations (k_refine).
#pragma once

#include "fast_select.h"
#include "kernels.h"

namespace hire {

template <typename K, int LOADS>
struct BatchKeys {
  using Keys = KeyRegs<K, LOADS, kSelThreads>;
  static_assert(LOADS * Keys::PER <= 32, "one bit per key of a lane");
};

// Window histogram of the registers' values below `anchor` (zeros are never counted) and the bin that holds the k-th
// largest of those.  false: fewer than k values in the window.  *bin: that bin; *above: the values counted in higher ones;
// *beyond: this thread has a value above the anchor, which is not counted.
template <typename Keys>
__device__ __forceinline__ bool window_bin(const Keys& kr, uint32_t anchor, int k, uint32_t* win,
                                           SelSharedT<kSelThreads>& sh, uint32_t* bin, int* above, bool* beyond) {
  uint32_t farthest = 0u;
#pragma unroll
  for (int e = 0; e < (int)(sizeof(kr.r) / sizeof(kr.r[0])); ++e)
#pragma unroll
    for (int q = 0; q < Keys::PER; ++q) {
      const uint32_t slot = anchor - fine_bin(kr.r[e][q]);  // (wraps above the anchor)
      farthest = max(farthest, slot);
      if (kr.r[e][q] != 0u && slot < (uint32_t)kWin) atomicAdd(&win[slot], 1u);
    }
  *beyond = farthest > anchor;
  __syncthreads();
  WinRegs<kSelThreads> wr;
  wr.issue(win);
  const WinWalk wk = walk_window<kSelThreads>(wr, k, sh);
  *bin = anchor - (uint32_t)wk.slot;
  *above = wk.above;
  return wk.found && *bin >= 1u && *bin <= anchor;  // uniform
}

// ---------------------------------------------------------------------------------------------------
// The window's anchor.  fp32 keys (the int4 scorers): sumabs[b], sum of the token's |int8 codes|, and *smax, the largest row
// scale of the int4 copy that the keys were scored with, bound them: key_j = fl(fl(acc_j) s_j) <= fl(7 sumabs smax),
// rounding being monotone (7 sumabs < 2^24).  fp64 keys (the low-rank scorer) have no bound at hand: their maximum, through
// one barrier more.
template <typename K>
struct KeysSelectShared {
  __align__(16) uint32_t win[kWin];
  SelSharedT<kSelThreads> sh;
  unsigned long long wave_top[kSelWaves];
  int wave_cnt[kSelWaves];
  int off_window;  // not 0: the window does not count every key that it should
  BinList<K> list;
};

inline bool keys_select_ok(const KeysSelect& p) {
  return p.N <= 32768 && p.stride % (p.f64 ? 2 : 4) == 0 &&
         reinterpret_cast<uintptr_t>(p.keys) % 16 == 0;
}

// The `want` largest of the registers' keys, ties to the lower index: bit e * PER + q.  vals: the same keys by index, in memory.
// The window is clear, and so are sh.list_n and off_window; all of it behind a barrier.
template <typename K, typename Keys>
__device__ __forceinline__ uint32_t keys_take(const Keys& kr, const void* vals, int want, uint32_t anchor,
                                              KeysSelectShared<K>& S, uint32_t* window_misses) {
  constexpr int PER = Keys::PER, LOADS = Keys::kLoads;
  const int lane = lane_id();
  auto& sh = S.sh;
  auto& list = S.list;
  HIRE_TS(11);
  uint32_t bin;
  int above;
  bool beyond;
  bool known = window_bin(kr, anchor, want, S.win, sh, &bin, &above, &beyond);
  if (beyond) S.off_window = 1;  // (row scales that do not belong to the codes)
  HIRE_TS(12);
  uint32_t take = 0u;  // this lane's selected keys, as in BinMasks
  if (known) {
    const BinMasks<K> bm = bin_masks<K>(kr, bin_floor<K>(bin), bin_floor<K>(bin + 1u));
    list_inside<K>(kr, bm.inside, &sh.list_n, list);
    __syncthreads();
    HIRE_TS(13);
    const int m = sh.list_n;
    known = m <= kFastAmbCap && S.off_window == 0;  // uniform
    if (known)
      take = bm.above | taken_of_list(kr, lane < m ? list.key[lane] : (K)0, lane < m ? list.idx[lane] : 0x7FFFFFFF, m,
                                      want - above);
    HIRE_TS(14);
  }
  if (!known) {  // threshold among the zeros or below the window, crowded bin: range narrowing
    WinRegs<kSelThreads> none{};
    const Selection<K> sel =
        fast_select<60>(kr, vals, want, none, 0u, false, sh, S.wave_cnt, window_misses, 0, want, true);
    take = 0u;
#pragma unroll
    for (int e = 0; e < LOADS; ++e)
#pragma unroll
      for (int q = 0; q < PER; ++q)
        take = take + take + (kr.valid(e, q) && cut_takes(sel.cut, kr.r[e][q], kr.index(e, q)) ? 1u : 0u);
  }
  return __brev(take) >> (32 - LOADS * PER);
}

// Adds the taken keys' bits to a bitmap: a word covers 32 consecutive indices, the keys of 32 / PER neighbouring lanes of one
// load.  Those lanes fold their bits together and one of them adds the word.
template <typename Keys>
__device__ __forceinline__ void add_bits(const Keys& kr, uint32_t take, uint32_t* bitmap) {
  constexpr int PER = Keys::PER, LOADS = Keys::kLoads, kLanes = 32 / PER;
  static_assert(kLanes == 8 || kLanes == 16, "lanes per word");
  const int lane = lane_id();
#pragma unroll
  for (int e = 0; e < LOADS; ++e) {
    uint32_t bits = (take >> (e * PER) & ((1u << PER) - 1u)) << (lane % kLanes * PER);
    bits |= dpp_move<0xB1, 0xF>(0u, bits);   // lanes 1, 0, 3, 2 of a quad
    bits |= dpp_move<0x4E, 0xF>(0u, bits);   // lanes 2, 3, 0, 1
    bits |= dpp_move<0x141, 0xF>(0u, bits);  // eight lanes mirrored: the other quad
    if constexpr (kLanes == 16) bits |= dpp_move<0x140, 0xF>(0u, bits);  // sixteen: the other eight
    if (lane % kLanes == 0 && bits != 0u) atomicOr(&bitmap[(kr.base + e * Keys::SPAN) / 32 + lane / kLanes], bits);
  }
}

// Token b, by the whole workgroup.
template <typename K, int LOADS>
__device__ __forceinline__ void keys_select_token(const KeysSelect& p, int b, KeysSelectShared<K>& S) {
  using Keys = typename BatchKeys<K, LOADS>::Keys;
  constexpr int PER = Keys::PER;
  const int tid = (int)threadIdx.x, lane = lane_id(), N = p.N, kprime = p.kprime;
  auto& sh = S.sh;
  auto& win = S.win;
  HIRE_TS(10);
  const K* row = static_cast<const K*>(p.keys) + (size_t)b * p.stride;
  Keys kr;
  kr.issue_clamped(row, N);  // rows are padded to whole vectors
  {
    uint4* z = reinterpret_cast<uint4*>(win) + 2 * tid;
    z[0] = z[1] = make_uint4(0, 0, 0, 0);
  }
  if (tid == 0) sh.list_n = S.off_window = 0;
  uint32_t anchor;
  if constexpr (sizeof(K) == 4) {
    anchor = fine_bin(__float_as_uint(7.0f * p.sumabs[b] * *p.smax));
    kr.finish();
    kr.mask_beyond(N);
    __syncthreads();
  } else {
    kr.finish();
    kr.mask_beyond(N);
    K top = 0;  // non-negative doubles order like their bits
#pragma unroll
    for (int e = 0; e < LOADS; ++e)
#pragma unroll
      for (int q = 0; q < PER; ++q) top = kr.r[e][q] > top ? kr.r[e][q] : top;
    top = wave_max(top);
    if (lane == 0) S.wave_top[wave_id()] = top;
    __syncthreads();
    anchor = fine_bin((K)wave_max((K)(lane < kSelWaves ? S.wave_top[lane] : 0)));
  }
  add_bits(kr, keys_take<K>(kr, row, kprime, anchor, S, p.window_misses), p.bitmap);
  HIRE_TS(15);
}

}  // namespace hire
