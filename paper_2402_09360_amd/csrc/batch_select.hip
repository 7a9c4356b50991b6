// The two selections of a batched FFN step (TopInd_k of arXiv 2402.09360 Sec. 3.1, both lines of Algorithm 1), one
// workgroup of sixteen waves per token, rows of up to 32768 units:
//
//   k_keys_select  the k' largest scorer keys of a token -> its bits of the union bitmap
//   k_refine       the k largest exact activations of a token from the filter stage's values (launch_filter_units,
//                  in unit order), recomputing in fp64 what lies around the threshold -> indices, values and the
//                  (row, coefficient) list of the second layer
//   k_refine_w2    the same with the second layer behind it, where the selected rows are few enough: several workgroups per
//                  token, each with some columns of y
//   k_refine_values  the same where the values are to be rounded from 64 bits and not only selected by them: several workgroups
//                  per token, each with some of the values; k_exact_values over the list where these are many
//
// The selections are chains of dependent steps on one compute unit: a barrier-separated section costs about its instruction
// count per thread times 16 cycles (four waves share a SIMD), so what counts is the number of sections and of passes
// over the register-resident row.  The window histogram (fast_select.h) is anchored at an a-priori bound of the
// row's values - no pass and no barrier for their maximum - and is built in LDS from the registers themselves, so the
// number of entries above the bin it proposes is exact and no counting pass confirms it, unless a value lies above the
// anchor, which whoever holds it sees.
#include "fast_select.h"
#include "kernels.h"
#include "keys_select.h"
#include "listed_rows.h"

namespace hire {

constexpr int kBsCap = 128;  // refined entries around the threshold kept in LDS

template <typename K, int LOADS>
__global__ __launch_bounds__(kSelThreads) void k_keys_select(KeysSelect p) {
  __shared__ KeysSelectShared<K> S;
  keys_select_token<K, LOADS>(p, (int)blockIdx.x, S);
}

// ---------------------------------------------------------------------------------------------------
struct RefineShared {
  SelSharedT<kSelThreads> sh;
  __align__(16) uint32_t win[kWin + 2 * kWave];  // window histogram; then the selected entries in order (k <= kWin / 2)
  unsigned long long l_val[kBsCap];  // refined values (fp64 bits) and their units
  int l_idx[kBsCap];
  int wave_cnt[kSelWaves], wave_eq[kSelWaves];
  float wave_max[kSelWaves];
  int cand_cnt[kSelWaves];
};

// What the histogram and the list cannot settle (threshold among the zeros, very many activations within the error of
// the threshold): exact, by streaming the row.  The k-th largest stored value among the candidates by range
// narrowing; everything within hw of it recomputed in fp64; then the k-th largest of the candidates' fp64 values (stored
// ones outside the band) with ties to the lower unit, packed into LDS in order.  The fp64 values lie in the order of the
// candidates; a wave owns the units [i_lo, i_hi) and so the candidates from c_lo on.  Workgroups that select for the same token
// share the scratch: each place is written once by each of them, with the same value, and read by its own writer behind a barrier.
// What all of them read again comes from the caches.  us per step with 400 copies of a unit near the threshold, one workgroup per token
// doing this / all of them: ~1B shape, 16 equal tokens, copies at random units 162.6 / 152.0, in a row 567.7 / 542.1, five tokens 165.9 / 154.7, 571.9 /
// 548.4; d = 800, 5003 units, 33 tokens 96.5 / 89.1; d = 1024, 8000 units, 64 tokens 113.0 / 105.2 (without copies 47.6 / 45.4, 45.7 / 44.0, 36.6 / 33.4,
// 37.3 / 32.5).
__device__ __forceinline__ void refine_streaming(const RefineParams& p, int b, const uint4* tok, RefineShared& L, double hw) {
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int N = p.N, k = p.k;
  const float* row = p.vals + (size_t)b * p.stride;
  double* h = p.h64 + (size_t)b * p.h_stride;
  auto candidate = [&](int i) { return ((p.bitmap[i >> 5] >> (i & 31)) & 1u) != 0u; };
  const int M = ((N + kSelWaves - 1) / kSelWaves + kWave - 1) / kWave * kWave, i_lo = w * M, i_hi = min(N, i_lo + M);
  int mine = 0;
#pragma unroll 1
  for (int i0 = i_lo; i0 < i_hi; i0 += kWave) mine += i0 + lane < i_hi && candidate(i0 + lane) ? 1 : 0;
  int n_units;
  const int incl = wg_scan_incl<kSelThreads>(mine, L.sh, &n_units);
  const int c_lo = __builtin_amdgcn_readfirstlane(incl - mine), c_hi = __builtin_amdgcn_readlane(incl, kWave - 1);
  const uint32_t okey = wg_kth_largest<uint32_t>(
      [&](auto&& f) {
#pragma unroll 1
        for (int i = tid; i < N; i += kSelThreads) f(candidate(i) ? order_key(row[i]) : 0u);
      },
      N, k, L.sh);
  const double cut0 = (double)key_value(okey);
  const double lo = cut0 - hw, hi = cut0 + hw;
  // the same positions are written and read by this workgroup only; a barrier orders them
  int run_c = c_lo;
#pragma unroll 1
  for (int i0 = i_lo; i0 < i_hi; i0 += kWave) {
    const int i = i0 + lane;
    const float v = i < i_hi ? row[i] : 0.0f;
    const bool cand = i < i_hi && candidate(i);
    const uint64_t cands = __ballot(cand);
    const int at = run_c + mask_prefix(cands);
    run_c += __popcll(cands);
    double stored = (double)v;
    // exact zeros are activations already; with k = all candidates nothing needs to be decided
    uint64_t band = __ballot(cand && k < n_units && v > 0.0f && (double)v >= lo && (double)v <= hi);
    while (band != 0ull) {
      const int s = __builtin_ctzll(band);
      band &= band - 1ull;
      const double r = wave_row_dot(p.W + (size_t)(i0 + s) * p.d, tok, p.d);
      stored = lane == s ? r : stored;
    }
    if (cand) h[at] = stored;
  }
  __syncthreads();
  const uint64_t t = wg_kth_largest<uint64_t>(
      [&](auto&& f) {
#pragma unroll 1
        for (int i = tid; i < n_units; i += kSelThreads) f(order_key(h[i]));
      },
      n_units, k, L.sh);
  int gt = 0, eq = 0;
#pragma unroll 1
  for (int c = c_lo + lane; c < c_hi; c += kWave) {
    const uint64_t key = order_key(h[c]);
    gt += key > t ? 1 : 0;
    eq += key == t ? 1 : 0;
  }
  gt = wave_sum(gt);
  eq = wave_sum(eq);
  __syncthreads();
  if (lane == 0) {
    L.wave_cnt[w] = gt;
    L.wave_eq[w] = eq;
  }
  __syncthreads();
  int run_gt = 0, run_eq = 0, all_gt = 0;
  for (int u = 0; u < kSelWaves; ++u) {
    run_gt += u < w ? L.wave_cnt[u] : 0;
    run_eq += u < w ? L.wave_eq[u] : 0;
    all_gt += L.wave_cnt[u];
  }
  const int need_eq = k - all_gt;
  run_c = c_lo;
#pragma unroll 1
  for (int i0 = i_lo; i0 < i_hi; i0 += kWave) {  // uniform trip count per wave
    const int i = i0 + lane;
    const bool cand = i < i_hi && candidate(i);
    const uint64_t cands = __ballot(cand);
    const double v = cand ? h[run_c + mask_prefix(cands)] : -1.0;
    run_c += __popcll(cands);
    const uint64_t key = order_key(v);
    const uint64_t mg = __ballot(cand && key > t), me = __ballot(cand && key == t);
    const int gt_before = run_gt + mask_prefix(mg), eq_before = run_eq + mask_prefix(me);
    run_gt += __popcll(mg);
    run_eq += __popcll(me);
    if (cand && (key > t || (key == t && eq_before < need_eq)))
      reinterpret_cast<uint2*>(L.win)[gt_before + min(eq_before, need_eq)] = make_uint2((uint32_t)i, __float_as_uint((float)v));
  }
}

// The stored values are within delta(b, j) = err_c |u_j| |x_b| of the activations.  With f and c the edges of the fine
// bin that holds the k-th largest stored value and hw = 2 err_c max|u| |x| >= 2 delta, the true k-th largest lies in
// [f - hw/2, c + hw/2): entries stored above H = c + hw are larger, entries stored below f - hw smaller, and what lies
// between is recomputed in fp64 (about fifteen entries at the ~1B shape).  With A entries above, the k - A largest recomputed
// ones complete the selection.  The outcome is checked and not taken on trust: if the (k - A)-th largest recomputed
// value r satisfies L + hw/2 <= r <= H - hw/2, every entry above H is at least r and every one below L less than r.
// Leaves the selected (unit, value) pairs in L.win, in order, behind a barrier.  tok_sh: room for the token, d <= kRefineTokenMax.
template <int LOADS>
__device__ __forceinline__ void refine_token(const RefineParams& p, int b, bool counts_misses, uint4* tok_sh, RefineShared& L) {
  using K = uint32_t;
  using Keys = typename BatchKeys<uint32_t, LOADS>::Keys;
  constexpr int PER = Keys::PER;
  const int tid = (int)threadIdx.x, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(wave_id());
  const int N = p.N, k = p.k, d = p.d;
  HIRE_TS(40);
  const float* row = p.vals + (size_t)b * p.stride;
  const uint4* tok = reinterpret_cast<const uint4*>(p.x + (size_t)b * d);
  Keys kr;
  kr.issue_clamped(row, N);
  uint32_t words[LOADS];  // the bitmap's words of this lane's units
#pragma unroll
  for (int e = 0; e < LOADS; ++e) words[e] = p.bitmap[min(kr.index(e, 0), N - 1) >> 5];
  if (d <= kRefineTokenMax) {
    for (int i = tid; i < d / 8; i += kSelThreads) tok_sh[i] = tok[i];
    tok = tok_sh;
  }
  const float xn = p.xnorm[b];
  float wn = 0.0f;
  for (int i = tid; i < p.wnorm_n; i += kSelThreads) wn = fmaxf(wn, p.wnorm_tiles[i]);
  wn = wave_max(wn);
  if (lane == 0) L.wave_max[w] = wn;
  {
    uint4* z = reinterpret_cast<uint4*>(L.win) + 2 * tid;
    z[0] = z[1] = make_uint4(0, 0, 0, 0);
  }
  if (tid == 0) L.sh.list_n = 0;
  kr.finish();
  kr.mask_beyond(N);
  if (p.all_rows) {  // uniform: units that no token shortlists have values as well
#pragma unroll
    for (int e = 0; e < LOADS; ++e) {
      const uint32_t bits = words[e] >> (kr.index(e, 0) & 31);  // four units, all in one word
#pragma unroll
      for (int q = 0; q < PER; ++q) kr.r[e][q] &= 0u - (bits >> q & 1u);
    }
  }
  __syncthreads();
  wn = wave_max(lane < kSelWaves ? L.wave_max[lane] : 0.0f);
  const uint32_t anchor = fine_bin(__float_as_uint(xn * wn * 1.001f));  // of a bound of every stored value
  const double hw = 2.0 * (double)p.err_c * (double)xn * (double)wn * 1.000001;
  HIRE_TS(41);
  uint32_t bin;
  int above_bin;
  bool beyond;
  const bool found = window_bin(kr, anchor, k, L.win, L.sh, &bin, &above_bin, &beyond);
  (void)above_bin;  // the window only proposes: the band's own counts decide
  (void)beyond;
  HIRE_TS(42);
  if (found) {  // uniform
    const double f = (double)__uint_as_float(bin << kFineShift), c = (double)__uint_as_float((bin + 1u) << kFineShift);
    const double lo_v = f - hw, hi_v = c + hw;
    const K lo_k = __float_as_uint(__double2float_rd(lo_v)), hi_k = __float_as_uint(__double2float_ru(hi_v));
    if (lo_v > 0.0) {  // uniform; non-negative floats order like their bit patterns
      // above: stored above hi_k; inside: in [lo_k, hi_k], the band
      const BinMasks<K> bm = bin_masks<K>(kr, lo_k, hi_k + 1u);
      for (uint32_t m = bm.inside; m != 0u;) {  // few lanes
        const int i = pop_first(kr, m), slot = atomicAdd(&L.sh.list_n, 1);
        if (slot < kBsCap) L.l_idx[slot] = i;
      }
      const int above = wave_sum(__popc(bm.above));
      if (lane == 0) L.wave_cnt[w] = above;
      __syncthreads();
      HIRE_TS(43);
      const int A = wave_sum(lane < kSelWaves ? L.wave_cnt[lane] : 0), C = L.sh.list_n, need = k - A;
      if (C <= kBsCap && need >= 1 && need <= C) {  // uniform
        for (int i = w; i < C; i += kSelWaves) {    // a wave per entry
          const double s = wave_row_dot(p.W + (size_t)L.l_idx[i] * d, tok, d);
          if (lane == 0) L.l_val[i] = (unsigned long long)__double_as_longlong(s);
        }
        __syncthreads();
        HIRE_TS(44);
        // Lane l holds entries l and l + 64.  A wave ranks (value descending, unit ascending) the entries of its own
        // part of the row only, one or two: as many as are ahead of them, by ballots.
        uint64_t kv[2], own[2], taken[2] = {0ull, 0ull};
        int ki[2], enough = 0, beyond = 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int i = lane + u * kWave;
          const bool in = i < C;
          kv[u] = in ? L.l_val[i] : 0ull;
          ki[u] = in ? L.l_idx[i] : 0x7FFFFFFF;
          const double v = __longlong_as_double((long long)kv[u]);
          enough += __popcll(__ballot(in && v >= lo_v + 0.5 * hw));
          beyond += __popcll(__ballot(in && v > hi_v - 0.5 * hw));
          own[u] = __ballot(in && ki[u] >= kr.base && ki[u] - kr.base < kr.len);
        }
        // this lane's key that list entry l of half u stands for, as a bit e * PER + q (0: another lane's)
        auto bit_here = [&](int u, int l) -> uint32_t {
          const int r = __builtin_amdgcn_readlane(ki[u], l) - kr.base;
          return lane == r % Keys::SPAN / PER ? 1u << (r / Keys::SPAN * PER + r % PER) : 0u;
        };
        uint32_t take = __brev(bm.above) >> (32 - LOADS * PER);
#pragma unroll
        for (int u = 0; u < 2; ++u)
          for (uint64_t m = own[u]; m != 0ull; m &= m - 1ull) {
            const int l = __builtin_ctzll(m), i = __builtin_amdgcn_readlane(ki[u], l);
            const uint64_t v = read_lane(kv[u], l);
            const int ahead = __popcll(__ballot(lane < C && ranks_ahead(kv[0], ki[0], v, i))) +
                              __popcll(__ballot(lane + kWave < C && ranks_ahead(kv[1], ki[1], v, i)));
            if (ahead < need) {  // uniform
              taken[u] |= 1ull << l;
              take |= bit_here(u, l);
            }
          }
        HIRE_TS(45);
        // the need-th largest value lies in [lo_v + hw/2, hi_v - hw/2]
        if (enough >= need && beyond < need) {  // uniform
          if (lane == 0) L.wave_eq[w] = above + __popcll(taken[0]) + __popcll(taken[1]);
          __syncthreads();
          const int pa = wave_scan_incl(lane < kSelWaves ? L.wave_eq[lane] : 0);
          int run = w > 0 ? __builtin_amdgcn_readlane(pa, w - 1) : 0;
          // This lane's selected keys of every load, counted in 16-bit fields (a wave holds at most 256 per load):
          // a prefix sum over the lanes gives the places of two loads at once.  A key that is not selected goes to a
          // place of its lane that nobody reads: a predicate per key would cost more than its store.
          uint2* pk = reinterpret_cast<uint2*>(L.win);
          constexpr uint32_t kField = (1u << PER) - 1u;
          int first[LOADS];
#pragma unroll
          for (int e0 = 0; e0 < LOADS; e0 += 2) {
            const int c0 = __popc(take >> (e0 * PER) & kField), c1 = __popc(take >> ((e0 + 1) * PER) & kField);
            const int incl = wave_scan_incl(c0 | c1 << 16), tot = __builtin_amdgcn_readlane(incl, kWave - 1);
            first[e0] = run + (incl & 0xFFFF) - c0;
            first[e0 + 1] = run + (tot & 0xFFFF) + (incl >> 16) - c1;
            run += (tot & 0xFFFF) + (tot >> 16);
          }
#pragma unroll
          for (int e = 0; e < LOADS; ++e) {
            int at = first[e];
#pragma unroll
            for (int q = 0; q < PER; ++q) {
              const bool in = (take >> (e * PER + q) & 1u) != 0u;
              pk[in ? at : kWin / 2 + lane] = make_uint2((uint32_t)kr.index(e, q), kr.r[e][q]);
              at += in ? 1 : 0;
            }
          }
          // recomputed values over the stored ones (a wave's stores to LDS stay in order)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            for (uint64_t m = taken[u]; m != 0ull; m &= m - 1ull) {
              const int l = __builtin_ctzll(m);
              const uint32_t bit = bit_here(u, l), v = __float_as_uint((float)__longlong_as_double((long long)read_lane(kv[u], l)));
              if (bit != 0u) {
                const int e = __builtin_ctz(bit) / PER;
                int at = first[0];
#pragma unroll
                for (int f = 1; f < LOADS; ++f) at = e == f ? first[f] : at;
                pk[at + __popc(take & (bit - 1u) & (kField << (e * PER)))].y = v;
              }
            }
          __syncthreads();
          HIRE_TS(46);
          return;
        }
      }
    }
  }
  if (tid == 0 && counts_misses && p.window_misses) atomicAdd(p.window_misses, 1u);
  __syncthreads();
  refine_streaming(p, b, tok, L, hw);
  __syncthreads();
}

// Where a kernel leaves a compute unit for it, one more workgroup lists the candidates meanwhile.
__device__ __forceinline__ void list_candidates(const RefineParams& p, RefineShared& L) {
  const int n = list_bitmap<kSelThreads>(p.bitmap, (p.N + 31) / 32, p.cand_out, p.cand_cap, L.sh);
  if (threadIdx.x == 0 && p.n_cand_out) *p.n_cand_out = n;
}

// Entries [t0, t1) of the packed ones -> the caller's columns.
__device__ __forceinline__ void write_selected(const RefineParams& p, int b, const RefineShared& L, int t0, int t1, uint2* list) {
  for (int t = t0 + (int)threadIdx.x; t < t1; t += kSelThreads) {
    const uint2 v = reinterpret_cast<const uint2*>(L.win)[t];
    const size_t o = (size_t)b * p.k + t;
    if (list) list[o] = v;
    if (p.idx_out) p.idx_out[o] = (int)v.x;
    if (p.val_out) p.val_out[o] = __uint_as_float(v.y);
  }
}

template <int LOADS>
__global__ __launch_bounds__(kSelThreads) void k_refine(RefineParams p) {
  __shared__ RefineShared L;
  extern __shared__ uint4 tok_sh[];
  const int b = (int)blockIdx.x;
  if (b == p.B) {
    list_candidates(p, L);
    return;
  }
  refine_token<LOADS>(p, b, true, tok_sh, L);
  write_selected(p, b, L, 0, p.k, p.list_out);
  HIRE_TS(47);
}

// Otherwise the list of the candidates is shared out over its workgroups, 64 units each.
// The bits come a word per thread (N <= 32768): issue() at the kernel's start, count() once they are surely there, write() behind
// a barrier.
struct CandidateShare {
  uint32_t bits;
  int upto;  // bits of the wave's words up to this lane's
  bool shared;
  __device__ __forceinline__ void issue(const RefineParams& p, int padded) {
    shared = p.cand_out != nullptr && (int)gridDim.x == padded;  // uniform
    if (shared) bits = p.bitmap[min((int)threadIdx.x, (p.N + 31) / 32 - 1)];
  }
  __device__ __forceinline__ void count(const RefineParams& p, RefineShared& L) {
    if (!shared) return;
    if ((int)threadIdx.x >= (p.N + 31) / 32) bits = 0u;
    upto = wave_scan_incl(__popc(bits));
    if (lane_id() == kWave - 1) L.cand_cnt[threadIdx.x / kWave] = upto;
  }
  __device__ __forceinline__ void write(const RefineParams& p, const RefineShared& L, int item, int n_items) const {
    if (!shared) return;
    const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id()), words = (p.N + 31) / 32;
    const int cnt = wave_scan_incl(lane < kSelWaves ? L.cand_cnt[lane] : 0);
    const int ahead = w > 0 ? __builtin_amdgcn_readlane(cnt, w - 1) : 0;
    for (int pair = item; 2 * pair < words; pair += n_items) {
      const int l = 2 * pair % kWave;  // (even: both words are the same wave's; beyond the end they are 0)
      if (2 * pair / kWave != w) continue;  // uniform
      const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)bits, l), b1 = (uint32_t)__builtin_amdgcn_readlane((int)bits, l + 1);
      const uint64_t m = (uint64_t)b1 << 32 | b0;
      const int at = ahead + __builtin_amdgcn_readlane(upto, l) - __popc(b0) + mask_prefix(m);
      if ((m >> lane & 1ull) != 0ull && at < p.cand_cap) p.cand_out[at] = pair * kWave + lane;
    }
    if (item == 0 && threadIdx.x == 0 && p.n_cand_out) *p.n_cand_out = __builtin_amdgcn_readlane(cnt, kSelWaves - 1);
  }
};

// The same selection with all values from 64 bits: several workgroups per token, each of which selects and forms the values of its
// share of the entries, a wave a row at a time.  Against k_exact_values behind k_refine it saves a boundary and the round trip
// through the list.
template <int LOADS>
__global__ __launch_bounds__(kSelThreads) void k_refine_values(RefineParams p, int parts) {
  __shared__ RefineShared L;
  extern __shared__ uint4 tok_sh[];
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int n_items = parts * p.B, padded = (n_items + 7) / 8 * 8;
  if ((int)blockIdx.x == padded) {
    list_candidates(p, L);
    return;
  }
  const int item = (int)(blockIdx.x & 7) * (padded / 8) + (int)(blockIdx.x >> 3);
  if (item >= n_items) return;  // uniform
  const int part = item / p.B, b = item % p.B;
  CandidateShare cand;
  cand.issue(p, padded);
  refine_token<LOADS>(p, b, part == 0, tok_sh, L);
  cand.count(p, L);
  const uint4* tok = p.d <= kRefineTokenMax ? tok_sh : reinterpret_cast<const uint4*>(p.x + (size_t)b * p.d);
  const int t1 = (int)((long long)p.k * (part + 1) / parts);
  for (int t = (int)((long long)p.k * part / parts) + w; t < t1; t += kSelWaves) {  // uniform
    const int unit = __builtin_amdgcn_readfirstlane((int)reinterpret_cast<const uint2*>(L.win)[t].x);
    const float v = (float)wave_row_dot<true>(p.W + (size_t)unit * p.d, tok, p.d);
    if (lane == 0) {
      const size_t o = (size_t)b * p.k + t;
      p.list_out[o] = make_uint2((uint32_t)unit, __float_as_uint(v));
      if (p.idx_out) p.idx_out[o] = unit;
      if (p.val_out) p.val_out[o] = v;
    }
  }
  lds_barrier();
  cand.write(p, L, item, n_items);
  HIRE_TS(47);
}

// The same selection and the second layer in one kernel: a workgroup has 8 LPR columns of one token, selects for it (every
// workgroup of a token does) and adds up the selected rows from the list in its own LDS.  Against k_refine and k_w2_list it saves
// a boundary and the lists' way through memory, and pays for the values and the band's rows being read by every slice's workgroup.
// Bound by the selection's chain (8.4 us at the ~1B shape), then by the rows (38 MB from HBM for 16 tokens in 7).
template <int LPR>
__global__ __launch_bounds__(kSelThreads) void k_refine_w2(RefineParams p, const uint16_t* __restrict__ W2, float* __restrict__ y) {
  constexpr int kCols = 8 * LPR, FL = 4;
  __shared__ RefineShared L;
  extern __shared__ uint4 dyn_sh[];  // the token; then the waves' sums
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int k = p.k, d = p.d;
  const int slices = (d + kCols - 1) / kCols, n_items = slices * p.B, padded = (n_items + 7) / 8 * 8;
  if ((int)blockIdx.x == padded) {
    list_candidates(p, L);
    return;
  }
  const int item = (int)(blockIdx.x & 7) * (padded / 8) + (int)(blockIdx.x >> 3);
  if (item >= n_items) return;  // uniform: the last dies' shares may be short
  const int slice = item / p.B, b = item % p.B;
  CandidateShare cand;
  cand.issue(p, padded);
  refine_token<4>(p, b, slice == 0, dyn_sh, L);
  const uint2* entries = reinterpret_cast<const uint2*>(L.win);
  const int sub = lane % LPR, first = w * (kWave / LPR) + lane / LPR;
  const int colc = min(slice * kCols + sub * 8, d - 8);
  float acc[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) acc[q] = 0.0f;
  auto entry = [&](int t) {
    const uint2 e = entries[min(t, k - 1)];
    return make_uint2(e.x, t < k ? e.y : 0u);
  };
  add_listed_rows<LPR, FL, kSelWaves>(W2 + colc, d, k, first, entry, acc);
  HIRE_TS(48);
  float* red = reinterpret_cast<float*>(dyn_sh);  // [kSelWaves][kCols]; the token was last read ahead of a barrier
  fold_lanes<LPR>(acc);
  if (lane < LPR) {
    float4* dst = reinterpret_cast<float4*>(&red[w * kCols + sub * 8]);
    dst[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
    dst[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
  }
  cand.count(p, L);
  __syncthreads();
  if (tid < kCols && slice * kCols + tid < d) {
    float s = 0.0f;
#pragma unroll
    for (int u = 0; u < kSelWaves; ++u) s += red[u * kCols + tid];
    y[(size_t)b * d + slice * kCols + tid] = s;
  }
  write_selected(p, b, L, (int)((long long)k * slice / slices), (int)((long long)k * (slice + 1) / slices), nullptr);
  cand.write(p, L, item, n_items);
  HIRE_TS(49);
}

// ---------------------------------------------------------------------------------------------------
// The activations of the selected (token, unit) pairs once more, in fp64 and rounded once: k_refine leaves the filter
// stage's fp32 values outside the band around the threshold, up to 2.3 half ulps off where one rounding is 1.0 at most
// (mean 0.39 to 0.50 against 0.34).  A wave per pair: bound by the round trips list -> row, 5.0 us for 33 tokens with 251
// units of d = 800 (13 MB), 6.1 for 8 with 819 of 2048 (27 MB); two rows per wave 0.3 to 1.4 us more, four 1 to 2.4.  A die
// takes an eighth of the (entries, token) pairs, entries first: neighbours in the lists are neighbours among the units, so
// that what tokens share comes from its L2.
constexpr int kEvThreads = 256;
constexpr int kEvEntries = kEvThreads / kWave;  // of a workgroup
__global__ __launch_bounds__(kEvThreads) void k_exact_values(uint2* __restrict__ lists, float* __restrict__ val_out,
                                                             const uint16_t* __restrict__ W,
                                                             const uint16_t* __restrict__ x, int B, int k, int d) {
  const int n_items = (k + kEvEntries - 1) / kEvEntries * B;
  const int item = (int)(blockIdx.x & 7) * ((n_items + 7) / 8) + (int)(blockIdx.x >> 3);
  if (item >= n_items) return;  // uniform: the last dies' shares may be short
  const int b = item % B, e = item / B * kEvEntries + __builtin_amdgcn_readfirstlane(wave_id());
  if (e >= k) return;
  const size_t at = (size_t)b * k + e;
  const float v = (float)wave_row_dot<true>(W + (size_t)lists[at].x * d, reinterpret_cast<const uint4*>(x + (size_t)b * d), d);
  if (lane_id() != 0) return;
  lists[at].y = __float_as_uint(v);
  if (val_out) val_out[at] = v;
}

// ---------------------------------------------------------------------------------------------------
// Both selections of a group-sparse step (groups of eight, eq. (6)), one workgroup per token: the k groups with the largest
// sums of eight absolute values, added in unit order in the values' own type.  A wave sums the groups of its own part of the
// row: whole vectors side by side, the lanes that share a group hand the sum on.  The sums stay in LDS for rows that need the
// narrowing.  Bound by the same chain as k_keys_select, behind a barrier more for the largest sum, the window's anchor.
// d = 512, 16000 units, 16 tokens 48.2 -> 37.8 us per step against the general selection, which reads the eight values a lane
// at a time; 64 tokens 96.9 -> 74.9; d = 1024, 6000 units, 16 tokens 42.8 -> 33.9; fp64 keys, 16000 units, 64 tokens 115 -> 81.
template <typename K, int LOADS>
struct GroupShared {
  using Keys = KeyRegs<K, LOADS, kSelThreads, false, true>;
  KeysSelectShared<K> s;
  __align__(16) K sums[Keys::CAPACITY + Keys::SPAN * LOADS];  // bit patterns, by group
};

template <typename K, int LOADS>
__global__ __launch_bounds__(kSelThreads) void k_group_select(GroupSelect p) {
  using Keys = typename GroupShared<K, LOADS>::Keys;
  constexpr int PER = Keys::PER, VPG = 8 * (int)sizeof(K) / 16, kVecs = LOADS * Keys::SPAN * VPG / kWave;  // vectors per group, lane
  extern __shared__ uint4 group_lds[];
  auto& G = *reinterpret_cast<GroupShared<K, LOADS>*>(group_lds);
  auto& S = G.s;
  const int b = (int)blockIdx.x, tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  Keys kr;
  kr.len = Keys::share(p.n_cap);
  kr.base = w * kr.len;
  const uint4* row = reinterpret_cast<const uint4*>(static_cast<const K*>(p.vals) + (size_t)b * p.stride);
  uint4 raw[kVecs];
#pragma unroll
  for (int i = 0; i < kVecs; ++i)
    if (i * kWave < kr.len * VPG) raw[i] = row[min(kr.base * VPG + i * kWave + lane, p.n_cap * VPG - 1)];  // uniform
  const int n = p.n_dev ? min(*p.n_dev, p.n_cap) : p.n_cap;
  {
    uint4* z = reinterpret_cast<uint4*>(S.win) + 2 * tid;
    z[0] = z[1] = make_uint4(0, 0, 0, 0);
  }
  if (tid == 0) S.sh.list_n = S.off_window = 0;
#pragma unroll
  for (int i = 0; i < kVecs; ++i)
    if (i * kWave < kr.len * VPG) {
      const int at = i * kWave + lane;  // vector of the wave's part
      K sum;
      if constexpr (sizeof(K) == 4) {
        const float x = fabsf(__uint_as_float(raw[i].x)), y = fabsf(__uint_as_float(raw[i].y)),
                    z = fabsf(__uint_as_float(raw[i].z)), u = fabsf(__uint_as_float(raw[i].w));
        const float before = dpp_move<0x111, 0xF>(0.0f, x + y + z + u);
        sum = __float_as_uint(before + x + y + z + u);
      } else {
        const double x = fabs(__hiloint2double((int)raw[i].y, (int)raw[i].x)), y = fabs(__hiloint2double((int)raw[i].w, (int)raw[i].z));
        double t = x + y;
#pragma unroll
        for (int q = 1; q < VPG; ++q) {
          const double before = dpp_move<0x111, 0xF>(0.0, t);
          t = lane % VPG == q ? before + x + y : t;
        }
        sum = (K)__double_as_longlong(t);
      }
      if (lane % VPG == VPG - 1 && at < kr.len * VPG) G.sums[kr.base + at / VPG] = sum;
    }
  __builtin_amdgcn_wave_barrier();  // a wave reads what it has written itself
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  K top = 0;
#pragma unroll
  for (int e = 0; e < LOADS; ++e)
#pragma unroll
    for (int q = 0; q < PER; ++q) kr.r[e][q] = G.sums[kr.index(e, q)];
  kr.mask_beyond(n);
#pragma unroll
  for (int e = 0; e < LOADS; ++e)
#pragma unroll
    for (int q = 0; q < PER; ++q) top = kr.r[e][q] > top ? kr.r[e][q] : top;
  top = wave_max(top);
  if (lane == 0) S.wave_top[w] = top;
  __syncthreads();
  const uint32_t anchor = fine_bin((K)wave_max((K)(lane < kSelWaves ? S.wave_top[lane] : 0)));
  const uint32_t take = keys_take<K>(kr, G.sums, p.k, anchor, S, p.window_misses);
  if (p.bitmap != nullptr) {
    add_bits(kr, take, p.bitmap);
    return;
  }
  // places of the selected groups in order; then their units, eight neighbouring threads a group
  __syncthreads();  // the narrowing's readers of wave_cnt are done
  const int mine = wave_sum(__popc(take));
  if (lane == 0) S.wave_cnt[w] = mine;
  __syncthreads();
  const int incl = wave_scan_incl(lane < kSelWaves ? S.wave_cnt[lane] : 0);
  int at = w > 0 ? __builtin_amdgcn_readlane(incl, w - 1) : 0;
  int* place = reinterpret_cast<int*>(S.win);  // (k <= kWin)
#pragma unroll
  for (int e = 0; e < LOADS; ++e) {
    const uint32_t bits = take >> (e * PER) & ((1u << PER) - 1u);
    const int c = __popc(bits), upto = wave_scan_incl(c);
    int o = at + upto - c;
#pragma unroll
    for (int q = 0; q < PER; ++q)
      if ((bits >> q & 1u) != 0u) place[o++] = kr.index(e, q);
    at += __builtin_amdgcn_readlane(upto, kWave - 1);
  }
  __syncthreads();
  const int units = 8 * p.k;
  const double* h = static_cast<const double*>(p.vals) + (size_t)b * p.stride;
  for (int t0 = tid; t0 < units; t0 += 4 * kSelThreads) {  // four position -> value chains in flight
    int group[4];
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = min(t0 + u * kSelThreads, units - 1), pos = place[t / 8];
      group[u] = p.map[pos];
      v[u] = h[(size_t)pos * 8 + t % 8];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + u * kSelThreads;
      if (t < units) {
        const size_t o = (size_t)b * units + t;
        p.list_out[o] = make_uint2((uint32_t)(group[u] * 8 + t % 8), __float_as_uint((float)v[u]));
        if (p.val_out) p.val_out[o] = (float)v[u];
        if (p.idx_out && t % 8 == 0) p.idx_out[(size_t)b * p.k + t / 8] = group[u];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------------
bool batch_select_supported(int N, int k) { return N >= 1 && N <= 2 * 16384 && k <= kWin / 2; }

hipError_t launch_keys_select(const KeysSelect& p, int B, hipStream_t s) {
  if (!keys_select_ok(p)) return hipErrorInvalidValue;
  if (p.f64)
    return launch(p.N <= 16384 ? k_keys_select<uint64_t, 8> : k_keys_select<uint64_t, 16>, dim3(B), dim3(kSelThreads), 0, s, p);
  return launch(p.N <= 16384 ? k_keys_select<uint32_t, 4> : k_keys_select<uint32_t, 8>, dim3(B), dim3(kSelThreads), 0, s, p);
}

hipError_t launch_group_select(const GroupSelect& p, int B, hipStream_t s) {
  if (p.n_cap < 1 || p.n_cap > kGroupSelectMax || p.k < 1 || p.k > p.n_cap || reinterpret_cast<uintptr_t>(p.vals) % 16 != 0 ||
      p.stride % 8 != 0 || (p.bitmap == nullptr && (!p.f64 || !p.map || !p.list_out)))
    return hipErrorInvalidValue;
  static std::atomic<size_t> raised_to[3] = {};
  auto go = [&](auto kernel, size_t lds, std::atomic<size_t>& raised) {
    if (const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, raised); e != hipSuccess)
      return e;
    return launch(kernel, dim3(B), dim3(kSelThreads), lds, s, p);
  };
  if (!p.f64) return go(k_group_select<uint32_t, 1>, sizeof(GroupShared<uint32_t, 1>), raised_to[0]);
  if (p.n_cap <= kGroupSelectMax / 2) return go(k_group_select<uint64_t, 1>, sizeof(GroupShared<uint64_t, 1>), raised_to[1]);
  return go(k_group_select<uint64_t, 2>, sizeof(GroupShared<uint64_t, 2>), raised_to[2]);
}

hipError_t launch_exact_values(uint2* lists, float* val_out, const uint16_t* W, const uint16_t* x, int B, int k, int d,
                               hipStream_t s) {
  const int items = (k + kEvEntries - 1) / kEvEntries * B;
  return launch(k_exact_values, dim3((items + 7) / 8 * 8), dim3(kEvThreads), 0, s, lists, val_out, W, x, B, k, d);
}

// Workgroups of a kernel whose items are shared out over the dies, and one for the list of the candidates if there is a compute
// unit for it.
static int refine_grid(int items, const RefineParams& p) {
  const int padded = (items + 7) / 8 * 8;
  return padded + (p.cand_out != nullptr && padded < 256 ? 1 : 0);
}

// Workgroups per token of k_refine_values, up to sixteen entries each where they are few: as many as one round has.  0: some wave would
// have more than three rows, one after the other, and k_exact_values, whose waves have one each, is as fast or faster.  us per step with that /
// with k_refine_values: d = 2048, k = 819 of 16384 units, 5 tokens 46.0 / 45.1, 8 51.3 / 50.0, 12 (three rows in some waves) 55.9 / 55.0, 15 57.0 /
// 56.5; k = 409 of 8191, 16 39.6 / 38.3, 27 44.2 / 43.7, 33 (four) 51.1 / 50.8, 64 (seven) 62.8 / 63.7; d = 4096, k = 409 of 8192, 5 54.4 / 52.7, 15 65.2 /
// 62.8; k = 51, 5 46.4 / 46.2; d = 1024, k = 400 of 8000, 8 29.5 / 27.9; k = 819 of 16383, 33 (seven) 57.7 / 60.7; k = 195 of 8001, 63 (four) 38.3 / 38.3; d = 800,
// k = 251 of 5003, 8 27.2 / 26.5, 33 33.2 / 32.7, k = 337, 33 (four) 34.3 / 34.9; d = 512, k = 2449 of 12000, 5 (four) 35.4 / 35.1; k = 1200 of 24000, 64
// 75.0 / 80.2; d = 256, k = 51 of 1024, 15 23.2 / 22.2, 64 25.3 / 24.5.  Requesting a wave's next two rows ahead, with the last one again past the
// end, was slower up to three rows (d = 800, 8 tokens 30.3 instead of 27.6).
static int refine_value_parts(int B, int k) {
  const int parts = min(256 / B, (k + kSelWaves - 1) / kSelWaves);  // (B <= 64)
  return (k + parts - 1) / parts > 3 * kSelWaves ? 0 : parts;
}

hipError_t launch_refine(const RefineParams& p, hipStream_t s) {
  if (!batch_select_supported(p.N, p.k) || p.stride % 4 != 0 || reinterpret_cast<uintptr_t>(p.vals) % 16 != 0 || p.d % 8 != 0)
    return hipErrorInvalidValue;
  const size_t lds = p.d <= kRefineTokenMax ? (size_t)p.d * 2 : 0;
  static std::atomic<size_t> raised_to[4] = {};
  auto go = [&](auto kernel, std::atomic<size_t>& raised) {
    if (const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, raised); e != hipSuccess)
      return e;
    return launch(kernel, dim3(p.B + (p.cand_out != nullptr ? 1 : 0)), dim3(kSelThreads), lds, s, p);
  };
  const int parts = refine_value_parts(p.B, p.k);
  if (p.exact_values && parts > 0) {
    auto values = [&](auto kernel, std::atomic<size_t>& raised) {
      if (const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, raised); e != hipSuccess)
        return e;
      return launch(kernel, dim3(refine_grid(parts * p.B, p)), dim3(kSelThreads), lds, s, p, parts);
    };
    return p.N <= 16384 ? values(k_refine_values<4>, raised_to[2]) : values(k_refine_values<8>, raised_to[3]);
  }
  const hipError_t e = p.N <= 16384 ? go(k_refine<4>, raised_to[0]) : go(k_refine<8>, raised_to[1]);
  return e == hipSuccess && p.exact_values ? launch_exact_values(p.list_out, p.val_out, p.W, p.x, p.B, p.k, p.d, s) : e;
}

template <int LPR>
static hipError_t refine_w2_launch(const RefineParams& p, const uint16_t* W2, float* y, hipStream_t s) {
  const size_t sums = (size_t)kSelWaves * 8 * LPR * sizeof(float), tok = p.d <= kRefineTokenMax ? (size_t)p.d * 2 : 0;
  const size_t lds = sums > tok ? sums : tok;
  static std::atomic<size_t> raised_to{0};
  if (const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(k_refine_w2<LPR>), lds, raised_to); e != hipSuccess)
    return e;
  const int items = (p.d + 8 * LPR - 1) / (8 * LPR) * p.B;
  return launch(k_refine_w2<LPR>, dim3(refine_grid(items, p)), dim3(kSelThreads), lds, s, p, W2, y);
}

// A workgroup fills a compute unit, and every one of them selects: one round of 256, of the narrowest slices that fit.
static int refine_w2_columns(int B, int d) {
  for (int cols = 64; cols <= 512; cols *= 2)
    if ((d + cols - 1) / cols * B <= 256) return cols;
  return 0;
}
// Where the rows are many (96 MB, several tokens' repeats counted) the caches bound the second layer, and k_w2_list's even shares of
// a die serve more of them from its L2: wide slices of one token per workgroup make two dies read the same columns, and 256 workgroups
// read values and band.  us per step with k_refine and k_w2_list / this kernel, d = 2048, k = 819 of 16384 units: 16 tokens 49.1 / 47.7,
// 24 55.6 / 54.4, 28 55.7 / 55.0 (94 MB), 32 58.8 / 59.5, 33 62.8 / 63.6, 48 64.6 / 65.6, 64 68.4 / 71.5 (with nine tenths in common 63.6 /
// 61.5); k = 327, 33 58.4 / 57.3, 64 62.7 / 62.6; k = 51, 64 50.5 / 52.0; d = 4096, k = 409 of 8192, 16 56.7 / 55.3, 32 59.8 / 59.7, k = 100, 16 46.6 / 45.0;
// d = 1024, k = 400 of 8000, 16 27.1 / 25.9, 33 31.4 / 30.0, 64 33.6 / 32.3; d = 512, k = 200 of 4000, 16 22.0 / 21.4, 64 26.4 / 26.0; d = 256, k = 51 of 2048,
// 16 20.7 / 19.9, 64 23.4 / 23.4; d = 64, k = 200 of 4000, 64 24.5 / 23.6.
constexpr long long kRefineW2Bytes = 96ll << 20;
bool refine_w2_supported(const RefineParams& p) {
  return p.N <= 16384 && !p.exact_values && refine_w2_columns(p.B, p.d) != 0 &&
         2ll * p.B * p.k * p.d <= kRefineW2Bytes;
}
hipError_t launch_refine_w2(const RefineParams& p, const uint16_t* W2, float* y, hipStream_t s) {
  if (!batch_select_supported(p.N, p.k) || !refine_w2_supported(p) || p.stride % 4 != 0 ||
      reinterpret_cast<uintptr_t>(p.vals) % 16 != 0 || p.d % 8 != 0)
    return hipErrorInvalidValue;
  switch (refine_w2_columns(p.B, p.d)) {
    case 64: return refine_w2_launch<8>(p, W2, y, s);
    case 128: return refine_w2_launch<16>(p, W2, y, s);
    case 256: return refine_w2_launch<32>(p, W2, y, s);
    default: return refine_w2_launch<64>(p, W2, y, s);
  }
}

}  // namespace hire

#ifdef HIRE_TIMESTAMPS
extern "C" int hire_debug_timestamps_batch_select(unsigned long long* host64) {
  return (int)hipMemcpyFromSymbol(host64, HIP_SYMBOL(hire_ts), sizeof(hire_ts));
}
#endif
