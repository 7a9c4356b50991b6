// Exact top-k selection kernels (TopInd_k / Top_k of arXiv 2402.09360 Sec. 3.1,
// used on both lines of Algorithm 1) and the bitmap compaction that forms the
// batch union of Sec. 3.4.1.
//
// One 1024-thread workgroup per score row.  Wave w owns the contiguous index
// range [w*M, (w+1)*M), M a multiple of 64, and walks it 64 at a time, so a
// wave ballot is a 64-bit slice of the selection mask in index order: ordered
// output positions come from popcounts, no sorting, and ties at the threshold
// go to the lowest indices by construction.
#include "fast_select.h"
#include "hist.h"
#include "kernels.h"
#include "select.h"

namespace hire {

constexpr int kItemsMax = 16;                       // most register-resident keys per thread
constexpr int kCachedMax = kSelThreads * kItemsMax; // 16384
constexpr int kRankMax = 4096;                      // largest k sorted into rank order
constexpr int kPackMax = 2048;                      // largest k emitted through the packed list in LDS
static_assert(kPackMax * (8 + 4) <= kHistWindow * 4, "the packed list reuses the window histogram's LDS");

template <typename V>
struct KeyOf;
template <>
struct KeyOf<float> {
  using K = uint32_t;
};
template <>
struct KeyOf<double> {
  using K = uint64_t;
};

// Selection of row b by one whole workgroup.  dyn: rank order only, K keys[k] then int pos[k], int rank[k].
// win: kHistWindow words of LDS for the window histogram, or nullptr to go straight to range narrowing.
// ITEMS: keys a thread keeps in registers (rows of at most ITEMS * 1024 entries), or 0 to stream the row from
// memory on every pass.
template <typename V, int ITEMS>
__device__ __forceinline__ void select_row(const SelectParams& p, int b, SelShared& sh, unsigned long long* dyn,
                                           uint32_t* win) {
  using K = typename KeyOf<V>::K;
  __shared__ int tot_gt[kSelWaves], tot_eq[kSelWaves];

  // Everything the kernel needs first goes out in one batch of loads: the device-side count, the keys and the
  // index map.  The keys are laid out over the waves by the host-known bound of the count, so that their
  // addresses do not wait for the count itself.
  const int nload = p.n_dev ? p.n_cap : p.n;
  const int k = p.k;
  const V* vals = reinterpret_cast<const V*>(p.vals) + (size_t)b * p.stride;
  const int32_t* map = p.map ? p.map + (size_t)b * p.map_stride : nullptr;
  const int lane = lane_id(), w = wave_id();
  const int M = (((nload + kSelWaves - 1) / kSelWaves) + kWave - 1) / kWave * kWave;
  const int base = w * M;
  const int iters = M / kWave;

  auto to_key = [&](V v) -> K {
    if (p.relu) v = v > (V)0 ? v : (V)0;
    return order_key(v);
  };
  auto load_key = [&](int i) -> K { return to_key(vals[i]); };

  HIRE_TS(0);
  const int n_raw = p.n_dev ? *p.n_dev : p.n;
  // Small selections are emitted in two phases: the selected (position, key) pairs are first packed into LDS in
  // output order, then one thread per output translates the position and stores; the index map is then read for
  // the selected positions only.  Otherwise the map is fetched for every position with the keys, because a load
  // inside the emission loop would cost one memory round trip per trip.
  const bool packed = win != nullptr && !p.rank_order && p.bitmap == nullptr && k <= kPackMax;
  constexpr bool CACHED = ITEMS > 0;
  constexpr int kItems = CACHED ? ITEMS : 1;
  K regs[kItems];
  int mapped[kItems];
  if (CACHED) {
    V raw[kItems];
#pragma unroll
    for (int e = 0; e < kItems; ++e) {  // clamped and unconditional, so that the loads do not wait for one another
      const int i = min(base + e * kWave + lane, nload - 1);
      raw[e] = vals[i];
      mapped[e] = (map && !p.rank_order && !packed) ? map[i] : base + e * kWave + lane;
    }
    const int n_now = p.n_dev ? min(n_raw, p.n_cap) : p.n;
#pragma unroll
    for (int e = 0; e < kItems; ++e) {
      const int i = base + e * kWave + lane;
      regs[e] = (e < iters && i < n_now) ? to_key(raw[e]) : (K)0;
    }
  }
  const int n = p.n_dev ? min(n_raw, p.n_cap) : p.n;
  HIRE_TS(9);
  // element visitor: f(e, i, key) for every owned, valid element in index order
  auto visit = [&](auto&& f) {
    if (CACHED) {
#pragma unroll
      for (int e = 0; e < kItems; ++e) {
        const int i = base + e * kWave + lane;
        if (e < iters && i < n) f(e, i, regs[e]);
      }
    } else {
      for (int e0 = 0; e0 < iters; e0 += 8) {  // eight clamped loads in flight, then their elements in index order
        K kk[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) kk[j] = load_key(min(base + (e0 + j) * kWave + lane, n - 1));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int i = base + (e0 + j) * kWave + lane;
          if (e0 + j < iters && i < n) f(e0 + j, i, kk[j]);
        }
      }
    }
  };

  // ---- the k-th largest key ----
  // First try: a fine histogram (2^14 order keys per bin) of the kHistWindow bins at and below the largest key,
  // built in LDS; the bin holding the k-th key follows from one walk, and the few keys inside it are ranked
  // directly.  Exact zeros are left out (after a ReLU they would all queue up on one counter).  When the window
  // does not answer - the k-th key lies below it or among the zeros, or its bin is crowded - the range narrowing
  // of select.h takes over.
  K T = 0;
  bool guided = false;
  if (win != nullptr) {
    const int tid = (int)threadIdx.x;
    K hi = 0;
    visit([&](int, int, K key) { hi = key > hi ? key : hi; });
    hi = wave_max(hi);
    __syncthreads();  // previous readers of red_a are done
    if (lane == 0) sh.red_a[w] = (unsigned long long)hi;
    for (int i = tid; i < kHistWindow; i += kSelThreads) win[i] = 0u;
    if (tid == 0) sh.list_n = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSelWaves; ++u) hi = (K)sh.red_a[u] > hi ? (K)sh.red_a[u] : hi;
    HIRE_TS(30);
    const int top_bin = (int)hist_bin(hi);
    const int base_bin = (top_bin | 7) - (kHistWindow - 1);  // a multiple of 8: the walk reads aligned groups
    const K zero_key = order_key((V)0);
    visit([&](int, int, K key) {
      const int rel = (int)hist_bin(key) - base_bin;
      if (rel >= 0 && key != zero_key) atomicAdd(&win[rel], 1u);
    });
    __syncthreads();
    const BinWalk wk = walk_histogram<kSelThreads>(win - base_bin, (uint32_t)top_bin, k, sh);
    HIRE_TS(31);
    if (wk.found && wk.cnt <= kSelSmall) {
      visit([&](int, int, K key) {
        if ((int)hist_bin(key) == wk.bin && key != zero_key) {
          const int q = atomicAdd(&sh.list_n, 1);
          if (q < kSelSmall) sh.list_key[q] = (unsigned long long)key;
        }
      });
      __syncthreads();
      const int m = min(sh.list_n, kSelSmall), need = k - wk.above;
      if (tid < m) {
        const K mine = (K)sh.list_key[tid];
        int cg = 0, cge = 0;
        for (int u0 = 0; u0 < m; u0 += 8) {  // eight LDS reads in flight
          K other[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) other[j] = (K)sh.list_key[min(u0 + j, m - 1)];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            cg += (u0 + j < m) && other[j] > mine;
            cge += (u0 + j < m) && other[j] >= mine;
          }
        }
        if (cg < need && need <= cge) sh.bc_key = (unsigned long long)mine;  // equal keys write the same value
      }
      __syncthreads();
      T = (K)sh.bc_key;
      guided = true;
      HIRE_TS(32);
    } else if (tid == 0 && p.window_misses != nullptr) {
      atomicAdd(p.window_misses, 1u);
    }
  }
  if (!guided) T = wg_kth_largest<K>([&](auto&& f) { visit([&](int, int, K key) { f(key); }); }, n, k, sh);

  // ---- ordered counts of keys above / equal to the threshold, per wave ----
  int cnt_gt = 0, cnt_eq = 0;
  visit([&](int, int, K key) {
    cnt_gt += key > T;
    cnt_eq += key == T;
  });
  cnt_gt = wave_sum(cnt_gt);
  cnt_eq = wave_sum(cnt_eq);
  __syncthreads();
  if (lane == 0) {
    tot_gt[w] = cnt_gt;
    tot_eq[w] = cnt_eq;
  }
  __syncthreads();
  int run_gt = 0, run_eq = 0, all_gt = 0;
  for (int u = 0; u < kSelWaves; ++u) {
    if (u < w) {
      run_gt += tot_gt[u];
      run_eq += tot_eq[u];
    }
    all_gt += tot_gt[u];
  }
  HIRE_TS(7);
  const int need_eq = k - all_gt;  // ties at the threshold that are taken, lowest indices first

  // ---- emission in index order ----
  K* rk_key = reinterpret_cast<K*>(dyn);
  int* rk_pos = reinterpret_cast<int*>(rk_key + (p.rank_order ? k : 0));
  // packed mode: the window histogram's LDS is free by now; K keys[kPackMax] then int pos[kPackMax]
  K* pk_key = reinterpret_cast<K*>(win);
  int* pk_pos = reinterpret_cast<int*>(pk_key + kPackMax);
  if (packed) __syncthreads();  // every wave is done with the window histogram
  // one step of 64 consecutive positions per wave; uniform trip count per wave, so the ballots are safe
  auto emit_step = [&](int e, K key_in, int mi) {
    const int i = base + e * kWave + lane;
    const bool valid = i < n;
    const K key = valid ? key_in : (K)0;
    const bool gt = valid && key > T, eq = valid && key == T;
    const uint64_t mg = __ballot(gt), me = __ballot(eq);
    const int gt_before = run_gt + mask_prefix(mg), eq_before = run_eq + mask_prefix(me);
    const bool sel = gt || (eq && eq_before < need_eq);
    const int out = gt_before + min(eq_before, need_eq);
    run_gt += __popcll(mg);
    run_eq += __popcll(me);
    const V v = key_value(key);
    if (p.bitmap) {
      const uint64_t ms = __ballot(sel);
      if (lane == 0 && (uint32_t)ms) atomicOr(&p.bitmap[(base + e * kWave) >> 5], (uint32_t)ms);
      if (lane == 32 && (uint32_t)(ms >> 32)) atomicOr(&p.bitmap[((base + e * kWave) >> 5) + 1], (uint32_t)(ms >> 32));
    }
    if (sel) {
      if (p.rank_order) {
        rk_key[out] = key;
        rk_pos[out] = i;
      } else if (packed) {
        pk_pos[out] = i;
        pk_key[out] = key;
      } else {
        if (p.idx_out) p.idx_out[(size_t)b * k + out] = mi;
        if (p.pos_out) p.pos_out[(size_t)b * k + out] = i;
        if (p.val_out) p.val_out[(size_t)b * k + out] = (float)v;
        if (p.list_out && p.gs == 0) p.list_out[(size_t)b * k + out] = make_uint2((uint32_t)mi, __float_as_uint((float)v));
      }
    }
  };
  if (CACHED) {
#pragma unroll
    for (int e = 0; e < kItems; ++e)  // unrolled: the register arrays are indexed statically
      if (e < iters) emit_step(e, regs[e], mapped[e]);
  } else {
    for (int e = 0; e < iters; ++e) {
      const int i = min(base + e * kWave + lane, n - 1);
      emit_step(e, load_key(i), (map && !p.rank_order) ? map[i] : base + e * kWave + lane);
    }
  }
  HIRE_TS(8);
  if (packed) {
    __syncthreads();
    for (int t = (int)threadIdx.x; t < k; t += kSelThreads) {
      const int i = pk_pos[t], mi = map ? map[i] : i;
      const float v = (float)key_value(pk_key[t]);
      if (p.idx_out) p.idx_out[(size_t)b * k + t] = mi;
      if (p.pos_out) p.pos_out[(size_t)b * k + t] = i;
      if (p.val_out) p.val_out[(size_t)b * k + t] = v;
      if (p.list_out && p.gs == 0) p.list_out[(size_t)b * k + t] = make_uint2((uint32_t)mi, __float_as_uint(v));
    }
  }
  if (p.list_out != nullptr && p.gs > 0) {  // the selected groups' units with their activations
    __syncthreads();  // pos_out of this row: written by this workgroup, visible after the barrier
    const int gmask = (1 << p.gs) - 1, ku = k << p.gs;
    const double* uh = p.unit_h + (size_t)b * p.unit_h_stride;
    for (int t0 = (int)threadIdx.x; t0 < ku; t0 += 4 * kSelThreads) {  // four position -> value chains in flight
      int ps[4], row[4];
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = min(t0 + u * kSelThreads, ku - 1) >> p.gs;
        ps[u] = packed ? pk_pos[t] : p.pos_out[(size_t)b * k + t];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int l = min(t0 + u * kSelThreads, ku - 1) & gmask;
        row[u] = ((map ? map[ps[u]] : ps[u]) << p.gs) + l;
        v[u] = uh[((size_t)ps[u] << p.gs) + l];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = t0 + u * kSelThreads;
        if (t < ku) {
          p.list_out[(size_t)b * ku + t] = make_uint2((uint32_t)row[u], __float_as_uint((float)v[u]));
          if (p.unit_val_out) p.unit_val_out[(size_t)b * ku + t] = (float)v[u];
        }
      }
    }
  }
  if (!p.rank_order) return;

  // ---- rank order: position of each selected entry among the k (value desc, index asc) ----
  constexpr int kPerThread = kRankMax / kSelThreads;
  // Up to two waves of entries: a lane each, and the workgroup's waves (of two, every other one) compare them with an equal part
  // of the others and add that up.  Beyond that by bins of the keys, or sorted where many share a bin.  us per call, compared /
  // by bins: 16 rows of 1000, 64 entries 5.9 / 6.9, 100 of them 7.9 / 8.0 (of equal values 7.9 / 16.7), 256 11.3 / 8.0, 512 28.0 /
  // 11.5; softmax step of two tokens through fp64 logits, 40000 classes, k = 100 31.2 / 32.4.
  int* rk_rank = rk_pos + k;
  const bool spread = k <= 2 * kWave;
  if (spread && (int)threadIdx.x < k) rk_rank[threadIdx.x] = 0;
  __syncthreads();
  auto spread_ranks = [&](auto entry_waves) __attribute__((always_inline)) {
    constexpr int kEntries = decltype(entry_waves)::value * kWave, kOthers = kEntries / (kSelThreads / kEntries);
    const int e = (int)threadIdx.x % kEntries, t = min(e, k - 1), first = (int)threadIdx.x / kEntries * kOthers;
    const K mine = rk_key[t];
    int rank = 0;
#pragma unroll
    for (int j0 = 0; j0 < kOthers; j0 += 4) {
      K other[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) other[j] = rk_key[min(first + j0 + j, k - 1)];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int u = first + j0 + j;  // the list is in index order, so u < t is "lower index"
        rank += u < k && (other[j] > mine || (other[j] == mine && u < t)) ? 1 : 0;
      }
    }
    if (e < k) atomicAdd(&rk_rank[t], rank);
    __syncthreads();
  };
  if (k <= kWave) {
    spread_ranks(std::integral_constant<int, 1>{});
  } else if (spread) {
    spread_ranks(std::integral_constant<int, 2>{});
  }
  int my_rank[kPerThread];
  V my_val[kPerThread];
#pragma unroll
  for (int q = 0; q < kPerThread; ++q) {
    my_rank[q] = -1;
    my_val[q] = (V)0;
  }
  auto put = [&](int q, int t, int rank) {
    const int i = rk_pos[t];
    const V v = key_value(rk_key[t]);
    if (p.idx_out) p.idx_out[(size_t)b * k + rank] = map ? map[i] : i;
    if (p.pos_out) p.pos_out[(size_t)b * k + rank] = i;
    if (p.val_out) p.val_out[(size_t)b * k + rank] = (float)v;
    my_rank[q] = rank;
    my_val[q] = v;
  };
  if (spread) {
    if ((int)threadIdx.x < k) put(0, (int)threadIdx.x, rk_rank[threadIdx.x]);
  } else {
    static_assert(kRankBins + kRankMax <= kHistWindow, "the bins and the list reuse the window's memory");
    int own[kPerThread];
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) own[u] = u * kSelThreads + (int)threadIdx.x;
    int* list = reinterpret_cast<int*>(win) + kRankBins;
    auto ahead = [&](int o, int t) { return rk_key[o] > rk_key[t] || (rk_key[o] == rk_key[t] && o < t); };  // index order
    using Item = std::conditional_t<sizeof(K) == 4, unsigned long long, KeyAndNumber>;  // key and place in the list
    constexpr int kMost = kHistWindow * 4 / (int)sizeof(Item);                           // as many as the window's memory holds
    const bool ranked = bucket_ranks<K>(
        k, own, [&](int t) { return rk_key[t]; }, ahead, win, list, k <= kMost ? rank_run(k) : k, sh, put);
    if (__builtin_expect(!ranked, 0)) {  // uniform
      Item* items = reinterpret_cast<Item*>(win);
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kPerThread; ++u)
        if (own[u] < k) {
          if constexpr (sizeof(K) == 4)
            items[own[u]] = (unsigned long long)~rk_key[own[u]] << 32 | (uint32_t)own[u];
          else
            items[own[u]] = Item{~rk_key[own[u]], (uint32_t)own[u]};
        }
      __syncthreads();
      if constexpr (sizeof(K) == 4)
        sort_list(items, k, ~0ull);
      else
        sort_list(items, k, Item{~0ull, ~0u});
#pragma unroll
      for (int u = 0; u < kPerThread; ++u)
        if (own[u] < k) {
          if constexpr (sizeof(K) == 4)
            put(u, (int)(uint32_t)items[own[u]], own[u]);
          else
            put(u, (int)items[own[u]].number, own[u]);
        }
    }
  }
  HIRE_TS(34);
  if (!p.prob_out) return;
  // ---- softmax over the k survivors: exp(z - zmax) / sum; the sorted values reuse the key array ----
  __syncthreads();
  V* sorted = reinterpret_cast<V*>(dyn);
#pragma unroll
  for (int q = 0; q < kPerThread; ++q)
    if (my_rank[q] >= 0) sorted[my_rank[q]] = my_val[q];
  __syncthreads();
  const double zmax = (double)sorted[0];
  double part = 0.0;
  for (int t = (int)threadIdx.x; t < k; t += kSelThreads) part += exp((double)sorted[t] - zmax);
  part = wave_sum(part);
  if (lane == 0) sh.red_a[w] = (unsigned long long)__double_as_longlong(part);
  __syncthreads();
  double sum = 0.0;
  for (int u = 0; u < kSelWaves; ++u) sum += __longlong_as_double((long long)sh.red_a[u]);
  for (int t = (int)threadIdx.x; t < k; t += kSelThreads)
    p.prob_out[(size_t)b * k + t] = (float)(exp((double)sorted[t] - zmax) / sum);
  HIRE_TS(35);
}

template <typename V, int ITEMS>
__global__ __launch_bounds__(kSelThreads) void k_select(SelectParams p) {
  __shared__ SelShared sh;
  __shared__ __align__(16) uint32_t win[kHistWindow];
  extern __shared__ unsigned long long dyn[];
  select_row<V, ITEMS>(p, (int)blockIdx.x, sh, dyn, win);
}

// ---------------------------------------------------------------------------
// Bitmap -> ascending index list, one workgroup.
template <int kPer>  // words per thread and round, loaded together
__device__ __forceinline__ void compact_bitmap_per(const uint32_t* bitmap, int words, int32_t* __restrict__ list_out,
                                                   int32_t* __restrict__ count_out, int32_t* __restrict__ count_out2,
                                                   uint32_t* zero_ptr, int zero_words, SelShared& sh) {
  const int tid = (int)threadIdx.x;
  if (zero_ptr)
    for (int i = tid; i < zero_words; i += kSelThreads) zero_ptr[i] = 0u;
  int base = 0;
  for (int r0 = 0; r0 < words; r0 += kSelThreads * kPer) {
    const int w0 = r0 + tid * kPer;
    uint32_t m[kPer];
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint32_t v = bitmap[min(w0 + j, words - 1)];  // clamped and unconditional: the loads go out together
      m[j] = w0 + j < words ? v : 0u;
      cnt += __popc(m[j]);
    }
    int total;
    const int incl = wg_scan_incl(cnt, sh, &total);
    int out = base + incl - cnt;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      uint32_t mm = m[j];
      while (mm) {
        const int bit = __ffs((int)mm) - 1;
        list_out[out++] = (w0 + j) * 32 + bit;
        mm &= mm - 1;
      }
    }
    base += total;
  }
  if (tid == 0) {
    count_out[0] = base;
    if (count_out2) count_out2[0] = base;
  }
}

// A short bitmap spreads one word per thread, so that the list is written by many threads.
__device__ __forceinline__ void compact_bitmap(const uint32_t* bitmap, int words, int32_t* __restrict__ list_out,
                                               int32_t* __restrict__ count_out, int32_t* __restrict__ count_out2,
                                               uint32_t* zero_ptr, int zero_words, SelShared& sh) {
  if (words <= 2 * kSelThreads)
    compact_bitmap_per<1>(bitmap, words, list_out, count_out, count_out2, zero_ptr, zero_words, sh);
  else
    compact_bitmap_per<8>(bitmap, words, list_out, count_out, count_out2, zero_ptr, zero_words, sh);
}

__global__ __launch_bounds__(kSelThreads) void k_bitmap_compact(const uint32_t* bitmap, int words,
                                                                int32_t* __restrict__ list_out,
                                                                int32_t* __restrict__ count_out,
                                                                int32_t* __restrict__ count_out2, uint32_t* zero_ptr,
                                                                int zero_words) {
  __shared__ SelShared sh;
  compact_bitmap(bitmap, words, list_out, count_out, count_out2, zero_ptr, zero_words, sh);
}

// ---------------------------------------------------------------------------
// Histogram-guided selection over many workgroups.  Grid (ceil(N / 4096), B): every workgroup of token b
// repeats the short walk over b's histogram (largest key from the producers' per-workgroup maxima, then the
// window of bins below it) and so knows the bin that holds the k'-th largest key; its own 4096 keys then fall
// into three classes: above that bin (selected: bit set in the union bitmap), inside it (listed for the
// resolving kernel), below (dropped).
constexpr int kMarkKeys = 4;  // keys per thread

// Largest key of token b from the producers' per-workgroup maxima, to all threads.
__device__ __forceinline__ uint32_t token_top_key(const MultiRegion& mr, int b, int slots, SelShared& sh) {
  const int tid = (int)threadIdx.x;
  const uint4 mx = reinterpret_cast<const uint4*>(mr.wgmax + (size_t)b * kWgMaxSlots)[tid];
  uint32_t top = 0u;
  top = (4 * tid + 0 < slots && mx.x > top) ? mx.x : top;
  top = (4 * tid + 1 < slots && mx.y > top) ? mx.y : top;
  top = (4 * tid + 2 < slots && mx.z > top) ? mx.z : top;
  top = (4 * tid + 3 < slots && mx.w > top) ? mx.w : top;
  return wg_max_u32(top, sh);
}

// Counting pass for long rows, where one atomic per key from the producer would pile up on the few cache lines
// that hold the populated bins.  Grid (ceil(N / 16384), B).  Bins are 2^shift order keys wide (coarser than the
// producer-side histogram); only the kHistWindow bins at and below the largest key's are counted, first in LDS,
// then with one global atomic per populated bin.
constexpr int kCountKeys = 16;  // keys per thread

__global__ __launch_bounds__(kSelThreads) void k_count_f32(const float* __restrict__ keys, int B, int N, int slots,
                                                           int shift, int relu, MultiRegion mr) {
  __shared__ SelShared sh;
  __shared__ uint32_t cnt[kHistWindow];
  if (!multi_hist_ok(mr.hdr, B)) return;
  const int b = (int)blockIdx.y, tid = (int)threadIdx.x;
  if (blockIdx.x == 0 && b == 0 && tid == 0) set_busy(mr.hdr);
  const float* row = keys + (size_t)b * N;
  const int i0 = (int)blockIdx.x * (kSelThreads * kCountKeys);
  float v[kCountKeys];
#pragma unroll
  for (int e = 0; e < kCountKeys; ++e) v[e] = row[min(i0 + e * kSelThreads + tid, N - 1)];
  if (relu) {
#pragma unroll
    for (int e = 0; e < kCountKeys; ++e) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
  }
  for (int i = tid; i < kHistWindow; i += kSelThreads) cnt[i] = 0u;
  const int top_bin = (int)(token_top_key(mr, b, slots, sh) >> shift);  // barriers inside: cnt is cleared
  const int lo_bin = top_bin - (kHistWindow - 1);
#pragma unroll
  for (int e = 0; e < kCountKeys; ++e) {
    const int rel = (int)(order_key(v[e]) >> shift) - lo_bin;
    if (i0 + e * kSelThreads + tid < N && rel >= 0) atomicAdd(&cnt[rel], 1u);
  }
  __syncthreads();
  uint32_t* hist = mr.hist + (size_t)b * kHistStride + kHistWindow + lo_bin;  // lo_bin >= -kHistWindow + 1: the apron
  for (int i = tid; i < kHistWindow; i += kSelThreads) {
    const uint32_t c = cnt[i];
    if (c) atomicAdd(&hist[i], c);
  }
}

__global__ __launch_bounds__(kSelThreads) void k_mark_f32(const float* __restrict__ keys, int B, int N, int kprime,
                                                          int slots, int shift, int relu, MultiRegion mr,
                                                          uint32_t* __restrict__ bitmap, long long bitmap_stride) {
  __shared__ SelShared sh;
  const int b = (int)blockIdx.y, tid = (int)threadIdx.x, lane = lane_id();
  bitmap += (size_t)b * bitmap_stride;  // stride 0: one bitmap for the union of all rows
  const bool ok = multi_hist_ok(mr.hdr, B);
  if (!ok) {  // histograms not usable yet: the resolving kernel selects by streaming and stamps the region
    if (blockIdx.x == 0 && tid == 0) {
      mr.walk[4 * b + 0] = kprime;
      mr.walk[4 * b + 1] = 0;
      mr.walk[4 * b + 2] = 0;
    }
    return;
  }
  const float* row = keys + (size_t)b * N;
  const int i0 = (int)blockIdx.x * (kSelThreads * kMarkKeys);
  float v[kMarkKeys];
#pragma unroll
  for (int e = 0; e < kMarkKeys; ++e) v[e] = row[min(i0 + e * kSelThreads + tid, N - 1)];
  if (relu) {
#pragma unroll
    for (int e = 0; e < kMarkKeys; ++e) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
  }
  const uint32_t top_bin = token_top_key(mr, b, slots, sh) >> shift;
  const BinWalk wk = walk_histogram<kSelThreads>(mr.hist + (size_t)b * kHistStride + kHistWindow, top_bin, kprime, sh);
  if (blockIdx.x == 0 && tid == 0) {
    mr.walk[4 * b + 0] = kprime - wk.above;
    mr.walk[4 * b + 1] = wk.found ? 1 : 0;
    mr.walk[4 * b + 2] = (int)top_bin;
  }
  if (!wk.found) return;
#pragma unroll
  for (int e = 0; e < kMarkKeys; ++e) {
    const int i = i0 + e * kSelThreads + tid;
    const uint32_t okey = order_key(v[e]);
    const int bin = (int)(okey >> shift);
    const bool valid = i < N;
    const uint64_t ms = __ballot(valid && bin > wk.bin);
    const int wbase = (i0 + e * kSelThreads + (tid & ~63)) >> 5;
    if (lane == 0 && (uint32_t)ms) atomicOr(&bitmap[wbase], (uint32_t)ms);
    if (lane == 32 && (uint32_t)(ms >> 32)) atomicOr(&bitmap[wbase + 1], (uint32_t)(ms >> 32));
    const bool amb = valid && bin == wk.bin;
    const uint64_t ma = __ballot(amb);
    if (ma) {
      int base = 0;
      if (lane == 0) base = (int)atomicAdd(&mr.amb_n[b], (uint32_t)__popcll(ma));
      base = __builtin_amdgcn_readfirstlane(base);
      const int pos = base + mask_prefix(ma);
      if (amb && pos < kAmbCap) mr.amb[(size_t)b * kAmbCap + pos] = AmbEntry{okey, i};
    }
  }
}

// Second half, grid (1 + cleaners, B).  Workgroup (0, b) ranks the listed keys of token b's threshold bin by (key
// descending, index ascending) and sets the bits of the first `need`; a token whose histogram did not answer
// (region not stamped, threshold outside the window, list overflow) is selected by the streaming kernel's
// method instead.  Workgroups (c > 0, b) put a slice of token b's histogram back to all-zero: only the bins
// its keys touched, or everything when the region is not stamped yet.
constexpr int kCleanKeys = 4096;  // keys per cleaning workgroup

__global__ __launch_bounds__(kSelThreads) void k_resolve_compact(const float* __restrict__ keys, int B, int N, int kprime,
                                                                 int shift, int relu, MultiRegion mr, uint32_t* bitmap,
                                                                 long long bitmap_stride) {
  __shared__ SelShared sh;
  __shared__ AmbEntry amb_sh[kAmbCap];
  __shared__ int rank_sh[kAmbCap];
  const int b = (int)blockIdx.y, tid = (int)threadIdx.x;
  bitmap += (size_t)b * bitmap_stride;  // stride 0: one bitmap for the union of all rows
  HIRE_TS(40);
  const bool ok = multi_hist_ok(mr.hdr, B);
  uint32_t* hist = mr.hist + (size_t)b * kHistStride;
  const float* row = keys + (size_t)b * N;
  if (blockIdx.x == 0) {
    const int need = mr.walk[4 * b + 0];
    const bool found = mr.walk[4 * b + 1] != 0;
    const int m = (int)mr.amb_n[b];
    if (ok && found && m <= kAmbCap) {
      HIRE_TS(41);
      for (int t = tid; t < m; t += kSelThreads) amb_sh[t] = mr.amb[(size_t)b * kAmbCap + t];
      __syncthreads();
      HIRE_TS(42);
      // rank of every listed key among the m, the comparisons of one key spread over as many threads as fit
      // (a wave issues an instruction every few cycles only, so a lone thread's m-step loop is slow)
      const int padded = (m + kWave - 1) / kWave * kWave;
      const int slices = padded <= kSelThreads ? kSelThreads / padded : 1;
      const int per = (m + slices - 1) / slices;
      for (int t = tid; t < kAmbCap; t += kSelThreads) rank_sh[t] = 0;
      __syncthreads();
      for (int t0 = 0; t0 < m; t0 += kSelThreads / slices) {
        const int t = t0 + tid % (kSelThreads / slices), sl = tid / (kSelThreads / slices);
        if (t < m && sl < slices) {
          const AmbEntry mine = amb_sh[t];
          const int u_lo = sl * per, u_hi = min(m, u_lo + per);
          int rank = 0;
          for (int u0 = u_lo; u0 < u_hi; u0 += 8) {  // eight LDS reads in flight
            AmbEntry o[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = amb_sh[min(u0 + j, m - 1)];
#pragma unroll
            for (int j = 0; j < 8; ++j)
              rank += (u0 + j < u_hi) && ((o[j].okey > mine.okey) || (o[j].okey == mine.okey && o[j].idx < mine.idx));
          }
          atomicAdd(&rank_sh[t], rank);
        }
      }
      __syncthreads();
      for (int t = tid; t < m; t += kSelThreads) {
        const int idx = amb_sh[t].idx;
        if (rank_sh[t] < need) atomicOr(&bitmap[idx >> 5], 1u << (idx & 31));
      }
    } else {
      SelectParams sp{};
      sp.vals = keys;
      sp.stride = N;
      sp.n = N;
      sp.n_cap = N;
      sp.k = kprime;
      sp.relu = relu;
      sp.bitmap = bitmap;
      select_row<float, 0>(sp, b, sh, nullptr, reinterpret_cast<uint32_t*>(amb_sh));  // the list's LDS is free here
      if (tid == 0 && ok) atomicAdd(&mr.hdr->fallbacks, 1u);
    }
    HIRE_TS(43);
    __syncthreads();  // every thread has read amb_n[b]
    if (tid == 0) mr.amb_n[b] = 0u;
    if (tid == 0 && b == 0) mr.hdr->busy = 0u;
    HIRE_TS(44);
  } else {
    const int c = (int)blockIdx.x - 1, nc = (int)gridDim.x - 1;
    if (ok && shift == kHistShift) {  // the producer counted every key
      for (int i = c * kSelThreads + tid; i < N; i += nc * kSelThreads)
        hist[kHistWindow + hist_bin(order_key(relu && row[i] < 0.0f ? 0.0f : row[i]))] = 0u;
    } else if (ok) {                  // the counting pass filled the window below the largest key only
      uint32_t* win = hist + kHistWindow + mr.walk[4 * b + 2] - (kHistWindow - 1);
      for (int i = c * kSelThreads + tid; i < kHistWindow; i += nc * kSelThreads) win[i] = 0u;
    } else {
      for (int i = c * kSelThreads + tid; i < kHistStride; i += nc * kSelThreads) hist[i] = 0u;
    }
  }
}

// ---------------------------------------------------------------------------
// topk_select on long rows: the same many-workgroup selection with a bitmap per row, framed by two small kernels.
// k_row_maxima (grid (ceil(N / 16384), B)) plays the producer: per-workgroup maxima of the keys, and it is the
// sequence's first kernel (clears the bitmaps, checks the layout signature).  k_emit_rows (one workgroup per row)
// turns the row's bitmap into the ascending index list with the values.
__global__ __launch_bounds__(kSelThreads) void k_row_maxima(const float* __restrict__ keys, int N, int relu, MultiRegion mr,
                                                            uint32_t* zero_ptr, long long zero_words, GeneralHeader* gh,
                                                            unsigned long long sig) {
  __shared__ SelShared sh;
  const long long gsz = (long long)gridDim.x * gridDim.y * kSelThreads;
  for (long long i = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * kSelThreads + threadIdx.x; i < zero_words; i += gsz)
    zero_ptr[i] = 0u;
  if (blockIdx.x == 0 && blockIdx.y == 0) general_header_check(gh, sig);
  const int b = (int)blockIdx.y, tid = (int)threadIdx.x;
  const float* row = keys + (size_t)b * N;
  const int i0 = (int)blockIdx.x * (kSelThreads * kCountKeys);
  float v[kCountKeys];
#pragma unroll
  for (int e = 0; e < kCountKeys; ++e) v[e] = row[min(i0 + e * kSelThreads + tid, N - 1)];  // clamped: a row's own key
  uint32_t m = 0u;
#pragma unroll
  for (int e = 0; e < kCountKeys; ++e) {
    const uint32_t ok = order_key(relu && v[e] < 0.0f ? 0.0f : v[e]);
    m = ok > m ? ok : m;
  }
  m = wg_max_u32(m, sh);
  if (tid == 0) mr.wgmax[(size_t)b * kWgMaxSlots + blockIdx.x] = m;
}

__global__ __launch_bounds__(kSelThreads) void k_emit_rows(const float* __restrict__ keys, int B, int N, int k, int relu,
                                                           MultiRegion mr, const uint32_t* __restrict__ bitmaps,
                                                           int words, int32_t* __restrict__ idx_out,
                                                           float* __restrict__ val_out, int32_t* __restrict__ counts) {
  __shared__ SelShared sh;
  const int b = (int)blockIdx.x;
  int32_t* list = idx_out + (size_t)b * k;
  compact_bitmap(bitmaps + (size_t)b * words, words, list, counts + b, nullptr, nullptr, 0, sh);
  if (b == 0 && threadIdx.x == 0 && !multi_hist_ok(mr.hdr, B)) {  // the histograms were cleared by the kernel before
    mr.hdr->fallbacks = 0u;
    mr.hdr->stamps += 1u;
    mr.hdr->layout_b = (uint32_t)B;
    mr.hdr->cookie = kMultiCookie;
  }
  if (val_out == nullptr) return;
  __syncthreads();  // the list is this workgroup's own: visible after the barrier
  const float* row = keys + (size_t)b * N;
  for (int t0 = 0; t0 < k; t0 += kSelThreads * 4) {  // four index -> value chains in flight per thread
    int j[4];
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) j[u] = list[min(t0 + u * kSelThreads + (int)threadIdx.x, k - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = row[j[u]];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + u * kSelThreads + (int)threadIdx.x;
      if (t < k) val_out[(size_t)b * k + t] = relu && v[u] < 0.0f ? 0.0f : (v[u] == 0.0f ? 0.0f : v[u]);
    }
  }
}

// Third part for bitmaps too long for the gather kernels to compact themselves, one workgroup: the union bitmap
// becomes the ascending candidate list, and a region that was not stamped is now (its histograms were cleared by
// the kernel before).  A kernel of its own rather than the last workgroup of the previous one: device-scope
// fences inside a kernel cost a write-back of the whole L2 here.
__global__ __launch_bounds__(kSelThreads) void k_union_compact(int B, MultiRegion mr, const uint32_t* bitmap, int words,
                                                               int32_t* __restrict__ list_out,
                                                               int32_t* __restrict__ count_out,
                                                               int32_t* __restrict__ count_out2, uint32_t* zero_ptr,
                                                               int zero_words) {
  __shared__ SelShared sh;
  compact_bitmap(bitmap, words, list_out, count_out, count_out2, zero_ptr, zero_words, sh);
  if (threadIdx.x == 0 && !multi_hist_ok(mr.hdr, B)) {
    mr.hdr->fallbacks = 0u;
    mr.hdr->stamps += 1u;
    mr.hdr->layout_b = (uint32_t)B;
    mr.hdr->cookie = kMultiCookie;
  }
}

// ---------------------------------------------------------------------------
// topk_select on long rows with few entries wanted (rows beyond 32768, k <= 2048): three kernels, without a histogram
// of the row.
//
//   k_tk_maxima  4096 disjoint groups of every row, interleaved (entry i belongs to group i % 4096): their largest keys
//   k_tk_gather  every workgroup of a row bounds the k-th largest key from below by the k-th largest of the maxima (the
//                lower edge of its fine bin: each maximum is a key of its own, so at least k keys reach it) and appends
//                its own keys at or above the bound to the row's list: about -4096 ln(1 - k / 4096) of them, 1180 for
//                k = 1024, in any order
//   k_tk_final   one workgroup per row ranks the list by (key descending, index ascending); the first k are the result,
//                in that order or once more ranked by index
//
// The list is counted, not trusted: a row that has no bound (its maxima spread beyond the window) or more such keys
// than the list holds (many equal ones) is selected from memory by the last kernel.  Interleaved groups, because the
// largest entries of rows with an order of their own are neighbours.  k = 2048 is half of the groups: 2840 entries.
// Bound: one read of the rows (16 x 256000: 16 MB) and the chain of the final kernel on one compute unit per row.
// Measured for 16 rows of 256000, k = 1024, rank order: 15.2 us per call (1.7 more with the lengths of all rows' lists in
// one line); the histogram route below took 45.
constexpr int kTkGroups = 4096;
constexpr int kTkMaxK = 2048;
constexpr int kTkMaxGroups = 256;
constexpr int kTkKeys = 16;  // keys per thread of the gathering kernel
static_assert(kTkGroups == kWgMaxSlots && kAmbCap % kSelThreads == 0, "the maxima and the list use the histogram route's places");
static_assert(kTkMaxK * (4 + 2 * 4) <= kAmbCap * (int)sizeof(AmbEntry), "rank order from memory: the list's LDS");

// The lengths of the rows' lists, in the place of the bitmaps that the longer sequence clears for itself: kilobytes apart, as
// the workgroups of all rows wait for what they add (side by side in one line 1.9 us longer for 16 rows of 256000).
struct TkCounts {
  uint32_t* first;
  int stride;
  __device__ __forceinline__ uint32_t* of(int b) const { return first + (size_t)b * stride; }
};

__device__ __forceinline__ uint32_t row_key(float v, int relu) { return order_key(relu && !(v > 0.0f) ? 0.0f : v); }

// Grid (16, B): 256 groups per workgroup, PARTS threads share one.  Also the sequence's first kernel: empties the rows' lists
// and checks the layout signature.
template <int PARTS>
__global__ __launch_bounds__(kTkMaxGroups * PARTS) void k_tk_maxima(const float* __restrict__ keys, int N, int relu,
                                                             MultiRegion mr, TkCounts cnt, GeneralHeader* gh,
                                                             unsigned long long sig) {
  constexpr int kStep = PARTS * kTkGroups;
  __shared__ uint32_t part_max[PARTS][kTkMaxGroups];
  if (blockIdx.x == 0 && blockIdx.y == 0) general_header_check(gh, sig);
  const int b = (int)blockIdx.y, tid = (int)threadIdx.x, own = tid % kTkMaxGroups, part = tid / kTkMaxGroups;
  const int g = (int)blockIdx.x * kTkMaxGroups + own, first = g + part * kTkGroups;
  const float* row = keys + (size_t)b * N;
  uint32_t m = 0u;
  for (int i0 = first; i0 < N; i0 += 16 * kStep) {  // sixteen loads in flight; those past the end repeat the first
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = row[i0 + u * kStep < N ? i0 + u * kStep : i0];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const uint32_t k = row_key(v[u], relu);
      m = k > m ? k : m;
    }
  }
  part_max[part][own] = m;
  __syncthreads();
  if (part != 0) return;
#pragma unroll
  for (int q = 1; q < PARTS; ++q) m = max(m, part_max[q][own]);
  mr.wgmax[(size_t)b * kWgMaxSlots + g] = m;
  if (g == 0) *cnt.of(b) = 0u;
}

// Grid (ceil(N / 16384), B).
__global__ __launch_bounds__(kSelThreads) void k_tk_gather(const float* __restrict__ keys, int N, int k, int relu,
                                                           MultiRegion mr, TkCounts counts) {
  __shared__ SelShared sh;
  __shared__ __align__(16) uint32_t win[kWin];
  __shared__ int base_sh;
  const int b = (int)blockIdx.y, tid = (int)threadIdx.x;
  const float* row = keys + (size_t)b * N;
  const int i0 = (int)blockIdx.x * (kSelThreads * kTkKeys);
  const uint4 mx4 = reinterpret_cast<const uint4*>(mr.wgmax + (size_t)b * kWgMaxSlots)[tid];
  float v[kTkKeys];
#pragma unroll
  for (int e = 0; e < kTkKeys; ++e) v[e] = row[min(i0 + e * kSelThreads + tid, N - 1)];
  {
    uint4* z = reinterpret_cast<uint4*>(win) + 2 * tid;
    z[0] = z[1] = make_uint4(0, 0, 0, 0);
  }
  const uint32_t mx[4] = {mx4.x, mx4.y, mx4.z, mx4.w};
  const uint32_t top = wg_max_u32(max(max(mx[0], mx[1]), max(mx[2], mx[3])), sh);  // barriers inside: win is clear
  const uint32_t anchor = top >> kFineShift;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t slot = anchor - (mx[q] >> kFineShift);
    if (slot < (uint32_t)kWin) atomicAdd(&win[slot], 1u);
  }
  __syncthreads();
  WinRegs<kSelThreads> wr;
  wr.issue(win);
  const WinWalk wk = walk_window<kSelThreads>(wr, k, sh);
  if (!wk.found) {  // uniform
    if (blockIdx.x == 0 && tid == 0) *counts.of(b) = kAmbCap + 1;
    return;
  }
  const uint32_t bound = max((anchor - (uint32_t)wk.slot) << kFineShift, 1u);  // key 0 stands for "past the end"
  uint32_t key[kTkKeys];
  int c = 0;
#pragma unroll
  for (int e = 0; e < kTkKeys; ++e) {
    key[e] = i0 + e * kSelThreads + tid < N ? row_key(v[e], relu) : 0u;
    c += key[e] >= bound ? 1 : 0;
  }
  int total;
  const int incl = wg_scan_incl(c, sh, &total);
  if (total == 0) return;  // uniform
  if (tid == 0) base_sh = (int)atomicAdd(counts.of(b), (uint32_t)total);
  __syncthreads();
  int at = base_sh + incl - c;
#pragma unroll
  for (int e = 0; e < kTkKeys; ++e)
    if (key[e] >= bound) {
      if (at < kAmbCap) mr.amb[(size_t)b * kAmbCap + at] = AmbEntry{key[e], i0 + e * kSelThreads + tid};
      ++at;
    }
}

__global__ __launch_bounds__(kSelThreads) void k_tk_final(const float* __restrict__ keys, int B, int N, int k, int relu,
                                                          int rank_order, MultiRegion mr, TkCounts counts,
                                                          int32_t* __restrict__ idx_out, float* __restrict__ val_out) {
  __shared__ SelShared sh;
  __shared__ __align__(16) uint32_t bins[kHistWindow];  // the ranking's; the window of a row selected from memory
  __shared__ __align__(16) AmbEntry list[kAmbCap];
  __shared__ AmbEntry chosen[kTkMaxK];
  const int b = (int)blockIdx.x, tid = (int)threadIdx.x;
  const int n = (int)*counts.of(b);
  const AmbEntry first = mr.amb[(size_t)b * kAmbCap + tid];  // asked for with the number that says whether it counts: 0.13 us
  int32_t* idx = idx_out + (size_t)b * k;
  float* val = val_out ? val_out + (size_t)b * k : nullptr;
  if (b == 0 && tid == 0 && !multi_hist_ok(mr.hdr, B)) {  // the workspace has taken this layout
    mr.hdr->fallbacks = 0u;
    mr.hdr->stamps += 1u;
    mr.hdr->layout_b = (uint32_t)B;
    mr.hdr->cookie = kMultiCookie;
  }
  if (n < k || n > kAmbCap) {  // uniform
    SelectParams sp{};
    sp.vals = keys;
    sp.stride = N;
    sp.n = N;
    sp.n_cap = N;
    sp.k = k;
    sp.relu = relu;
    sp.rank_order = rank_order;
    sp.idx_out = idx_out;
    sp.val_out = val_out;
    select_row<float, 0>(sp, b, sh, reinterpret_cast<unsigned long long*>(list), bins);
    if (tid == 0) atomicAdd(&mr.hdr->fallbacks, 1u);
    return;
  }
  AmbEntry own[kAmbCap / kSelThreads];
  own[0] = first;
#pragma unroll
  for (int u = 1; u < kAmbCap / kSelThreads; ++u)
    if (u * kSelThreads < n) own[u] = mr.amb[(size_t)b * kAmbCap + u * kSelThreads + tid];  // uniform; places past n hold old entries
  unsigned long long* both = reinterpret_cast<unsigned long long*>(list);  // of rows with many equal keys: sorted in one word
  static_assert(sizeof(AmbEntry) == sizeof(unsigned long long), "in the list's place");
  auto place = [&](int, const AmbEntry& e, int rank) {
    if (rank >= k) return;
    if (rank_order) {
      idx[rank] = e.idx;
      if (val) val[rank] = key_value(e.okey);
    } else {
      chosen[rank] = e;
    }
  };
  auto larger = [](const AmbEntry& o, const AmbEntry& e) { return o.okey > e.okey || (o.okey == e.okey && o.idx < e.idx); };
  const bool ranked = bucket_ranks<uint32_t>(n, own, [](const AmbEntry& e) { return e.okey; }, larger, bins, list, rank_run(n), sh, place);
  if (__builtin_expect(!ranked, 0)) {  // uniform
#pragma unroll
    for (int u = 0; u < kAmbCap / kSelThreads; ++u)
      if (u * kSelThreads + tid < n) both[u * kSelThreads + tid] = (unsigned long long)~own[u].okey << 32 | (uint32_t)own[u].idx;
    __syncthreads();
    sort_list(both, n, ~0ull);
    for (int t = tid; t < min(n, k); t += kSelThreads) place(0, AmbEntry{~(uint32_t)(both[t] >> 32), (int32_t)(uint32_t)both[t]}, t);
  }
  if (rank_order) return;
  __syncthreads();
  AmbEntry mine[kTkMaxK / kSelThreads];
#pragma unroll
  for (int u = 0; u < kTkMaxK / kSelThreads; ++u) mine[u] = chosen[min(u * kSelThreads + tid, k - 1)];
  auto write = [&](int, const AmbEntry& e, int rank) {
    idx[rank] = e.idx;
    if (val) val[rank] = key_value(e.okey);
  };
  auto lower = [](const AmbEntry& o, const AmbEntry& e) { return o.idx < e.idx; };
  const bool listed = bucket_ranks<uint32_t>(
      k, mine, [](const AmbEntry& e) { return ~(uint32_t)e.idx; }, lower, bins, list, rank_run(k), sh, write);
  if (__builtin_expect(!listed, 0)) {  // uniform
#pragma unroll
    for (int u = 0; u < kTkMaxK / kSelThreads; ++u)
      if (u * kSelThreads + tid < k) both[u * kSelThreads + tid] = (unsigned long long)(uint32_t)mine[u].idx << 32 | mine[u].okey;
    __syncthreads();
    sort_list(both, k, ~0ull);
    for (int t = tid; t < k; t += kSelThreads) write(0, AmbEntry{(uint32_t)both[t], (int32_t)(both[t] >> 32)}, t);
  }
}

// ---------------------------------------------------------------------------
// The same selection for rows of non-negative values (scorer keys and activations after a ReLU) of at most 16384
// entries, in index order: the leaner machinery of fast_select.h.  The values' bit patterns are the keys, entries
// at and beyond the row's length are zeroed once, so no pass tests validity; the largest key's bin anchors a
// window histogram that is built in LDS, the walk proposes the threshold bin, two comparisons per key count what
// lies above it and find its own few keys, which every wave ranks for itself.  Selected positions go to a bitmap
// (the lanes that share a word fold their bits, one atomic per non-zero word) or, packed in LDS in output order,
// to the index / position / value outputs.  Irregular rows (all zero, threshold among the zeros, crowded bin) take the narrowing of
// select.h inside fast_select.
struct LeanShared {
  SelShared sh;
  uint32_t win[kWin];  // the window histogram; afterwards the row's bitmap, or the packed outputs
  int wave_cnt[kSelWaves];
  uint32_t wmax[kSelWaves];
};

// The row's keys are in kr (loaded, masked beyond n): anchor, window histogram, selection of the k largest.
template <int TB, typename K, int LOADS, bool FR>
__device__ __forceinline__ Selection<K> lean_select(const KeyRegs<K, LOADS, kSelThreads, FR>& kr, const void* vals, int k,
                                                    LeanShared& L, uint32_t* window_misses) {
  using Keys = KeyRegs<K, LOADS, kSelThreads, FR>;
  const int tid = (int)threadIdx.x, lane = lane_id(), w = wave_id();
  {
    uint4* z = reinterpret_cast<uint4*>(L.win) + 2 * tid;
    z[0] = z[1] = make_uint4(0, 0, 0, 0);
  }
  K mx = 0;
#pragma unroll
  for (int e = 0; e < LOADS; ++e)
#pragma unroll
    for (int q = 0; q < Keys::PER; ++q) mx = kr.r[e][q] > mx ? kr.r[e][q] : mx;
  mx = wave_max(mx);
  if (lane == 0) L.wmax[w] = fine_bin(mx);
  __syncthreads();
  const uint32_t anchor = wave_max(lane < kSelWaves ? L.wmax[lane] : 0u);  // bin of the row's largest key
  HIRE_TS(TB + 1);
#pragma unroll
  for (int e = 0; e < LOADS; ++e)
#pragma unroll
    for (int q = 0; q < Keys::PER; ++q) {
      const uint32_t slot = anchor - fine_bin(kr.r[e][q]);
      if (kr.r[e][q] != (K)0 && slot < (uint32_t)kWin) atomicAdd(&L.win[slot], 1u);  // zeros are never counted
    }
  __syncthreads();
  WinRegs<kSelThreads> wr;
  wr.issue(L.win);
  HIRE_TS(TB + 2);
  // (the window's LDS is free again once the walk inside has passed its first barrier)
  const Selection<K> sel = fast_select<TB + 3>(kr, vals, k, wr, anchor, anchor != 0u, L.sh, L.wave_cnt, window_misses, 0,
                                               k, true);
  HIRE_TS(TB + 6);
  return sel;
}

// The selected entries, packed in LDS in output order, to the index / position / value outputs.
// emit_all(fn): calls fn(position, output slot, value as float) for every selected entry.
template <typename EmitAll>
__device__ __forceinline__ void lean_outputs(const SelectParams& p, int b, int k, LeanShared& L, EmitAll&& emit_all) {
  const int tid = (int)threadIdx.x;
  int* pk_pos = reinterpret_cast<int*>(L.win);  // k <= kWin / 2
  float* pk_val = reinterpret_cast<float*>(L.win + kWin / 2);
  emit_all([&](int i, int out, float v) {
    pk_pos[out] = i;
    pk_val[out] = v;
  });
  __syncthreads();
  const int32_t* map = p.map ? p.map + (size_t)b * p.map_stride : nullptr;
  for (int t = tid; t < k; t += kSelThreads) {
    const int i = pk_pos[t], mi = map ? map[i] : i;
    const float v = pk_val[t];
    if (p.idx_out) p.idx_out[(size_t)b * k + t] = mi;
    if (p.pos_out) p.pos_out[(size_t)b * k + t] = i;
    if (p.val_out) p.val_out[(size_t)b * k + t] = v;
    if (p.list_out) p.list_out[(size_t)b * k + t] = make_uint2((uint32_t)mi, __float_as_uint(v));
  }
}

// One row: load, select, write the outputs.
template <int TB, typename V>
__device__ __forceinline__ void lean_row(const SelectParams& p, int b, const V* vals, LeanShared& L) {
  using K = typename KeyOf<V>::K;
  constexpr int LOADS = sizeof(V) == 4 ? 4 : 8;  // 16 waves x loads x 256 (128) keys = 16384
  using Keys = KeyRegs<K, LOADS, kSelThreads, sizeof(V) == 8>;  // the fp64 instance is short of registers
  static_assert(Keys::CAPACITY == kCachedMax, "rows of up to 16384 entries");
  const int cap = p.n_dev ? p.n_cap : p.n, k = p.k;
  const int n_raw = p.n_dev ? *p.n_dev : p.n;
  Keys kr;
  kr.issue_clamped(vals, cap);
  kr.finish();
  const int n = p.n_dev ? min(n_raw, p.n_cap) : p.n;
  kr.mask_beyond(n);
  const Selection<K> sel = lean_select<TB>(kr, vals, k, L, p.window_misses);
  if (p.bitmap != nullptr) {
    // A bitmap word covers 32 consecutive indices: the keys of 32 / PER neighbouring lanes of one load.  Those
    // lanes fold their bits together and one of them adds the word to the union: no ranks, no LDS, no barrier.
    constexpr int PER = Keys::PER, LPW = 32 / PER;
    const int lane = lane_id();
#pragma unroll
    for (int e = 0; e < LOADS; ++e) {
      uint32_t bits = 0u;
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const bool take = sel.plain ? kr.r[e][q] >= sel.cut.key
                                    : (kr.valid(e, q) && cut_takes(sel.cut, kr.r[e][q], kr.index(e, q)));
        bits |= take ? 1u << q : 0u;
      }
      bits <<= (lane % LPW) * PER;
#pragma unroll
      for (int m = 1; m < LPW; m <<= 1) bits |= (uint32_t)__shfl_xor((int)bits, m);
      if (lane % LPW == 0 && bits != 0u) atomicOr(&p.bitmap[(kr.base + e * Keys::SPAN) / 32 + lane / LPW], bits);
    }
  }
  if (p.idx_out != nullptr || p.pos_out != nullptr || p.val_out != nullptr || p.list_out != nullptr) {
    lean_outputs(p, b, k, L, [&](auto&& put) {
      fast_emit(kr, sel, 0, k, [&](int i, int out, K bits, int, int) {
        V v;
        __builtin_memcpy(&v, &bits, sizeof(V));
        put(i, out, (float)v);
      });
    });
  }
  HIRE_TS(TB + 7);
}

template <typename V>
__global__ __launch_bounds__(kSelThreads) void k_select_nonneg(SelectParams p) {
  __shared__ LeanShared L;
  constexpr int TB = sizeof(V) == 4 ? 10 : 40;  // stamps of the profiling build: the two instances apart
  HIRE_TS(TB);
  lean_row<TB, V>(p, (int)blockIdx.x, reinterpret_cast<const V*>(p.vals) + (size_t)blockIdx.x * p.stride, L);
}

// fp64 dot products of up to four bf16 rows (the first nr count; the others must point at readable rows) and a bf16
// token by one wave: products exact in fp32, sums in fp64; all loads of a 256-chunk slice are in flight together.
__device__ __forceinline__ void wave_rows_dot_f64(const uint16_t* const (&row)[4], int nr, const uint16_t* tok, int d,
                                                  double (&out)[4]) {
  const int cpr = d / 8, lane = lane_id();
  const uint4* t4 = reinterpret_cast<const uint4*>(tok);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma nounroll
  for (int c0 = 0; c0 < cpr; c0 += 2 * kWave) {
    uint4 wv[4][2], xv[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int c = min(c0 + v * kWave + lane, cpr - 1);
      xv[v] = t4[c];
#pragma unroll
      for (int u = 0; u < 4; ++u) wv[u][v] = reinterpret_cast<const uint4*>(row[u])[c];
    }
#pragma unroll
    for (int v = 0; v < 2; ++v)
      if (c0 + v * kWave + lane < cpr) {
        const uint32_t xd[4] = {xv[v].x, xv[v].y, xv[v].z, xv[v].w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (u < nr) {  // uniform
            const uint32_t wd[4] = {wv[u][v].x, wv[u][v].y, wv[u][v].z, wv[u][v].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              acc[u] += (double)(bf16_lo(wd[q]) * bf16_lo(xd[q]));
              acc[u] += (double)(bf16_hi(wd[q]) * bf16_hi(xd[q]));
            }
          }
        }
      }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) out[u] = wave_sum(acc[u]);
}

// ---------------------------------------------------------------------------
// Filter and refine for the classifier (Algorithm 1 with phi = identity, then eq. (2)): the row holds fp32 logits
// within err_c |w| |x| of the true ones.  With t~ the k-th largest stored value, every entry stored below
// t~ - 2 err_c |x| max|w| has a true logit below that of k others, so only the entries at or above that mark -
// k and a few - are recomputed in fp64 (a wave per row), ranked (value descending, position ascending) and the
// first k kept, in rank order, with the softmax over them.  A lower bound of t~ serves as well: the k-th largest of
// the maxima that the filter stage left (up to 1024 per token; each is a value of an entry of its own), or the lower
// edge of its fine bin.  With M maxima about -M ln(1 - k/M) entries reach it, 66 for k = 64 of 1024; the row itself
// is passed over once, against the mark.  The entries go through an LDS list of kSmList; rows with more of them (many
// equal logits, fewer maxima than k) take several rounds, each merged with the best k so far.
// Measured at 64 tokens, 57600 entries: 12.5 + 6.8 us, 16 tokens, 16000 entries: 8.5 + 6.9.  One kernel with one
// workgroup per token and a histogram of the whole row: 31 and 21 us, half of it the products and a ranking loop of
// one thread per entry.  With 1024 slots instead of 2048 the parts of k = 512 overflow: 2048 shortlisted classes per token,
// 16 tokens 168 instead of 125 us per step (when one workgroup recomputed all that overflowed).
constexpr int kSmList = 2048;
constexpr int kSmSpan = 64 * kSelThreads;  // entries that one 64-bit mask per thread stands for
constexpr int kSmFirst = 256;              // entries of the first round, where 2 k are not more
static_assert(2 * kSoftmaxRefineMaxK <= kSmList, "the first round's entries");

// Two kernels.  k_softmax_parts: every workgroup of a token takes an equal part of the row, finds the bound from the
// maxima itself, recomputes its own part's entries at or above the mark and leaves them in its slots.
// k_softmax_refine (one workgroup per token) ranks them and takes the softmax.  One compute unit alone would be bound
// by the fp64 products of some 75 rows (160 vector instructions per row and wave, 8 us at 64 tokens).
//
// A part with more such entries than slots (a token of zeros, thousands of equal classes, fewer maxima than k) still recomputes
// them, its share of the work, and leaves their logits by position.  The second kernel then goes through the row's
// entries at or above the mark in rounds of up to 2048, and of a round only what ranks ahead of the k-th best so far is ranked
// anew; the first round is a small one, and what it finds raises the mark.  us per step with one token of zeros among 64, or one with
// a shortlist of equal classes, through fp64 logits / with all of that recomputed and ranked by one workgroup, 2048 against 2048 /
// so: 256000 classes of d = 2048, k' = 1200, k = 100 1030 / 18997 / 538, 1181 / 934 / 795 (other tokens 681 / 205 / 205); 100000 of
// 512, k' = 1100, k = 64 404 / 11265 / 202, 493 / 432 / 304; 140000 of 512, 16 tokens, k' = 5000 356 / 13782 / 245, 541 / 1417 / 487.
constexpr int kSpThreads = 256;
constexpr int kSpWinBins = 2048;  // bins of 2^kSpShift order keys
constexpr int kSpShift = 16;
struct SmEntry {
  unsigned long long key;  // order key of the fp64 logit
  int pos, pad;
};
// Slots of a token (kSmList in all, shared out evenly over its parts) behind the parts' counts.
__host__ __device__ inline int softmax_parts(int B) { return B > 32 ? 16 : 32; }
constexpr int kSpMaxParts = 32;
size_t softmax_refine_slot_bytes(int B) { return (size_t)B * (kSpMaxParts * sizeof(int) + kSmList * sizeof(SmEntry)); }
__device__ __forceinline__ int* sp_counts(void* slots, int b) { return static_cast<int*>(slots) + b * kSpMaxParts; }
__device__ __forceinline__ SmEntry* sp_entries(void* slots, int B, int b) {
  return reinterpret_cast<SmEntry*>(static_cast<int*>(slots) + B * kSpMaxParts) + (size_t)b * kSmList;
}

// What every workgroup of a token finds by itself, the same in each: the order key that an entry's stored value has to reach, and how
// far a true logit may be from that value.
template <int NT>
struct SmMark {
  SelSharedT<NT> sh;
  uint32_t win[kSpWinBins], wave_a[NT / kWave], wave_b[NT / kWave];
};
struct SmMarked {
  uint32_t key;
  double reach;
  bool zero_rows_ok;  // the largest row norm is finite: a token of zeros has no other logits than 0
};
template <int NT>
__device__ __forceinline__ SmMarked softmax_mark(const SelectParams& p, int b, SmMark<NT>& S) {
  constexpr int NW = NT / kWave, kPer = kFilterMaxima / NT, kBins = kSpWinBins / NT;
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  float mx[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) mx[u] = p.maxima[(size_t)b * kFilterMaxima + min(tid + u * NT, p.n_maxima - 1)];
  const float tile_norm = p.wnorm_tiles[min(tid, p.wnorm_n - 1)];  // wnorm_n <= 256
#pragma unroll
  for (int u = 0; u < kBins; ++u) S.win[u * NT + tid] = 0u;
  if (tid == 0) S.sh.list_n = 0;
  uint32_t key[kPer], top = 0u;  // order keys of the maxima; none: 0, below every number
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    key[u] = tid + u * NT < p.n_maxima && mx[u] > -__builtin_inff() ? order_key(mx[u]) : 0u;
    top = key[u] > top ? key[u] : top;
  }
  const uint32_t wa = wave_max(top), wb = wave_max(__float_as_uint(tile_norm));  // non-negative floats order like their bits
  if (lane == 0) {
    S.wave_a[w] = wa;
    S.wave_b[w] = wb;
  }
  __syncthreads();
  const int anchor = (int)(wave_max(lane < NW ? S.wave_a[lane] : 0u) >> kSpShift);
  const float wn = __uint_as_float(wave_max(lane < NW ? S.wave_b[lane] : 0u));
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int s = anchor - (int)(key[u] >> kSpShift);
    if (key[u] != 0u && s < kSpWinBins) atomicAdd(&S.win[s], 1u);
  }
  __syncthreads();
  int c[kBins], mine = 0;
#pragma unroll
  for (int u = 0; u < kBins; ++u) {
    c[u] = (int)S.win[kBins * tid + u];
    mine += c[u];
  }
  int total, run = wg_scan_incl<NT>(mine, S.sh, &total) - mine;
  if (run < p.k && p.k <= run + mine) {
#pragma unroll
    for (int u = 0; u < kBins; ++u) {
      if (run < p.k && p.k <= run + c[u]) S.sh.bc_bin = kBins * tid + u;
      run += c[u];
    }
  }
  __syncthreads();
  SmMarked r{1u, (double)p.err_c * (double)p.xnorm[b] * (double)wn * 1.000001, wn < __builtin_inff()};
  if (total >= p.k) {  // uniform; with fewer maxima than k inside the window it is every entry
    const uint32_t floor_key = (uint32_t)max(anchor - S.sh.bc_bin, 0) << kSpShift;
    if (floor_key != 0u) r.key = order_key(__double2float_rd((double)key_value(floor_key) - 2.0 * r.reach));
  }
  return r;
}

// Whether all logits of a token are 0, whatever its candidates: to all threads of the workgroup.
template <int NT>
__device__ __forceinline__ bool softmax_all_zero(const SmMarked& mark, const uint16_t* tok, int d) {
  uint32_t bits = 0u;
  for (int i = (int)threadIdx.x; i < d / 8; i += NT) {
    const uint4 v = reinterpret_cast<const uint4*>(tok)[i];
    bits |= (v.x | v.y | v.z | v.w) & 0x7FFF7FFFu;
  }
  return !__syncthreads_or(bits != 0u) && mark.zero_rows_ok;
}

__global__ __launch_bounds__(kSpThreads) void k_softmax_parts(SelectParams p) {
  constexpr int NW = kSpThreads / kWave;
  __shared__ SmMark<kSpThreads> S;
  __shared__ int l_pos[kSmList / 8];
  __shared__ unsigned long long l_key[kSmList / 8];
  const int part = (int)blockIdx.x, P = (int)gridDim.x, b = (int)blockIdx.y, B = (int)gridDim.y;
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int cap = kSmList / P;
  const int n = p.n_dev ? min(*p.n_dev, p.n_cap) : p.n;
  const SmMarked mark = softmax_mark<kSpThreads>(p, b, S);
  // This part's entries: a wave's 64 of the row out of every P.  (Neighbours in the row, whose logits may all be the same, are
  // several parts' work.)  Eight loads of a wave at a time.
  const float* vals = reinterpret_cast<const float*>(p.vals) + (size_t)b * p.stride;
  const int first = part * kWave + lane, step = P * kWave;
  for (int j0 = w; j0 * step + part * kWave < n; j0 += 8 * NW) {  // uniform
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = vals[min(first + (j0 + u * NW) * step, n - 1)];  // clamped, unconditional
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = first + (j0 + u * NW) * step;
      if (i < n && order_key(v[u]) >= mark.key) {
        const int slot = atomicAdd(&S.sh.list_n, 1);
        if (slot < cap) l_pos[slot] = i;
      }
    }
  }
  __syncthreads();
  const int m = S.sh.list_n;
  if (tid == 0) sp_counts(p.refine_slots, b)[part] = m;
  const int32_t* map = p.map + (size_t)b * p.map_stride;
  const uint16_t* tok = p.refine_x + (size_t)b * p.refine_d;
  if (m > cap) {  // uniform: the logits only, for the second kernel
    if (softmax_all_zero<kSpThreads>(mark, tok, p.refine_d)) return;  // uniform: it needs none
    unsigned long long* keys = p.refine_keys + (size_t)b * p.refine_keys_stride;
    for (int i0 = part * kWave + w * step; i0 < n; i0 += NW * step) {
      const int i = min(i0 + lane, n - 1), cls = map[i];
      for (uint64_t in = __ballot(i0 + lane < n && order_key(vals[i]) >= mark.key); in != 0ull;) {  // uniform
        const uint16_t* row[4];
        int at[4], nr = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          at[u] = u > 0 ? at[u - 1] : 0;
          if (in != 0ull) {
            nr = u + 1;
            at[u] = __builtin_ctzll(in);
            in &= in - 1ull;
          }
          row[u] = p.refine_w + (size_t)__builtin_amdgcn_readlane(cls, at[u]) * p.refine_d;
        }
        double s4[4];
        wave_rows_dot_f64(row, nr, tok, p.refine_d, s4);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (lane == 0 && u < nr) keys[i0 + at[u]] = order_key(s4[u]);
      }
    }
    return;
  }
  for (int e0 = w; e0 < m; e0 += 4 * NW) {  // a wave per row, four rows in flight per wave
    const uint16_t* row[4];
    int nr = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * NW;
      if (e < m) nr = u + 1;
      row[u] = p.refine_w + (size_t)map[l_pos[min(e, m - 1)]] * p.refine_d;
    }
    double s4[4];
    wave_rows_dot_f64(row, nr, tok, p.refine_d, s4);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (lane == 0 && u < nr) l_key[e0 + u * NW] = order_key(s4[u]);  // -0 counts as +0
  }
  __syncthreads();
  SmEntry* out = sp_entries(p.refine_slots, B, b) + part * cap;
  for (int t = tid; t < m; t += kSpThreads) out[t] = SmEntry{l_key[t], l_pos[t], 0};
}

__global__ __launch_bounds__(kSelThreads) void k_softmax_refine(SelectParams p) {
  __shared__ SmMark<kSelThreads> S;
  __shared__ unsigned long long l_key[kSmList];  // order keys of fp64 logits
  __shared__ int l_pos[kSmList];
  __shared__ int b_pos[2][kSoftmaxRefineMaxK];
  __shared__ unsigned long long b_key[2][kSoftmaxRefineMaxK];
  __shared__ int l_n;
  const int b = (int)blockIdx.x, tid = (int)threadIdx.x, lane = lane_id(), w = wave_id();
  const int k = p.k;
  HIRE_TS(50);
  const int32_t* map = p.map + (size_t)b * p.map_stride;
  // what the parts left: thread t holds slots t and t + 1024; the valid ones move together
  constexpr int kOwn = kSmList / kSelThreads;
  const int P = softmax_parts((int)gridDim.x), cap = kSmList / P;
  int have_n[kOwn];
  SmEntry entry[kOwn];
#pragma unroll
  for (int u = 0; u < kOwn; ++u) {
    have_n[u] = sp_counts(p.refine_slots, b)[(tid + u * kSelThreads) / cap];
    entry[u] = sp_entries(p.refine_slots, (int)gridDim.x, b)[tid + u * kSelThreads];
  }
  unsigned long long pending = 0ull;  // bit i: value i counts and has not been listed yet
  int ready = 0;                      // entries from the slots
  int first = 0, end = 0;             // the span of the row that the mask stands for, the row's length (0: the slots served it)
  SmMarked mark{1u, 0.0, false};
  int have = 0, cur = 0;              // entries of the best list so far, and which of its two copies holds them
  const float* vals = reinterpret_cast<const float*>(p.vals) + (size_t)b * p.stride;
  unsigned long long* keys = p.refine_keys + (size_t)b * p.refine_keys_stride;
  auto scan = [&]() {  // value i of thread t is entry first + t + 1024 i
    const int n = min(end - first, kSmSpan);
    for (int i0 = 0; kSelThreads * i0 < n; i0 += 16) {  // uniform
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = vals[first + min(tid + kSelThreads * (i0 + u), n - 1)];  // clamped, unconditional
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (order_key(v[u]) >= mark.key && tid + kSelThreads * (i0 + u) < n) pending |= 1ull << (i0 + u);
    }
  };
  const int few = max(2 * k, kSmFirst);  // entries that are ranked as they are; of more of them, these come first
  int place[kOwn] = {-1, -1};            // of the slots' entries
  if (!__syncthreads_or(have_n[0] > cap || have_n[1] > cap)) {
    static_assert(kOwn == 2, "two slots per thread");
    const uint64_t vm[kOwn] = {__ballot(tid % cap < have_n[0]), __ballot((tid + kSelThreads) % cap < have_n[1])};
    if (lane == 0) S.wave_a[w] = (uint32_t)(__popcll(vm[0]) + __popcll(vm[1]));
    __syncthreads();
    const int incl = wave_scan_incl(lane < kSelWaves ? (int)S.wave_a[lane] : 0);
    ready = __builtin_amdgcn_readlane(incl, kSelWaves - 1);
    const int ws = __builtin_amdgcn_readfirstlane(w);
    int at = ws > 0 ? __builtin_amdgcn_readlane(incl, ws - 1) : 0;
#pragma unroll
    for (int u = 0; u < kOwn; ++u) {
      if (((vm[u] >> lane) & 1ull) != 0ull) {
        place[u] = at + mask_prefix(vm[u]);
        if (place[u] < few) {
          l_key[place[u]] = entry[u].key;
          l_pos[place[u]] = entry[u].pos;
        }
      }
      at += __popcll(vm[u]);
    }
  } else {
    // the parts that have not more than their slots: theirs by position too, behind the next barriers
#pragma unroll
    for (int u = 0; u < kOwn; ++u)
      if ((tid + u * kSelThreads) % cap < have_n[u] && have_n[u] <= cap) keys[entry[u].pos] = entry[u].key;
    mark = softmax_mark<kSelThreads>(p, b, S);
    HIRE_TS(51);
    if (softmax_all_zero<kSelThreads>(mark, p.refine_x + (size_t)b * p.refine_d, p.refine_d)) {  // uniform
      for (int t = tid; t < k; t += kSelThreads) {
        b_pos[0][t] = t;
        b_key[0][t] = order_key(0.0);
      }
      have = k;
      __syncthreads();
    } else {
      end = p.n_dev ? min(*p.n_dev, p.n_cap) : p.n;
      scan();
    }
    HIRE_TS(52);
  }
  while (end > 0 || have < k || ready > few) {  // uniform
    __syncthreads();  // the list and the counters of the round before have been read
    const bool full = have == k;  // uniform: there is a k-th best to compare with
    int listed = min(ready, few);
    if (full || end > 0) {  // uniform
      if (tid == 0) l_n = 0;
      __syncthreads();
      uint64_t key[kOwn];
      int pos[kOwn];
      bool stays[kOwn];
      if (end == 0) {  // the other slots
#pragma unroll
        for (int u = 0; u < kOwn; ++u) {
          stays[u] = place[u] >= few;
          pos[u] = entry[u].pos;
          key[u] = entry[u].key;
        }
      } else {
        const int room = full ? kSmList - k : few - have;
        while (pending != 0ull) {
          const int i = __builtin_ctzll(pending);
          const int slot = atomicAdd(&l_n, 1);
          if (slot >= room) break;
          l_pos[slot] = first + tid + kSelThreads * i;
          pending &= pending - 1ull;
        }
        __syncthreads();
        HIRE_TS(53);
        const int fresh = min(l_n, room);
#pragma unroll
        for (int u = 0; u < kOwn; ++u) {
          const int e = tid + u * kSelThreads;
          stays[u] = e < fresh;
          pos[u] = stays[u] ? l_pos[e] : 0;
          key[u] = keys[pos[u]];
        }
        __syncthreads();
        if (tid == 0) l_n = 0;
        __syncthreads();
      }
      // once there is a k-th best, only what ranks ahead of it is listed
#pragma unroll
      for (int u = 0; u < kOwn; ++u)
        if (stays[u] && !(full && !ranks_ahead(key[u], pos[u], (uint64_t)b_key[cur][k - 1], b_pos[cur][k - 1]))) {
          const int slot = atomicAdd(&l_n, 1);
          l_key[slot] = key[u];
          l_pos[slot] = pos[u];
        }
      __syncthreads();
      listed = l_n;
    }
    HIRE_TS(54);
    if (listed > 0) {  // uniform
      // the best so far join the list, then every entry is ranked among all of them, sixteen lanes per entry
      for (int t = tid; t < have; t += kSelThreads) {
        l_pos[listed + t] = b_pos[cur][t];
        l_key[listed + t] = b_key[cur][t];
      }
      __syncthreads();
      const int m = listed + have, sub = tid & 15;
      for (int t0 = 0; t0 < m; t0 += kSelThreads / 16) {  // uniform
        const int t = min(t0 + tid / 16, m - 1);
        const uint64_t mine = l_key[t];
        const int mine_pos = l_pos[t];
        int rank = 0;
        for (int u0 = sub; u0 < m; u0 += 64) {  // four LDS reads in flight
          uint64_t ok[4];
          int op[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            ok[j] = l_key[min(u0 + 16 * j, m - 1)];
            op[j] = l_pos[min(u0 + 16 * j, m - 1)];
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) rank += u0 + 16 * j < m && ranks_ahead(ok[j], op[j], mine, mine_pos) ? 1 : 0;
        }
        auto add = [](int a, int b) { return a + b; };
        rank = add(rank, dpp_move<0x111, 0xF>(0, rank));  // the row's last lane holds the sum of its sixteen
        rank = add(rank, dpp_move<0x112, 0xF>(0, rank));
        rank = add(rank, dpp_move<0x114, 0xF>(0, rank));
        rank = add(rank, dpp_move<0x118, 0xF>(0, rank));
        if (sub == 15 && t0 + tid / 16 < m && rank < k) {
          b_pos[cur ^ 1][rank] = mine_pos;
          b_key[cur ^ 1][rank] = mine;
        }
      }
      have = min(k, m);
      cur ^= 1;
    }
    const bool left = __syncthreads_or(pending != 0ull) || (!full && ready > few), next = !left && end - first > kSmSpan;  // uniform
    if (!left && !next) break;
    if (end > 0 && have == k && (next || !full)) {  // what is stored further below the k-th best than a logit can be off is not among the best
      const double lowest = key_value((uint64_t)b_key[cur][k - 1]) - mark.reach;
      if (lowest == lowest) mark.key = max(mark.key, order_key(__double2float_rd(lowest)));
      if (!next) {
        const unsigned long long unlisted = pending;
        pending = 0ull;
        scan();
        pending &= unlisted;
      }
    }
    if (next) {
      first += kSmSpan;
      scan();
    }
  }
  HIRE_TS(55);
  // the k survivors in rank order; softmax: exp(z - zmax) / sum
  const double zmax = key_value((uint64_t)b_key[cur][0]);
  double part = 0.0;
  for (int t = tid; t < k; t += kSelThreads) part += exp(key_value((uint64_t)b_key[cur][t]) - zmax);
  part = wave_sum(part);
  if (lane == 0) S.sh.red_a[w] = (unsigned long long)__double_as_longlong(part);
  __syncthreads();
  double sum = 0.0;
  for (int u = 0; u < kSelWaves; ++u) sum += __longlong_as_double((long long)S.sh.red_a[u]);
  for (int t = tid; t < k; t += kSelThreads) {
    const double z = key_value((uint64_t)b_key[cur][t]);
    if (p.idx_out) p.idx_out[(size_t)b * k + t] = map[b_pos[cur][t]];
    if (p.val_out) p.val_out[(size_t)b * k + t] = (float)z;
    if (p.prob_out) p.prob_out[(size_t)b * k + t] = (float)(exp(z - zmax) / sum);
  }
  HIRE_TS(56);
}

hipError_t launch_softmax_refine(const SelectParams& p, int B, hipStream_t s) {
  const int cap = p.n_dev ? p.n_cap : p.n;
  if (cap < 1 || cap > kSoftmaxRefineMaxRow || p.k < 1 || p.k > kSoftmaxRefineMaxK || !p.refine_w || !p.refine_x ||
      p.refine_d % 8 != 0 || !p.map || !p.xnorm || !p.wnorm_tiles || !p.maxima || !p.refine_slots || p.n_maxima > kFilterMaxima ||
      p.wnorm_n > kSpThreads || p.n_maxima < 1 || p.wnorm_n < 1 || !p.vals || !p.refine_keys || p.refine_keys_stride < cap)
    return hipErrorInvalidValue;
  const hipError_t e = launch(k_softmax_parts, dim3(softmax_parts(B), B), dim3(kSpThreads), 0, s, p);
  if (e != hipSuccess) return e;
  return launch(k_softmax_refine, dim3(B), dim3(kSelThreads), 0, s, p);
}

// ---------------------------------------------------------------------------
template <typename V>
static bool select_is_lean(const SelectParams& p) {
  const int cap = p.n_dev ? p.n_cap : p.n;
  return p.nonneg && !p.rank_order && p.gs == 0 && !p.relu && cap > kSelThreads && cap <= kCachedMax &&
         p.k <= kWin / 2 && reinterpret_cast<uintptr_t>(p.vals) % 16 == 0 && (p.stride * (long long)sizeof(V)) % 16 == 0;
}
template <typename V>
static hipError_t launch_select(const SelectParams& p, int B, hipStream_t s) {
  size_t lds = 0;
  if (p.rank_order) lds = (size_t)p.k * (sizeof(typename KeyOf<V>::K) + 2 * sizeof(int));
  const int cap = p.n_dev ? p.n_cap : p.n;
  if (select_is_lean<V>(p)) return launch(k_select_nonneg<V>, dim3(B), dim3(kSelThreads), 0, s, p);
  if (cap <= kSelThreads) return launch(k_select<V, 1>, dim3(B), dim3(kSelThreads), lds, s, p);
  if (cap <= 4 * kSelThreads) return launch(k_select<V, 4>, dim3(B), dim3(kSelThreads), lds, s, p);
  if (cap <= kCachedMax) return launch(k_select<V, kItemsMax>, dim3(B), dim3(kSelThreads), lds, s, p);
  return launch(k_select<V, 0>, dim3(B), dim3(kSelThreads), lds, s, p);
}

hipError_t launch_select_f32(const SelectParams& p, int B, hipStream_t s) { return launch_select<float>(p, B, s); }
hipError_t launch_select_f64(const SelectParams& p, int B, hipStream_t s) { return launch_select<double>(p, B, s); }

size_t multi_body_bytes_host(int B) { return multi_body_bytes(B); }
size_t general_fallbacks_offset(int which) {
  switch (which) {
    case 0: return offsetof(GeneralHeader, multi) + offsetof(MultiHeader, fallbacks);
    case 1: return offsetof(GeneralHeader, window_misses);
    default: return offsetof(GeneralHeader, multi) + offsetof(MultiHeader, stamps);
  }
}

bool multi_producer_counts(int N, int B) { return (long long)N * B <= kDirectCountMaxKeys; }
int multi_hist_shift(int N, int B) { return multi_producer_counts(N, B) ? kHistShift : kCoarseShift; }

// Shared by the step (one union bitmap, keys already passed through phi) and topk_select on long rows (a bitmap per
// row, ReLU applied on the fly, always counted by the pass of its own).
static hipError_t mark_rows(const float* keys, int B, int N, int k, int slots, bool own_count, int relu,
                            const MultiRegion& mr, uint32_t* bitmap, long long bitmap_stride, hipStream_t s) {
  const int shift = own_count ? kCoarseShift : kHistShift;
  if (own_count) {
    const int chunks = (N + kSelThreads * kCountKeys - 1) / (kSelThreads * kCountKeys);
    const hipError_t e = launch(k_count_f32, dim3(chunks, B), dim3(kSelThreads), 0, s, keys, B, N, slots, shift, relu, mr);
    if (e != hipSuccess) return e;
  }
  const int chunks = (N + kSelThreads * kMarkKeys - 1) / (kSelThreads * kMarkKeys);
  return launch(k_mark_f32, dim3(chunks, B), dim3(kSelThreads), 0, s, keys, B, N, k, slots, shift, relu, mr, bitmap,
                bitmap_stride);
}

static hipError_t resolve_rows(const float* keys, int B, int N, int k, bool own_count, int relu, const MultiRegion& mr,
                               uint32_t* bitmap, long long bitmap_stride, hipStream_t s) {
  // per-key cleaning spreads over up to 64 workgroups; the window of the counting pass needs few
  const int cleaners = own_count ? 2 : min(64, (N + kCleanKeys - 1) / kCleanKeys);
  return launch(k_resolve_compact, dim3(1 + cleaners, B), dim3(kSelThreads), 0, s, keys, B, N, k,
                own_count ? kCoarseShift : kHistShift, relu, mr, bitmap, bitmap_stride);
}

hipError_t launch_mark_f32(const float* keys, int B, int N, int kprime, int slots, const HistRefs& hr, uint32_t* bitmap,
                           hipStream_t s) {
  return mark_rows(keys, B, N, kprime, slots, !multi_producer_counts(N, B), 0, multi_of(hr, B), bitmap, 0, s);
}

hipError_t launch_resolve_compact(const float* keys, int B, int N, int kprime, const HistRefs& hr, uint32_t* bitmap,
                                  int words, int32_t* list_out, int32_t* count_out, int32_t* count_out2,
                                  uint32_t* zero_ptr, int zero_words, hipStream_t s) {
  const MultiRegion mr = multi_of(hr, B);
  const hipError_t e = resolve_rows(keys, B, N, kprime, !multi_producer_counts(N, B), 0, mr, bitmap, 0, s);
  if (e != hipSuccess || list_out == nullptr) return e;  // no list wanted: the gather compacts the bitmap itself
  return launch(k_union_compact, dim3(1), dim3(kSelThreads), 0, s, B, mr, bitmap, words, list_out, count_out,
                count_out2, zero_ptr, zero_words);
}

bool topk_rows_supported(int N, int k) { return N > 8 * kTkGroups && k <= kTkMaxK; }

hipError_t launch_topk_rows(const float* scores, int B, int N, int k, int relu, int rank_order, int32_t* idx_out,
                            float* val_out, void* general_header, void* body, unsigned long long sig, hipStream_t s) {
  GeneralHeader* gh = static_cast<GeneralHeader*>(general_header);
  const MultiRegion mr = carve_multi(&gh->multi, body, B);
  const TkCounts counts{reinterpret_cast<uint32_t*>(static_cast<char*>(body) + multi_body_bytes(B)), (N + 31) / 32 + 2};
  auto maxima = [&](auto kernel, int parts) {
    return launch(kernel, dim3(kTkGroups / kTkMaxGroups, B), dim3(kTkMaxGroups * parts), 0, s, scores, N, relu, mr, counts, gh, sig);
  };
  // as many threads per group as have sixteen entries each: one round of loads.  16 rows of 256000: 18.0, 17.0, 16.9 us for the
  // three kernels with one, two, four; of 131072: 15.1, 14.8, 15.3; of 40000: 13.6, 13.6, 14.2
  hipError_t e = N > 32 * kTkGroups ? maxima(k_tk_maxima<4>, 4)
                                    : (N > 16 * kTkGroups ? maxima(k_tk_maxima<2>, 2) : maxima(k_tk_maxima<1>, 1));
  if (e != hipSuccess) return e;
  const int chunks = (N + kSelThreads * kTkKeys - 1) / (kSelThreads * kTkKeys);
  e = launch(k_tk_gather, dim3(chunks, B), dim3(kSelThreads), 0, s, scores, N, k, relu, mr, counts);
  if (e != hipSuccess) return e;
  return launch(k_tk_final, dim3(B), dim3(kSelThreads), 0, s, scores, B, N, k, relu, rank_order, mr, counts, idx_out, val_out);
}

size_t topk_long_workspace_bytes(int B, int N) {
  const size_t words = (size_t)(N + 31) / 32 + 2;
  return multi_body_bytes(B) + (B * words * 4 + 255) / 256 * 256 + ((size_t)B * 4 + 255) / 256 * 256;
}

hipError_t launch_topk_long(const float* scores, int B, int N, int k, int relu, int32_t* idx_out, float* val_out,
                            void* general_header, void* body, unsigned long long sig, hipStream_t s) {
  const int words = (N + 31) / 32 + 2;
  const MultiRegion mr = carve_multi(&static_cast<GeneralHeader*>(general_header)->multi, body, B);
  char* after = static_cast<char*>(body) + multi_body_bytes(B);
  uint32_t* bitmaps = reinterpret_cast<uint32_t*>(after);
  int32_t* counts = reinterpret_cast<int32_t*>(after + ((size_t)B * words * 4 + 255) / 256 * 256);
  const int chunks = (N + kSelThreads * kCountKeys - 1) / (kSelThreads * kCountKeys);
  if (chunks > kWgMaxSlots) return hipErrorInvalidValue;
  hipError_t e = launch(k_row_maxima, dim3(chunks, B), dim3(kSelThreads), 0, s, scores, N, relu, mr, bitmaps,
                        (long long)B * words, static_cast<GeneralHeader*>(general_header), sig);
  if (e != hipSuccess) return e;
  if ((e = mark_rows(scores, B, N, k, chunks, true, relu, mr, bitmaps, words, s)) != hipSuccess) return e;
  if ((e = resolve_rows(scores, B, N, k, true, relu, mr, bitmaps, words, s)) != hipSuccess) return e;
  return launch(k_emit_rows, dim3(B), dim3(kSelThreads), 0, s, scores, B, N, k, relu, mr, bitmaps, words, idx_out, val_out,
                counts);
}

hipError_t launch_bitmap_compact(const uint32_t* bitmap, int words, int32_t* list_out, int32_t* count_out,
                                 int32_t* count_out2, uint32_t* zero_ptr, int zero_words, hipStream_t s) {
  return launch(k_bitmap_compact, dim3(1), dim3(kSelThreads), 0, s, bitmap, words, list_out, count_out,
                     count_out2, zero_ptr, zero_words);
}

}  // namespace hire

#ifdef HIRE_TIMESTAMPS
extern "C" int hire_debug_timestamps_select(unsigned long long* host64) {
  return (int)hipMemcpyFromSymbol(host64, HIP_SYMBOL(hire_ts), sizeof(hire_ts));
}
#endif
