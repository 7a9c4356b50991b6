// Workgroup-cooperative exact selection: the k-th largest key of a set that a
// workgroup of NT threads holds in registers or streams from memory.
//
// Method (range narrowing): keep a closed key interval [lo, hi] known to
// contain the k-th largest key together with `need` = its rank inside the
// interval.  Each round bins the interval into 2048 bins in LDS, walks the
// bins from the top to the one holding the rank, and tightens [lo, hi] to the
// keys of that bin.  The first round bins linearly in *value* space (a bell
// shaped distribution then spreads over all bins and LDS atomics rarely
// collide); later rounds bin the integer key space, which removes at least 11
// bits of range per round and therefore terminates.  Once at most 64 keys are
// left they are ranked directly.  Bin 0 is never counted with atomics (ReLU
// zeros would all collide there); its population follows from the total.
#pragma once

#include "device_utils.h"

// Phase stamps for a profiling build (-DHIRE_TIMESTAMPS): thread 0 of workgroup (0, 0) stores the 100 MHz wall
// clock at numbered points of the selecting kernels; each translation unit keeps its own table and exports a
// reader.  Compiled out of the product build.
#ifdef HIRE_TIMESTAMPS
static __device__ unsigned long long hire_ts[128];  // [i]: 100 MHz wall clock; [64 + i]: shader clock cycles
#define HIRE_TS(i)                                                 \
  do {                                                             \
    if (threadIdx.x == 0 && blockIdx.x == 0 && blockIdx.y == 0) {  \
      hire_ts[i] = wall_clock64();                                 \
      hire_ts[64 + (i)] = clock64();                               \
    }                                                              \
  } while (0)
#else
#define HIRE_TS(i) ((void)0)
#endif

namespace hire {

constexpr int kSelThreads = 1024;  // workgroup size of the general selection kernels
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kSelBins = 2048;
constexpr int kSelSmall = 64;

template <int NT>
struct SelSharedT {
  static constexpr int NW = NT / kWave;
  uint32_t hist[kSelBins];
  unsigned long long red_a[NW];
  unsigned long long red_b[NW];
  int wave_tot[NW];
  int bc_bin, bc_above, bc_cnt;
  unsigned long long bc_key;
  int list_n;
  unsigned long long list_key[kSelSmall];
};
using SelShared = SelSharedT<kSelThreads>;

// min and max over the workgroup; every thread gets both.
template <typename K, int NT>
__device__ __forceinline__ void wg_minmax(K& vmin, K& vmax, SelSharedT<NT>& sh) {
  constexpr int NW = NT / kWave;
  K a = wave_min(vmin), b = wave_max(vmax);
  __syncthreads();  // previous readers of red_a/red_b are done
  if (lane_id() == 0) {
    sh.red_a[wave_id()] = (unsigned long long)a;
    sh.red_b[wave_id()] = (unsigned long long)b;
  }
  __syncthreads();
  a = (K)sh.red_a[0];
  b = (K)sh.red_b[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    K x = (K)sh.red_a[w], y = (K)sh.red_b[w];
    a = x < a ? x : a;
    b = y > b ? y : b;
  }
  vmin = a;
  vmax = b;
}

// Inclusive prefix sum over the NT threads in thread order; *total (optional) receives the sum of all.
// Wave totals go through LDS once; every wave then scans them itself in registers.
// FRESH: no thread can still be reading wave_tot from an earlier use, so the leading barrier is left out.
template <int NT, bool FRESH = false>
__device__ __forceinline__ int wg_scan_incl(int v, SelSharedT<NT>& sh, int* total = nullptr) {
  constexpr int NW = NT / kWave;
  const int incl = wave_scan_incl(v);
  if (!FRESH) __syncthreads();  // previous readers of wave_tot are done
  if (lane_id() == kWave - 1) sh.wave_tot[wave_id()] = incl;
  __syncthreads();
  const int t = lane_id() < NW ? sh.wave_tot[lane_id()] : 0;
  const int p = wave_scan_incl(t);
  const int w = __builtin_amdgcn_readfirstlane(wave_id());
  const int base = w > 0 ? __builtin_amdgcn_readlane(p, w - 1) : 0;
  if (total) *total = __builtin_amdgcn_readlane(p, NW - 1);
  return incl + base;
}

// Largest of one value per thread, to all threads.
template <int NT>
__device__ __forceinline__ uint32_t wg_max_u32(uint32_t m, SelSharedT<NT>& sh) {
  constexpr int NW = NT / kWave;
  m = wave_max(m);
  __syncthreads();
  if (lane_id() == 0) sh.wave_tot[wave_id()] = (int)m;
  __syncthreads();
  return wave_max(lane_id() < NW ? (uint32_t)sh.wave_tot[lane_id()] : 0u);
}

template <typename K>
struct KeyTraits;
template <>
struct KeyTraits<uint32_t> {
  using V = float;
};
template <>
struct KeyTraits<uint64_t> {
  using V = double;
};

// for_each(f): calls f(key) for every key this thread owns.  n keys in total
// over the workgroup, 1 <= k <= n.  Returns the k-th largest key to all threads.
// Keys are order keys (device_utils.h), so key_value() recovers the number.
template <typename K, int NT, typename ForEach>
__device__ K wg_kth_largest(ForEach&& for_each, int n, int k, SelSharedT<NT>& sh) {
  using V = typename KeyTraits<K>::V;
  constexpr int kBinsPerThread = kSelBins / NT;
  static_assert(kBinsPerThread >= 2 && kSelBins % NT == 0, "each thread walks a whole number of bins");
  K lo = ~(K)0, hi = 0;
  for_each([&](K key) {
    lo = key < lo ? key : lo;
    hi = key > hi ? key : hi;
  });
  HIRE_TS(1);
  wg_minmax(lo, hi, sh);
  HIRE_TS(2);
  int need = k, nact = n;
  bool value_round = true;
  const int tid = (int)threadIdx.x;
  while (true) {
    if (lo == hi) return lo;
    if (nact <= kSelSmall) break;
    // ---- histogram of the active interval ----
    for (int b = tid; b < kSelBins; b += NT) sh.hist[b] = 0;
    __syncthreads();
    const V vlo = key_value(lo);
    const V vscale = (V)(kSelBins - 1) / (key_value(hi) - vlo);
    const int shift = max(0, ilog2_u64((uint64_t)(hi - lo)) + 1 - 11);
    auto bin_of = [&](K key) -> int {
      if (value_round) {
        int b = (int)((key_value(key) - vlo) * vscale);
        return min(max(b, 0), kSelBins - 1);
      }
      return (int)((key - lo) >> shift);
    };
    for_each([&](K key) {
      if (key >= lo && key <= hi) {
        int b = bin_of(key);
        if (b) atomicAdd(&sh.hist[b], 1u);
      }
    });
    __syncthreads();
    HIRE_TS(3);
    // ---- walk the bins from the top: thread t owns the kBinsPerThread bins ending at bin 2047 - t*kBinsPerThread ----
    const int b_top = kSelBins - 1 - kBinsPerThread * tid;
    int c[kBinsPerThread], s = 0;
#pragma unroll
    for (int q = 0; q < kBinsPerThread; ++q) {
      c[q] = (int)sh.hist[b_top - q];
      s += c[q];
    }
    int total;
    const int incl = wg_scan_incl(s, sh, &total);
    int run = incl - s;
    if (run < need && need <= incl) {
#pragma unroll
      for (int q = 0; q < kBinsPerThread; ++q) {
        if (run < need && need <= run + c[q]) {
          sh.bc_bin = b_top - q;
          sh.bc_above = run;
          sh.bc_cnt = c[q];
        }
        run += c[q];
      }
    }
    if (tid == 0 && total < need) {  // the rank falls into the uncounted bin 0
      sh.bc_bin = 0;
      sh.bc_above = total;
      sh.bc_cnt = nact - total;
    }
    __syncthreads();
    const int beta = sh.bc_bin;
    need -= sh.bc_above;
    nact = sh.bc_cnt;
    HIRE_TS(4);
    // ---- tighten [lo, hi] to the keys of bin beta ----
    K nlo = ~(K)0, nhi = 0;
    for_each([&](K key) {
      if (key >= lo && key <= hi && bin_of(key) == beta) {
        nlo = key < nlo ? key : nlo;
        nhi = key > nhi ? key : nhi;
      }
    });
    wg_minmax(nlo, nhi, sh);
    lo = nlo;
    hi = nhi;
    value_round = false;
    HIRE_TS(5);
  }
  // ---- at most 64 keys left in [lo, hi]: rank them directly ----
  __syncthreads();
  if (tid == 0) sh.list_n = 0;
  __syncthreads();
  for_each([&](K key) {
    if (key >= lo && key <= hi) {
      int p = atomicAdd(&sh.list_n, 1);
      if (p < kSelSmall) sh.list_key[p] = (unsigned long long)key;
    }
  });
  __syncthreads();
  const int m = min(sh.list_n, kSelSmall);
  if (tid < m) {
    const K mine = (K)sh.list_key[tid];
    int cg = 0, cge = 0;
    for (int u = 0; u < m; ++u) {
      const K other = (K)sh.list_key[u];
      cg += other > mine;
      cge += other >= mine;
    }
    if (cg < need && need <= cge) sh.bc_key = (unsigned long long)mine;  // equal keys write the same value
  }
  __syncthreads();
  HIRE_TS(6);
  return (K)sh.bc_key;
}

// Consumer-side compaction of a bitmap: the workgroup finds the indices of the set bits with ranks
// [r0, r0 + R) in ascending order and learns the total number of set bits, without a pass of its own kernel.
// Wave w owns a contiguous block of words and reads it 64 words at a time (one coalesced load per step, kept
// in registers); the waves' totals give every wave the rank of its first bit, and only a wave whose ranks meet
// the wanted ones walks its steps again, from registers, with a wave prefix sum per step.  out_sh[r - r0]
// receives the index of rank r; entries at and past the total are left alone.  words <= NT / 64 * 64 * STEPS;
// callers with short bitmaps take the variant with few steps, whose unrolled loops are correspondingly short.
constexpr int kLocateSteps = 32;       // 64-word steps per wave
constexpr int kLocateStepsShort = 4;

// range(total, r0, R) names the wanted ranks once the total is known.
template <int NT, int STEPS, typename Range>
__device__ __forceinline__ int union_locate_range(const uint32_t* __restrict__ bitmap, int words, SelSharedT<NT>& sh,
                                                  Range&& range, int32_t* out_sh) {
  constexpr int NW = NT / kWave;
  const int lane = lane_id(), w = wave_id();
  const int per_wave = ((words + NW - 1) / NW + kWave - 1) / kWave * kWave;
  const int w0 = w * per_wave, w1 = min(words, w0 + per_wave);
  const int steps = max(0, (w1 - w0 + kWave - 1) / kWave);  // <= STEPS
  uint32_t keep[STEPS];
  int cnt = 0;
#pragma unroll
  for (int st = 0; st < STEPS; ++st) {
    keep[st] = 0u;
    // uniform over the wave, clamped, and nothing done to the value yet: the loads of the block go out together
    if (st < steps) keep[st] = bitmap[min(w0 + st * kWave + lane, words - 1)];
  }
#pragma unroll
  for (int st = 0; st < STEPS; ++st) {
    keep[st] = w0 + st * kWave + lane < w1 ? keep[st] : 0u;
    cnt += __popc(keep[st]);
  }
  const int mine = wave_sum(cnt);
  __syncthreads();  // previous readers of wave_tot are done
  if (lane == 0) sh.wave_tot[w] = mine;
  __syncthreads();
  int base = 0, total = 0;
#pragma unroll
  for (int u = 0; u < NW; ++u) {
    const int t = sh.wave_tot[u];
    base += u < w ? t : 0;
    total += t;
  }
  int r0, R;
  range(total, r0, R);
  if (base < r0 + R && base + mine > r0) {  // this wave's bits meet the wanted ranks (uniform over the wave)
    int run = base;
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      if (st < steps && run < r0 + R) {
        uint32_t m = keep[st];
        const int c = __popc(m);
        const int incl = wave_scan_incl(c);
        const int tot = __builtin_amdgcn_readlane(incl, kWave - 1);
        if (run + tot > r0) {
          int rank = run + incl - c;  // rank of this lane's first bit
          const int q = w0 + st * kWave + lane;
          while (m) {
            const int bit = __ffs((int)m) - 1;
            if (rank >= r0 && rank < r0 + R) out_sh[rank - r0] = q * 32 + bit;
            ++rank;
            m &= m - 1;
          }
        }
        run += tot;
      }
    }
  }
  __syncthreads();
  return total;
}

template <int NT, int STEPS = kLocateSteps>
__device__ __forceinline__ int union_locate(const uint32_t* __restrict__ bitmap, int words, SelSharedT<NT>& sh,
                                            int first, int count, int32_t* out_sh) {
  return union_locate_range<NT, STEPS>(
      bitmap, words, sh,
      [&](int, int& r0, int& R) {
        r0 = first;
        R = count;
      },
      out_sh);
}

// The set bits of a bitmap as an ascending list of at most cap entries, by one workgroup (NT threads, words <= 16 NT).
template <int NT>
__device__ __forceinline__ int list_bitmap(const uint32_t* __restrict__ bitmap, int words, int32_t* __restrict__ out, int cap,
                                           SelSharedT<NT>& sh) {
  const int tid = (int)threadIdx.x;
  int base = 0;
  for (int w0 = 0; w0 < words; w0 += NT * 4) {
    uint32_t m[4];
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t v = bitmap[min(w0 + tid * 4 + j, words - 1)];
      m[j] = w0 + tid * 4 + j < words ? v : 0u;
      cnt += __popc(m[j]);
    }
    int total;
    int at = base + wg_scan_incl<NT>(cnt, sh, &total) - cnt;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      for (uint32_t mm = m[j]; mm != 0u && at < cap; mm &= mm - 1u) out[at++] = (w0 + tid * 4 + j) * 32 + __builtin_ctz(mm);
    base += total;
  }
  return base;
}

// A 64-bit key that ranks smaller ones first, ties by a number.
struct KeyAndNumber {
  unsigned long long key;
  uint32_t number;
};
__device__ __forceinline__ bool comes_first(unsigned long long a, unsigned long long b) { return a < b; }
__device__ __forceinline__ bool comes_first(const KeyAndNumber& a, const KeyAndNumber& b) {
  return a.key < b.key || (a.key == b.key && a.number < b.number);
}
__device__ __forceinline__ unsigned long long lane_xor(unsigned long long v, int m) { return __shfl_xor(v, m); }
__device__ __forceinline__ KeyAndNumber lane_xor(const KeyAndNumber& v, int m) {
  return KeyAndNumber{__shfl_xor(v.key, m), (uint32_t)__shfl_xor((int)v.number, m)};
}

// The n items of a list in LDS in ascending order, by one workgroup: Batcher's exchanges with the first step of every merge mirrored,
// so that the smaller item always belongs to the lower place.  A wave has 128 places in registers, two per lane, while the pairs lie
// within those; `last`: no item is larger.  The list must be visible; ends behind a barrier.  16 rows, us per call of topk_select for k
// equal values, with all items of a bin compared with one another / so: 1000 values, k = 256 31.0 / 11.1, 512 55.2 / 12.7; 16384, k =
// 1024 131.7 / 36.3 (of it 22 before the ranking).
template <typename T>
__device__ __forceinline__ void sort_list(T* list, int n, const T& last) {
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  auto cross = [&](T& v, int m) {  // lanes l and l ^ m, the smaller one to the lower lane
    const T other = lane_xor(v, m);
    if (comes_first(other, v) == (lane < (lane ^ m))) v = other;
  };
  for (int size = 2 * kWave;; size <<= 1) {  // uniform
    for (int s = size >> 1; s >= 2 * kWave; s >>= 1) {
      for (int p = (int)threadIdx.x; 2 * (p & -s) < n; p += kSelThreads) {
        const int at = p & (s - 1), lo = 2 * p - at, hi = 2 * s == size ? lo + 2 * (s - at) - 1 : lo + s;
        if (hi < n) {  // (places past n would hold what comes last)
          const T a = list[lo], b = list[hi];
          if (comes_first(b, a)) {
            list[lo] = b;
            list[hi] = a;
          }
        }
      }
      __syncthreads();
    }
    for (int i = 2 * kWave * w + lane; i - lane < n; i += 2 * kSelThreads) {  // uniform over the wave
      T a = i < n ? list[i] : last, b = i + kWave < n ? list[i + kWave] : last;
      if (size == 2 * kWave) {
        for (int z = 2; z <= kWave; z <<= 1) {
          cross(a, z - 1);
          cross(b, z - 1);
          for (int s = z >> 2; s > 0; s >>= 1) {
            cross(a, s);
            cross(b, s);
          }
        }
        b = lane_xor(b, kWave - 1);  // mirrored: place 127 - l beside place l
      }
      if (comes_first(b, a)) {
        const T t = a;
        a = b;
        b = t;
      }
      // (b may stay mirrored: what follows within its 64 places sorts them from any order that is bitonic)
      for (int s = kWave / 2; s > 0; s >>= 1) {
        cross(a, s);
        cross(b, s);
      }
      if (i < n) list[i] = a;
      if (i + kWave < n) list[i + kWave] = b;
    }
    __syncthreads();
    if (size >= n) break;
  }
}

// Ranks of n <= PER * 1024 items, of which thread t holds the t-th, the (1024 + t)-th and so on, in a total order whose keys are
// key(item), larger ahead; ahead(a, b) says whether item a comes before item b (consulted between items of one bin only).  The keys
// between the smallest and the largest go to 4096 equal bins; the addition that counts a bin's items gives each its place in the
// bin, a scan gives every bin's first rank, the items are listed bin by bin and each counts those ahead of it inside its bin: a few
// instead of n comparisons per item.  emit(u, item, rank) is called once per item, a thread's u-th.  Where a bin has more than
// longest_run items (equal keys, or all near each other and one far off) nothing is emitted and the result is false: the caller sorts
// them, in memory of its own or, behind a barrier, in that of bins and list.  bins: kRankBins words of LDS, 16-byte aligned; list: n
// items of LDS.  All threads call this; what key() reads of LDS must be visible, and sh.red_a and sh.red_b free.
// Bound: the chain of barriers and LDS round trips on one compute unit.  16 rows of 256000, in us per call of topk_select: k = 1024
// 17.4 (2048 bins, the items' numbers listed, by a second pass of additions) -> 15.6 (this, 2048 bins) -> 15.1 (4096 bins: the keys
// are densest at the threshold); k = 2048 27.1 -> 21.2 -> 18.8.
constexpr int kRankBins = 4096;
// The longest run of items that is compared: it takes 0.1 us per item of the run, sorting 3 us for 256 items and 10 for 2000 (16
// rows of 256000 values rounded to bf16, k = 1024, runs of about 60: 22.9 us per call compared, 26.0 sorted).
__device__ __forceinline__ int rank_run(int n) { return 48 + n / 32; }
template <typename K, typename T, int PER, typename Key, typename Ahead, typename Emit>
__device__ __forceinline__ bool bucket_ranks(int n, const T (&own)[PER], Key&& key, Ahead&& ahead, uint32_t* bins, T* list,
                                             int longest_run, SelShared& sh, Emit&& emit) {
  static_assert(kRankBins == 4 * kSelThreads && PER * kSelThreads < 65536, "four bins per thread; first rank and length in one word");
  const int tid = (int)threadIdx.x;
  uint4* quad = reinterpret_cast<uint4*>(bins) + tid;
  *quad = make_uint4(0, 0, 0, 0);
  K lo = ~(K)0, hi = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (u * kSelThreads + tid < n) {
      const K k = key(own[u]);
      lo = k < lo ? k : lo;
      hi = k > hi ? k : hi;
    }
  lo = wave_min(lo);
  hi = wave_max(hi);
  if (lane_id() == 0) {
    sh.red_a[wave_id()] = (unsigned long long)lo;
    sh.red_b[wave_id()] = (unsigned long long)hi;
  }
  __syncthreads();
  lo = wave_min((K)sh.red_a[lane_id() % kSelWaves]);
  hi = wave_max((K)sh.red_b[lane_id() % kSelWaves]);
  const int shift = hi > lo ? max(0, ilog2_u64((uint64_t)(hi - lo)) + 1 - 12) : 0;
  int bin[PER], at[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (u * kSelThreads + tid < n) {
      bin[u] = (int)((hi - key(own[u])) >> shift);
      at[u] = (int)atomicAdd(&bins[bin[u]], 1u);
    }
  __syncthreads();
  const uint4 c = *quad;
  const uint32_t sum = c.x + c.y + c.z + c.w;
  // (in the same scan, above the sums: the threads with a bin that has too many)
  constexpr int kTooMany = 1 << 20;
  const int mine = (int)sum + (max(max(c.x, c.y), max(c.z, c.w)) > (uint32_t)longest_run ? kTooMany : 0);
  int total;
  const uint32_t s0 = (uint32_t)(wg_scan_incl(mine, sh, &total) & (kTooMany - 1)) - sum, s1 = s0 + c.x, s2 = s1 + c.y, s3 = s2 + c.z;
  if (total >= kTooMany) return false;  // uniform
  *quad = make_uint4(s0 << 16 | c.x, s1 << 16 | c.y, s2 << 16 | c.z, s3 << 16 | c.w);
  __syncthreads();
  uint32_t run[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (u * kSelThreads + tid < n) {
      run[u] = bins[bin[u]];
      list[(run[u] >> 16) + at[u]] = own[u];
    }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (u * kSelThreads + tid < n) {
      const int first = (int)(run[u] >> 16), end = first + (int)(run[u] & 0xFFFFu);
      int rank = first;
      for (int i0 = first; i0 < end; i0 += 4) {  // four LDS reads in flight
        T other[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) other[j] = list[min(i0 + j, end - 1)];
#pragma unroll
        for (int j = 0; j < 4; ++j) rank += i0 + j < end && ahead(other[j], own[u]) ? 1 : 0;
      }
      emit(u, own[u], rank);
    }
  return true;
}

}  // namespace hire
