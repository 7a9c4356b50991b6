// HiRE-FFN with Algorithm 2's sharded selection (arXiv 2402.09360) for batches and for long shards: the scorer, the filter
// stage and the second layer of the unsharded step, and between them the selections of every (token, shard) by a wave of
// its own.
//
//   k_scorer_int4_mfma  keys of all tokens
//   k_shard_keys        the k'/s largest keys of every token in every shard -> bits of the union
//   k_filter_units      the union's activations on the bf16 matrix cores, within a proven distance
//   k_shard_refine      the k/s largest activations of every token in every shard, by their fp64 values
//   k_exact_values      the selected activations, rounded once from fp64
//   k_w2_list           y
//
// k_ffn_shard (ffn_shard.hip) keeps a shard in one workgroup for the whole step and takes the tokens four at a time: nothing
// is handed over, but a step of many tokens is as long as they are many, and few shards leave most of the chip idle; more than
// 64 units are ranked by comparing each with all.  ffn_shard_batch says where this sequence is the faster one.  Bound by
// the launches' own latencies up to 16 tokens (six of them, 4 to 6 us each), then by the passes over the weights.  us per
// step, that kernel / this sequence, 16 and 64 tokens of d = 2048: 256 shards of 64 units 109 / 54, 400 / 103; 16 shards of
// 128 186 / 33, 728 / 45.
#include "kernels.h"
#include "select.h"

namespace hire {

constexpr int kSbWaves = 4;  // waves, each with its own (token, shard), of a workgroup

// The `want` largest of a wave's keys (E per lane, entry e * 64 + lane; keys of entries that do not count are 0 and `counts`
// says which do, at least `want` of them), ties to the lower index: masks by e.  Bit by bit from the top: the candidate
// threshold that exactly `want` keys reach ends the search, after a dozen bits for ordinary rows.
template <typename K, int E>
__device__ __forceinline__ void wave_top(const K (&key)[E], const uint64_t (&counts)[E], int want, uint64_t (&take)[E]) {
  constexpr int kBits = 8 * (int)sizeof(K);
  K t = 0;
  bool exact = false;
  for (int bit = kBits - 2; bit >= 0 && !exact; --bit) {  // (the sign bit is clear)
    const K c = t | (K)1 << bit;
    int n = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) n += __popcll(__ballot(key[e] >= c) & counts[e]);
    if (n >= want) t = c;
    exact = n == want;
  }
  int above = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    take[e] = __ballot(exact ? key[e] >= t : key[e] > t) & counts[e];
    above += __popcll(take[e]);
  }
  if (exact) return;
  int need = want - above;  // of those equal to the threshold the first
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint64_t eq = __ballot(key[e] == t) & counts[e];
    take[e] |= __ballot(((eq >> lane_id()) & 1ull) != 0ull && mask_prefix(eq) < need);
    need -= min(need, (int)__popcll(eq));
  }
}

// Entries of a shard that exist, by e.
template <int E>
__device__ __forceinline__ void shard_mask(int Ls, uint64_t (&m)[E]) {
#pragma unroll
  for (int e = 0; e < E; ++e) m[e] = Ls - 64 * e >= 64 ? ~0ull : (Ls > 64 * e ? (1ull << (Ls - 64 * e)) - 1ull : 0ull);
}

struct ShardBatch {
  const float* vals;   // [B, stride]: keys, then the filter stage's values
  long long stride;
  int B, d, Ls, shards;
  int kps, ks;
  uint32_t* bitmap;    // union over the units
  // k_shard_refine
  const uint16_t* W;
  const uint16_t* x;
  const float* xnorm;
  const float* wnorm_tiles;
  int wnorm_n;
  float err_c;
  uint2* list;         // [B, shards ks]
  int32_t* idx_out;    // optional, the same places
  int32_t* cand;       // optional [shards, cap]
  int cap;
  int32_t* n_cand;     // optional [shards]
};

template <int E>
__global__ __launch_bounds__(kWave * kSbWaves) void k_shard_keys(ShardBatch p) {
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int sh = (int)blockIdx.x, b = (int)blockIdx.y * kSbWaves + w, u0 = sh * p.Ls;
  __shared__ uint64_t masks[kSbWaves][E];
  uint64_t real[E], take[E];
  shard_mask(p.Ls, real);
#pragma unroll
  for (int e = 0; e < E; ++e) take[e] = 0ull;
  if (b < p.B) {  // uniform over the wave
    uint32_t key[E];
#pragma unroll
    for (int e = 0; e < E; ++e) key[e] = __float_as_uint(p.vals[(size_t)b * p.stride + u0 + min(64 * e + lane, p.Ls - 1)]);
    wave_top(key, real, p.kps, take);
  }
  if (lane == 0) {
#pragma unroll
    for (int e = 0; e < E; ++e) masks[w][e] = take[e];
  }
  lds_barrier();
  // the tokens' masks together; entry e * 64 is bit u0 + e * 64 of the union: three words at most
  for (int i = (int)threadIdx.x; i < 3 * E; i += kWave * kSbWaves) {
    const int e = i / 3, j = i - 3 * e, at = u0 + 64 * e, off = at & 31;
    uint64_t m = 0ull;
#pragma unroll
    for (int v = 0; v < kSbWaves; ++v) m |= masks[v][e];
    const uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
    const uint32_t bits = j == 0 ? lo << off : (j == 1 ? (off != 0 ? lo >> (32 - off) : 0u) | hi << off : (off != 0 ? hi >> (32 - off) : 0u));
    if (bits != 0u) atomicOr(&p.bitmap[(at >> 5) + j], bits);
  }
}

// The stored values are within hw / 2 of the activations (hw = 2 err_c max|u| |x|; zeros are exact).  With v the ks-th largest
// stored value of the shard's candidates, the ks-th largest activation lies in [v - hw / 2, v + hw / 2]: what is stored
// above v + hw is selected, what is stored below v - hw is not, and what lies between - the ks-th itself and seldom another -
// is recomputed in fp64 (zeros excepted) and decides by (value descending, unit ascending).
template <int E>
__global__ __launch_bounds__(kWave * kSbWaves) void k_shard_refine(ShardBatch p) {
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int sh = (int)blockIdx.x, b = (int)blockIdx.y * kSbWaves + w, u0 = sh * p.Ls;
  if (b >= p.B) return;  // uniform over the wave
  float v[E];
  uint32_t word[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = u0 + min(64 * e + lane, p.Ls - 1);
    v[e] = p.vals[(size_t)b * p.stride + i];
    word[e] = p.bitmap[i >> 5];
  }
  const float xn = p.xnorm[b];
  const uint4* tok = reinterpret_cast<const uint4*>(p.x + (size_t)b * p.d);
  float wn = 0.0f;
  for (int i = lane; i < p.wnorm_n; i += kWave) wn = fmaxf(wn, p.wnorm_tiles[i]);
  wn = wave_max(wn);
  uint64_t cand[E], take[E];
  shard_mask(p.Ls, cand);
#pragma unroll
  for (int e = 0; e < E; ++e) cand[e] &= __ballot((word[e] >> ((u0 + 64 * e + lane) & 31) & 1u) != 0u);
  if (b == 0) {  // the shard's candidates, for the caller
    int n = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int at = n + mask_prefix(cand[e]);
      if (p.cand != nullptr && ((cand[e] >> lane) & 1ull) != 0ull && at < p.cap) p.cand[(size_t)sh * p.cap + at] = u0 + 64 * e + lane;
      n += __popcll(cand[e]);
    }
    if (p.n_cand != nullptr && lane == 0) p.n_cand[sh] = n;
  }
  uint32_t key[E];
#pragma unroll
  for (int e = 0; e < E; ++e) key[e] = ((cand[e] >> lane) & 1ull) != 0ull ? __float_as_uint(v[e]) : 0u;
  wave_top(key, cand, p.ks, take);
  uint32_t least = ~0u;  // the ks-th largest stored value: the smallest taken
#pragma unroll
  for (int e = 0; e < E; ++e) least = ((take[e] >> lane) & 1ull) != 0ull ? min(least, key[e]) : least;
  const double hw = 2.0 * (double)p.err_c * (double)xn * (double)wn * 1.000001, vk = (double)__uint_as_float(wave_min(least));
  uint64_t sure[E], band[E];
  int n_sure = 0, n_band = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const double s = (double)v[e];
    sure[e] = __ballot(s > vk + hw) & cand[e];
    band[e] = __ballot(!(s < vk - hw) && !(s > vk + hw)) & cand[e];  // without a finite bound everything
    n_sure += __popcll(sure[e]);
    n_band += __popcll(band[e]);
  }
  const int need = p.ks - n_sure;
  if (need != n_band) {  // (otherwise the whole band is selected)
    uint64_t act[E];     // the band's activations: non-negative doubles order like their bits
#pragma unroll
    for (int e = 0; e < E; ++e) {
      act[e] = 0ull;
      uint64_t open = band[e] & __ballot(v[e] > 0.0f);
      while (open != 0ull) {
        const int l = __builtin_ctzll(open);
        open &= open - 1ull;
        const double r = wave_row_dot<true>(p.W + (size_t)(u0 + 64 * e + l) * p.d, tok, p.d);
        if (lane == l) act[e] = (uint64_t)__double_as_longlong(r);
      }
    }
    wave_top(act, band, need, take);
#pragma unroll
    for (int e = 0; e < E; ++e) band[e] = take[e];
  }
  int at = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint64_t m = sure[e] | band[e];
    const int place = at + mask_prefix(m);
    if (((m >> lane) & 1ull) != 0ull && place < p.ks) {
      const size_t o = ((size_t)b * p.shards + sh) * p.ks + place;
      p.list[o] = make_uint2((uint32_t)(u0 + 64 * e + lane), 0u);
      if (p.idx_out) p.idx_out[o] = u0 + 64 * e + lane;
    }
    at += __popcll(m);
  }
}

// ---------------------------------------------------------------------------------------------------
// us per step, k_ffn_shard / this sequence.  Shards of up to 64 units, four tokens: d = 512, 16 x 32 units 12.8 / 21.7,
// d = 2048, 256 x 64 29.1 / 39.2; six tokens: d = 512, 16 x 32 19.9 / 22.2, 16 x 64 23.8 / 22.4; d = 1024, 64 x 32 24.6 /
// 26.0; d = 2048, 16 x 32 29.9 / 27.0, 256 x 64 50.8 / 42.6.  Longer ones: d = 512, 16 x 128, two tokens 20.6 / 23.9, three
// 26.4 / 24.2; 16 x 256, one 24.0 / 24.1, two 38.5 / 25.3; 16 x 512, one 49.2 / 37.4; of 32768 units, whose filter stage
// needs two rounds of workgroups, 256 x 128, four 34.6 / 45.4, six 58.8 / 47.6; 64 x 512, one 49.9 / 57.9, two 84.1 / 60.3.
// d = 4096, 16 x 100, two 32.8 / 39.4, three 45.5 / 40.4.
bool ffn_shard_batch(int B, int N, int d, int shards) {
  const int Ls = N / shards;
  if (Ls <= kWave) return B > 4 && (long long)B * d * Ls >= 3 << 16;
  return B > 4 || B * Ls >= (N > 16384 ? 640 : (d > 2048 ? 256 : 384));
}

template <int E>
static hipError_t shard_selections(const FfnShardArgs& a, const ShardBatch& p, const FfnShardBuffers& f, hipStream_t s) {
  const dim3 grid(p.shards, (p.B + kSbWaves - 1) / kSbWaves);
  hipError_t e = launch(k_shard_keys<E>, grid, dim3(kWave * kSbWaves), 0, s, p);
  if (e != hipSuccess) return e;
  e = launch_filter_units(a.w1u, a.x, a.B, a.d, f.bitmap, nullptr, a.N, f.vals, f.stride, f.xnorm, f.wnorm_tiles, nullptr, s);
  if (e != hipSuccess) return e;
  return launch(k_shard_refine<E>, grid, dim3(kWave * kSbWaves), 0, s, p);
}

hipError_t launch_ffn_shard_batch(const FfnShardArgs& a, const FfnShardBuffers& f, hipStream_t s) {
  ScorerTokens tok{f.xq, nullptr, false, nullptr, f.bitmap, f.zero_words, nullptr, 0ull};
  hipError_t e = hipSuccess;
  if (scorer_mfma_quantises(a.B, a.N, a.d, false)) tok.x = a.x;
  else e = launch_quantize_tokens(a.x, false, a.B, a.d, f.xq, nullptr, f.bitmap, f.zero_words, nullptr, 0ull, s);
  if (e != hipSuccess) return e;
  e = launch_scorer_int4_mfma(static_cast<const uint32_t*>(a.q4), a.q4_scale, tok, a.B, a.N, a.d, 1, f.vals, f.stride,
                              a.scorer_acc, HistRefs{nullptr, nullptr}, s);
  if (e != hipSuccess) return e;
  ShardBatch p{};
  p.vals = f.vals; p.stride = f.stride;
  p.B = a.B; p.d = a.d; p.shards = a.shards; p.Ls = a.N / a.shards;
  p.kps = (a.kprime + a.shards - 1) / a.shards; p.ks = (a.k + a.shards - 1) / a.shards;
  p.bitmap = f.bitmap;
  p.W = a.w1u; p.x = a.x;
  p.xnorm = f.xnorm; p.wnorm_tiles = f.wnorm_tiles; p.wnorm_n = filter_tiles(a.N); p.err_c = gather_filter_error(a.B);
  p.list = f.list; p.idx_out = a.topk_idx;
  p.cand = a.cand; p.n_cand = a.n_cand;
  p.cap = (int)((long long)a.B * p.kps < (long long)p.Ls ? a.B * p.kps : p.Ls);
  if (p.Ls <= 64) e = shard_selections<1>(a, p, f, s);
  else if (p.Ls <= 128) e = shard_selections<2>(a, p, f, s);
  else if (p.Ls <= 256) e = shard_selections<4>(a, p, f, s);
  else e = shard_selections<16>(a, p, f, s);
  if (e != hipSuccess) return e;
  const int k = p.shards * p.ks;
  e = launch_exact_values(f.list, a.topk_val, a.w1u, a.x, a.B, k, a.d, s);
  if (e != hipSuccess) return e;
  return launch_w2_list(a.w2u, a.d, a.B, k, f.list, nullptr, 0, nullptr, a.y, s);
}

}  // namespace hire
