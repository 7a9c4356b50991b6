// HiRE-FFN step for two to four tokens, groups of eight up to eight (arXiv 2402.09360, Algorithm 1 + eq. (4)):
// the scorer and the gather of the batch-1 sequence (ffn_fast.hip) for several tokens at once; the second layer is that
// sequence's own kernel, a row of workgroups per token.
//
// The two selections of the longer sequence for batches keep one compute unit per token busy for 6 and 10 us.  Here nothing
// runs on a unit per token.  The scorer
// counts every token's keys into a window histogram in memory; every workgroup of the gather walks all tokens'
// histograms, knows which of its own 64 units are shortlisted, and forms their activations for all tokens in fp64 on
// the matrix cores, so that no band around the threshold has to be computed again.
#include "ffn_fast.h"

namespace hire {

constexpr int kTT = kRowsThreads;
constexpr int kTW = kTT / kWave;
constexpr int kTokRows = 64;  // rows of a workgroup of the scorer

// ---------------------------------------------------------------------------------------------------
// Kernel 1: scorer.  Every workgroup quantises the tokens itself (a kernel for that alone costs 3.3 us), kTW / TT waves
// per token, then scores 64 rows on the int8 matrix cores, four rows per wave: v_mfma_i32_4x4x4 takes row l % 4 and
// token l % 4 from lane l and adds up sixteen blocks of columns l / 4 separately, so that a load covers 256 bytes of
// four adjacent rows and a wave's loads one piece of memory.  At the ~1B shape and four tokens 5.9 us until the
// keys are stored, and 1.3 more than a kernel boundary takes until the 33000 counts have reached memory (4.5 with the
// counters of adjacent bins side by side, see spread_slot); 3.3 more with the quantisation in front.  The kernel 8.5 us (12.0
// with the counters side by side).
// TT: tokens rounded up to four or eight; VECS: 16-byte vectors of a token per thread.  LRQ: as in k_fast_score_int4.
struct FastScoreTokens {
  const uint4* q4;
  const float* scale;
  const void* x;       // [B, d] bf16 (LRQ: fp32)
  int B, N, d;
  float* keys;         // [B, stride]
  long long stride;
  int32_t* acc_out;    // optional [B, N]
  FastRegion* fr;
  float* gkeys;        // groups of eight: [B, gstride] their activations, which are ranked instead of the units' keys
  long long gstride;
  const uint4* xn;     // LRQ: the tokens, [B, xn_d]
  int xn_d;
  const float* umax;
};

template <bool LRQ, int TT, int VECS>
__global__ __launch_bounds__(kTT) void k_fast_score_tokens(FastScoreTokens p) {
  constexpr int kWPT = kTW / TT;  // waves per token
  extern __shared__ uint4 xs[];              // [TT][d / 16 + 1] int8 codes
  __shared__ float red[kTW], isum[kTW], xsqs[kTW];
  __shared__ float sxs[TT];
  __shared__ int part[4][TT][kTokRows];      // columns' share, token, row
  __shared__ float unit_keys[TT][kTokRows];
  HIRE_TS(30);
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int B = p.B, N = p.N, d = p.d;
  const int cpr = d / 32, xstride = d / 16 + 1;
  const unsigned long long cookie = p.fr->cookie;  // (workgroup 0 takes it away)
  const float smax = __uint_as_float(p.q4[(size_t)N * cpr].x);  // largest row scale, kept behind the codes
  // the windows of the activations, filled by the next kernel, start from zero
  for (int i = (int)blockIdx.x * kTT + tid; i < B * kWin; i += (int)gridDim.x * kTT)
    p.fr[i / kWin].hist2[i % kWin] = 0u;
  const int t = w / kWPT, lt = w % kWPT * kWave + lane, nvec = d / 8;
  auto token_vec = [&](int i) -> uint4 {
    const size_t at = (size_t)min(t, B - 1) * nvec + min(i, nvec - 1);
    if constexpr (!LRQ) {
      return reinterpret_cast<const uint4*>(p.x)[at];
    } else {
      return bf16_pairs(reinterpret_cast<const uint4*>(p.x)[2 * at], reinterpret_cast<const uint4*>(p.x)[2 * at + 1]);
    }
  };
  // All loads are unconditional: the wait for the tokens must not become one for the weights, which are issued next.
  uint4 xv[VECS];
#pragma unroll
  for (int m = 0; m < VECS; ++m) xv[m] = token_vec(m * kWPT * kWave + lt);
  // the wave's rows, sixteen chunks of sixteen bytes per load, four loads at a time
  const int nsl = (cpr + 15) / 16;
  const uint4* wrow = p.q4 + (size_t)min((int)blockIdx.x * kTokRows + w * 4 + (lane & 3), N - 1) * cpr;
  uint4 wv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) wv[i] = load_streaming(&wrow[min(i * 16 + (lane >> 2), cpr - 1)]);
  const float row_scale = p.scale[min((int)blockIdx.x * kTokRows + lane, N - 1)];

  float amax = 0.0f;
#pragma unroll
  for (int m = 0; m < VECS; ++m) {
    const uint32_t ud[4] = {xv[m].x, xv[m].y, xv[m].z, xv[m].w};
#pragma unroll
    for (int q = 0; q < 4; ++q) amax = fmaxf(amax, fmaxf(fabsf(bf16_lo(ud[q])), fabsf(bf16_hi(ud[q]))));
  }
  amax = wave_max(amax);
  if (lane == 0) red[w] = amax;
  if constexpr (LRQ) {
    float xsq = 0.0f;
    for (int i = lt; i < p.xn_d / 8; i += kWPT * kWave) {
      const uint4 u = p.xn[(size_t)min(t, B - 1) * (p.xn_d / 8) + i];
      const uint32_t ud[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float a = bf16_lo(ud[q]), b = bf16_hi(ud[q]);
        xsq = fmaf(a, a, xsq);
        xsq = fmaf(b, b, xsq);
      }
    }
    xsq = wave_sum(xsq);
    if (lane == 0) xsqs[w] = xsq;
  }
  lds_barrier();
  HIRE_TS(31);
  amax = wave_max(lane < kWPT ? red[t * kWPT + lane] : 0.0f);
  const TokenScale ts = token_scale(amax);
  float sabs = 0.0f;
#pragma unroll
  for (int m = 0; m < VECS; ++m)
    if (m * kWPT * kWave < nvec) {  // uniform
      float sum8;
      const uint2 codes = quantise8(xv[m], ts, &sum8);
      const int i = m * kWPT * kWave + lt;
      if (i < nvec) {
        sabs += sum8;
        reinterpret_cast<uint2*>(xs + t * xstride)[i] = codes;
      }
    }
  sabs = wave_sum(sabs);
  if (lane == 0) {
    isum[w] = sabs;
    if (w % kWPT == 0) sxs[t] = ts.sx;
  }
  lds_barrier();
  HIRE_TS(32);

  // Wave b will take the 64 keys of token b; its bounds, those of k_fast_score_int4, while the weights are under way.
  const int b = w, bt = min(w, TT - 1);
  const bool here = b < B;
  const float sumabs = wave_sum(lane < kWPT ? isum[bt * kWPT + lane] : 0.0f);
  const float group_factor = p.gkeys != nullptr ? 8.001f : 1.0f;
  const float bound1 = 7.0f * sumabs * smax * group_factor;
  float bound2 = smax * sxs[bt] * (7.6f * sumabs + 3.8f * (float)d + 1.0f) * 1.01f * group_factor;
  if constexpr (LRQ) {
    const float xsq = wave_sum(lane < kWPT ? xsqs[bt * kWPT + lane] : 0.0f);
    bound2 = sqrtf(xsq * (1.0f + (float)p.xn_d * 0x1p-22f)) * 1.0001f * p.umax[0] * 1.0001f * group_factor;
  }
  FastRegion* fr = p.fr + min(b, B - 1);
  const uint32_t anchor1 = fine_bin(__float_as_uint(bound1)), anchor2 = fine_bin(__float_as_uint(bound2));
  if (here && blockIdx.x == 0 && lane == 0) {
    fr->anchor1 = anchor1;
    fr->anchor2 = anchor2;
    fr->beyond2 = 0u;
    if (b == 0) take_cookie(p.fr, cookie);
  }

  constexpr int kTok4 = TT / 4;
  v4i acc[kTok4];
#pragma unroll
  for (int f = 0; f < kTok4; ++f) acc[f] = v4i{0, 0, 0, 0};
  for (int s0 = 0; s0 < nsl; s0 += 4) {
    if (s0 > 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) wv[i] = load_streaming(&wrow[min((s0 + i) * 16 + (lane >> 2), cpr - 1)]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (s0 + i < nsl) {  // uniform
        const int c = (s0 + i) * 16 + (lane >> 2), cc = min(c, cpr - 1);
        const uint32_t keep = c < cpr ? 0xFFFFFFFFu : 0u;  // past the row's end: zeros
        const uint4 codes = make_uint4(wv[i].x & keep, wv[i].y & keep, wv[i].z & keep, wv[i].w & keep);
#pragma unroll
        for (int f = 0; f < kTok4; ++f) {
          const uint4* xr = xs + (f * 4 + (lane & 3)) * xstride + 2 * cc;
          int4_rows_by_tokens(codes, xr[0], xr[1], acc[f]);
        }
      }
  }
  HIRE_TS(33);
#pragma unroll
  for (int f = 0; f < kTok4; ++f)
#pragma unroll
    for (int r = 0; r < 4; ++r) {  // row r, token l % 4: the four blocks of sixteen lanes
      int v = acc[f][r];
      v += dpp_move<0x124, 0xF>(0, v);
      v += dpp_move<0x128, 0xF>(0, v);
      if ((lane & 12) == 0) part[lane >> 4][f * 4 + (lane & 3)][w * 4 + r] = v;
    }
  lds_barrier();

  if (b >= TT) {
    if (p.gkeys != nullptr) lds_barrier();
    return;
  }
  auto count_key = [&](float key) { count_in_window<true>(__float_as_uint(key), anchor1, fr->hist1, &fr->beyond1); };
  const int j = (int)blockIdx.x * kTokRows + lane;
  int sum = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) sum += part[q][b][lane];
  sum >>= 4;  // every partial is a multiple of 16
  float key = (float)sum * row_scale;
  key = key > 0.0f ? key : 0.0f;  // ReLU, and -0 -> +0
  if (here && j < N) {
    if (p.acc_out) p.acc_out[(size_t)b * N + j] = sum;
    if (p.gkeys == nullptr) {
      p.keys[(size_t)b * p.stride + j] = key;
      count_key(key);
    }
  }
  if (p.gkeys != nullptr) {
    unit_keys[b][lane] = key;
    lds_barrier();
    const int J = (int)blockIdx.x * (kTokRows / 8) + lane;
    if (here && lane < kTokRows / 8 && J * 8 < N) {
      float s = 0.0f;
#pragma unroll
      for (int l = 0; l < 8; ++l) s += fabsf(unit_keys[b][lane * 8 + l]);
      p.gkeys[(size_t)b * p.gstride + J] = s;
      count_key(s);
    }
  }
  HIRE_TS(34);
}

// ---------------------------------------------------------------------------------------------------
// Kernel 2: the shortlists and their exact pre-activations, as k_fast_gather, for all tokens.
struct FastGatherTokens {
  const void* keys;           // [B, stride] fp32 (fp64), rows at multiples of 16 bytes
  long long stride;
  int B, N, kprime, d;        // kprime: selected entries (units or groups) per token
  FastRegion* fr;
  const uint16_t* W1;         // [N, d] bf16
  const uint4* x;             // [B, d] bf16
  float* h32;                 // [B, entries] activations, 0 where no token shortlists the entry
  double* h64;                // the same in fp64, -1 there
  int entries;                // N >> gs up to a whole workgroup
  int gs;                     // 3: groups of eight units, as in FastGatherParams
  float* u32;                 // groups: [B, entries << gs] the units' activations
  uint32_t* bitmap;           // union of the shortlists, (N >> gs) bits
  // dense units: own_blocks workgroups take `share` each beside their own units, further workgroups kDenseRows each
  int own_blocks, share;
  const uint16_t* Wd;
  int m1;
  double* hd;                 // [B, m1]
};
constexpr int kDenseRows = 32;

// Where the selection of the k largest of n keys in memory cuts them, without a histogram.
template <typename K>
__device__ __forceinline__ Cut<K> streaming_cut(const K* keys, int n, int k, SelSharedT<kTT>& sh, int* wave_gt,
                                                int* wave_eq) {
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const K t = KeyIO<K>::from_order_key(wg_kth_largest<K>(
      [&](auto&& f) {
#pragma unroll 1
        for (int i = tid; i < n; i += kTT) f(KeyIO<K>::to_order_key(keys[i]));
      },
      n, k, sh));
  const int M = ((n + kTW - 1) / kTW + kWave - 1) / kWave * kWave, lo = w * M, hi = min(n, lo + M);
  int gt = 0, eq = 0;
#pragma unroll 1
  for (int i = lo + lane; i < hi; i += kWave) {
    gt += keys[i] > t ? 1 : 0;
    eq += keys[i] == t ? 1 : 0;
  }
  gt = wave_sum(gt);
  eq = wave_sum(eq);
  __syncthreads();
  if (lane == 0) {
    wave_gt[w] = gt;
    wave_eq[w] = eq;
  }
  __syncthreads();
  int all_gt = 0, before = 0;
  for (int u = 0; u < kTW; ++u) {
    all_gt += wave_gt[u];
    before += u < w ? wave_eq[u] : 0;
  }
  const int need = k - all_gt;  // >= 1: t itself is selected
  if (before < need && need <= before + eq) {  // one wave
    int run = before;
#pragma unroll 1
    for (int i0 = lo; i0 < hi; i0 += kWave) {
      const uint64_t m = __ballot(i0 + lane < hi && keys[min(i0 + lane, n - 1)] == t);
      if (((m >> lane) & 1ull) != 0ull && run + mask_prefix(m) + 1 == need) sh.bc_bin = i0 + lane;
      run += __popcll(m);
    }
  }
  __syncthreads();
  Cut<K> c;
  c.key = t;
  c.idx = sh.bc_bin;
  return c;
}

// K: the keys' bit patterns.  TT: tokens rounded up to four or eight.
// Measured at the ~1B shape and four tokens, from the first wave's start: 4.2 us until the rows are known, the 9600 rows of the
// union until 13.2 (40 MB, 4.5 TB/s), 1.2 for the outputs; half the workgroups have ended by 14.3 and the last by 17.6, one
// that has two keys of threshold bins to settle (19.8 when they were settled ahead of the rows).  The kernel 17.3 us.
template <typename K, int TT>
__global__ __launch_bounds__(kTT) void k_fast_gather_tokens(FastGatherTokens p) {
  constexpr int kWPT = kTW / TT, kChunks = kWin / 256, kMine = kChunks / kWPT;  // 256 counters per wave and load
  __shared__ SelSharedT<kTT> sh;
  __shared__ int wave_gt[kTW], wave_eq[kTW];
  __shared__ int chunk_sum[TT][kChunks], slot[TT];
  // units of the workgroup that only have keys of threshold bins: key, unit and token, keys ahead of it by wave.  More than four
  // tokens come with groups of eight, whose first units stand for them.
  constexpr int kOpen = TT <= 4 ? TT * kOwnUnits : TT * kOwnUnits / 8;
  __shared__ K open_key[kOpen];
  __shared__ int open_unit[kOpen], open_ahead[kOpen][kTW];
  __shared__ int unit_of[kOwnUnits];
  __shared__ double unit_h[TT][kOwnUnits];
  extern __shared__ double red[];  // partial sums of rows_by_tokens
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int g = (int)blockIdx.x, nvec = p.d / 8, gs = p.gs, B = p.B;
  HIRE_TS(10);
  const bool sparse = g < p.own_blocks;  // uniform
  // this workgroup's dense units
  const int r0 = sparse ? g * p.share : p.own_blocks * p.share + (g - p.own_blocks) * kDenseRows;
  const int dense = max(0, min(sparse ? p.share : kDenseRows, p.m1 - r0));
  const int u0 = g * kOwnUnits;  // first unit of the workgroup
  uint64_t rows = 0ull, taken = 0ull;  // units of the workgroup: whose rows are read; that any token shortlists
  int opens = 0;                       // (unit, token) pairs that settle the difference
  const int n = p.N >> gs;
  if (sparse) {
    uint4 wr[kMine];
    const int tw = w / kWPT, wt = w % kWPT;  // the token whose window this wave helps to walk, its part of it
    {
      const uint4* hist = reinterpret_cast<const uint4*>(p.fr[min(tw, B - 1)].hist1);
#pragma unroll
      for (int u = 0; u < kMine; ++u) wr[u] = hist[spread_slot(((wt * kMine + u) * kWave + lane) * 4) / 4];
    }
    const int entry = (u0 + lane) >> gs;  // lane's unit, or its group
    const bool valid = u0 + lane < p.N;
    K own[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) own[t] = reinterpret_cast<const K*>(p.keys)[min(t, B - 1) * p.stride + min(entry, n - 1)];
    const uint32_t a1 = p.fr[min(lane, B - 1)].anchor1;  // lane t: token t's
    const int clean = (int)p.fr->clean;
    const uint32_t beyond1 = p.fr[min(tw, B - 1)].beyond1;
    const bool hist_ok = (tw < clean) & (beyond1 == 0u);  // (both asked for at once, behind the window: no branch between the two)
    if (tid < TT) slot[tid] = -1;
    // walk: sums of 256 counters, the chunk that holds the k'-th key, its lane, its counter
    int s[kMine];
#pragma unroll
    for (int u = 0; u < kMine; u += 2) {  // (sums of counters fit sixteen bits: 16384 keys at most)
      s[u] = (int)(wr[u].x + wr[u].y + wr[u].z + wr[u].w);
      s[u + 1] = (int)(wr[u + 1].x + wr[u + 1].y + wr[u + 1].z + wr[u + 1].w);
      const uint32_t tot = wave_sum((uint32_t)s[u] | (uint32_t)s[u + 1] << 16);
      if (lane == 0) {
        chunk_sum[tw][wt * kMine + u] = (int)(tot & 0xFFFFu);
        chunk_sum[tw][wt * kMine + u + 1] = (int)(tot >> 16);
      }
    }
    lds_barrier();
    HIRE_TS(11);
    {
      const int v = lane < kChunks ? chunk_sum[tw][lane] : 0, incl = wave_scan_incl(v);
      const uint64_t at = __ballot(lane < kChunks && incl - v < p.kprime && p.kprime <= incl);
      if (at != 0ull && hist_ok) {  // uniform; tokens without an exact histogram have no slot
        const int q = __builtin_ctzll(at), run0 = __builtin_amdgcn_readlane(incl - v, q);
#pragma unroll
        for (int u = 0; u < kMine; ++u)
          if (q == wt * kMine + u) {  // uniform: one wave
            const int run = run0 + wave_scan_incl(s[u]) - s[u];
            if (run < p.kprime && p.kprime <= run + s[u]) {  // one lane
              const int c[4] = {(int)wr[u].x, (int)wr[u].y, (int)wr[u].z, (int)wr[u].w};
              int rr = run;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                if (rr < p.kprime && p.kprime <= rr + c[e]) slot[tw] = (q * kWave + lane) * 4 + e;
                rr += c[e];
              }
            }
          }
      }
    }
    lds_barrier();
    HIRE_TS(15);
    uint32_t unresolved = 0u;  // tokens
    uint64_t in_bin[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      in_bin[t] = 0ull;
      if (t < B) {  // uniform
        const int sl = __builtin_amdgcn_readfirstlane(slot[t]);
        const uint32_t anchor = (uint32_t)__builtin_amdgcn_readlane((int)a1, t), bin = anchor - (uint32_t)sl;
        if (sl >= 0 && bin >= 1u && bin <= anchor) {  // uniform
          const K lo = bin_floor<K>(bin), up = bin_floor<K>(bin + 1u);
          rows |= __ballot(valid && own[t] >= up);
          in_bin[t] = __ballot(valid && own[t] >= lo && own[t] < up);
        } else {
          unresolved |= 1u << t;
        }
      }
    }
    for (uint32_t m = unresolved; m != 0u; m &= m - 1u) {  // fresh workspace, threshold among the zeros or below the
      const int t = __builtin_ctz(m);                      // window
      if (g == 0 && tid == 0 && t < clean) atomicAdd(&p.fr->fallbacks[0], 1u);
      const K* row = reinterpret_cast<const K*>(p.keys) + (size_t)t * p.stride;
      __syncthreads();
      const Cut<K> cut = streaming_cut<K>(row, n, p.kprime, sh, wave_gt, wave_eq);
      rows |= __ballot(valid && cut_takes(cut, row[min(entry, n - 1)], entry));
    }
    // every wave notes the undecided units (the same values) and reads its own notes; of a group its first unit.  Their rows
    // are read with the others.
    uint64_t undecided = 0ull;
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const uint64_t m = in_bin[t] & ~rows & (gs != 0 ? 0x0101010101010101ull : ~0ull);
      if (((m >> lane) & 1ull) != 0ull) {
        open_key[opens + mask_prefix(m)] = own[t];
        open_unit[opens + mask_prefix(m)] = lane * TT + t;
      }
      opens += __popcll(m);
      undecided |= m;
    }
    taken = rows;
    rows |= gs != 0 ? undecided * 0xFFull : undecided;  // (of a group its first unit's bit)
  }
  HIRE_TS(12);
  const int cnt = __popcll(rows);
  // every wave notes all rows (the same values) and reads its own notes
  if (((rows >> lane) & 1ull) != 0ull) unit_of[mask_prefix(rows)] = lane;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  HIRE_TS(13);
  auto count_h = [&](int t, double v) {  // the scorer kernel of this step has cleared the windows
    count_in_window<true>((uint64_t)__double_as_longlong(v), p.fr[t].anchor2, p.fr[t].hist2, &p.fr[t].beyond2);
  };
  if (sparse && gs == 0 && w < B && ((rows >> lane) & 1ull) == 0ull) {
    p.h32[(size_t)w * p.entries + u0 + lane] = 0.0f;
    p.h64[(size_t)w * p.entries + u0 + lane] = -1.0;
  }
  // (one base and an offset: between two pointers the compiler selects where they are stored, and every row's loads
  // wait for the load of an address)
  const char* base = reinterpret_cast<const char*>(p.W1);
  const long long row_bytes = 2ll * p.d, own_at = u0 * row_bytes,
                  dense_at = reinterpret_cast<const char*>(p.Wd) - base + (r0 - cnt) * row_bytes;
  rows_sums<TT>(
      cnt + dense,
      [&](int r) {
        const int at = r < cnt ? unit_of[min(r, kOwnUnits - 1)] : r;
        return reinterpret_cast<const uint4*>(base + ((r < cnt ? own_at : dense_at) + at * row_bytes));
      },
      p.x, B, nvec, red);
  // A unit that only has keys of threshold bins, of which some are selected: its key is compared with all others of the token.
  // One workgroup in six has such a unit, and then one or two, and would be the last to end.  Its rows are read with the others,
  // and a wave that has its rows asks for its part of the keys while other waves still wait for theirs: ahead of the rows, or
  // beside their first loads, the keys cost 2 to 5 us instead of one.  Where rows repeat and a workgroup has many such units, they
  // follow one another; the next one's keys requested ahead of the comparison are slower there as well: the ~1B shape, four
  // tokens, 40 distinct rows 83.9 us per step (85.7), all rows equal 595 (625), no repeated rows 37.7 (37.9).
#pragma unroll 1
  for (int j = 0; j < opens; ++j) {  // uniform over the workgroup
    constexpr int PER = KeyIO<K>::PER, kLoads = 16 / PER;  // the row of 16384 keys at a time
    const int unit = __builtin_amdgcn_readfirstlane(open_unit[j]), vecs = (n + PER - 1) / PER, at = (u0 + unit / TT) >> gs;
    const uint4* row = reinterpret_cast<const uint4*>(reinterpret_cast<const K*>(p.keys) + (size_t)(unit % TT) * p.stride);
    uint4 raw[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) raw[u] = row[min(u * kTT + tid, vecs - 1)];
    const K mine = open_key[j];
    int ahead = 0;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int i = (u * kTT + tid) * PER;
      K k[PER];
      KeyIO<K>::unpack(raw[u], k);
#pragma unroll
      for (int q = 0; q < PER; ++q) ahead += i + q < n && k[q] >= mine + (i + q < at ? 0u : 1u) ? 1 : 0;
    }
    ahead = wave_sum(ahead);
    if (lane == 0) open_ahead[j][w] = ahead;
  }
  lds_barrier();
  HIRE_TS(17);
#pragma unroll 1
  for (int j = 0; j < opens; ++j)
    if (wave_sum(lane < kTW ? open_ahead[j][lane] : 0) < p.kprime)
      taken |= (gs != 0 ? 0xFFull : 1ull) << (__builtin_amdgcn_readfirstlane(open_unit[j]) / TT);
  rows_out<TT>(
      cnt + dense, B, nvec, red,
      [&](int r, int t, double v) {
        if (r >= cnt) {
          p.hd[(size_t)t * p.m1 + r0 + r - cnt] = v;
          return;
        }
        const int pos = unit_of[r];
        if (gs != 0) {
          unit_h[t][pos] = v;
        } else {
          const bool in = ((taken >> pos) & 1ull) != 0ull;
          p.h32[(size_t)t * p.entries + u0 + pos] = in ? (float)v : 0.0f;
          p.h64[(size_t)t * p.entries + u0 + pos] = in ? v : -1.0;
          if (in) count_h(t, v);
        }
      });
  if (!sparse) return;
  if (gs != 0) {  // exact group activations, units added in order; wave t: token t
    __syncthreads();
    if (w < B) {
      p.u32[(size_t)w * (p.entries << gs) + u0 + lane] = ((taken >> lane) & 1ull) != 0ull ? (float)unit_h[w][lane] : 0.0f;
      if (lane < kOwnUnits >> gs) {
        const bool in = ((taken >> (lane << gs)) & 1ull) != 0ull;
        double e = 0.0;
        if (in)
          for (int l = 0; l < (1 << gs); ++l) e += fabs(unit_h[w][(lane << gs) + l]);
        const size_t at = (size_t)w * p.entries + (u0 >> gs) + lane;
        p.h32[at] = in ? (float)e : 0.0f;
        p.h64[at] = in ? e : -1.0;
        if (in) count_h(w, e);
      }
    }
  }
  if (tid == 0) {  // the workgroup's part of the union
    if (gs == 0) {
      p.bitmap[2 * g] = (uint32_t)taken;
      p.bitmap[2 * g + 1] = (uint32_t)(taken >> 32);
    } else {
      uint32_t bits = 0u;
      for (int J = 0; J < kOwnUnits >> gs; ++J) bits |= (uint32_t)((taken >> (J << gs)) & 1ull) << J;
      uint8_t* bytes = reinterpret_cast<uint8_t*>(p.bitmap);
      bytes[g] = (uint8_t)bits;
      if (g == p.own_blocks - 1)
        for (int i = g + 1; (i & 3) != 0; ++i) bytes[i] = 0u;  // the last word is read whole
    }
  }
  HIRE_TS(14);
}

// ---------------------------------------------------------------------------------------------------
static int token_slots(int B) { return B <= 4 ? 4 : 8; }

// Steps on units: up to four tokens.  With more the fp64 products and two windows of counters per wave outweigh the
// selections saved: the longer sequence (its values rounded from 64 bits like these, k' = N / 5) against this one in us per step,
// int4 scorer, for 2 / 3 / 4 and 5 / 6 / 7 / 8 tokens
//   d =  256,  1024 units  27.9 24.3 24.5   21.4 22.1 23.8 and 24.2 24.6 24.4 24.7   25.8 26.8 27.9 29.0
//   d = 1024,  4096 units  32.5 29.2 29.0   24.4 25.1 27.1 and 29.3 29.7 29.6 29.8   31.2 32.5 33.5 36.0
//   d =  800,  5003 units  31.3 28.8 28.8   23.6 24.8 26.8 and 29.0 29.1 29.2 29.4   30.8 31.8 32.9 33.9
//   d = 4096,  8192 units  48.9 51.1 52.4   35.9 39.9 45.8 and 54.7 55.2   56.8 59.4
//   d = 2048,  8192 units  37.5 35.7 36.1   28.6 30.0 33.7 and 36.5 36.8   41.5 43.9
//   d =  512, 16000 units  34.0 30.5 31.0   28.0 30.6 34.5
//   d = 2048, 16384 units  42.7 44.3 46.4   34.0 37.8 43.7
// Groups of eight, whose longer sequence forms its activations in fp64 too, gain up to eight where they have dense units beside
// them or many units (ffn_group_step_impl holds the line).  The scorer keeps a token in four vectors per thread.
bool ffn_fast_tokens_supported(int B, int d, bool groups) {
  if (B < 2 || B > kFastTokens || token_slots(B) * d > 32768) return false;
  return groups || B <= 4;
}

hipError_t launch_fast_score_tokens(const FfnFastArgs& a, const void* x, bool lrq, hipStream_t s) {
  FastScoreTokens p{};
  p.q4 = reinterpret_cast<const uint4*>(lrq ? a.lr_b : a.q4);
  p.scale = lrq ? a.lr_b_scale : a.q4_scale;
  p.x = x;
  p.B = a.B; p.N = a.N; p.d = lrq ? a.r : a.d;
  p.keys = a.keys; p.stride = a.key_stride;
  p.acc_out = a.scorer_acc;
  p.fr = reinterpret_cast<FastRegion*>(a.fast_region);
  p.gkeys = a.gs ? a.gkeys : nullptr;
  p.gstride = a.gkey_stride;
  p.xn = reinterpret_cast<const uint4*>(a.x); p.xn_d = a.d; p.umax = a.norm_bounds;
  const size_t lds = (size_t)token_slots(a.B) * (p.d / 16 + 1) * sizeof(uint4);
  const dim3 grid((a.N + kTokRows - 1) / kTokRows);
  static std::atomic<size_t> raised_to[7] = {};
  auto go = [&](auto kernel, int i) -> hipError_t {
    if (const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, raised_to[i]); e != hipSuccess)
      return e;
    return launch(kernel, grid, dim3(kTT), lds, s, p);
  };
  const bool four = token_slots(a.B) == 4;
  if (lrq) return four ? go(k_fast_score_tokens<true, 4, 1>, 0) : hipErrorInvalidValue;  // r <= 1024
  const int values = token_slots(a.B) * p.d;  // a workgroup loads 8192 of them at a time
  if (values <= 8192) return four ? go(k_fast_score_tokens<false, 4, 1>, 1) : go(k_fast_score_tokens<false, 8, 1>, 2);
  if (values <= 16384) return four ? go(k_fast_score_tokens<false, 4, 2>, 3) : go(k_fast_score_tokens<false, 8, 2>, 4);
  return four ? go(k_fast_score_tokens<false, 4, 4>, 5) : go(k_fast_score_tokens<false, 8, 4>, 6);
}

hipError_t launch_fast_gather_tokens(const FfnFastArgs& a, hipStream_t s) {
  FastGatherTokens p{};
  p.keys = a.lowrank ? static_cast<const void*>(a.gs ? a.gkeys64 : a.keys64) : (a.gs ? a.gkeys : a.keys);
  p.stride = a.gs ? a.gkey_stride : a.key_stride;
  p.B = a.B; p.N = a.N; p.kprime = a.kprime >> a.gs; p.d = a.d;
  p.fr = reinterpret_cast<FastRegion*>(a.fast_region);
  p.W1 = a.w1u; p.x = reinterpret_cast<const uint4*>(a.x);
  p.h32 = a.h32; p.h64 = a.h; p.entries = ffn_fast_entries(a.N, a.gs); p.gs = a.gs; p.u32 = a.u32;
  p.bitmap = a.bitmap;
  p.own_blocks = (a.N + kOwnUnits - 1) / kOwnUnits;
  p.Wd = a.dense_w1u; p.m1 = a.m1; p.hd = a.h_dense;
  // dense units go to the compute units left over first (a workgroup more than there are units waits for a whole
  // workgroup's time), then to the workgroups of the sparse ones, then to workgroups of their own after all
  const int spare = max(0, 256 - p.own_blocks) * kDenseRows;
  p.share = min(kMostRows - kOwnUnits, (max(0, a.m1 - spare) + p.own_blocks - 1) / p.own_blocks);
  const int rest = max(0, a.m1 - p.own_blocks * p.share);
  const size_t lds = (size_t)kTW * (kMostRows / 4) * (token_slots(a.B) / 4) * 16 * sizeof(double);
  const dim3 grid(p.own_blocks + (rest + kDenseRows - 1) / kDenseRows);
  static std::atomic<size_t> raised_to[3] = {};
  auto go = [&](auto kernel, int i) -> hipError_t {
    if (const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, raised_to[i]); e != hipSuccess)
      return e;
    return launch(kernel, grid, dim3(kTT), lds, s, p);
  };
  if (a.lowrank) return token_slots(a.B) == 4 ? go(k_fast_gather_tokens<uint64_t, 4>, 2) : hipErrorInvalidValue;
  switch (token_slots(a.B)) {
    case 4: return go(k_fast_gather_tokens<uint32_t, 4>, 0);
    default: return go(k_fast_gather_tokens<uint32_t, 8>, 1);
  }
}

}  // namespace hire

#ifdef HIRE_TIMESTAMPS
extern "C" int hire_debug_timestamps_fast_tokens(unsigned long long* host64) {
  return (int)hipMemcpyFromSymbol(host64, HIP_SYMBOL(hire_ts), sizeof(hire_ts));
}
#endif
