// HiRE-Q scorer for batches (arXiv 2402.09360, Algorithm 1 line 1 with the int4 Zapprox of Sec. 3.2) on the
// int8 matrix cores: acc[b, j] = sum_i q_j[i] xq[b, i] as 16x16x64 MFMA tiles, 16 tokens by 16 weight rows.
//
// The packed layout (scorer.hip) turns one dword into two registers of four signed bytes equal to 16*code with two ANDs
// and a shift; these feed the MFMA directly and the sums are shifted back by four bits at the end (every partial is a
// multiple of 16, so this is exact).  Which 16 of a row's codes a lane contributes to which MFMA does not matter as
// long as its token operand holds the activations of the same 16 positions: a dot product does not care about the
// order of its terms.
//
// Operand roles: tokens are the A matrix (rows), weights the B matrix (columns), so lane l of the result holds
// weight row l % 16 for tokens 4 * (l / 16) .. + 3, and the 16 lanes of a DPP row store 16 consecutive keys
// of one token.
#include "device_utils.h"
#include "hist.h"
#include "kernels.h"
#include "rows_mfma.h"

namespace hire {

struct ScorerBatch {
  const uint4* q4;
  const float* scale;
  ScorerTokens tok;
  int B, N, d, relu;
  float* keys;
  long long stride;
  int32_t* acc_out;  // optional [B, N]
  uint32_t* wgmax;   // optional [B, kWgMaxSlots]
  int seg_steps;     // steps of 128 codes of a K segment, whose codes of all tokens are in LDS
  int parts;         // PARTS: of the tokens
};

enum ScorerSource { kCodes, kBf16, kF32 };

// A workgroup has RW x KW waves: RW groups of RT row tiles of 16 rows, the steps of a K segment shared out over KW waves,
// whose integer sums are added in LDS.  CT: token tiles of 16 (batch <= 16 CT).  P: steps (16 bytes per lane and tile)
// requested together.
//
// KW > 1 (rows of the FFN and of the low-rank factors): a workgroup has one group of tiles and sixteen waves, so that the
// staging of the tokens, the unpacking and the epilogue are each a sixteenth of the work: the kernel is bound by that chain
// and not by memory.  In steps whose weights come from HBM, averages under rocprofv3 (as all times here): d = 2048, 16384 rows,
// 16 / 32 / 64 tokens 7.4 / 8.0 / 9.5 us, where a workgroup of four waves with whole rows each took 8.9 / 12.5 / 13.4; 5003 rows
// of 800 codes, 33 tokens 5.8, 10.8 (7.9 with the quantisation in it, against 5.5 + 3.6 and a kernel boundary).
//
// KW = 1 (vocabularies): a workgroup of eight waves per compute unit stages the tokens once and runs on from tile to tile,
// the next request always out ahead of the current product.  No load there sits behind a branch: the wait for one request
// would become one for the next (64 to 68 us instead of 52 to 54 for 256000 rows of 2048 codes and 16 tokens).  16 / 32 / 64
// tokens: 52 / 58 / 73 to 80 us (54 / 80 / 124 with a workgroup's tile in registers as a whole and four waves); the 263 MB alone
// take 42 us with loads of this pattern, the keys 8 to 12 more, and from 33 tokens on the products (30 us of matrix cores and
// LDS) and the stores that a wave waits for between its tiles are not hidden by two waves per SIMD.
//
// kBf16, kF32: the workgroup quantises the tokens itself.  VECS: 16-byte vectors (of bf16 values, or of codes) of a token
// per lane.
// PARTS: a workgroup has sixteen of the tokens, one to quantise per wave, and so many more rows; the workgroups with the same rows
// are on one die, whose L2 has the codes.
template <int CT, int RT, int RW, int KW, int P, int SRC, int VECS, bool PARTS = false>
__global__ __launch_bounds__(64 * RW * KW) void k_scorer_int4_mfma(ScorerBatch p) {
  constexpr int NW = RW * KW, NT = kWave * NW, kTok = 16 * CT, kRows = 16 * RT * RW;
  static_assert(RT == 1 || KW == 1, "tiles of a wave");
  static_assert(SRC == kCodes || KW > 1, "vocabularies: a kernel in front quantises");
  static_assert(!PARTS || (SRC == kBf16 && CT == 1), "a token per wave");
  extern __shared__ uint4 xs[];  // [kTok][8 seg_steps + 1]: a token row's first chunk in another bank than its neighbours'
  const int tid = (int)threadIdx.x, lane = lane_id(), jl = lane & 15, g = lane >> 4;
  // known to be uniform: a matrix-core instruction must never sit behind a branch that is lowered to lane masking
  const int w = __builtin_amdgcn_readfirstlane(wave_id()), rw = w % RW, kw = w / RW;
  int first_tile = (int)blockIdx.x, tok0 = 0;
  if constexpr (PARTS) {
    const int at = (int)blockIdx.x % (8 * p.parts);
    first_tile = (int)blockIdx.x / (8 * p.parts) * 8 + at % 8;
    tok0 = at / 8 * kTok;
  }
  const int B = PARTS ? min(p.B - tok0, kTok) : p.B, N = p.N, cpr = p.d / 32;  // 16-byte chunks per packed row
  const int steps = (cpr + 3) / 4, seg_steps = p.seg_steps, nseg = (steps + seg_steps - 1) / seg_steps;
  const int per = (seg_steps + KW - 1) / KW, nblk = (per + P - 1) / P;  // steps, requests of a wave per segment
  const int xstride = 8 * seg_steps + 1;

  struct Request {
    uint4 v[P][RT];
    float sj[RT];
  };
  // A wave's request: P steps of its tiles and their row scales.  Past the row's end a lane loads its last chunk (the
  // tokens' codes are zero there), past the matrix its last row (nothing is stored).
  auto request = [&](Request& q, int tile, int seg, int blk) __attribute__((always_inline)) {
    const int s0 = seg * seg_steps + kw * per + blk * P;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int row = min(tile * kRows + (rw * RT + rt) * 16 + jl, N - 1);
      q.sj[rt] = p.scale[row];
      const uint4* wrow = p.q4 + (size_t)row * cpr;
#pragma unroll
      for (int u = 0; u < P; ++u) q.v[u][rt] = wrow[min((s0 + u) * 4 + g, cpr - 1)];
    }
  };

  // The tokens' codes of a segment into LDS, a wave whole tokens: load_tokens ahead of the first request (loads return in
  // order), stage behind it.
  constexpr int TPW = kTok / NW;  // tokens of a wave
  constexpr int kMost = SRC == kCodes ? 4 : (SRC == kF32 ? 4 / VECS : TPW), kAhead = TPW > kMost ? kMost : TPW;  // (registers)
  static_assert(TPW >= 1 && TPW % kAhead == 0 && (SRC != kCodes || VECS == 2), "whole tokens, segments of 256 vectors");
  uint4 tv[kAhead][VECS], tv2[kAhead][SRC == kF32 ? VECS : 1];
  const int segq = 8 * seg_steps, xv = p.d / 16, nvec = p.d / 8;
  auto load_codes = [&](uint4 (&v)[kAhead][VECS], int seg, int q0) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
#pragma unroll
      for (int m = 0; m < VECS; ++m)
        v[q][m] = reinterpret_cast<const uint4*>(p.tok.xq)[(size_t)min(w + (q0 + q) * NW, B - 1) * xv +
                                                           min(seg * segq + m * kWave + lane, xv - 1)];
  };
  auto store_codes = [&](const uint4 (&v)[kAhead][VECS], int seg, int q0) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
#pragma unroll
      for (int m = 0; m < VECS; ++m) {
        const int t = w + (q0 + q) * NW, i = m * kWave + lane;
        if (i < segq) xs[t * xstride + i] = t < B && seg * segq + i < xv ? v[q][m] : make_uint4(0, 0, 0, 0);
      }
  };
  auto load_values = [&](int q0) __attribute__((always_inline)) {
    const uint4* x4 = reinterpret_cast<const uint4*>(p.tok.x) + (size_t)tok0 * nvec;
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
#pragma unroll
      for (int m = 0; m < VECS; ++m) {
        const size_t at = (size_t)min(w + (q0 + q) * NW, B - 1) * nvec + min(m * kWave + lane, nvec - 1);
        tv[q][m] = x4[SRC == kF32 ? 2 * at : at];
        if constexpr (SRC == kF32) tv2[q][m] = x4[2 * at + 1];
      }
  };
  auto load_tokens = [&](int seg) __attribute__((always_inline)) {
    if constexpr (SRC == kCodes) load_codes(tv, seg, 0);
    else load_values(0);
  };
  auto stage = [&](int seg) __attribute__((always_inline)) {
    if constexpr (SRC == kCodes) {
      store_codes(tv, seg, 0);
#pragma unroll
      for (int q0 = kAhead; q0 < TPW; q0 += kAhead) {
        uint4 v[kAhead][VECS];
        load_codes(v, seg, q0);
        store_codes(v, seg, q0);
      }
    } else {  // one segment
#pragma unroll
      for (int at = 0; at < TPW; ++at) {
        const int q = at % kAhead, t = w + at * NW;
        if (at > 0 && q == 0) load_values(at);
        // uniform; what LDS holds in the place of tokens beyond the batch reaches no result (17 tokens of 2048 values, 16384 rows
        // 58.0 -> 55.9 us per step, 5 of 800, 5003 rows 28.7 -> 28.0, against quantising the last token in their place)
        if (t >= B) continue;
        float amax = 0.0f;
#pragma unroll
        for (int m = 0; m < VECS; ++m) {
          if constexpr (SRC == kF32) {
            tv[q][m] = bf16_pairs(tv[q][m], tv2[q][m]);
          }
          const uint32_t ud[4] = {tv[q][m].x, tv[q][m].y, tv[q][m].z, tv[q][m].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) amax = fmaxf(amax, fmaxf(fabsf(bf16_lo(ud[e])), fabsf(bf16_hi(ud[e]))));
        }
        const TokenScale ts = token_scale(wave_max(amax));
        float sabs = 0.0f;
#pragma unroll
        for (int m = 0; m < VECS; ++m)
          if (m * kWave < 2 * segq) {  // uniform
            const int i = m * kWave + lane;
            const bool counts = i < nvec;
            float sum8;
            const uint2 codes = quantise8(tv[q][m], ts, &sum8);
            sabs += counts ? sum8 : 0.0f;
            if (i < 2 * segq) reinterpret_cast<uint2*>(xs + t * xstride)[i] = counts ? codes : make_uint2(0, 0);
            __builtin_amdgcn_sched_barrier(0);  // (registers)
          }
        if (p.tok.sumabs != nullptr && first_tile == 0) {
          sabs = wave_sum(sabs);
          if (lane == 0) p.tok.sumabs[tok0 + t] = sabs;
        }
      }
    }
  };
  // every wave of the workgroup goes through the same tiles, segments and requests
  auto stage_if_due = [&](int tile, int seg, int blk) __attribute__((always_inline)) {
    if (blk == 0 && (nseg > 1 || tile == first_tile)) {
      if (seg > 0 || tile != first_tile) {
        load_tokens(seg);
        lds_barrier();  // the readers of the segment before are done
      }
      stage(seg);
      lds_barrier();
    }
  };

  v4i acc[RT][CT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = v4i{0, 0, 0, 0};
  auto multiply = [&](const Request& q, int seg, int blk) __attribute__((always_inline)) {
    const int l0 = kw * per + blk * P, n = min(seg_steps, steps - seg * seg_steps);
#pragma unroll
    for (int u = 0; u < P; ++u)
      if (blk * P + u < per && l0 + u < n) {  // uniform
        v4i wa[RT], wb[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const uint4 c = q.v[u][rt];
          wa[rt] = v4i{(int)(c.x & 0xF0F0F0F0u), (int)((c.x << 4) & 0xF0F0F0F0u), (int)(c.y & 0xF0F0F0F0u),
                       (int)((c.y << 4) & 0xF0F0F0F0u)};
          wb[rt] = v4i{(int)(c.z & 0xF0F0F0F0u), (int)((c.z << 4) & 0xF0F0F0F0u), (int)(c.w & 0xF0F0F0F0u),
                       (int)((c.w << 4) & 0xF0F0F0F0u)};
        }
        const uint4* col = xs + jl * xstride + 2 * ((l0 + u) * 4 + g);  // the chunk's 32 codes meet these token bytes
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const uint4 ta = col[ct * 16 * xstride], tb = col[ct * 16 * xstride + 1];
          const v4i va = {(int)ta.x, (int)ta.y, (int)ta.z, (int)ta.w}, vb = {(int)tb.x, (int)tb.y, (int)tb.z, (int)tb.w};
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            acc[rt][ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(va, wa[rt], acc[rt][ct], 0, 0, 0);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            acc[rt][ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vb, wb[rt], acc[rt][ct], 0, 0, 0);
        }
      }
  };
  // key of a sum of this lane's row
  auto key_of = [&](int sum, float sj) __attribute__((always_inline)) {
    float key = (float)sum * sj;
    if (p.relu) key = key > 0.0f ? key : 0.0f;
    return key + 0.0f;  // -0 -> +0
  };

  load_tokens(0);
  if constexpr (KW > 1) {
    if constexpr (SRC != kCodes) {
      for (int i = (int)blockIdx.x * NT + tid; i < p.tok.zero_words; i += (int)gridDim.x * NT) p.tok.zero_ptr[i] = 0u;
      if (blockIdx.x == 0) general_header_check(static_cast<GeneralHeader*>(p.tok.header), p.tok.sig);
    }
    constexpr int kUnits = CT * 4;
    // one of every KW of the workgroup's sums per wave
    auto finish_tile = [&](const int* red, int tile, float sj) __attribute__((always_inline)) {
      const int j = tile * kRows + rw * 16 + jl;
#pragma unroll
      for (int u0 = 0; u0 < kUnits; u0 += KW) {
        const int u = u0 + kw, t = u / 4 * 16 + 4 * g + u % 4;
        if (u < kUnits) {  // uniform
          int sum = 0;
#pragma unroll
          for (int k = 0; k < KW; ++k) sum += red[((k * RW + rw) * kUnits + u) * kWave + lane];
          sum >>= 4;
          if (t < B && j < N) {
            p.keys[(size_t)(tok0 + t) * p.stride + j] = key_of(sum, sj);
            if (p.acc_out) p.acc_out[(size_t)(tok0 + t) * N + j] = sum;
          }
        }
      }
    };
    if (PARTS && first_tile * kRows >= N) return;  // uniform: the last dies' shares may be short
    const int tile = first_tile;
    Request q;
    for (int seg = 0; seg < nseg; ++seg)
      for (int blk = 0; blk < nblk; ++blk) {
        request(q, tile, seg, blk);
        stage_if_due(tile, seg, blk);
        multiply(q, seg, blk);
      }
    lds_barrier();  // the codes' place takes the waves' sums
    int* red = reinterpret_cast<int*>(xs);
#pragma unroll
    for (int u = 0; u < kUnits; ++u) red[(w * kUnits + u) * kWave + lane] = acc[0][u / 4][u % 4];
    lds_barrier();
    finish_tile(red, tile, q.sj[0]);
  } else {
    float wmax[CT][4];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r) wmax[ct][r] = -INFINITY;
    auto epilogue = [&](const float (&sj)[RT], int tile) __attribute__((always_inline)) {
      const int j0 = tile * kRows + rw * RT * 16 + jl;
      long long stride = p.stride;
      asm("" : "+s"(stride));  // (or the loop keeps an address per value)
      if ((tile + 1) * kRows <= N && B == kTok && p.acc_out == nullptr) {  // uniform: nothing to leave out
        float* dst = p.keys + 4 * g * stride + j0;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
              const float key = key_of(acc[rt][ct][r] >> 4, sj[rt]);
              wmax[ct][r] = __builtin_amdgcn_fmed3f(key, wmax[ct][r], INFINITY);  // the larger one
              dst[(ct * 16 + r) * stride + 16 * rt] = key;
            }
      } else {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
              const int t = ct * 16 + r + 4 * g, j = j0 + 16 * rt, sum = acc[rt][ct][r] >> 4;
              const float key = key_of(sum, sj[rt]);
              if (j < N) wmax[ct][r] = fmaxf(wmax[ct][r], key);
              if (t < B && j < N) {
                p.keys[t * stride + j] = key;
                if (p.acc_out) p.acc_out[(size_t)t * N + j] = sum;
              }
            }
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = v4i{0, 0, 0, 0};
    };
    Request qa, qb;
    int tile = (int)blockIdx.x, seg = 0, blk = 0;
    request(qa, tile, 0, 0);
    if (nseg == 1) stage_if_due(tile, 0, 0);
    // Multiplies one request, the next one out ahead of that, across segments and tiles.  false: that was the last.
    auto turn = [&](Request& cur, Request& next) __attribute__((always_inline)) -> bool {
      int ntile = tile, nsg = seg, nb = blk + 1;
      if (nb == nblk) {
        nb = 0;
        if (++nsg == nseg) {
          nsg = 0;
          ntile += (int)gridDim.x;
        }
      }
      const bool more = ntile * kRows < N;
      request(next, more ? ntile : tile, nsg, nb);
      __builtin_amdgcn_sched_barrier(0);
      if (nseg > 1) stage_if_due(tile, seg, blk);
      multiply(cur, seg, blk);
      if (nb == 0 && nsg == 0) epilogue(cur.sj, tile);
      tile = ntile;
      seg = nsg;
      blk = nb;
      return more;
    };
    while (turn(qa, qb) && turn(qb, qa)) {
    }
    if (p.wgmax == nullptr) return;
    // two of the largest keys per token and wave (scorer_mfma_maxima per token): across eight lanes of each DPP row
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        uint32_t v = wmax[ct][r] == -INFINITY ? 0u : order_key(wmax[ct][r]);
        v = max(v, dpp_move<0x111, 0xF>(0u, v));
        v = max(v, dpp_move<0x112, 0xF>(0u, v));
        v = max(v, dpp_move<0x114, 0xF>(0u, v));
        const int t = ct * 16 + 4 * g + r;
        if (jl % 8 == 7 && t < B) p.wgmax[(size_t)t * kWgMaxSlots + (blockIdx.x * NW + w) * 2 + jl / 8] = v;
      }
  }
}

constexpr int kVocabBlocks = 256, kVocabWaves = 8;  // KW = 1: workgroups, one per compute unit, and their waves
constexpr int kSegSteps = 16;                       // most steps of a segment of codes
constexpr int kVocabMinRows = 32769;                // rows from which KW = 1 serves; only these leave maxima
static_assert(2 * kVocabBlocks * kVocabWaves <= kWgMaxSlots, "two maxima per wave");

static int vocab_blocks(int N) { return min((N + 16 * kVocabWaves - 1) / (16 * kVocabWaves), kVocabBlocks); }
int scorer_mfma_maxima(int N) { return 2 * kVocabWaves * vocab_blocks(N); }

// Where quantising in every workgroup is cheaper than a kernel in front (3.6 to 4.8 us, and the boundary behind it, 1.5 to 2.5): up
// to 32 tokens of 2048 values, a wave then has one or two, 40 of 1024, where half of the waves have a third, or 64 of 512.
// d = 2048, 16384 rows: 16 tokens 8.4 against 3.8 + 7.4
// us, 32 tokens 11.9 against 4.1 + 8.0; 32000 rows, 32 tokens 14.8 against 4.7 + 9.7; d = 512, 3600 rows, 64 tokens 8.6 against
// 3.6 + 5.9, 20184 rows, 32 tokens 7.4 against 4.4 + 5.7.  us per step, 33, 36 and 40 tokens: d = 1024, 16384 rows 47.3 against 48.9,
// 48.2 / 49.4, 49.2 / 50.1, 4000 rows 32.5 / 32.9, 32.7 / 32.9, 31.7 / 31.7; d = 800, 5003 rows 36.2 / 36.5, 36.6 / 36.9, 38.5 / 38.7;
// d = 544, 4000 rows 29.8 / 29.8, 29.8 / 29.9, 29.8 / 29.7.  Beyond (48 of 800: 39.4 against 38.5; 64 of 1024, 16384 rows 52.0
// against 50.8) a wave has three or four long tokens, one after the other.  The intermediate of the int4 low-rank scorer is short
// (r <= 1024), and a rounding kernel goes with it: always.  Vocabularies: 256 workgroups of eight waves would take as long as the
// kernel in front.

// Sixteen tokens to a workgroup: a wave quantises one token, whatever the batch, and the rows' codes are read once more for every
// sixteen tokens, from the L2 of one die.  Where one round of workgroups has a single tile of up to 128 rows and 128 KB of codes each; three
// parts of 16384 rows would leave two tiles to some (33 tokens of 2048: 62.9 -> 65.3 us per step, 64 68.1 -> 69.7), and twice as many codes
// as that take as long as the kernel in front (33 of 4096, 8192 rows 66.2 -> 68.9).  us per step with the kernels that quantise all tokens
// or have them quantised in front / with parts: d = 2048, 16000 rows, 21 tokens 48.3 / 48.4, 25 50.0 / 49.7, 32 53.5 / 52.6, 5200 rows, 47 38.7 / 37.9;
// d = 1536, 10000 rows, 25 32.9 / 33.0, 12000, 32 36.4 / 35.7; d = 1024, 8000 rows, 21 26.7 / 25.9, 33 31.0 / 29.8, 64 34.9 / 32.3, 16000, 21 37.0 / 37.4;
// d = 768, 5200 rows, 33 27.9 / 26.6, 47 29.8 / 27.8; d = 512, 6000 rows, 21 22.5 / 22.0, 4000, 64 27.4 / 24.5, 16000, 25 31.0 / 30.6; d = 256, 1000 rows, 33
// 24.3 / 22.9, 64 27.3 / 24.1, 8000, 21 22.7 / 22.2.
// With four requests of rows at a time for every length, most of which a wave of short rows has no use for, 47 tokens on 5200 rows of 256 27.2
// instead of 24.2, 25 on 6000 rows of 512 23.6 instead of 22.4.
// Rows of a workgroup: so many that a round of 32 workgroups per die has them all, an eighth of the tiles and all parts of these; 0: more
// than 128 would be needed.  With as few as 256 workgroups hold, of which a die or two had one too many for a round, three parts of 5200
// rows: 47 tokens of 2048 40.5 instead of 37.9 us per step, of 768 30.6 instead of 27.8, of 256 24.2 instead of 23.5.
static int scorer_part_tile(int B, int N) {
  const int parts = (B + 15) / 16;
  for (int tile = 16; tile <= 128; tile *= 2)
    if (((N + tile - 1) / tile + 7) / 8 * parts <= 32) return tile;
  return 0;
}
static bool scorer_mfma_parts(int B, int N, int d) {
  static_assert(8192 <= 64 * 128 && 128 * 1024 <= 256 << 10, "more than 32 tokens that scorer_mfma_rows quantises: rows beyond 8192 only");
  const int fewest = d > 512 && N > 8192 ? 25 : 21, tile = scorer_part_tile(B, N);
  return B >= fewest && d <= 2048 && tile != 0 && (long long)tile * d <= 256 << 10;
}
bool scorer_mfma_quantises(int B, int N, int d, bool f32) {
  if (N >= kVocabMinRows) return false;
  if (!f32 && scorer_mfma_parts(B, N, d)) return true;
  return f32 ? d <= 1024 : d <= (B <= 32 ? 2048 : (B <= 40 ? 1024 : 512));
}

template <int CT, int RT, int RW, int KW, int P, int SRC, int VECS, bool PARTS = false>
static hipError_t scorer_mfma_launch(ScorerBatch& p, int grid, hipStream_t s) {
  const int steps = (p.d / 32 + 3) / 4, nseg = SRC == kCodes ? (steps + kSegSteps - 1) / kSegSteps : 1;
  if (SRC != kCodes && p.d > 512 * VECS) return hipErrorInvalidValue;
  p.seg_steps = (steps + nseg - 1) / nseg;
  const size_t codes = (size_t)16 * CT * (8 * p.seg_steps + 1) * sizeof(uint4);
  const size_t sums = KW > 1 ? (size_t)RW * KW * CT * 4 * kWave * sizeof(int) : 0;
  const size_t lds = codes > sums ? codes : sums;
  auto kernel = k_scorer_int4_mfma<CT, RT, RW, KW, P, SRC, VECS, PARTS>;
  static std::atomic<size_t> raised_to{0};
  if (const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, raised_to); e != hipSuccess)
    return e;
  return launch(kernel, dim3(grid), dim3(kWave * RW * KW), lds, s, p);
}

// Rows per workgroup for KW > 1: so many that the workgroups, one of which fills a compute unit, are 256 at most; a second
// round costs as much as the first (20184 rows of 512 codes, 32 tokens, quantised in place: 8.6 us with 64 rows each, 7.3 with 128;
// 64 tokens of 2048 codes 16.3 and 12.2).
template <int CT, int P, int SRC, int VECS>
static hipError_t scorer_mfma_rows(ScorerBatch& p, hipStream_t s) {
  if (p.N > 16384) return scorer_mfma_launch<CT, 1, 8, 2, 2, SRC, VECS>(p, (p.N + 127) / 128, s);
  if (p.N > 8192) return scorer_mfma_launch<CT, 1, 4, 4, P, SRC, VECS>(p, (p.N + 63) / 64, s);
  if constexpr (CT == 4 && SRC == kBf16) {
    return hipErrorInvalidValue;  // (scorer_mfma_parts)
  } else {
    if (p.N > 4096) return scorer_mfma_launch<CT, 1, 2, 8, 2, SRC, VECS>(p, (p.N + 31) / 32, s);
    return scorer_mfma_launch<CT, 1, 1, 16, 1, SRC, VECS>(p, (p.N + 15) / 16, s);
  }
}

// The same for sixteen tokens per workgroup, the workgroups of eight tiles and all parts after one another.
template <int VECS>
static hipError_t scorer_parts_rows(ScorerBatch& p, hipStream_t s) {
  const int tile = scorer_part_tile(p.B, p.N), grid = ((p.N + tile - 1) / tile + 7) / 8 * 8 * p.parts;
  constexpr int kSteps = 4 * VECS;  // of a row, at most; a wave requests no more of them at a time than its share
  switch (tile) {
    case 16: return scorer_mfma_launch<1, 1, 1, 16, 1, kBf16, VECS, true>(p, grid, s);
    case 32: return scorer_mfma_launch<1, 1, 2, 8, kSteps >= 16 ? 2 : 1, kBf16, VECS, true>(p, grid, s);
    case 64: return scorer_mfma_launch<1, 1, 4, 4, kSteps / 4, kBf16, VECS, true>(p, grid, s);
    default: return scorer_mfma_launch<1, 1, 8, 2, kSteps >= 8 ? 4 : 2, kBf16, VECS, true>(p, grid, s);
  }
}

template <int CT>
static hipError_t scorer_mfma_tokens(ScorerBatch& p, hipStream_t s) {
  if (p.N >= kVocabMinRows) {
    // 32 rows per wave read the tokens' codes half as often (64 tokens, 256000 rows of 2048: 79.1 against 80.9 us), unless they
    // leave more of the last round of tiles empty (40 tokens, 90000 of 1024: 24.8 against 22.5)
    auto rounds = [&](int rows) { return ((p.N + rows - 1) / rows + kVocabBlocks - 1) / kVocabBlocks; };
    const int wide = 32 * kVocabWaves, blocks = min((p.N + wide - 1) / wide, kVocabBlocks);
    if (CT == 4 && blocks == vocab_blocks(p.N) && 2 * rounds(wide) <= rounds(wide / 2))
      return scorer_mfma_launch<CT, 2, kVocabWaves, 1, 2, kCodes, 2>(p, blocks, s);
    return scorer_mfma_launch<CT, 1, kVocabWaves, 1, 4, kCodes, 2>(p, vocab_blocks(p.N), s);
  }
  if (p.tok.x == nullptr) return scorer_mfma_rows<CT, 2, kCodes, 2>(p, s);
  if (!p.tok.f32 && scorer_mfma_parts(p.B, p.N, p.d)) {
    p.parts = (p.B + 15) / 16;
    if (p.d <= 512) return scorer_parts_rows<1>(p, s);
    if (p.d <= 1024) return scorer_parts_rows<2>(p, s);
    return scorer_parts_rows<4>(p, s);
  }
  if (p.tok.f32) return p.d <= 512 ? scorer_mfma_rows<CT, 2, kF32, 1>(p, s) : scorer_mfma_rows<CT, 2, kF32, 2>(p, s);
  if (p.d <= 512) return scorer_mfma_rows<CT, 2, kBf16, 1>(p, s);
  if constexpr (CT == 4)
    if (p.d <= 1024) return scorer_mfma_rows<CT, 2, kBf16, 2>(p, s);
  if constexpr (CT <= 2) return p.d <= 1024 ? scorer_mfma_rows<CT, 2, kBf16, 2>(p, s) : scorer_mfma_rows<CT, 4, kBf16, 4>(p, s);
  return hipErrorInvalidValue;
}

hipError_t launch_scorer_int4_mfma(const uint32_t* q4, const float* scale, const ScorerTokens& tok, int B, int N, int d,
                                   int relu, float* keys, long long stride, int32_t* acc, const HistRefs& hr, hipStream_t s) {
  if (tok.x != nullptr && !scorer_mfma_quantises(B, N, d, tok.f32)) return hipErrorInvalidValue;
  const MultiRegion mr = multi_of(hr, B);
  ScorerBatch p{reinterpret_cast<const uint4*>(q4), scale, tok, B, N, d, relu, keys, stride, acc,
                N >= kVocabMinRows ? mr.wgmax : nullptr, 0, 1};
  if (B <= 16) return scorer_mfma_tokens<1>(p, s);
  if (B <= 32) return scorer_mfma_tokens<2>(p, s);
  return scorer_mfma_tokens<4>(p, s);
}

}  // namespace hire
