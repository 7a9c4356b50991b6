// Building blocks of kernels that take a few tokens at a time (ffn_fast_tokens.hip, ffn_shard.hip): int8 codes of a token,
// and the exact pre-activations of rows for all tokens of a workgroup of sixteen waves.
#pragma once

#include "select.h"

namespace hire {

constexpr int kRowsThreads = 1024;
constexpr int kRowsWaves = kRowsThreads / kWave;
constexpr int kMostRows = 96;  // rows of one call of rows_by_tokens

// Int8 codes of a token: rint(x / sx), sx = amax / 127, the quotient correctly rounded.  With the correctly rounded
// reciprocal of a divisor whose significand is not all ones, one residual corrects the product (Markstein, IBM J. Res.
// Dev. 34, 1990); the division itself where that does not apply or the residual could underflow.
struct TokenScale {
  float sx, rs;
  bool plain;
};
__device__ __forceinline__ TokenScale token_scale(float amax) {
  TokenScale t;
  t.sx = __fdiv_rn(amax, 127.0f);
  if (amax == 0.0f) t.sx = 1.0f;
  t.rs = __fdiv_rn(1.0f, t.sx);
  t.plain = t.sx > 0x1p-100f && t.sx < 0x1p100f && (__float_as_uint(t.sx) & 0x7FFFFFu) != 0x7FFFFFu;
  return t;
}
// Eight values; *sum8: the sum of the codes' absolute values.  Adding 1.5 2^23 rounds to whole numbers, half to even, and leaves
// them in the lowest bits in two's complement; bytes are gathered and summed four at a time.  With rintf, a conversion and an
// addition per value instead, us per step with that / this at the ~1B shape: 16 tokens 49.3 / 49.1, 20 54.6 / 54.2, the int4 low-rank scorer
// with 16 51.3 / 51.0; four tokens 38.15 / 38.05.
__device__ __forceinline__ uint2 quantise8(const uint4& v, const TokenScale& t, float* sum8) {
  const uint32_t ud[4] = {v.x, v.y, v.z, v.w};
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float f = (e & 1) != 0 ? bf16_hi(ud[e / 2]) : bf16_lo(ud[e / 2]), y = f * t.rs;
    r[e] = fmaf(fmaf(-y, t.sx, f), t.rs, y);
  }
  if (__ballot(!t.plain) != 0ull) {
    asm volatile("");  // keeps the compiler from dividing always and selecting
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = __fdiv_rn((e & 1) != 0 ? bf16_hi(ud[e / 2]) : bf16_lo(ud[e / 2]), t.sx);
  }
  uint32_t packed[2], sum = 0u;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint32_t b[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = __float_as_uint(fminf(fmaxf(r[4 * h + e], -127.0f), 127.0f) + 0x1.8p23f);
    packed[h] = __builtin_amdgcn_perm(b[1], b[0], 0x0C0C0400u) | __builtin_amdgcn_perm(b[3], b[2], 0x04000C0Cu);
    sum = __builtin_amdgcn_sad_u8(packed[h] ^ 0x80808080u, 0x80808080u, sum);
  }
  *sum8 = (float)sum;
  return make_uint2(packed[0], packed[1]);
}

// Adds to acc what four rows of packed int4 codes (lane l: sixteen bytes of row l % 4) have in common with four tokens
// (lane l: the same 32 columns of token l % 4 as int8), blocks of columns l / 4 separately: acc[r] is sixteen times the
// sum of row r with token l % 4.
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void int4_rows_by_tokens(const uint4& wv, const uint4& ta, const uint4& tb, v4i& acc) {
  const uint32_t wd[4] = {wv.x, wv.y, wv.z, wv.w};
  const int xd[8] = {(int)ta.x, (int)ta.y, (int)ta.z, (int)ta.w, (int)tb.x, (int)tb.y, (int)tb.z, (int)tb.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    acc = __builtin_amdgcn_mfma_i32_4x4x4i8((int)(wd[q] & 0xF0F0F0F0u), xd[2 * q], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_i32_4x4x4i8((int)((wd[q] << 4) & 0xF0F0F0F0u), xd[2 * q + 1], acc, 0, 0, 0);
  }
}

// out(r, t, relu(<row r, x_t>)) for r < cnt <= kMostRows rows and all tokens, by the workgroup.  v_mfma_f64_4x4x4: four
// rows and four tokens at a time, in lane l row l % 4 of A, token l % 4 of B and column chunk l / 4 of both, element by
// element of the sixteen-byte chunks (the order of the columns does not matter to a dot product).  A wave has SL slices
// of sixteen chunks of the columns, whose token values stay in its registers as fp64, and runs over its share of the
// rows, four at a time, eight loads in flight; nothing goes through LDS but the waves' sums.  SL as large as the
// registers allow: a wave then reads up to a KB of a row (9.9 us for the rows of four tokens at the ~1B shape with 256
// bytes, 8.6 with a KB, 7.8 with whole rows).  red: [parts of the columns][groups of four rows][TT / 4][16] sums, added
// in a fixed order.
// The waves' sums; rows_out, behind a barrier, adds them up.
template <int TT, int SL = 16 / TT, int kDepth = 8 / SL, typename RowOf>
__device__ __forceinline__ void rows_sums(int cnt, RowOf&& row_of, const uint4* __restrict__ x, int B, int nvec, double* red) {
  constexpr int kTok4 = TT / 4, kMaxGroups = kMostRows / 4;
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int nsl = (nvec + 15) / 16, ng = (cnt + 3) / 4;
  int ps = 1;  // waves side by side over the columns: sixteen parts are enough (TT d <= 32768)
  while (ps * SL < nsl) ps <<= 1;
  const int s0 = (w & (ps - 1)) * SL, rp = w / ps, step = kRowsWaves / ps;
  uint4 ring[kDepth][SL];
  // No load sits behind a branch, or the wait for one group's rows would become one for all that is under way: in the place of
  // groups past the end a wave asks for the first token again, which is in the caches.
  auto load = [&](int q, uint4 (&v)[SL]) __attribute__((always_inline)) {
    const uint4* row = row_of(min(q * 4 + (lane & 3), cnt - 1));
    if (q >= ng) row = x;  // uniform
#pragma unroll
    for (int j = 0; j < SL; ++j) v[j] = load_streaming(row + min((s0 + j) * 16 + (lane >> 2), nvec - 1));
    __builtin_amdgcn_sched_barrier(0);
  };
  uint4 xr[SL][kTok4];  // asked for ahead of the rows: loads return in order
#pragma unroll
  for (int j = 0; j < SL; ++j)
#pragma unroll
    for (int f = 0; f < kTok4; ++f)
      xr[j][f] = x[(size_t)min(f * 4 + (lane & 3), B - 1) * nvec + min((s0 + j) * 16 + (lane >> 2), nvec - 1)];
  __builtin_amdgcn_sched_barrier(0);
  if (s0 < nsl && rp < ng) {  // uniform over the wave
#pragma unroll
    for (int i = 0; i < kDepth; ++i) load(rp + i * step, ring[i]);
    double xd[SL][kTok4][8];
    uint32_t keep[SL];  // past the row's end: zeros
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      const int c = (s0 + j) * 16 + (lane >> 2);
      keep[j] = c < nvec ? 0xFFFFFFFFu : 0u;
#pragma unroll
      for (int f = 0; f < kTok4; ++f) {
        const uint4 u = xr[j][f];
        const uint32_t ud[4] = {u.x & keep[j], u.y & keep[j], u.z & keep[j], u.w & keep[j]};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          xd[j][f][2 * q] = (double)bf16_lo(ud[q]);
          xd[j][f][2 * q + 1] = (double)bf16_hi(ud[q]);
        }
      }
    }
    auto multiply = [&](int q, const uint4 (&v)[SL]) __attribute__((always_inline)) {
      double acc[kTok4];
#pragma unroll
      for (int f = 0; f < kTok4; ++f) acc[f] = 0.0;
#pragma unroll
      for (int j = 0; j < SL; ++j) {
        const uint4 u = v[j];
        const uint32_t wd[4] = {u.x & keep[j], u.y & keep[j], u.z & keep[j], u.w & keep[j]};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double wf = (double)((e & 1) != 0 ? bf16_hi(wd[e / 2]) : bf16_lo(wd[e / 2]));
#pragma unroll
          for (int f = 0; f < kTok4; ++f) acc[f] = __builtin_amdgcn_mfma_f64_4x4x4f64(wf, xd[j][f][e], acc[f], 0, 0, 0);
        }
      }
#pragma unroll
      for (int f = 0; f < kTok4; ++f) {  // row l / 16, token l % 4: the four blocks of columns
        double t = acc[f] + dpp_move<0x124, 0xF>(0.0, acc[f]);
        t += dpp_move<0x128, 0xF>(0.0, t);
        if ((lane & 12) == 0)
          red[(((size_t)(w & (ps - 1)) * kMaxGroups + q) * kTok4 + f) * 16 + (lane >> 4) * 4 + (lane & 3)] = t;
      }
    };
    int q0 = rp;
    for (; q0 + kDepth * step < ng; q0 += kDepth * step) {  // uniform
#pragma unroll
      for (int i = 0; i < kDepth; ++i) {
        multiply(q0 + i * step, ring[i]);  // (all groups of this trip are there)
        load(q0 + (kDepth + i) * step, ring[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < kDepth; ++i)
      if (q0 + i * step < ng) multiply(q0 + i * step, ring[i]);  // uniform
  }
  HIRE_TS(16);
}
template <int TT, int SL = 16 / TT, typename Out>
__device__ __forceinline__ void rows_out(int cnt, int B, int nvec, const double* red, Out&& out) {
  constexpr int kTok4 = TT / 4, kMaxGroups = kMostRows / 4;
  const int tid = (int)threadIdx.x, nsl = (nvec + 15) / 16, ng = (cnt + 3) / 4;
  for (int o = tid; o < ng * kTok4 * 16; o += kRowsThreads) {
    const int r = o / (kTok4 * 16) * 4 + (o >> 2 & 3), t = o / 16 % kTok4 * 4 + (o & 3);
    double v = 0.0;
    for (int j = 0; j * SL < nsl; ++j) v += red[(size_t)j * kMaxGroups * kTok4 * 16 + o];
    if (r < cnt && t < B) out(r, t, v > 0.0 ? v : 0.0);  // ReLU, and -0 -> +0
  }
}

template <int TT, int SL = 16 / TT, int kDepth = 8 / SL, typename RowOf, typename Out>
__device__ __forceinline__ void rows_by_tokens(int cnt, RowOf&& row_of, const uint4* __restrict__ x, int B, int nvec,
                                               double* red, Out&& out) {
  rows_sums<TT, SL, kDepth>(cnt, row_of, x, B, nvec, red);
  lds_barrier();
  HIRE_TS(17);
  rows_out<TT, SL>(cnt, B, nvec, red, out);
}

}  // namespace hire
