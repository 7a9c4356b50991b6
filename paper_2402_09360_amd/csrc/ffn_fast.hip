// Batch-1 HiRE-FFN step in three kernels (arXiv 2402.09360, Algorithm 1 + eq. (4)),
// laid out so that no stage runs on a single workgroup:
//
//   k_fast_score   int8 token quantisation (redone by every workgroup, 4 KB), int4 scorer, keys to memory and
//                  a fine histogram of the keys (integer atomics; a bin is 2^14 consecutive fp32 bit patterns,
//                  i.e. exponent and nine mantissa bits, so that few keys share a counter)
//   k_fast_gather  every workgroup walks the histogram from the top to the bin of the k'-th key and computes the exact
//                  pre-activations of those of its own 64 units that belong to the shortlist; histogram of h the
//                  same way
//   k_fast_w2      the same selection on h (exact top-k), then sum_j h_j v_j over all selected rows for the
//                  workgroup's 32 columns, reduced inside the workgroup in a fixed order: y itself, no
//                  kernel follows.  Clears the key histogram (the next step's scorer kernel clears the h
//                  histogram, which nobody reads in between).
//
// A kernel boundary is the cheapest device-wide synchronisation on this machine (a spinning grid barrier
// costs several microseconds per round with 256 workgroups), hence separate kernels instead of one
// persistent kernel.  Selection work is duplicated in every workgroup instead of being serialised in one.
// What the selecting heads cost is their chain of dependent memory round trips (~1 us each) and their serial
// sections: a SIMD issues one vector instruction every four cycles, so with sixteen waves on a CU each wave
// gets one every ~16 cycles and a section of a hundred instructions takes 0.7 us.  Hence
//
//  * both run sixteen waves per workgroup: fewer were measured slower for the same work (the serial sections of a
//    lone wave run at 10 to 15 cycles per instruction);
//  * The histograms are windows of 8192 bins at FIXED addresses: slot s counts the keys of bin anchor - s.
//    The anchors are rigorous upper bounds of the keys and of the activations that the scorer kernel derives
//    from the quantised token alone (sum |xq|) and the layer's largest row scale (kept behind the packed int4
//    codes), so every workgroup of every kernel knows them without waiting for any maximum, and a consumer
//    requests its histogram window together with its keys as its very first instructions.
//  * Key arrays are zero-padded to whole 16-byte vectors and lanes beyond the end read a vector of zeros, so
//    the passes over the register-resident keys need no validity tests: every comparison is against a
//    positive threshold.
//
// ReLU makes every key and every h non-negative, so their IEEE bit patterns already order like the numbers
// and are used as integer keys directly.
//
// The key histogram must be all zero when a step starts.  The second-layer kernel of every step leaves it so
// and stamps a cookie into the workspace, which the next step's scorer kernel takes away again; on a workspace without
// the cookie (first use, arbitrary contents, a step that ended half-way) the first selection of one step takes a slower
// histogram-free route, and so does a selection whose keys are not all at or below their anchor (ffn_fast.h).  The h
// histogram is cleared by the scorer kernel of the step that uses it.  No kernel waits for, or counts, the workgroups of
// another.
#include "ffn_fast.h"

namespace hire {

// ---------------------------------------------------------------------------------------------------
// Kernel 1: scorer.
constexpr int kRPW = 4;     // rows per wave and pass
constexpr int kST = 1024;   // threads per scorer workgroup: one workgroup per CU, the token is quantised once per CU
constexpr int kSW = kST / kWave;

// Code of a value, scale sx, by the division itself: a thread has one word of codes to form.  (quantise8 of rows_mfma.h, whose
// eight values per thread leave most waves idle, is slower in the one-token kernels: 18 steps at the ~1B shape 435 us against 430,
// four steps of the int4 low-rank scorer there 102.5 against 101.6.)
__device__ __forceinline__ int code_of(float f, float sx) {
  return (int)fminf(fmaxf(rintf(__fdiv_rn(f, sx)), -127.0f), 127.0f);
}

// LRQ (the int4 low-rank scorer's second product): the "token" is the fp32 intermediate t of the first product,
// rounded to bf16 here as it is loaded, the rows are those of the int4 copy of Z2, and the activations' bound comes
// from the real token's norm and the layer's largest row norm (xn, xn_d, umax) instead of from the int4 codes.
template <bool LRQ>
__global__ __launch_bounds__(kST) void k_fast_score_int4(const uint4* __restrict__ q4, const float* __restrict__ scale,
                                                         const uint32_t* __restrict__ x, int N, int d,
                                                         float* __restrict__ keys, int32_t* __restrict__ acc_out,
                                                         FastRegion* __restrict__ fr,
                                                         unsigned long long* __restrict__ clocks,
                                                         float* __restrict__ gkeys, const uint4* __restrict__ xn,
                                                         int xn_d, const float* __restrict__ umax) {
  // gkeys != nullptr (group-sparse step, groups of eight adjacent units, eq. (6)): what is handed on and counted
  // in the histogram is the group activation gkeys[J] = sum_{l<8} |key[8J + l]| (fp32, unit order) instead of
  // the unit keys; a workgroup's 64 consecutive rows are eight whole groups.
  extern __shared__ uint32_t lds[];  // raw token, d/2 dwords of bf16 pairs; then d/4 dwords of int8 quads
  __shared__ float red[kSW];
  __shared__ int isum[kSW];
  __shared__ float unit_keys[kSW * kRPW];
  if (clocks && threadIdx.x == 0) clocks[2 * blockIdx.x] = wall_clock64();
  HIRE_TS(30);
  uint32_t* xraw = lds;
  uint32_t* xq = lds + d / 2;
  const int tid = (int)threadIdx.x, lane = lane_id(), w = wave_id();
  const int cpr = d / 32;
  const int total_waves = (int)gridDim.x * kSW;
  const int gw = (int)blockIdx.x * kSW + w;

  // token first (loads return in order, and the token is needed first), then the first rows' weights and
  // scales: all of these loads are in flight together
  const unsigned long long cookie = fr->cookie;  // (workgroup 0 takes it away)
  const float smax = __uint_as_float(q4[(size_t)N * cpr].x);  // largest row scale, kept behind the codes
  // the window of the activations, filled by the next kernel, starts from zero (its last reader was the step before)
  for (int i = (int)blockIdx.x * kST + tid; i < kWin; i += (int)gridDim.x * kST) fr->hist2[i] = 0u;
  const uint4* x4 = reinterpret_cast<const uint4*>(x);
  const int xvecs = d / 8;
  // eight token values as bf16 pairs: as they are, or (LRQ) two vectors of four floats rounded to nearest even
  auto token_vec = [&](int i) -> uint4 {
    if constexpr (!LRQ) {
      return x4[i];
    } else {
      return bf16_pairs(x4[2 * i], x4[2 * i + 1]);
    }
  };
  const uint4 xv0 = token_vec(min(tid, xvecs - 1));
  const int cl = min(lane, cpr - 1);
  uint4 pre[kRPW];
#pragma unroll
  for (int rr = 0; rr < kRPW; ++rr) pre[rr] = load_streaming(&q4[(size_t)min(gw * kRPW + rr, N - 1) * cpr + cl]);
  const float pre_scale = scale[min(gw * kRPW + (lane >> 4), N - 1)];
  float amax = 0.0f;
  for (int i = tid; i < xvecs; i += kST) {
    const uint4 u = i == tid ? xv0 : token_vec(i);
    reinterpret_cast<uint4*>(xraw)[i] = u;
    const uint32_t ud[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) amax = fmaxf(amax, fmaxf(fabsf(bf16_lo(ud[q])), fabsf(bf16_hi(ud[q]))));
  }
  amax = wave_max(amax);
  if (lane == 0) red[w] = amax;
  __syncthreads();
  HIRE_TS(31);
  amax = wave_max(lane < kSW ? red[lane] : 0.0f);
  float sx = __fdiv_rn(amax, 127.0f);
  if (amax == 0.0f) sx = 1.0f;
  int sabs = 0;  // this thread's share of sum |xq|
  for (int i = tid; i < d / 4; i += kST) {
    const uint32_t a = xraw[2 * i], b = xraw[2 * i + 1];
    const float f[4] = {bf16_lo(a), bf16_hi(a), bf16_lo(b), bf16_hi(b)};
    uint32_t packed = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = code_of(f[e], sx);
      sabs += abs(c);
      packed |= ((uint32_t)c & 0xFFu) << (8 * e);
    }
    xq[i] = packed;
  }
  sabs = wave_sum(sabs);
  if (lane == 0) isum[w] = sabs;
  __syncthreads();
  HIRE_TS(32);
  // Upper bounds that hold for every unit of the layer, from the token alone.  With codes |q| <= 7, |xq| <= 127:
  //   key_j = fl(fl(acc_j) s_j) <= fl(7 sum|xq| smax)                       (rounding is monotone; 7 sum|xq| < 2^24)
  //   <u_j, x> = s_j sx sum (q + dq)(xq + dx), |dq|, |dx| <= 1/2 (+ rounding of the two divisions)
  //           <= smax sx (7.5 sum|xq| + 3.75 d + ...), taken with a margin that also covers the fp32 arithmetic
  // The group activations of eq. (6) are sums of eight such terms.
  const int sumabs = wave_sum(lane < kSW ? isum[lane] : 0);
  const float group_factor = gkeys != nullptr ? 8.001f : 1.0f;
  const float bound1 = (float)(7 * sumabs) * smax * group_factor;
  float bound2 = smax * sx * (7.6f * (float)sumabs + 3.8f * (float)d + 1.0f) * 1.01f * group_factor;
  if constexpr (LRQ) {  // Cauchy-Schwarz: <u_j, x> <= |u_j| |x|, both rounded up by more than their error
    float xsq = 0.0f;
    for (int i = tid; i < xn_d / 8; i += kST) {
      const uint4 u = xn[i];
      const uint32_t ud[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float a = bf16_lo(ud[q]), b = bf16_hi(ud[q]);
        xsq = fmaf(a, a, xsq);
        xsq = fmaf(b, b, xsq);
      }
    }
    xsq = wave_sum(xsq);
    __syncthreads();  // red's readers above are done
    if (lane == 0) red[w] = xsq;
    __syncthreads();
    xsq = wave_sum(lane < kSW ? red[lane] : 0.0f);
    bound2 = sqrtf(xsq * (1.0f + (float)xn_d * 0x1p-22f)) * 1.0001f * umax[0] * 1.0001f * group_factor;
  }
  const uint32_t anchor1 = fine_bin(__float_as_uint(bound1)), anchor2 = fine_bin(__float_as_uint(bound2));
  if (blockIdx.x == 0 && tid == 0) {
    fr->anchor1 = anchor1;
    fr->anchor2 = anchor2;
    fr->beyond2 = 0u;
    take_cookie(fr, cookie);
  }
  {  // zero padding of the handed-on key array up to a whole 16-byte vector
    float* arr = gkeys != nullptr ? gkeys : keys;
    const int n = gkeys != nullptr ? N / 8 : N;
    if (blockIdx.x == 0 && tid < ((4 - (n & 3)) & 3)) arr[n + tid] = 0.0f;
  }
  auto count_key = [&](float key) { count_in_window<false>(__float_as_uint(key), anchor1, fr->hist1, &fr->beyond1); };

  const uint4* xq4 = reinterpret_cast<const uint4*>(xq);
  for (int g = gw; g * kRPW < N; g += total_waves) {
    const int j0 = g * kRPW;
    int acc[kRPW];
#pragma unroll
    for (int rr = 0; rr < kRPW; ++rr) acc[rr] = 0;
    for (int c = lane; c < cpr; c += kWave) {
      uint4 wv[kRPW];
      if (g == gw && c == lane) {
#pragma unroll
        for (int rr = 0; rr < kRPW; ++rr) wv[rr] = pre[rr];
      } else {
#pragma unroll
        for (int rr = 0; rr < kRPW; ++rr) wv[rr] = load_streaming(&q4[(size_t)min(j0 + rr, N - 1) * cpr + c]);
      }
      const uint4 xa = xq4[2 * c], xb = xq4[2 * c + 1];
      const int xd[8] = {(int)xa.x, (int)xa.y, (int)xa.z, (int)xa.w, (int)xb.x, (int)xb.y, (int)xb.z, (int)xb.w};
#pragma unroll
      for (int rr = 0; rr < kRPW; ++rr) {
        const uint32_t wd[4] = {wv[rr].x, wv[rr].y, wv[rr].z, wv[rr].w};
        int a = acc[rr];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          a = __builtin_amdgcn_sdot4((int)(wd[t] & 0xF0F0F0F0u), xd[2 * t], a, false);
          a = __builtin_amdgcn_sdot4((int)((wd[t] << 4) & 0xF0F0F0F0u), xd[2 * t + 1], a, false);
        }
        acc[rr] = a;
      }
    }
    HIRE_TS(33);
    // lanes 15, 31, 47, 63 take rows j0 + 0, 1, 2, 3
    const int s = wave_sum4(acc[0], acc[1], acc[2], acc[3]);
    const int j = j0 + (lane >> 4);
    if ((lane & 15) == 15 && j < N) {
      const int sum = s >> 4;  // every partial is a multiple of 16
      float key = (float)sum * (g == gw ? pre_scale : scale[j]);
      key = key > 0.0f ? key : 0.0f;  // ReLU, and -0 -> +0
      if (acc_out) acc_out[j] = sum;
      if (gkeys != nullptr) {
        unit_keys[w * kRPW + (lane >> 4)] = key;  // one pass per workgroup here (N <= 64 * gridDim.x)
      } else {
        keys[j] = key;
        count_key(key);
      }
    }
  }
  if (gkeys != nullptr) {
    __syncthreads();
    const int J = (int)blockIdx.x * (kSW * kRPW / 8) + tid;
    if (tid < kSW * kRPW / 8 && J * 8 < N) {
      float sum = 0.0f;
#pragma unroll
      for (int l = 0; l < 8; ++l) sum += fabsf(unit_keys[tid * 8 + l]);
      gkeys[J] = sum;
      count_key(sum);
    }
  }
  HIRE_TS(34);
  if (clocks) {
    __syncthreads();
    if (tid == 0) clocks[2 * blockIdx.x + 1] = wall_clock64();
  }
}

// ---------------------------------------------------------------------------------------------------
// Kernel 1 for the int4 low-rank scorer where both products fit one kernel: every workgroup quantises the token, forms all r
// sums of the first product itself - the codes of Z1 transposed, r d / 2 bytes, come from L2 - rounds them to bf16, quantises
// them, and scores its own 64 rows of Z2 with sixteen lanes per row.  Everything that does not depend on a result (the
// token, a wave's rows of Z1 up to d = 2048, its rows of Z2) is requested at the start.  With a kernel for the first product in
// front, and a wave's lanes on four rows of Z2 together, a step takes, us, that / this: d = 2048, 16384 units, r = 128 28.8 /
// 25.4, r = 256 28.6 / 28.5; d = 256, 4000 units, r = 64 21.3 / 17.4, r = 256 22.5 / 20.9; r = 512 (eight rows at a time,
// d = 1024, 8000 units) 23.5 / 26.6.
// ROWS: rows of Z1 per wave, all of them requested at once (r <= 16 ROWS).
constexpr int kLrqFusedRank = 256;         // largest r
constexpr int kLrqFusedBytes = 256 << 10;  // most bytes of Z1's codes

// sum of a chunk of 32 codes with its activations (two vectors of sixteen)
__device__ __forceinline__ int chunk_dot(const uint4& v, const uint4& xa, const uint4& xb, int a) {
  const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
  const int xd[8] = {(int)xa.x, (int)xa.y, (int)xa.z, (int)xa.w, (int)xb.x, (int)xb.y, (int)xb.z, (int)xb.w};
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    a = __builtin_amdgcn_sdot4((int)(wd[t] & 0xF0F0F0F0u), xd[2 * t], a, false);
    a = __builtin_amdgcn_sdot4((int)((wd[t] << 4) & 0xF0F0F0F0u), xd[2 * t + 1], a, false);
  }
  return a;
}

template <int ROWS>
__global__ __launch_bounds__(kST) void k_fast_score_lrq(const uint4* __restrict__ q1, const float* __restrict__ scale1,
                                                        const uint4* __restrict__ q2, const float* __restrict__ scale2,
                                                        const uint4* __restrict__ x, int N, int d, int r,
                                                        float* __restrict__ keys, FastRegion* __restrict__ fr,
                                                        unsigned long long* __restrict__ clocks,
                                                        const float* __restrict__ umax, float* __restrict__ gkeys) {
  extern __shared__ uint4 tok[];  // the token, d/8 vectors of bf16; then its codes, d/16
  __shared__ float red[kSW], sq[kSW], t_sh[kLrqFusedRank];
  __shared__ __align__(16) uint32_t tq[kLrqFusedRank / 4];  // the intermediate's codes
  __shared__ int isum[kSW];
  __shared__ float unit_keys[kSW * kRPW];  // groups, as in k_fast_score_int4
  if (clocks && threadIdx.x == 0) clocks[2 * blockIdx.x] = wall_clock64();
  HIRE_TS(30);
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int cpr1 = d / 32, cpr2 = r / 32, xvecs = d / 8;
  const int sub = lane & 15, per = (r + kSW - 1) / kSW, ja = w * per;  // rows of Z1 of this wave: [ja, min(ja + per, r))
  const unsigned long long cookie = fr->cookie;
  const float smax = __uint_as_float(q2[(size_t)N * cpr2].x), um = umax[0];
  for (int i = (int)blockIdx.x * kST + tid; i < kWin; i += (int)gridDim.x * kST) fr->hist2[i] = 0u;
  const uint4 xv = x[min(tid, xvecs - 1)];  // d <= 8192: one vector per thread
  uint4 z1[ROWS], z2;
  auto load_z1 = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < ROWS; ++i) z1[i] = q1[(size_t)min(ja + min(i, per - 1), r - 1) * cpr1 + c];
  };
  load_z1(min(lane, cpr1 - 1));
  float z1_scale[ROWS / 4];
#pragma unroll
  for (int q = 0; q < ROWS / 4; ++q) z1_scale[q] = scale1[min(ja + 4 * q + (lane >> 4), r - 1)];
  auto load_z2 = [&](int g) __attribute__((always_inline)) {
    z2 = load_streaming(&q2[(size_t)min(4 * g + (lane >> 4), N - 1) * cpr2 + min(sub, cpr2 - 1)]);
  };
  const int gw = (int)blockIdx.x * kSW + w, waves = (int)gridDim.x * kSW;
  load_z2(gw);
  float row_scale = scale2[min(4 * gw + (lane >> 4), N - 1)];
  {  // largest value, and the sum of squares of the token
    const uint32_t ud[4] = {xv.x, xv.y, xv.z, xv.w};
    float amax = 0.0f, xsq = 0.0f;
    if (tid < xvecs) {
      tok[tid] = xv;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float a = bf16_lo(ud[q]), b = bf16_hi(ud[q]);
        amax = fmaxf(amax, fmaxf(fabsf(a), fabsf(b)));
        xsq = fmaf(a, a, xsq);
        xsq = fmaf(b, b, xsq);
      }
    }
    amax = wave_max(amax);
    xsq = wave_sum(xsq);
    if (lane == 0) {
      red[w] = amax;
      sq[w] = xsq;
    }
  }
  lds_barrier();  // the codes stay under way
  HIRE_TS(31);
  uint32_t* xq = reinterpret_cast<uint32_t*>(tok + xvecs);
  {
    const float amax = wave_max(lane < kSW ? red[lane] : 0.0f), sx = amax == 0.0f ? 1.0f : __fdiv_rn(amax, 127.0f);
    const uint2* raw = reinterpret_cast<const uint2*>(tok);
    for (int i = tid; i < d / 4; i += kST) {
      const uint2 v = raw[i];
      xq[i] = ((uint32_t)code_of(bf16_lo(v.x), sx) & 0xFFu) | ((uint32_t)code_of(bf16_hi(v.x), sx) & 0xFFu) << 8 |
              ((uint32_t)code_of(bf16_lo(v.y), sx) & 0xFFu) << 16 | (uint32_t)code_of(bf16_hi(v.y), sx) << 24;
    }
  }
  lds_barrier();
  const uint4* xq4 = reinterpret_cast<const uint4*>(xq);
  {
    int acc[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) acc[i] = 0;
    for (int c0 = 0; c0 < cpr1; c0 += kWave) {  // uniform
      const int c = c0 + lane, cc = min(c, cpr1 - 1);
      if (c0 > 0) load_z1(cc);
      const uint4 xa = xq4[2 * cc], xb = xq4[2 * cc + 1];
      if (c < cpr1) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) acc[i] = chunk_dot(z1[i], xa, xb, acc[i]);
      }
    }
#pragma unroll
    for (int q = 0; q < ROWS / 4; ++q) {  // lanes 15, 31, 47, 63: rows 4 q + 0, 1, 2, 3
      const int sum = wave_sum4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]) >> 4;  // multiples of 16
      const int i = 4 * q + (lane >> 4);
      if (sub == 15 && i < per && ja + i < r) {
        const uint32_t u = __float_as_uint((float)sum * z1_scale[q] + 0.0f);  // -0 -> +0
        t_sh[ja + i] = __uint_as_float(f32_to_bf16_rne(u) << 16);
      }
    }
  }
  lds_barrier();
  HIRE_TS(32);
  {
    float tmax = 0.0f;
    for (int i = lane; i < r; i += kWave) tmax = fmaxf(tmax, fabsf(t_sh[i]));
    tmax = wave_max(tmax);
    const float st = tmax == 0.0f ? 1.0f : __fdiv_rn(tmax, 127.0f);
    int sabs = 0;
    if (w * kWave < r / 4) {  // uniform over the wave
      const int i = min(tid, r / 4 - 1);
      const float4 v = reinterpret_cast<const float4*>(t_sh)[i];
      const int c[4] = {code_of(v.x, st), code_of(v.y, st), code_of(v.z, st), code_of(v.w, st)};
      if (tid < r / 4) {
        tq[i] = ((uint32_t)c[0] & 0xFFu) | ((uint32_t)c[1] & 0xFFu) << 8 | ((uint32_t)c[2] & 0xFFu) << 16 | (uint32_t)c[3] << 24;
        sabs = abs(c[0]) + abs(c[1]) + abs(c[2]) + abs(c[3]);
      }
      sabs = wave_sum(sabs);
    }
    if (lane == 0) isum[w] = sabs;
  }
  lds_barrier();
  // bounds as in k_fast_score_int4
  const int sumabs = wave_sum(lane < kSW ? isum[lane] : 0);
  const float xsq = wave_sum(lane < kSW ? sq[lane] : 0.0f);
  const float group_factor = gkeys != nullptr ? 8.001f : 1.0f;
  const float bound1 = (float)(7 * sumabs) * smax * group_factor;
  const float bound2 = sqrtf(xsq * (1.0f + (float)d * 0x1p-22f)) * 1.0001f * um * 1.0001f * group_factor;
  const uint32_t anchor1 = fine_bin(__float_as_uint(bound1));
  if (blockIdx.x == 0 && tid == 0) {
    fr->anchor1 = anchor1;
    fr->anchor2 = fine_bin(__float_as_uint(bound2));
    fr->beyond2 = 0u;
    take_cookie(fr, cookie);
  }
  {
    float* arr = gkeys != nullptr ? gkeys : keys;
    const int n = gkeys != nullptr ? N / 8 : N;
    if (blockIdx.x == 0 && tid < ((4 - (n & 3)) & 3)) arr[n + tid] = 0.0f;
  }
  auto count_key = [&](float key) { count_in_window<false>(__float_as_uint(key), anchor1, fr->hist1, &fr->beyond1); };
  const uint4* tq4 = reinterpret_cast<const uint4*>(tq);
  for (int g = gw; 4 * g < N; g += waves) {  // uniform
    if (g != gw) {
      load_z2(g);
      row_scale = scale2[min(4 * g + (lane >> 4), N - 1)];
    }
    int acc = 0;
    if (sub < cpr2) acc = chunk_dot(z2, tq4[2 * sub], tq4[2 * sub + 1], acc);
    auto add = [](int a, int b) { return a + b; };
    acc = add(acc, dpp_move<0x111, 0xF>(0, acc));  // the last of the row's sixteen lanes has its sum
    acc = add(acc, dpp_move<0x112, 0xF>(0, acc));
    acc = add(acc, dpp_move<0x114, 0xF>(0, acc));
    acc = add(acc, dpp_move<0x118, 0xF>(0, acc));
    const int j = 4 * g + (lane >> 4);
    if (sub == 15 && j < N) {
      float key = (float)(acc >> 4) * row_scale;
      key = key > 0.0f ? key : 0.0f;  // ReLU, and -0 -> +0
      if (gkeys != nullptr) {
        unit_keys[w * kRPW + (lane >> 4)] = key;  // one pass per workgroup here
      } else {
        keys[j] = key;
        count_key(key);
      }
    }
  }
  if (gkeys != nullptr) {
    __syncthreads();
    const int J = (int)blockIdx.x * (kSW * kRPW / 8) + tid;
    if (tid < kSW * kRPW / 8 && J * 8 < N) {
      float sum = 0.0f;
#pragma unroll
      for (int l = 0; l < 8; ++l) sum += fabsf(unit_keys[tid * 8 + l]);
      gkeys[J] = sum;
      count_key(sum);
    }
  }
  HIRE_TS(34);
  if (clocks) {
    __syncthreads();
    if (tid == 0) clocks[2 * blockIdx.x + 1] = wall_clock64();
  }
}

// ---------------------------------------------------------------------------------------------------
// Kernel 1 for the low-rank scorer (HiRE-LR, Sec. 3.2): keys[j] = relu(<Z2[j, :], t>) in fp64 with
// t = bf16(Z1^T x) from k_lr_project.  The anchors are
// Cauchy-Schwarz bounds: key_j <= |Z2_j| |t| and <u_j, x> <= |u_j| |x| with the layer's largest row norms
// (bounds[1], bounds[0]: upper bounds, prepared once per layer) and the norms of t and x formed here in fp32 and
// rounded up by more than their own error.  Sixteen lanes share a row, four rows a wave: a workgroup's 64 rows take one trip.
// (From r = 136 on a whole wave per row, in four trips: d = 2048, 16384 units, r = 256, one token 33.4 against 30.5 us per
// step, four 58.1 against 51.6; d = 256, 1200 units, r = 160, four 35.8 against 28.8.)
// TT: tokens, 1 or up to 4; kSW / TT waves per token form the norms.
template <int TT>
__global__ __launch_bounds__(kST) void k_fast_score_lr(const uint16_t* __restrict__ t_in,
                                                       const uint16_t* __restrict__ z2, const uint4* __restrict__ x,
                                                       int B, int N, int d, int r, const float* __restrict__ bounds,
                                                       double* __restrict__ keys, long long stride,
                                                       FastRegion* __restrict__ fr, int groups) {
  // groups != 0: keys are the activations of groups of eight adjacent units, keys[J] = sum_{l<8} |key[8J + l]|
  constexpr int kWPT = kSW / TT;
  __shared__ uint4 ts[TT][128];  // t as raw bf16: r <= 1024
  __shared__ float red_t[kSW], red_x[kSW];
  constexpr int kRowLanes = 16, kRows = kWave / kRowLanes;  // lanes per row, rows per wave and trip
  __shared__ double unit_keys[TT][kSW * kRows];
  const int tid = (int)threadIdx.x, lane = lane_id(), w = wave_id();
  const int sub = lane % kRowLanes, rw = lane / kRowLanes;
  const int cpr = r / 8, n_keys = groups ? N / 8 : N;
  const float group_factor = groups ? 8.001f : 1.0f;
  HIRE_TS(30);
  const unsigned long long cookie = fr->cookie;  // (workgroup 0 takes it away)
  const float umax = bounds[0], zmax = bounds[1];
  for (int i = (int)blockIdx.x * kST + tid; i < B * kWin; i += (int)gridDim.x * kST) fr[i / kWin].hist2[i % kWin] = 0u;
  const int mine = min(w / kWPT, B - 1), lt = w % kWPT * kWave + lane;  // the token this wave prepares
  float tsq = 0.0f, xsq = 0.0f;
  uint16_t* t16 = reinterpret_cast<uint16_t*>(ts[w / kWPT]);
  for (int p = lt; p < r; p += kWPT * kWave) {
    const uint16_t tb = t_in[(size_t)mine * r + p];
    t16[p] = tb;
    const float tf = bf16_to_f32(tb);
    tsq = fmaf(tf, tf, tsq);
  }
  for (int i = lt; i < d / 8; i += kWPT * kWave) {
    const uint4 u = x[(size_t)mine * (d / 8) + i];
    const uint32_t ud[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float a = bf16_lo(ud[q]), b = bf16_hi(ud[q]);
      xsq = fmaf(a, a, xsq);
      xsq = fmaf(b, b, xsq);
    }
  }
  tsq = wave_sum(tsq);
  xsq = wave_sum(xsq);
  if (lane == 0) {
    red_t[w] = tsq;
    red_x[w] = xsq;
  }
  __syncthreads();
  HIRE_TS(32);
  uint32_t anchor1[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    const float tt = wave_sum(lane < kWPT ? red_t[t * kWPT + lane] : 0.0f);
    const float xx = wave_sum(lane < kWPT ? red_x[t * kWPT + lane] : 0.0f);
    const float tnorm = sqrtf(tt * (1.0f + (float)r * 0x1p-22f)) * 1.0001f;
    const float xnorm = sqrtf(xx * (1.0f + (float)d * 0x1p-22f)) * 1.0001f;
    const float bound1 = tnorm * zmax * 1.0001f * group_factor, bound2 = xnorm * umax * 1.0001f * group_factor;
    anchor1[t] = fine_bin(__float_as_uint(bound1));
    if (blockIdx.x == 0 && tid == 0 && t < B) {
      fr[t].anchor1 = anchor1[t];
      fr[t].anchor2 = fine_bin(__float_as_uint(bound2));
      fr[t].beyond2 = 0u;
      if (t == 0) take_cookie(fr, cookie);
      if (n_keys & 1) keys[t * stride + n_keys] = 0.0;  // zero padding of the handed-on keys up to a whole 16-byte vector
    }
  }
  for (int b0 = (int)blockIdx.x * kSW * kRows; b0 < N; b0 += (int)gridDim.x * kSW * kRows) {  // uniform over the workgroup
    const int j = b0 + w * kRows + rw;
    const uint4* row = reinterpret_cast<const uint4*>(z2 + (size_t)min(j, N - 1) * r);
    double acc[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[t] = 0.0;
    for (int c0 = 0; c0 < cpr; c0 += kRowLanes) {
      const int c = c0 + sub;
      const uint4 wv = row[min(c, cpr - 1)];
      const uint32_t keep = c < cpr ? 0xFFFFFFFFu : 0u;
      const uint32_t wd[4] = {wv.x & keep, wv.y & keep, wv.z & keep, wv.w & keep};
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        const uint4 tv = ts[t][min(c, cpr - 1)];
        const uint32_t td[4] = {tv.x, tv.y, tv.z, tv.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[t] += (double)(bf16_lo(wd[q]) * bf16_lo(td[q]));
          acc[t] += (double)(bf16_hi(wd[q]) * bf16_hi(td[q]));
        }
      }
    }
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      // prefix sum along the sixteen lanes of a DPP row: the row's last lane holds its total
      auto add = [](double a, double b) { return a + b; };
      double s = acc[t];
      s = add(s, dpp_move<0x111, 0xF>(0.0, s));
      s = add(s, dpp_move<0x112, 0xF>(0.0, s));
      s = add(s, dpp_move<0x114, 0xF>(0.0, s));
      s = add(s, dpp_move<0x118, 0xF>(0.0, s));
      if (sub == kRowLanes - 1 && j < N && t < B) {
        s = s > 0.0 ? s : 0.0;  // ReLU, and -0 -> +0
        if (groups) {
          unit_keys[t][w * kRows + rw] = s;
        } else {
          keys[t * stride + j] = s;
          count_in_window<(TT > 1)>((uint64_t)__double_as_longlong(s), anchor1[t], fr[t].hist1, &fr[t].beyond1);
        }
      }
    }
    if (groups) {  // (N is a multiple of eight, like a trip's rows)
      constexpr int kGroups = kSW * kRows / 8;
      lds_barrier();
      const int t = tid / kGroups, J = b0 / 8 + tid % kGroups;
      if (t < min(TT, B) && J < n_keys) {
        double sum = 0.0;
#pragma unroll
        for (int l = 0; l < 8; ++l) sum += fabs(unit_keys[t][tid % kGroups * 8 + l]);
        keys[t * stride + J] = sum;
        uint32_t anchor = 0u;
#pragma unroll
        for (int u = 0; u < TT; ++u) anchor = t == u ? anchor1[u] : anchor;
        count_in_window<(TT > 1)>((uint64_t)__double_as_longlong(sum), anchor, fr[t].hist1, &fr[t].beyond1);
      }
      lds_barrier();
    }
  }
  HIRE_TS(34);
}

// ---------------------------------------------------------------------------------------------------
// Kernel 2: the shortlist and its exact pre-activations.  A workgroup owns 64 adjacent units, about a fifth of which
// are shortlisted: with the threshold bin known from the walk, a ballot over its 64 keys names its rows, and their loads
// go out at once - nothing is counted, listed or placed first.  Only a workgroup that holds a key of the threshold bin
// itself looks through all keys for that bin's others, while its rows are in flight, and settles which of its own belong
// to the shortlist.  Activations are left by unit (fp32 for the selection that follows, fp64 for its ties; 0 and -1
// where a unit is not shortlisted), so no list of candidates is needed in between; the caller's is written beside
// kernel 3 (a 257th workgroup here would wait for a compute unit).  K: the keys' bit patterns, 32 bits for the int4
// scorer's fp32 keys, 64 for the low-rank scorer's fp64 ones; LOADS: 16-byte loads of keys per thread.
// Measured at the ~1B shape: 7.6 us against 10.5 when every workgroup selected all of the shortlist for an equal share of
// its rows.  Inside: 2.3 until the window is walked, 0.5 until the rows are known, 1.3 for the rows; workgroups that own a
// key of the threshold bin need 1.6 more for its list and are the last to end.
constexpr int kGT = 1024;
constexpr int kGW = kGT / kWave;
using GatherShared = SelSharedT<kGT>;

struct FastGatherParams {
  const void* keys;           // [N >> gs] fp32 (fp64), zero up to the next multiple of 4 (2)
  int N, kprime, d;           // units; selected entries (units or groups)
  FastRegion* fr;
  const uint16_t* W1;         // [N, d] bf16
  const uint4* x;             // token, d/8 uint4
  int32_t* n_cand;            // optional
  float* h32;                 // [N >> gs, up to a multiple of 64] activations, 0 where not shortlisted
  double* h64;                // the same in fp64, -1 where not shortlisted
  // gs = 3 (group-sparse step): keys are group activations, kprime counts groups of eight units, h32 / h64 hold the
  // groups' exact activations sum_l |h|, which are what is counted in the histogram and ranked by the next kernel, and
  // u32 [N, up to a multiple of 64] the units'.  gs = 0: units.
  int gs;
  float* u32;
  // workgroups from own_blocks on (CommonPath, eq. (7)): the activations of the m1 dense units, kGW rows per workgroup:
  // hd[r] = relu(<Wd[r, :], x>).
  int own_blocks;
  const uint16_t* Wd;
  int m1;
  double* hd;
};

// relu(<row, x>) by a wave, the token as fp32 in LDS: sixteen bytes per lane and load, 256 chunks in flight; every bf16
// product is exact in fp32 and the sums run in fp64.
__device__ __forceinline__ double row_dot_relu(const uint4* row, RowChunks first, const float* __restrict__ xtok, int cpr) {
  const int lane = lane_id();
  double acc = 0.0;
  for (int c0 = 0; c0 < cpr; c0 += 4 * kWave) {
    if (c0 > 0) first.issue(row, c0, cpr);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u * kWave + lane;
      if (c < cpr) {
        const float4 xa = reinterpret_cast<const float4*>(xtok)[2 * c], xb = reinterpret_cast<const float4*>(xtok)[2 * c + 1];
        const float xf[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
        const uint32_t wd[4] = {first.v[u].x, first.v[u].y, first.v[u].z, first.v[u].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc += (double)(bf16_lo(wd[q]) * xf[2 * q]);
          acc += (double)(bf16_hi(wd[q]) * xf[2 * q + 1]);
        }
      }
    }
  }
  const double s = wave_sum(acc);
  return s > 0.0 ? s : 0.0;  // ReLU, and -0 -> +0
}

__device__ __forceinline__ void token_to_lds(const uint4* __restrict__ x, int xvecs, float* xtok) {
  const int tid = (int)threadIdx.x;
  const uint4 xv0 = x[min(tid, xvecs - 1)];
  for (int i = tid; i < xvecs; i += kGT) {
    const uint4 u = i == tid ? xv0 : x[i];
    const float f[8] = {bf16_lo(u.x), bf16_hi(u.x), bf16_lo(u.y), bf16_hi(u.y),
                        bf16_lo(u.z), bf16_hi(u.z), bf16_lo(u.w), bf16_hi(u.w)};
#pragma unroll
    for (int q = 0; q < 8; ++q) xtok[8 * i + q] = f[q];
  }
}

// ROWS: rows that a wave has under way at a time (launch_ffn_fast).
template <typename K, int LOADS, int ROWS>
__global__ __launch_bounds__(kGT) void k_fast_gather(FastGatherParams p) {
  using Keys = KeyRegs<K, LOADS, kGT, false, true>;
  __shared__ GatherShared sh;
  __shared__ int wave_cnt[kGW];
  __shared__ BinList<K> list;
  __shared__ double unit_h[kOwnUnits];  // group-sparse: the units' activations
  extern __shared__ float xtok[];       // token as fp32, d floats
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int g = (int)blockIdx.x, xvecs = p.d / 8, gs = p.gs;
  if (g >= p.own_blocks) {  // dense common-path units: a row per wave
    token_to_lds(p.x, xvecs, xtok);
    const int r = (g - p.own_blocks) * kGW + w;
    const uint4* row = reinterpret_cast<const uint4*>(p.Wd + (size_t)min(r, p.m1 - 1) * p.d);
    RowChunks first;
    first.issue(row, 0, xvecs);
    __syncthreads();
    if (r >= p.m1) return;
    const double s = row_dot_relu(row, first, xtok, xvecs);
    if (lane == 0) p.hd[r] = s;
    return;
  }
  HIRE_TS(10);
  // every load of the selection goes out here, before the first wait
  const int n = p.N >> gs;
  WinRegs<kGT> wr;
  wr.issue(p.fr->hist1);
  const uint32_t clean = p.fr->clean, beyond1 = p.fr->beyond1, anchor1 = p.fr->anchor1, anchor2 = p.fr->anchor2;
  const int u0 = g * kOwnUnits;                // first unit of the workgroup
  const int entry = (u0 + lane) >> gs;         // lane's unit, or its group
  const bool valid = u0 + lane < p.N;
  const K own = reinterpret_cast<const K*>(p.keys)[min(entry, n - 1)];
  Keys kr;
  kr.issue(p.keys, n, p.fr->zeros);
  token_to_lds(p.x, xvecs, xtok);
  if (tid == 0) sh.list_n = 0;
  if (tid < kOwnUnits) unit_h[tid] = 0.0;
  const bool hist_ok = (clean > 0u) & (beyond1 == 0u);  // (both asked for at once: no branch between the two)
  kr.finish();
  HIRE_TS(11);
  uint64_t taken = 0ull, rows = 0ull;  // units of the workgroup: shortlisted; whose rows are read
  WinWalk wk{0, 0, false};
  if (hist_ok) wk = walk_window<kGT>(wr, p.kprime, sh);
  HIRE_TS(15);
  const uint32_t bin = anchor1 - (uint32_t)wk.slot;
  const bool found = wk.found && bin >= 1u && bin <= anchor1;  // uniform
  bool known = false;  // which of the workgroup's units are shortlisted is
  int cnt = 0;         // rows
  struct Row {  // of the wave: unit of the workgroup, address, first loads
    int pos;
    const uint4* row;
    RowChunks first;
  } wave_row[ROWS];
  auto aim = [&](Row& a, int r) {  // the r-th unit of `rows`
    a.pos = __builtin_ctzll(__ballot(((rows >> lane) & 1ull) != 0ull && mask_prefix(rows) == r));
    a.row = reinterpret_cast<const uint4*>(p.W1 + (size_t)(u0 + a.pos) * p.d);
    a.first.issue(a.row, 0, xvecs);
  };
  auto aim_all = [&](int r) {
#pragma unroll
    for (int u = 0; u < ROWS; ++u)
      if (r + u * kGW < cnt) aim(wave_row[u], r + u * kGW);
  };
  // The keys have arrived by now.  Said to the compiler here, before the rows' loads go out: where paths with and without
  // those meet, it would otherwise wait for the youngest loads, the rows, wherever a key is used.
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  if (found) {
    const K lo = bin_floor<K>(bin), up = bin_floor<K>(bin + 1u);
    taken = __ballot(valid && own >= up);
    const uint64_t open = __ballot(valid && own >= lo && own < up);
    rows = taken | open;
    cnt = __popcll(rows);
    aim_all(w);
    __builtin_amdgcn_sched_barrier(0);  // the rows' loads are not sunk below what follows
    if (open != 0ull) {                 // uniform over the workgroup
      list_inside<K>(kr, bin_masks<K>(kr, lo, up).inside, &sh.list_n, list);
      lds_barrier();
      const int m = sh.list_n, need = p.kprime - wk.above;
      known = m <= kFastAmbCap && need >= 1 && need <= m;  // uniform
      if (known) {
        const K mine_k = lane < m ? list.key[lane] : (K)0;
        const int mine_i = lane < m ? list.idx[lane] : 0x7FFFFFFF;
        for (uint64_t o = open; o != 0ull;) {
          const int l = __builtin_ctzll(o), e = (u0 + l) >> gs;
          const uint64_t units = (gs != 0 ? 0xFFull : 1ull) << l;  // (whole groups: l is a multiple of eight)
          if (list_takes<K>(mine_k, mine_i, m, need, read_lane(own, l), e)) taken |= units & open;
          o &= ~units;
        }
      }
    } else {
      known = true;  // no unit of this workgroup depends on the cut
    }
  }
  HIRE_TS(12);
  if (!known) {  // fresh workspace, threshold among the zeros or below the window, crowded bin: range narrowing
    const Selection<K> sel = fast_select<60>(kr, p.keys, p.kprime, wr, anchor1, false, sh, wave_cnt,
                                             hist_ok ? &p.fr->fallbacks[0] : static_cast<uint32_t*>(nullptr), 0, p.kprime);
    taken = __ballot(valid && cut_takes(sel.cut, own, entry));
  }
  if (!found) {
    rows = taken;
    cnt = __popcll(rows);
    aim_all(w);
  }
  HIRE_TS(13);
  auto count_h = [&](double v) {  // the scorer kernel of this step has cleared the window
    count_in_window<false>((uint64_t)__double_as_longlong(v), anchor2, p.fr->hist2, &p.fr->beyond2);
  };
  if (!found) __syncthreads();  // the token in LDS
  for (int r = w; r < cnt; r += ROWS * kGW) {  // uniform over the wave
    if (r > w) aim_all(r);
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      if (r + u * kGW >= cnt) break;
      const int pos = wave_row[u].pos;
      const double s = row_dot_relu(wave_row[u].row, wave_row[u].first, xtok, xvecs);
      const bool in = ((taken >> pos) & 1ull) != 0ull;
      if (lane == 0) {
        if (gs != 0) {
          unit_h[pos] = s;
        } else {
          p.h32[u0 + pos] = in ? (float)s : 0.0f;
          p.h64[u0 + pos] = in ? s : -1.0;
          if (in) count_h(s);
        }
      }
    }
  }
  if (gs == 0) {
    if (w == kGW - 1 && ((rows >> lane) & 1ull) == 0ull) {
      p.h32[u0 + lane] = 0.0f;
      p.h64[u0 + lane] = -1.0;
    }
  } else {  // exact group activations, units added in order
    __syncthreads();
    if (tid < kOwnUnits) p.u32[u0 + tid] = ((taken >> tid) & 1ull) != 0ull ? (float)unit_h[tid] : 0.0f;
    if (tid < kOwnUnits >> gs) {
      const bool in = ((taken >> (tid << gs)) & 1ull) != 0ull;
      double e = 0.0;
      for (int l = 0; l < (1 << gs); ++l) e += fabs(unit_h[(tid << gs) + l]);
      p.h32[(u0 >> gs) + tid] = in ? (float)e : 0.0f;
      p.h64[(u0 >> gs) + tid] = in ? e : -1.0;
      if (in) count_h(e);
    }
  }
  if (g == 0 && tid == 0) {
    if (p.n_cand) *p.n_cand = p.kprime;
    p.fr->bin1 = found ? bin : 0u;
    p.fr->need1 = (uint32_t)(p.kprime - wk.above);
  }
  HIRE_TS(14);
}

// ---------------------------------------------------------------------------------------------------
// Kernel 3: exact top-k of the activations, then sum_j h_j v_j over the selected rows for this workgroup's 32 columns
// (64 bytes of every selected row: four lanes per row, sixteen rows per wave and load).  Every wave lists the selected
// units of its own part of the row in LDS and adds up their rows, so no barrier and no prefix over the waves lies between
// the cut and the rows' loads; the workgroup then reduces inside itself in a fixed order and writes y.  CommonPath's
// dense units (eq. (7)) are shared out over the waves behind the selected ones.  One more workgroup writes the selected
// entries and their values for the caller.
//
// The selection works on the activations rounded to fp32 (rounding is monotone; the coefficients of the second layer are
// these values anyway); the keys of the threshold bin, and a selection without histogram, go by the fp64 values.
// Measured at the ~1B shape: 7.8 us (8.1 with a branch around every load of rows; four tokens 10.8, 12.1), with the reduction over the
// waves and the lists for the caller in it (9.0 with the lists' keys placed by code unrolled over all of a lane's, whose workgroups were the last to end).  Inside: window walked 1.6,
// masks 0.6, bin settled 0.5, rows listed 0.5, rows 1.0 (from HBM 2.8), reduction 1.0.
constexpr int kWT = 1024;
constexpr int kWW = kWT / kWave;
using W2Shared = SelSharedT<kWT>;
constexpr int kW2Batch = 8;  // loads a lane has in flight
constexpr int kFastMaxUnits = 16384;

struct FastW2Params {    // (what the first loads need comes first)
  FastRegion* fr;        // of the first token
  const float* h32;      // [B, entries] activations by unit (gs = 3: by group), 0: not shortlisted
  const double* h64;     // the same in fp64, -1: not shortlisted
  int n, k, d, entries;  // entries ranked, selected; columns; n up to a whole workgroup of the gather
  int col_slices;
  int out_block;         // the workgroup that writes topk_idx / topk_val; -1: none
  int list_block;        // the workgroup that writes the shortlist; -1: none
  int shared_out;        // != 0 (several tokens, groups): the slices' workgroups write both beside their columns
  // gs = 3 (group-sparse step): entries are groups of eight units, u32 holds the units' activations.
  int gs;
  const float* u32;      // [B, entries << gs]
  const uint16_t* W2;    // [N, d] bf16
  float* y;              // [B, d]
  const uint16_t* W2d;   // CommonPath: y += fl32(hd[r]) * W2d[r, :], r < m1
  const double* hd;      // [B, m1]
  int m1;
  int B;                 // tokens, a row of workgroups each
  int32_t* topk_idx;     // optional [B, k]
  float* topk_val;       // optional [B, k << gs]
  // the shortlist, ascending: the kprime largest of the n keys; of several tokens the union, with its length
  const void* keys;
  int kprime;
  int32_t* cand_out;
  const uint32_t* bitmap;
  int32_t* n_cand;
};

// Column slice of a workgroup: slices 2i and 2i+1 are the two halves of the same 128-byte lines; they go to
// workgroups b and b + 8, which the dispatcher places on the same die (workgroups go round the eight dies),
// so that the second half of a line is found in that die's L2.
__device__ __forceinline__ int slice_of(int b, int slices) {
  if (slices % 16 != 0) return b;
  return 2 * (b % 8) + (b / 8) % 2 + 16 * (b / 16);
}

// Several tokens: the union of the shortlists in ascending order and its length, for the caller, a share of its words by one
// wave of every workgroup that writes columns: issue() among the kernel's first loads, write() when the wave has nothing
// else to do.  (A workgroup of its own would wait for a compute unit where the slices take all of them.)
struct UnionShare {
  static constexpr int kSteps = kFastMaxUnits / 32 / kWave;
  uint32_t word[kSteps];
  __device__ __forceinline__ void issue(const FastW2Params& p) {
    const int words = (p.n + 31) / 32;
#pragma unroll
    for (int u = 0; u < kSteps; ++u) word[u] = p.bitmap[min(u * kWave + lane_id(), words - 1)];
  }
  __device__ __forceinline__ void write(const FastW2Params& p) const {
    const int lane = lane_id(), words = (p.n + 31) / 32, blocks = p.col_slices * p.B;
    const int per = ((words + blocks - 1) / blocks + 1) / 2 * 2;  // an even number
    const int lo = ((int)blockIdx.y * p.col_slices + (int)blockIdx.x) * per;
    int ahead = 0, all = 0;
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const int c = u * kWave + lane < words ? __popc(word[u]) : 0;
      ahead += u * kWave + lane < lo ? c : 0;
      all += c;
    }
    if (lo == 0 && p.n_cand) {
      all = wave_sum(all);
      if (lane == 0) *p.n_cand = all;
    }
    int at = wave_sum(ahead);
    const int cap = min(p.B * p.kprime, p.n);
    for (int i = lo; i < min(lo + per, words); i += 2) {  // uniform
      const uint32_t v = p.bitmap[min(i + (lane >> 5), words - 1)];
      const bool in = i + (lane >> 5) < words && (v >> (lane & 31) & 1u) != 0u;
      const uint64_t m = __ballot(in);
      const int place = at + mask_prefix(m);
      if (in && place < cap) p.cand_out[place] = i * 32 + lane;
      at += __popcll(m);
    }
  }
};

// The shortlist in ascending order, for the caller, by one workgroup: K, LK as in the gathering kernel.
template <typename K, int LK>
__device__ __forceinline__ void list_shortlist(const FastW2Params& p, W2Shared& sh, int* wave_cnt, BinList<K>& list) {
  using Keys = KeyRegs<K, LK, kWT, false, true>;
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const uint32_t bin = p.fr->bin1;
  const int need = (int)p.fr->need1;
  Keys kr;
  kr.issue(p.keys, p.n, p.fr->zeros);
  if (tid == 0) sh.list_n = 0;
  kr.finish();
  __syncthreads();
  uint32_t take = 0u;  // this lane's selected keys, as in BinMasks
  bool known = false;
  if (bin != 0u) {  // uniform
    const BinMasks<K> bm = bin_masks<K>(kr, bin_floor<K>(bin), bin_floor<K>(bin + 1u));
    list_inside<K>(kr, bm.inside, &sh.list_n, list);
    __syncthreads();
    const int m = sh.list_n;
    known = m <= kFastAmbCap && need >= 1 && need <= m;  // uniform
    if (known) {
      const K mine_k = lane < m ? list.key[lane] : (K)0;
      const int mine_i = lane < m ? list.idx[lane] : 0x7FFFFFFF;
      take = bm.above | taken_of_list<Keys>(kr, mine_k, mine_i, m, need);
    }
  }
  if (!known) {
    WinRegs<kWT> none{};
    const Selection<K> sel = fast_select<60>(kr, p.keys, p.kprime, none, 0u, false, sh, wave_cnt,
                                             static_cast<uint32_t*>(nullptr), 0, p.kprime);
    take = 0u;
#pragma unroll
    for (int e = 0; e < LK; ++e)
#pragma unroll
      for (int q = 0; q < Keys::PER; ++q)
        take = take + take + (kr.valid(e, q) && cut_takes(sel.cut, kr.r[e][q], kr.index(e, q)) ? 1u : 0u);
  }
  const int mine = wave_sum(__popc(take));
  __syncthreads();
  if (lane == 0) wave_cnt[w] = mine;
  __syncthreads();
  const int before = wave_scan_incl(lane < kWW ? wave_cnt[lane] : 0);
  place_taken<Keys>(__brev(take) >> (32 - LK * Keys::PER), w > 0 ? __builtin_amdgcn_readlane(before, w - 1) : 0,
                    [&](int at, int e, int q) {
                      if (at < p.kprime) p.cand_out[at] = kr.index(e, q);
                    });
}

// KEY: the scorer keys' bit patterns (what the candidate list is selected from); LOADS: 16-byte loads of fp32
// activations per thread.
// Selected rows: streaming loads where a workgroup reads whole lines; slices of 32 columns read half of them, and the other
// half is another workgroup's, which has to find the line in L2 (one token at the ~1B shape 24.0 us per step, 24.3 with
// streaming loads; four tokens in slices of 64 42.4 with, 43.0 without).  Dense rows are every token's: plain loads (2736 of them
// and four tokens, groups of eight: 46.5 -> 40.5 us per step, one token 30.3 -> 25.7).
// SHARED: p.shared_out may be set (kernels without it are free of its branches).
template <typename KEY, int LOADS, int COLS, bool SHARED = false>
__global__ __launch_bounds__(kWT) void k_fast_w2(FastW2Params p) {
  auto load_w2 = [](const uint4* row) { return COLS == 32 ? *row : load_streaming(row); };
  using K = uint32_t;
  using Keys = KeyRegs<K, LOADS, kWT, false, true>;
  constexpr int PER = Keys::PER;
  __shared__ W2Shared sh;
  __shared__ BinList<KEY> list;
  __shared__ int wave_cnt[kWW], wave_eq[kWW];
  constexpr int kRowLanes = COLS / 8;                // lanes that share a row: 16 bytes each
  constexpr int kRowsPerLoad = kWave / kRowLanes;    // rows a wave covers with one load instruction
  constexpr int kSegRows = kRowsPerLoad * kW2Batch;  // rows a wave lists at a time
  static_assert((kRowLanes == 4 || kRowLanes == 8 || kRowLanes == 16) && kWW == 16, "whole DPP rows, 64 rows to reduce");
  __shared__ int seg[kWW][kSegRows];                 // selected entries of every wave
  __shared__ float red[4 * kWW][COLS];
  __shared__ float red2[8][COLS];
  const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const bool output = (int)blockIdx.x == p.out_block;  // uniform
  if ((int)blockIdx.x == p.list_block && p.B > 1) {
    if (blockIdx.y > 0) return;
    const int cnt = list_bitmap<kWT>(p.bitmap, (p.n + 31) / 32, p.cand_out, min(p.B * p.kprime, p.n), sh);
    if (tid == 0 && p.n_cand) *p.n_cand = cnt;
    return;
  }
  if ((int)blockIdx.x == p.list_block) {
    list_shortlist<KEY, LOADS * (int)(sizeof(KEY) / 4)>(p, sh, wave_cnt, list);
    return;
  }
  if ((int)blockIdx.x >= p.col_slices && !output) return;  // (the grid is padded)
  const int cs = COLS == 32 ? slice_of((int)blockIdx.x, p.col_slices) : (int)blockIdx.x;
  const size_t b = blockIdx.y;  // token
  FastRegion* fr = p.fr + b;
  const float* h32 = p.h32 + b * p.entries;
  const double* h64 = p.h64 + b * p.entries;
  const float* u32 = p.u32 + (b * p.entries << p.gs);  // (gs = 3 only)
  HIRE_TS(24);
  const uint32_t anchor2 = fr->anchor2;
  const bool whole = fr->beyond2 == 0u;     // the window counts every activation that it should
  const int clean = (int)p.fr->clean;       // (asked for here: at the end its latency would count)
  WinRegs<kWT> wr;
  wr.issue(fr->hist2, p.B > 1);
  Keys kr;
  kr.issue(h32, p.n, p.fr->zeros);
  if (tid == 0) sh.list_n = 0;
  kr.finish();
  const bool lists = SHARED && p.shared_out != 0 && w == kWW - 1 && p.cand_out != nullptr;  // uniform over the wave
  UnionShare share;
  if (lists) share.issue(p);
  // rows of the wave: slot-th of every sixteen, eight columns per lane
  const int slot = lane / kRowLanes, part = lane % kRowLanes;
  const int colc = min(cs * COLS + part * 8, p.d - 8);
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  auto add_row = [&](const uint4& wv, float cf) {
    const float wf[8] = {bf16_lo(wv.x), bf16_hi(wv.x), bf16_lo(wv.y), bf16_hi(wv.y),
                         bf16_lo(wv.z), bf16_hi(wv.z), bf16_lo(wv.w), bf16_hi(wv.w)};
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = fmaf(cf, wf[q], acc[q]);
  };
  // what lies behind a list's end adds nothing, were its weight infinite
  auto only_if = [&](bool counts, uint4& wv, auto& cf) __attribute__((always_inline)) {
    cf = counts ? cf : 0;
    wv = counts ? wv : make_uint4(0, 0, 0, 0);
  };
  // the activations' window is valid on any workspace: this step's scorer kernel cleared it, its gather filled it
  const WinWalk wk = walk_window<kWT>(wr, p.k, sh);
  HIRE_TS(20);
  const uint32_t bin = anchor2 - (uint32_t)wk.slot;
  const bool found = whole && wk.found && bin >= 1u && bin <= anchor2;  // uniform
  uint32_t take = 0u;  // this lane's selected keys, as in BinMasks
  bool known = false;
  if (found) {
    const K lo = bin_floor<K>(bin), up = bin_floor<K>(bin + 1u);
    const BinMasks<K> bm = bin_masks<K>(kr, lo, up);
    for (uint32_t m = bm.inside; m != 0u;) {  // few lanes of few waves
      const int i = pop_first(kr, m), at = atomicAdd(&sh.list_n, 1);
      if (at < kFastAmbCap) list.idx[at] = i;
    }
    __syncthreads();
    HIRE_TS(21);
    const int m = sh.list_n, need = p.k - wk.above;
    known = m <= kFastAmbCap && need >= 1 && need <= m;  // uniform
    if (known) {
      // the fp64 values of the bin's keys: they order what fp32 cannot
      const int mine_i = lane < m ? list.idx[lane] : 0x7FFFFFFF;
      const uint64_t mine_k = lane < m ? (uint64_t)__double_as_longlong(h64[mine_i]) : 0ull;
      take = bm.above | taken_of_list<Keys>(kr, mine_k, mine_i, m, need);
    }
    HIRE_TS(22);
  }
  if (!known) {  // range narrowing over the fp64 values, ties to the lower index
    __syncthreads();
    if (blockIdx.x == 0 && tid == 0) atomicAdd(&p.fr->fallbacks[1], 1u);
    const uint64_t t = wg_kth_largest<uint64_t>(
        [&](auto&& f) {
#pragma unroll 1
          for (int i = tid; i < p.n; i += kWT) f(order_key(h64[i]));
        },
        p.n, p.k, sh);
    int gt = 0, eq = 0;
#pragma unroll
    for (int e = 0; e < LOADS; ++e)
#pragma unroll
      for (int q = 0; q < PER; ++q)
        if (kr.valid(e, q)) {
          const uint64_t key = order_key(h64[kr.index(e, q)]);
          gt += key > t ? 1 : 0;
          eq += key == t ? 1 : 0;
        }
    gt = wave_sum(gt);
    eq = wave_sum(eq);
    __syncthreads();
    if (lane == 0) {
      wave_cnt[w] = gt;
      wave_eq[w] = eq;
    }
    __syncthreads();
    int all_gt = 0, run_eq = 0;
    for (int u = 0; u < kWW; ++u) {
      all_gt += wave_cnt[u];
      run_eq += u < w ? wave_eq[u] : 0;
    }
    __syncthreads();  // wave_cnt is free: a wave without selected keys is far ahead of the others when it counts them below
    const int need_eq = p.k - all_gt;
#pragma unroll
    for (int e = 0; e < LOADS; ++e) {
      uint64_t key[PER];
      int c = 0;
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        key[q] = kr.valid(e, q) ? order_key(h64[kr.index(e, q)]) : 0ull;
        c += key[q] == t ? 1 : 0;
      }
      const int incl = wave_scan_incl(c);
      int before = run_eq + incl - c;  // equal values ahead of this lane's
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        take = take + take + (key[q] > t || (key[q] == t && before < need_eq) ? 1u : 0u);
        before += key[q] == t ? 1 : 0;
      }
      run_eq += __builtin_amdgcn_readlane(incl, kWave - 1);
    }
  }
  const int gs = p.gs;
  // the selected entries and their activations, ascending: every wave its own, once the waves' numbers are in wave_cnt
  auto write_selected = [&](bool units) {
    const int before = wave_scan_incl(lane < kWW ? wave_cnt[lane] : 0);
    const int run = w > 0 ? __builtin_amdgcn_readlane(before, w - 1) : 0;
    place_few<Keys>(kr, take, run, [&](int at, int i, int j) {
      if (at >= p.k) return;  // (never; but whatever the workspace holds, nothing is written past the token's row)
      if (p.topk_idx) p.topk_idx[b * p.k + at] = i;
      if (p.topk_val == nullptr) return;
      if (units) {
        p.topk_val[b * p.k + at] = __uint_as_float(key_at<0, LOADS * PER>(kr, j));
      } else {  // groups of eight: their units' activations
        const float4* act = reinterpret_cast<const float4*>(u32 + ((size_t)i << 3));
        const float4 lo = act[0], hi = act[1];
        const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        float* out = p.topk_val + ((b * p.k + at) << 3);
#pragma unroll
        for (int l = 0; l < 8; ++l) out[l] = v[l];
      }
    });
  };
  if (output) {
    const int mine = wave_sum(__popc(take));
    if (lane == 0) wave_cnt[w] = mine;
    __syncthreads();
    write_selected(gs == 0);
  } else {
    // The wave's selected entries go to LDS lane by lane (any fixed order will do), at most kSegRows rows at a time;
    // their coefficients are loaded with the rows.
    const int mine_n = __popc(take), incl = wave_scan_incl(mine_n);
    const int rows = __builtin_amdgcn_readlane(incl, kWave - 1) << gs;
    const float* coef = gs == 0 ? h32 : u32;
    for (int c0 = 0; c0 < rows; c0 += kSegRows) {  // uniform over the wave; one trip for most
      int at = incl - mine_n - (c0 >> gs);
      for (uint32_t m = take; m != 0u; ++at) {
        const int i = pop_first(kr, m);
        if (at >= 0 && at < kSegRows >> gs) seg[w][at] = i;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      HIRE_TS(26);
      const int m = min(kSegRows, rows - c0);
      // One piece of code for each number of loads, without a branch between them: with each behind a branch of its own the wait
      // for the first row was one for all that were under way.  18 layers of the ~1B shape, us per pass: one token 410.1 -> 402.8,
      // four 669.3 -> 646.3; four of the low-rank int4 scorer, one token, 95.4 -> 93.7.  (The dense rows gained nothing by it.)
      auto add_rows = [&](auto loads) __attribute__((always_inline)) {
        constexpr int kLoads = decltype(loads)::value;
        uint4 wv[kLoads];
        float raw[kLoads];
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
          const int rc = min(u * kRowsPerLoad + slot, m - 1);
          const int unit = (seg[w][rc >> gs] << gs) + (rc & ((1 << gs) - 1));
          wv[u] = load_w2(reinterpret_cast<const uint4*>(p.W2 + (size_t)unit * p.d + colc));
          raw[u] = coef[unit];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
          if (u < kLoads - 1 || u * kRowsPerLoad + slot < m) add_row(wv[u], raw[u]);  // (only the last load may not be whole)
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      static_assert(kW2Batch == 8, "the cases below");
      switch ((m + kRowsPerLoad - 1) / kRowsPerLoad) {  // uniform
        case 1: add_rows(std::integral_constant<int, 1>{}); break;
        case 2: add_rows(std::integral_constant<int, 2>{}); break;
        case 3: add_rows(std::integral_constant<int, 3>{}); break;
        case 4: add_rows(std::integral_constant<int, 4>{}); break;
        case 5: add_rows(std::integral_constant<int, 5>{}); break;
        case 6: add_rows(std::integral_constant<int, 6>{}); break;
        case 7: add_rows(std::integral_constant<int, 7>{}); break;
        default: add_rows(std::integral_constant<int, 8>{});
      }
    }
    for (int r0 = w * kRowsPerLoad; r0 < p.m1; r0 += kWW * kRowsPerLoad * kW2Batch) {  // dense units, uniform
      uint4 wv[kW2Batch];
      double raw[kW2Batch];  // (nothing is done with a load before all are out)
#pragma unroll
      for (int u = 0; u < kW2Batch; ++u)
        if (r0 + u * kWW * kRowsPerLoad < p.m1) {  // uniform
          const int rc = min(r0 + u * kWW * kRowsPerLoad + slot, p.m1 - 1);
          wv[u] = *reinterpret_cast<const uint4*>(p.W2d + (size_t)rc * p.d + colc);
          raw[u] = p.hd[b * p.m1 + rc];
        }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < kW2Batch; ++u)
        if (r0 + u * kWW * kRowsPerLoad < p.m1) {
          const int left = p.m1 - r0 - u * kWW * kRowsPerLoad;
          if (left < kRowsPerLoad) only_if(slot < left, wv[u], raw[u]);  // uniform
          add_row(wv[u], (float)raw[u]);
        }
    }
    HIRE_TS(27);
    // fixed-order reduction: the slots of a DPP row (its last lanes then hold their sums), the rows of all
    // waves in eight groups, the groups
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if constexpr (kRowLanes == 4) acc[q] += dpp_move<0x114, 0xF>(0.0f, acc[q]);
      if constexpr (kRowLanes <= 8) acc[q] += dpp_move<0x118, 0xF>(0.0f, acc[q]);
    }
    if ((lane & 15) >= 16 - kRowLanes) {
      float4* dst = reinterpret_cast<float4*>(&red[w * 4 + (lane >> 4)][part * 8]);
      dst[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
      dst[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    }
    // one of the token's workgroups writes the selected groups behind its columns
    const bool writes = SHARED && p.shared_out != 0 && blockIdx.x == 0 && (p.topk_idx != nullptr || p.topk_val != nullptr);  // uniform
    if (writes) {
      const int mine = wave_sum(__popc(take));
      if (lane == 0) wave_cnt[w] = mine;
    }
    __syncthreads();
    if (tid < 8 * COLS) {
      const int c = tid % COLS, j = tid / COLS;
      float t = 0.0f;
#pragma unroll
      for (int u = 0; u < 8; ++u) t += red[j * 8 + u][c];
      red2[j][c] = t;
    }
    __syncthreads();
    if (tid < COLS) {
      const int c = cs * COLS + tid;
      if (c < p.d) {
        float t = 0.0f;
#pragma unroll
        for (int u = 0; u < 8; ++u) t += red2[u][tid];
        p.y[b * p.d + c] = t;
      }
    }
    if (lists) share.write(p);
    if (writes) write_selected(false);
    HIRE_TS(28);
  }
  // The key histogram has served its purpose: the workgroups clear it between them and say so in the
  // cookie (the same value from each; the next kernel that looks at either starts after this one has ended).
  for (int i = (int)blockIdx.x * kWT + tid; i < kWin; i += p.col_slices * kWT) fr->hist1[i] = 0u;
  if (tid == 0) {
    fr->beyond1 = 0u;
    give_cookie(p.fr, clean, p.B);
  }
}

// ---------------------------------------------------------------------------------------------------
size_t ffn_fast_fallbacks_offset() { return offsetof(FastRegion, fallbacks); }
void ffn_fast_state_layout(size_t* cookie_off, unsigned long long* cookie, size_t* hist1_off, size_t* hist2_off,
                           size_t* hist_words) {
  *cookie_off = offsetof(FastRegion, cookie);
  *cookie = kCookie + 1;
  *hist1_off = offsetof(FastRegion, hist1);
  *hist2_off = offsetof(FastRegion, hist2);
  *hist_words = kWin;
}
int ffn_fast_score_blocks(int N) { return min(((N + kRPW - 1) / kRPW + kSW - 1) / kSW, 1024); }


// Entries (units or groups) of the arrays of activations: whole workgroups of the gather write them.
int ffn_fast_entries(int N, int gs) { return ((N + kOwnUnits - 1) / kOwnUnits * kOwnUnits) >> gs; }

// Group-sparse step with groups of eight: N, k, k' count units.  The selections see N/8, k'/8 and k/8 entries.
bool ffn_fast_group8_supported(int B, int N, int d, int k, int kprime) {
  return N % 8 == 0 && k % 8 == 0 && kprime % 8 == 0 && ffn_fast_supported(B, N, d, k, kprime, true);
}

bool ffn_fast_supported(int B, int N, int d, int k, int kprime, bool groups) {
  return N <= kFastMaxUnits && d % 32 == 0 && d >= 64 && d <= 8192 && k >= 1 && kprime <= N &&
         (B == 1 || ffn_fast_tokens_supported(B, d, groups));
}

hipError_t launch_ffn_fast(const FfnFastArgs& a, hipStream_t s) {
  hipError_t e;
  FastRegion* fr = reinterpret_cast<FastRegion*>(a.fast_region);
  auto mark = [&](int i) -> hipError_t { return a.stage_events ? hipEventRecord(a.stage_events[i], s) : hipSuccess; };
  if ((e = mark(0)) != hipSuccess) return e;
  const int score_blocks = ffn_fast_score_blocks(a.N);
  const int gs = a.gs;  // 0, or 3 for groups of eight units
  // what the selections rank: units with their keys and activations, or groups with their summed ones
  const int n_sel = a.N >> gs, kp_sel = a.kprime >> gs, k_sel = a.k >> gs;
  const bool lowrank = a.lowrank, several = a.B > 1;
  const void* sel_keys = lowrank ? static_cast<const void*>(gs ? a.gkeys64 : a.keys64) : (gs ? a.gkeys : a.keys);
  if (lowrank) {
    if (a.r < 8 || a.r > 1024 || a.r % 8 != 0) return hipErrorInvalidValue;
    e = launch_lr_project(static_cast<const uint16_t*>(a.lr_a), a.x, a.B, a.d, a.r, a.t, nullptr, 0, nullptr, 0ull, s);
    if (e != hipSuccess) return e;
    const uint4* x4 = reinterpret_cast<const uint4*>(a.x);
    auto go = [&](auto kernel) {
      return launch(kernel, dim3(score_blocks), dim3(kST), 0, s, static_cast<const uint16_t*>(a.t), static_cast<const uint16_t*>(a.lr_b),
                    x4, a.B, a.N, a.d, a.r, a.norm_bounds, gs ? a.gkeys64 : a.keys64, gs ? a.gkey_stride : a.key_stride, fr, gs);
    };
    e = several ? go(k_fast_score_lr<4>) : go(k_fast_score_lr<1>);
    if (e != hipSuccess) return e;
    if ((e = mark(1)) != hipSuccess) return e;
  } else if (a.lrq) {
    // first product: the r rows of the int4 copy of Z1^T against the token (no phi), fp32 intermediate; then the
    // scorer kernel on the int4 copy of Z2 with that intermediate as its token
    if (a.r < 32 || a.r > 1024 || a.r % 32 != 0) return hipErrorInvalidValue;
    if (several) {
      ScorerTokens tok{};
      if (scorer_mfma_quantises(a.B, a.r, a.d, false)) {
        tok.x = a.x;
      } else {
        if ((e = launch_quantize_tokens(a.x, false, a.B, a.d, a.xq, nullptr, nullptr, 0, nullptr, 0ull, s)) != hipSuccess) return e;
        tok.xq = a.xq;
      }
      e = launch_scorer_int4_mfma(reinterpret_cast<const uint32_t*>(a.lr_a), a.lr_a_scale, tok, a.B, a.r, a.d, 0, a.keys_t,
                                  a.r, nullptr, HistRefs{nullptr, nullptr}, s);
      if (e != hipSuccess) return e;
      if ((e = launch_fast_score_tokens(a, a.keys_t, true, s)) != hipSuccess) return e;
    } else if (a.r <= kLrqFusedRank && a.r * a.d / 2 <= kLrqFusedBytes) {
      auto go = [&](auto kernel) {
        return launch(kernel, dim3(score_blocks), dim3(kST), (size_t)a.d * 3, s, reinterpret_cast<const uint4*>(a.lr_a),
                      a.lr_a_scale, reinterpret_cast<const uint4*>(a.lr_b), a.lr_b_scale, reinterpret_cast<const uint4*>(a.x),
                      a.N, a.d, a.r, a.keys, fr, a.scorer_clocks, a.norm_bounds, gs ? a.gkeys : static_cast<float*>(nullptr));
      };
      if ((e = a.r <= 128 ? go(k_fast_score_lrq<8>) : go(k_fast_score_lrq<16>)) != hipSuccess) return e;
    } else {
      e = launch_scorer_int4_fused(reinterpret_cast<const uint32_t*>(a.lr_a), a.lr_a_scale, a.x, false, a.r, a.d, 0,
                                   a.keys_t, nullptr, HistRefs{nullptr, nullptr}, nullptr, 0, 0ull, s);
      if (e != hipSuccess) return e;
      const size_t lds = (size_t)a.r * 2 + (size_t)a.r;
      e = launch(k_fast_score_int4<true>, dim3(score_blocks), dim3(kST), lds, s, reinterpret_cast<const uint4*>(a.lr_b),
                 a.lr_b_scale, reinterpret_cast<const uint32_t*>(a.keys_t), a.N, a.r, a.keys, static_cast<int32_t*>(nullptr),
                 fr, a.scorer_clocks, gs ? a.gkeys : static_cast<float*>(nullptr), reinterpret_cast<const uint4*>(a.x), a.d,
                 a.norm_bounds);
      if (e != hipSuccess) return e;
    }
    if ((e = mark(1)) != hipSuccess) return e;
  } else if (several) {
    if ((e = launch_fast_score_tokens(a, a.x, false, s)) != hipSuccess) return e;
    if ((e = mark(1)) != hipSuccess) return e;
  } else {
    const size_t lds = (size_t)a.d * 2 + (size_t)a.d;
    e = launch(k_fast_score_int4<false>, dim3(score_blocks), dim3(kST), lds, s, reinterpret_cast<const uint4*>(a.q4),
               a.q4_scale, reinterpret_cast<const uint32_t*>(a.x), a.N, a.d, a.keys, a.scorer_acc, fr, a.scorer_clocks,
               gs ? a.gkeys : static_cast<float*>(nullptr), static_cast<const uint4*>(nullptr), 0,
               static_cast<const float*>(nullptr));
    if (e != hipSuccess) return e;
    if ((e = mark(1)) != hipSuccess) return e;
  }
  if (several) {
    if ((e = launch_fast_gather_tokens(a, s)) != hipSuccess) return e;
    if ((e = mark(2)) != hipSuccess) return e;
  } else {
    FastGatherParams p{};
    p.keys = sel_keys; p.N = a.N; p.kprime = kp_sel; p.d = a.d;
    p.fr = fr; p.W1 = a.w1u; p.x = reinterpret_cast<const uint4*>(a.x);
    p.n_cand = a.n_cand; p.h32 = a.h32; p.h64 = a.h; p.gs = gs; p.u32 = a.u32;
    p.own_blocks = (a.N + kOwnUnits - 1) / kOwnUnits;
    p.Wd = a.dense_w1u; p.m1 = a.m1; p.hd = a.h_dense;
    const dim3 grid(p.own_blocks + (a.m1 + kGW - 1) / kGW);
    const size_t lds = (size_t)a.d * 4;
    auto go = [&](auto kernel) { return launch(kernel, grid, dim3(kGT), lds, s, p); };
    // The fewest loads that hold the keys: every pass over them is as long as a thread's share.
    // Units: two rows of a wave at a time.  At k' = N / 5 every eighth workgroup has more than sixteen rows, and a second trip
    // would make it the last to end.  Groups of eight, whose rows come by eights: one.  us per step, one / two rows at a time:
    // units of the int4 scorer, k' = 0.1, 0.2, 0.3 N: 1000 of d = 2048 15.5 / 15.5, 16.6 / 16.5, 16.9 / 17.1; 4000 16.0 / 16.0,
    // 17.2 / 17.1, 18.2 / 18.1; 16384 19.7 / 19.8, 22.2 / 22.0, 24.3 / 24.5; k' = N / 5: 8192 of d = 1024 17.4 / 17.0, of
    // d = 4096 22.9 / 22.6; fp64 keys, 4000 of d = 2048 18.6 / 18.8, 20.1 / 20.0, 21.3 / 21.4; 16384 24.3 / 24.5, 27.0 / 27.2,
    // 29.9 / 29.8.  Groups, int4: 16384 units of d = 2048 21.9 / 22.6; fp64 keys: 13648 units of d = 2048, r = 32 21.9 / 22.4,
    // r = 128 23.6 / 24.5, with 2736 dense units 28.8 / 29.9; 8192 of d = 4096 29.2 / 30.3.
    static_assert(kFastMaxUnits / 8 <= 4096, "groups need the fewest loads");
    if (lowrank)
      e = gs ? go(k_fast_gather<uint64_t, 2, 1>)
             : (n_sel <= 4096 ? go(k_fast_gather<uint64_t, 2, 2>)
                              : (n_sel <= 8192 ? go(k_fast_gather<uint64_t, 4, 2>) : go(k_fast_gather<uint64_t, 8, 2>)));
    else
      e = gs ? go(k_fast_gather<uint32_t, 1, 1>)
             : (n_sel <= 4096 ? go(k_fast_gather<uint32_t, 1, 2>)
                              : (n_sel <= 8192 ? go(k_fast_gather<uint32_t, 2, 2>) : go(k_fast_gather<uint32_t, 4, 2>)));
    if (e != hipSuccess) return e;
    if ((e = mark(2)) != hipSuccess) return e;
  }
  {
    FastW2Params p{};
    p.h32 = a.h32; p.h64 = a.h; p.n = n_sel; p.k = k_sel; p.d = a.d; p.fr = fr; p.W2 = a.w2u;
    p.topk_idx = a.topk_idx; p.topk_val = a.topk_val; p.y = a.y;
    p.B = a.B; p.entries = ffn_fast_entries(a.N, gs); p.bitmap = a.bitmap; p.n_cand = a.n_cand;
    // The narrowest slices whose workgroups fit the compute units, one each: what is left over would wait for a whole
    // workgroup's time (registers do not admit two).  Two workgroups more per token write the selected entries and the
    // shortlist; where slices of half the width fit without them, the slices' workgroups do it for groups of eight (four tokens
    // of d = 2048 with 2736 dense units: 39.2 us per step against 40.4, eight: 52.8 against 58.3).  Not for units, us per step
    // without / with it: four tokens at the ~1B shape 35.3 / 35.2, with the rows in the caches 35.2 / 35.6, 8192 units 30.6 / 31.1, 4000
    // 28.9 / 29.5; eight of d = 1024, 8000 units 28.1 / 29.5; two of d = 4096, 8192 units 33.5 / 34.2.
    const int extra = (a.topk_idx || a.topk_val ? 1 : 0) + (a.cand_out || (several && a.n_cand) ? 1 : 0);
    int cols = 32, cols_alone = 32;  // with the extra workgroups, without
    while (cols < 128 && ((a.d + cols - 1) / cols + extra) * a.B > 256) cols *= 2;
    while (cols_alone < cols && (a.d + cols_alone - 1) / cols_alone * a.B > 256) cols_alone *= 2;
    p.shared_out = several && gs != 0 && cols_alone < cols ? 1 : 0;
    if (p.shared_out) cols = cols_alone;
    if (lowrank && !several) cols = 32;
    p.col_slices = (a.d + cols - 1) / cols;
    int blocks = p.col_slices;
    p.out_block = !p.shared_out && (a.topk_idx || a.topk_val) ? blocks++ : -1;
    p.list_block = !p.shared_out && (a.cand_out || (several && a.n_cand)) ? blocks++ : -1;
    // several tokens read the dense rows of a slice: on one die (workgroups go round the eight), so that they come from
    // its L2 for all but the first
    if (several && a.m1 > 0) blocks = (blocks + 7) / 8 * 8;
    p.keys = sel_keys; p.kprime = kp_sel;
    p.cand_out = a.cand_out || !several || !a.n_cand ? a.cand_out : a.cand_scratch;  // (the length is wanted: listed)
    p.gs = gs; p.u32 = a.u32;
    p.W2d = a.dense_w2u; p.hd = a.h_dense; p.m1 = a.m1;
    auto go = [&](auto kernel) { return launch(kernel, dim3(blocks, a.B), dim3(kWT), 0, s, p); };
    auto by_cols = [&](auto k32, auto k64, auto k128) { return cols == 32 ? go(k32) : (cols == 64 ? go(k64) : go(k128)); };
    if (lowrank && !several)  // (its list of the shortlist reads the fp64 keys)
      e = n_sel <= 4096 ? go(k_fast_w2<uint64_t, 1, 32>)
                        : (n_sel <= 8192 ? go(k_fast_w2<uint64_t, 2, 32>) : go(k_fast_w2<uint64_t, 4, 32>));
    else if (p.shared_out)  // groups: 2048 at most
      e = cols == 32 ? go(k_fast_w2<uint32_t, 1, 32, true>) : go(k_fast_w2<uint32_t, 1, 64, true>);
    else if (n_sel <= 4096)
      e = by_cols(k_fast_w2<uint32_t, 1, 32>, k_fast_w2<uint32_t, 1, 64>, k_fast_w2<uint32_t, 1, 128>);
    else if (n_sel <= 8192)
      e = by_cols(k_fast_w2<uint32_t, 2, 32>, k_fast_w2<uint32_t, 2, 64>, k_fast_w2<uint32_t, 2, 128>);
    else
      e = by_cols(k_fast_w2<uint32_t, 4, 32>, k_fast_w2<uint32_t, 4, 64>, k_fast_w2<uint32_t, 4, 128>);
    if (e != hipSuccess) return e;
  }
  return mark(3);
}

}  // namespace hire

#ifdef HIRE_TIMESTAMPS
extern "C" int hire_debug_timestamps_fast(unsigned long long* host64) {
  return (int)hipMemcpyFromSymbol(host64, HIP_SYMBOL(hire_ts), sizeof(hire_ts));
}
#endif
