// Exact pre-activations on the candidate union for batches (arXiv 2402.09360, Algorithm 1 line 2):
//   h[b, t] = phi(<z_{U[t]}, x_b>),  t < |U|,
// on the fp64 matrix cores.  A workgroup owns 16 candidate rows and 16 tokens and accumulates their 16 x 16
// tile with 16x16x4 MFMAs: tokens are the A matrix, candidate rows the B matrix, so lane l of the result holds
// candidate l % 16 for tokens l / 16 + 4 r, r = 0..3.  Every lane converts its own bf16 operands: lane (j, g)
// reads 16-byte chunks 4 * it + g of candidate row j and of token j - no sharing between lanes, hence no LDS
// staging - and feeds the eight values of a chunk to eight consecutive MFMAs.  Which position of the row goes
// to which MFMA is free as long as both operands agree, since the order of a sum's terms is.
//
// The four waves of the workgroup split the row's chunks between them (a union of a few thousand rows gives
// too few tiles to occupy the machine otherwise) and add their partial tiles through LDS in a fixed order.
//
// fp64 accumulation of products that are exact (bf16 x bf16 fits fp32, let alone fp64) keeps the ranking that
// follows independent of the summation order up to the last bits of a double.
#include "device_utils.h"
#include "hist.h"
#include "kernels.h"
#include "keys_select.h"

namespace hire {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kGmBatch = 2;  // 16-byte chunks per lane in flight for each operand

// TOK: tokens per tile.  16: the 16x16x4 MFMA as described.  4 (batches of at most four): the 4x4x4 MFMA of four
// independent blocks - lane l then holds candidate l % 16 (block l / 4 % 4, column l % 4) and K group l / 16 on
// the weight side as before, token l % 4 on the token side, and the result for candidate l % 16 and token l / 16 -
// a quarter of the matrix-core time of a 16-token tile that is three quarters padding.
// gs > 0 (group-sparse FFN, eq. (6)): list entries are groups of 2^gs <= 16 adjacent rows, a tile covers 16 >> gs
// of them, and the result of row l of entry e goes to column e * 2^gs + l of h.  Counts stay in entries.
template <int TOK>
__global__ __launch_bounds__(256) void k_gather_dot_mfma(const uint16_t* __restrict__ W, const uint16_t* __restrict__ x,
                                                         int B, int d, const int32_t* __restrict__ list, int n_host,
                                                         const int32_t* __restrict__ n_dev, int n_cap, int relu,
                                                         double* __restrict__ h, long long stride_h,
                                                         GatherUnion un, int gs) {
  constexpr int kAcc = TOK == 16 ? 4 : 1;  // result values per lane
  __shared__ double red[3][kAcc][kWave];
  __shared__ SelSharedT<256> sh;
  __shared__ int32_t rows_sh[16];
  HIRE_TS(50);
  const int tile = (int)blockIdx.x;
  const int lane = lane_id(), w = wave_id(), jl = lane & 15, g = lane >> 4;
  const int ept = 16 >> gs, e0 = tile * ept;  // entries per tile, the tile's first entry
  int n;                                      // entries
  if (un.bitmap != nullptr) {  // the workgroup finds its candidates in the union bitmap itself
    n = un.words <= 4 * 64 * kLocateStepsShort ? union_locate<256, kLocateStepsShort>(un.bitmap, un.words, sh, e0, ept, rows_sh)
                                               : union_locate<256>(un.bitmap, un.words, sh, e0, ept, rows_sh);
    n = min(n, n_cap);
    if (blockIdx.y == 0) {
      if (tile == 0) publish_union(un, n);
      const int t = (int)threadIdx.x;
      if (t < ept && e0 + t < n) un.list_out[e0 + t] = rows_sh[t];
    }
  } else {
    n = n_dev ? min(*n_dev, n_cap) : n_host;
  }
  n <<= gs;  // rows from here on
  HIRE_TS(51);
  const int tok = (int)blockIdx.y * TOK + (TOK == 16 ? jl : (jl & 3));
  const bool live = tile * 16 < n;  // uniform over the workgroup
  const int t_idx = tile * 16 + jl;
  v4d acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = acc0;  // two independent chains (16 tokens)
  double sacc0 = 0.0, sacc1 = 0.0;                 // the same for 4 tokens
  if (live) {
    const int cpr = d / 8;  // 16-byte chunks per row
    const int tc = min(t_idx, n - 1);
    const int te = tc >> gs;  // the row's entry
    const int cand = ((un.bitmap != nullptr ? rows_sh[te - e0] : (list != nullptr ? list[te] : te)) << gs) +
                     (tc & ((1 << gs) - 1));
    const uint4* wrow = reinterpret_cast<const uint4*>(W + (size_t)cand * d);
    const uint4* xrow = reinterpret_cast<const uint4*>(x + (size_t)min(tok, B - 1) * d);
    const int nit = (cpr + 3) / 4;
    const int per_wave = (nit + 3) / 4;
    const int it_lo = w * per_wave, it_hi = min(nit, it_lo + per_wave);

    auto fetch = [&](int it0, uint4 (&wv)[kGmBatch], uint4 (&tv)[kGmBatch]) {
#pragma unroll
      for (int u = 0; u < kGmBatch; ++u) {
        const int c = (it0 + u) * 4 + g;
        const int cc = min(c, cpr - 1);
        // clamped and unconditional: the loads of a batch must not wait for one another.  Plain loads: consecutive
        // loads share cache lines (64 bytes of a row each)
        wv[u] = wrow[cc];
        tv[u] = xrow[cc];
      }
    };

    auto mac = [&](int it0, const uint4 (&wv)[kGmBatch], const uint4 (&tv)[kGmBatch]) {
#pragma unroll
      for (int u = 0; u < kGmBatch; ++u) {
        // past the wave's share or the row's end: zero weights, the product vanishes whatever the token holds
        const uint32_t keep = (it0 + u < it_hi && (it0 + u) * 4 + g < cpr) ? 0xFFFFFFFFu : 0u;
        const uint32_t wd[4] = {wv[u].x & keep, wv[u].y & keep, wv[u].z & keep, wv[u].w & keep};
        const uint32_t td[4] = {tv[u].x, tv[u].y, tv[u].z, tv[u].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (TOK == 16) {
            acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)bf16_lo(td[q]), (double)bf16_lo(wd[q]), acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)bf16_hi(td[q]), (double)bf16_hi(wd[q]), acc1, 0, 0, 0);
          } else {
            sacc0 = __builtin_amdgcn_mfma_f64_4x4x4f64((double)bf16_lo(td[q]), (double)bf16_lo(wd[q]), sacc0, 0, 0, 0);
            sacc1 = __builtin_amdgcn_mfma_f64_4x4x4f64((double)bf16_hi(td[q]), (double)bf16_hi(wd[q]), sacc1, 0, 0, 0);
          }
        }
      }
    };

    // two register sets in turn: the loads of the next batch are issued before the current one is consumed (the
    // scheduling barriers keep the compiler from sinking them to their first use)
    uint4 wa[kGmBatch], ta[kGmBatch], wb[kGmBatch], tb[kGmBatch];
    fetch(it_lo, wa, ta);
    HIRE_TS(52);
    for (int it0 = it_lo; it0 < it_hi; it0 += 2 * kGmBatch) {
      fetch(it0 + kGmBatch, wb, tb);
      __builtin_amdgcn_sched_barrier(0);
      mac(it0, wa, ta);
      __builtin_amdgcn_sched_barrier(0);
      fetch(it0 + 2 * kGmBatch, wa, ta);
      __builtin_amdgcn_sched_barrier(0);
      mac(it0 + kGmBatch, wb, tb);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  HIRE_TS(53);
  double acc[kAcc];
  if constexpr (TOK == 16) {
    const v4d a = acc0 + acc1;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = a[r];
  } else {
    acc[0] = sacc0 + sacc1;
  }
  if (w > 0) {
#pragma unroll
    for (int r = 0; r < kAcc; ++r) red[w - 1][r][lane] = acc[r];
  }
  __syncthreads();
  if (w > 0) return;
#pragma unroll
  for (int r = 0; r < kAcc; ++r) {
    // 16-token tiles interleave the rows over the lane groups; a 4-token tile has token l / 16 in lane l
    const int tk = (int)blockIdx.y * TOK + g + 4 * r;
    double s = ((acc[r] + red[0][r][lane]) + red[1][r][lane]) + red[2][r][lane];
    if (relu) s = s > 0.0 ? s : 0.0;
    if (s == 0.0) s = 0.0;
    const bool valid = live && tk < B && t_idx < n;
    if (valid) h[(size_t)tk * stride_h + t_idx] = s;
  }
  HIRE_TS(54);
}

// ---------------------------------------------------------------------------------------------------
// Low-rank scorer for batches: keys[b, j] = phi(<Z2[j, :], t_b>) over all rows of Z2, the operands as in
// k_gather_dot_mfma.  The rows are short (r values), so a wave has sixteen rows to itself and no share of the columns:
// no LDS, no barrier, eight 16-byte chunks of both operands requested together.  Measured at r = 128, 16384 rows, 16
// tokens: 5.0 us, against 9.4 with k_gather_dot_mfma, whose four waves had 32 columns each and added their tiles in LDS.
constexpr int kLsThreads = 256;
__global__ __launch_bounds__(kLsThreads) void k_lr_score_mfma(const uint16_t* __restrict__ z2, const uint16_t* __restrict__ t,
                                                              int B, int N, int r, int relu, double* __restrict__ keys,
                                                              long long stride) {
  constexpr int kDepth = 4;
  const int lane = lane_id(), jl = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(wave_id());  // uniform for the matrix cores
  const int j0 = ((int)blockIdx.x * (kLsThreads / kWave) + w) * 16, j = j0 + jl, cpr = r / 8;
  if (j0 >= N) return;  // uniform
  const uint4* zrow = reinterpret_cast<const uint4*>(z2 + (size_t)min(j, N - 1) * r);
  const uint4* trow = reinterpret_cast<const uint4*>(t + (size_t)min((int)blockIdx.y * 16 + jl, B - 1) * r);
  v4d acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
  for (int c0 = 0; c0 < cpr; c0 += 4 * kDepth) {
    uint4 zv[kDepth], tv[kDepth];
#pragma unroll
    for (int u = 0; u < kDepth; ++u) {
      const int c = min(c0 + 4 * u + g, cpr - 1);
      zv[u] = zrow[c];
      tv[u] = trow[c];
    }
#pragma unroll
    for (int u = 0; u < kDepth; ++u)
      if (c0 + 4 * u < cpr) {  // uniform
        const uint32_t keep = c0 + 4 * u + g < cpr ? 0xFFFFFFFFu : 0u;  // past the row's end: zeros
        const uint32_t zd[4] = {zv[u].x & keep, zv[u].y & keep, zv[u].z & keep, zv[u].w & keep};
        const uint32_t td[4] = {tv[u].x & keep, tv[u].y & keep, tv[u].z & keep, tv[u].w & keep};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)bf16_lo(td[q]), (double)bf16_lo(zd[q]), acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)bf16_hi(td[q]), (double)bf16_hi(zd[q]), acc[1], 0, 0, 0);
        }
      }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int b = (int)blockIdx.y * 16 + g + 4 * i;
    double s = acc[0][i] + acc[1][i];
    if (relu) s = s > 0.0 ? s : 0.0;
    if (s == 0.0) s = 0.0;
    if (b < B && j < N) keys[(size_t)b * stride + j] = s;
  }
}

hipError_t launch_lr_score_mfma(const uint16_t* z2, const uint16_t* t, int B, int N, int r, int relu, double* keys,
                                long long stride, hipStream_t s) {
  constexpr int kRows = 16 * kLsThreads / kWave;
  return launch(k_lr_score_mfma, dim3((N + kRows - 1) / kRows, (B + 15) / 16), dim3(kLsThreads), 0, s, z2, t, B, N, r, relu,
                keys, stride);
}

// ---------------------------------------------------------------------------------------------------
// Filter stage of the exact pre-activations for batches (filter and refine): candidate rows times tokens on the
// bf16 matrix cores, 50 times the fp64 rate, so the stage is a read of the candidate rows.  Tokens are the A matrix,
// candidate rows the B matrix of a 16x16x32 MFMA: lane (j, g) feeds 16-byte chunk 4 it + g of token j and of
// candidate j as they come from memory, no conversion; result value i of lane l belongs to token 4 (l / 16) + i
// and candidate l % 16.
//
// What is stored is not the activation but a value within a proven distance of it.  Every MFMA (with more than
// 32 tokens, where the fp64 additions pace the kernel: every second one) starts from a zero accumulator, so a
// segment is the sum of S = 32 (64) products, each exact in fp32, after at most S roundings, each bounded - whether the hardware rounds to nearest, truncates, or aligns the products to the
// largest before adding - by 2^-23 of a running sum that never exceeds the segment's sum of |u_i x_i|.  The
// segments are added in fp64, whose own error is below 2^-40 of the same sums, and the total is rounded to fp32
// (2^-24 of it).  Hence, with a factor two of margin and Cauchy-Schwarz:
//   |stored - <u_j, x_b>| <= delta(b, j) = S 2^-22 |u_j| |x_b| = 2^-17 (2^-16) |u_j| |x_b|,   whatever d.
// The squared norms are the diagonals of two more MFMA chains (rows times rows, tokens times tokens; sums of
// non-negative terms, so their d roundings cost at most d 2^-23 relatively: rounded up by more than that).
// Stored per (token, candidate), as fp32 - with phi = identity (RELU false: the classifier) the sum itself; with
// the ReLU: the sum if it is positive (never rounded to zero); the smallest
// positive float if it lies in (-2 delta, 0], where the true activation may still be positive; exactly 0 below
// that, where the true activation is exactly 0.  The selection (k_refine) recomputes in fp64 the entries
// whose stored value lies within 2 max_j delta(b, j) of the k-th largest stored value and selects on the result:
// the selected set is that of the fp64 values.  xnorm[b] receives an upper bound of |x_b|, wnorm_tiles[i] one of the
// largest |u_j| over workgroup i's candidates (or, without it, *wnorm_max over all: float bits, atomic max).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& u) {
  bf16x8 v;
  __builtin_memcpy(&v, &u, sizeof(v));
  return v;
}
__device__ __forceinline__ float pick4(const f32x4& v, int i) {
  return i == 0 ? v[0] : (i == 1 ? v[1] : (i == 2 ? v[2] : v[3]));
}

// Layout.  A workgroup owns 64 candidates and all of the batch's tokens (TT tiles of 16): 4 groups of 16
// candidates times TG shares of the token tiles times KS shares of every stage's K steps, one wave each (the K shares
// are added in fp64 at the end).  K goes by in stages of 128 elements: 256 bytes of
// every row, brought into LDS by asynchronous 16-byte loads that bypass the registers (a wave's instruction fills 1
// KiB, four rows), kStages deep: a stage is requested three stages before it is used, and one barrier per stage
// (which also waits for this wave's share of it) is all the synchronisation.  LDS position p of a row holds its chunk
// p ^ (row % 16), so that the sixteen lanes that read one chunk column of sixteen rows hit different banks; the
// permutation is applied to the addresses the lanes load from (inside two cache lines).  Rows past the candidates'
// end repeat the last one and tokens past the batch the last token: their results are dropped.
//
// k_filter_units (the FFN): the workgroup's candidates are the set bits of its own 64 units' bitmap words, so nothing has to be
// located and nothing mapped back: stored values go to h[token][unit], zeros where a unit is no candidate (a ReLU
// activation of zero never displaces a positive one; the selection asks the bitmap where zeros are selected).
//
// Bound: HBM; one workgroup per compute unit keeps 48 KB of rows in flight.  Measured at d = 2048: 16 tokens, 15900
// candidates (65 MB) 14.5 us (17.4 with all workgroups starting in the same columns, see launch_filter_units), 64 tokens,
// 16384 candidates 19.7 us (of which the stages 12: 5.6 TB/s).  The kernel before this one staged through registers and
// located its candidates by rank: 22.4 us at 16 tokens, 30 at 64.  KS = 1: 17.6 and 19.9, not turned.
constexpr int kFtRows = 64;        // candidates per workgroup
constexpr int kFtChunks = 16;      // 16-byte chunks of a row per stage
constexpr int kFtStages = 4;
constexpr int kFtRowBytes = 16 * kFtChunks;
constexpr int kFtSteps = kFtChunks / 4;  // MFMA steps per stage
constexpr int ft_stage_bytes(int TT) { return (kFtRows + 16 * TT) * kFtRowBytes; }

// Asynchronous load of 16 bytes per lane into LDS: lane l's go to lds_off + 16 l.  Not tracked by the compiler: the
// barrier below waits for it.
__device__ __forceinline__ void load_to_lds(const void* g, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g),
               "s"(__builtin_amdgcn_readfirstlane((int)lds_off))
               : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}
// Workgroup barrier behind which everything but this wave's N youngest loads has arrived and every LDS read of the
// workgroup is done.
template <int N>
__device__ __forceinline__ void stage_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
// The same for the ST - 2 youngest stages of ci <= CI candidate and TI token loads (uniform; everything unless `whole`).
template <int CI, int TI, int ST = kFtStages>
__device__ __forceinline__ void stage_barrier_loads(int ci, bool whole) {
  if (!whole) {
    stage_barrier<0>();
  } else if constexpr (CI == 1) {
    stage_barrier<(ST - 2) * (1 + TI)>();
  } else {
    if (ci >= CI) stage_barrier<(ST - 2) * (CI + TI)>();
    else stage_barrier_loads<CI - 1, TI, ST>(ci, true);
  }
}

// Geometry of the filter kernels and what a wave accumulates.
template <int TT, int TG, int KS>
struct FtShape {
  static constexpr int NW = 4 * TG * KS, NT = 64 * NW, TTW = TT / TG;
  static constexpr int kSteps = kFtSteps / KS;                              // MFMA steps per wave and stage
  static constexpr int CI = kFtRows / (4 * NW);                             // load instructions per wave and stage:
  static constexpr int TI = 16 * TT > 4 * NW ? 16 * TT / (4 * NW) : 1;      // candidates, tokens (fewer than one per
                                                                            // wave: loaded twice)
  static constexpr int kStage = ft_stage_bytes(TT);
  static constexpr int kSegSteps = filter_segment_steps(16 * TT);           // MFMA steps per fp32 segment
  static_assert(TT % TG == 0 && CI >= 1 && 4 * CI * NW == kFtRows && kSteps % kSegSteps == 0, "equal shares");
  static_assert(4 * TI * NW == 16 * TT || 4 * NW % (16 * TT) == 0, "whole token rows");
  static_assert(4 * NW % 16 == 0, "a lane's chunk is the same for all of its load instructions");
};
template <int TTW>
struct FtAcc {
  double sum[TTW][4];
  f32x4 ww, xx[TTW];  // rows times rows (waves of the first token share); tokens times tokens (group 0's waves)
};

// One stage of one wave: slot: the stage in LDS; left: chunks of the rows from this stage on.
template <int TT, int TG, int KS>
__device__ __forceinline__ void ft_stage(const unsigned char* slot, int cw, int tt0, int kh, int left, bool token_norms,
                                         FtAcc<TT / TG>& a) {
  using S = FtShape<TT, TG, KS>;
  constexpr int TTW = S::TTW, kSteps = S::kSteps, kSegSteps = S::kSegSteps, kSeg = kSteps / kSegSteps;
  const int lane = lane_id(), jl = lane & 15, g = lane >> 4;
  const unsigned char* wcol = slot + (16 * cw + jl) * kFtRowBytes;
  const unsigned char* xcol = slot + (kFtRows + 16 * tt0 + jl) * kFtRowBytes;
  bf16x8 wk[kSteps], tk[TTW][kSteps];
#pragma unroll
  for (int u = 0; u < kSteps; ++u) {
    const int o = ((4 * (u + kh * kSteps) + g) ^ jl) * 16;
    wk[u] = as_bf16x8(*reinterpret_cast<const uint4*>(wcol + o));
#pragma unroll
    for (int t = 0; t < TTW; ++t) tk[t][u] = as_bf16x8(*reinterpret_cast<const uint4*>(xcol + t * 16 * kFtRowBytes + o));
  }
  if (left < kFtChunks) {  // uniform: the row ends inside the stage
#pragma unroll
    for (int u = 0; u < kSteps; ++u)
      if (4 * (u + kh * kSteps) + g >= left) {
        wk[u] = as_bf16x8(make_uint4(0, 0, 0, 0));
#pragma unroll
        for (int t = 0; t < TTW; ++t) tk[t][u] = as_bf16x8(make_uint4(0, 0, 0, 0));
      }
  }
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 part[TTW][kSeg];
#pragma unroll
  for (int v = 0; v < kSegSteps; ++v)
#pragma unroll
    for (int t = 0; t < TTW; ++t)
#pragma unroll
      for (int q = 0; q < kSeg; ++q)
        part[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tk[t][kSegSteps * q + v], wk[kSegSteps * q + v],
                                                             v == 0 ? zero : part[t][q], 0, 0, 0);
  if (tt0 == 0) {  // uniform
#pragma unroll
    for (int u = 0; u < kSteps; ++u) a.ww = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wk[u], wk[u], a.ww, 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < TTW; ++t) {
    if (cw == 0 && token_norms) {  // uniform
#pragma unroll
      for (int u = 0; u < kSteps; ++u)
        a.xx[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tk[t][u], tk[t][u], a.xx[t], 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < kSeg; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) a.sum[t][r] += (double)part[t][q][r];
  }
}

struct FilterUnits {
  const uint16_t* W;
  const uint16_t* x;
  int B, d;
  const uint32_t* bitmap;  // candidates; nullptr: every row below the count
  const int32_t* n_dev;    // optional count
  int n_cap;
  float* h;
  long long stride_h;
  float* xnorm;
  float* wnorm_tiles;
  uint32_t* wnorm_max;
  float err_c;
  int turn;                // the workgroups of a die start in different stages (launch_filter_units)
};

// The 64 units of a tile, by a workgroup; lds: kFtStages stages.
template <int TT, int TG, int KS, bool TURN>
__device__ __forceinline__ void filter_units_tile(const FilterUnits& p, int tile, unsigned char* lds) {
  using S = FtShape<TT, TG, KS>;
  constexpr int NW = S::NW, NT = S::NT, TTW = S::TTW, CI = S::CI, TI = S::TI, kStage = S::kStage;
  __shared__ int32_t rows_sh[kFtRows];
  __shared__ float xsq[KS][TT][16];
  __shared__ float wmx[4];
  const uint16_t* __restrict__ W = p.W;
  const uint16_t* __restrict__ x = p.x;
  const uint32_t* __restrict__ bitmap = p.bitmap;
  float* __restrict__ h = p.h;
  const long long stride_h = p.stride_h;
  const int B = p.B, d = p.d;
  const float err_c = p.err_c;
  const int tid = (int)threadIdx.x, lane = lane_id(), jl = lane & 15, g = lane >> 4;
  // known to be uniform: a matrix-core instruction must never sit behind a branch that is lowered to lane masking
  const int w = __builtin_amdgcn_readfirstlane(wave_id());
  const int e0 = tile * kFtRows;  // first unit of the workgroup
  const int cpr = d / 8;          // 16-byte chunks per row
  HIRE_TS(55);
  uint64_t m;
  if (bitmap != nullptr) {
    m = reinterpret_cast<const uint64_t*>(bitmap)[tile];  // padded to whole 64-bit words, no bits past the rows
  } else {  // every row below the count
    const int left = (p.n_dev != nullptr ? min(*p.n_dev, p.n_cap) : p.n_cap) - e0;
    m = left >= 64 ? ~0ull : (left > 0 ? (1ull << left) - 1ull : 0ull);
  }
  m = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(m >> 32)) << 32) |
      (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
  const int c = __popcll(m);  // candidates of the workgroup
  // The tokens' norms that p.xnorm receives are the first tile's, which reads its first unit's row where it has no candidate: a
  // norm's last bits go by the stage that its sum starts in, and k_refine's band must not go by which workgroup ends last.
  const int rows = max(c, tile == 0 ? 1 : 0);  // read
  if (w == 0 && ((m >> lane) & 1ull)) rows_sh[mask_prefix(m)] = e0 + lane;
  else if (tid == 0 && c == 0) rows_sh[0] = e0;
  __syncthreads();
  HIRE_TS(56);
  const int cw = w & 3, tt0 = (w >> 2) % TG * TTW, kh = (w >> 2) / TG;  // this wave's candidates, tokens, steps (uniform)
  FtAcc<TTW> acc{};
  if (rows > 0) {
    const uint32_t base = lds_offset(lds);
    const int nst = (cpr + kFtChunks - 1) / kFtChunks;
    const int ci = (rows + 4 * NW - 1) / (4 * NW);  // candidate loads of a stage: groups without candidates are left out
    // instruction i of this wave fills rows 4 NW i + 4 w .. + 3 of the candidates' (tokens') part of a stage
    const char* wptr[CI];
    const char* xptr[TI];
    const int r4 = 4 * w + g, ch = jl ^ (r4 & 15);  // lane's row inside an instruction's stripe, its chunk of a stage
#pragma unroll
    for (int i = 0; i < CI; ++i)
      wptr[i] = reinterpret_cast<const char*>(W + (size_t)rows_sh[min(4 * NW * i + r4, rows - 1)] * d);
#pragma unroll
    for (int i = 0; i < TI; ++i) xptr[i] = reinterpret_cast<const char*>(x + (size_t)min((4 * NW * i + r4) % (16 * TT), B - 1) * d);
    auto request = [&](int st, int slot) {
      const int at = kFtChunks * st + ch;
      const int off = 16 * (at < cpr ? at : 0);  // past the row's end: its first chunk, masked when it is used
      const uint32_t to = base + slot * kStage + 1024 * w;
      const uint32_t to_tok = base + slot * kStage + kFtRows * kFtRowBytes + 1024 * w % (16 * TT * kFtRowBytes);
#pragma unroll
      for (int i = 0; i < CI; ++i)
        if (i < ci) load_to_lds(wptr[i] + off, to + 1024 * NW * i);
#pragma unroll
      for (int i = 0; i < TI; ++i) load_to_lds(xptr[i] + off, to_tok + 1024 * NW * i);
    };
    // the stages in order, or (TURNED) from stage `from` on round the end of the row
    auto run = [&](auto turned, int from) __attribute__((always_inline)) {
      constexpr bool TURNED = decltype(turned)::value;
      auto stage_of = [&](int st) { return !TURNED ? st : (st + from < nst ? st + from : st + from - nst); };
#pragma unroll
      for (int st = 0; st < kFtStages - 1; ++st)
        if (st < nst) request(stage_of(st), st);
      int slot = 0;
      for (int st = 0; st < nst; ++st) {
        stage_barrier_loads<CI, TI>(ci, st + kFtStages - 2 < nst);
        if (st + kFtStages - 1 < nst) request(stage_of(st + kFtStages - 1), slot == 0 ? kFtStages - 1 : slot - 1);
        if (16 * cw < rows)  // uniform
          ft_stage<TT, TG, KS>(lds + slot * kStage, cw, tt0, kh, cpr - kFtChunks * stage_of(st), true, acc);
        slot = slot == kFtStages - 1 ? 0 : slot + 1;
      }
    };
    if (TURN && p.turn && c > 3 * kFtRows / 4) run(std::true_type{}, tile / 8 % nst);  // uniform
    else run(std::false_type{}, 0);
  }
  HIRE_TS(57);
  // LDS from here on: the result tile [16 TT][64], the rows' squared norms [KS][64], the other K shares' sums
  float* tile_out = reinterpret_cast<float*>(lds);
  float* wsq = tile_out + 16 * TT * kFtRows;
  double* shares = reinterpret_cast<double*>(wsq + KS * kFtRows);  // [KS - 1][4 TG][TTW * 4][64]
  static_assert((16 * TT + KS) * kFtRows * 4 + (KS - 1) * 4 * TG * TTW * 4 * kWave * 8 <= kFtStages * kStage, "LDS");
  __syncthreads();  // the stages' memory is free
  // entry (i, i) of a 16 x 16 result sits in value i % 4 of lane 16 (i / 4) + i.  Token norms from group 0's waves,
  // candidate norms from those of the first token share
  if (cw == 0 && (jl >> 2) == g) {
#pragma unroll
    for (int t = 0; t < TTW; ++t) xsq[kh][tt0 + t][jl] = pick4(acc.xx[t], jl & 3);
  }
  if (tt0 == 0 && (jl >> 2) == g) wsq[kh * kFtRows + 16 * cw + jl] = pick4(acc.ww, jl & 3);
  if (KS > 1 && kh > 0) {
#pragma unroll
    for (int t = 0; t < TTW; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        shares[((((kh - 1) * TG + tt0 / TTW) * 4 + cw) * TTW * 4 + t * 4 + r) * kWave + lane] = acc.sum[t][r];
  }
  for (int i = tid; i < 16 * TT * kFtRows / 4; i += NT) reinterpret_cast<float4*>(tile_out)[i] = make_float4(0, 0, 0, 0);
  __syncthreads();
  const float up = 1.0f + (float)d * 0x1p-22f;  // more than the relative error of the norms' sums
  const int ce = 16 * cw + jl;                  // this lane's candidate
  float wn2 = 0.0f;
#pragma unroll
  for (int q = 0; q < KS; ++q) wn2 += wsq[q * kFtRows + ce];
  wn2 *= up;
  if (w < 4) {  // tt0 == 0, kh == 0
    float m = ce < c ? wn2 : 0.0f;
    m = fmaxf(m, __shfl_xor(m, 1));
    m = fmaxf(m, __shfl_xor(m, 2));
    m = fmaxf(m, __shfl_xor(m, 4));
    m = fmaxf(m, __shfl_xor(m, 8));
    if (lane == 0) wmx[cw] = m;
  }
  if (kh == 0) {
    const double four_err2 = 4.001 * (double)err_c * (double)err_c * (double)wn2;
#pragma unroll
    for (int t = 0; t < TTW; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int tl = 4 * g + r, tk = 16 * (tt0 + t) + tl;
        double s = acc.sum[t][r];
#pragma unroll
        for (int q = 1; q < KS; ++q)
          s += shares[((((q - 1) * TG + tt0 / TTW) * 4 + cw) * TTW * 4 + t * 4 + r) * kWave + lane];
        float xn2 = 0.0f;
#pragma unroll
        for (int q = 0; q < KS; ++q) xn2 += xsq[q][tt0 + t][tl];
        const float tiny = __uint_as_float(1u);  // the smallest positive float
        float v = 0.0f;
        if (s > 0.0) v = fmaxf((float)s, tiny);
        else if (s * s < four_err2 * (double)(xn2 * up)) v = tiny;  // s > -2 delta: the true activation may be positive
        if (ce < c) tile_out[tk * kFtRows + rows_sh[ce] - e0] = v;
      }
  }
  __syncthreads();
  // 64 units of every token, 16 bytes per lane where the rows are aligned
  if (stride_h % 4 == 0) {
    for (int i = tid; i < B * (kFtRows / 4); i += NT) {
      const int t = i / (kFtRows / 4), q = 4 * (i % (kFtRows / 4));
      if (e0 + q < stride_h) *reinterpret_cast<float4*>(h + (size_t)t * stride_h + e0 + q) = *reinterpret_cast<float4*>(tile_out + 4 * i);
    }
  } else {
    for (int i = tid; i < B * kFtRows; i += NT) {
      const int t = i / kFtRows, q = i % kFtRows;
      if (e0 + q < stride_h) h[(size_t)t * stride_h + e0 + q] = tile_out[i];
    }
  }
  if (tid == 0) {  // a place per workgroup: 256 atomics on one address at the kernel's end took 7 us
    const float m = c > 0 ? sqrtf(fmaxf(fmaxf(wmx[0], wmx[1]), fmaxf(wmx[2], wmx[3]))) * 1.0001f : 0.0f;
    if (p.wnorm_tiles != nullptr) p.wnorm_tiles[tile] = m;
    else atomicMax(p.wnorm_max, __float_as_uint(m));
  }
  if (tile == 0)  // uniform
    for (int t = tid; t < B; t += NT) {
      float xn2 = 0.0f;
#pragma unroll
      for (int q = 0; q < KS; ++q) xn2 += xsq[q][t / 16][t % 16];
      p.xnorm[t] = sqrtf(xn2 * up) * 1.0001f;
    }
  HIRE_TS(58);
}

template <int TT, int TG, int KS>
__global__ __launch_bounds__(256 * TG * KS) void k_filter_units(FilterUnits p) {
  extern __shared__ __align__(16) unsigned char lds[];
  filter_units_tile<TT, TG, KS, TT <= 2>(p, (int)blockIdx.x, lds);
}

// The selection of the k' largest keys and the filter stage at once: the first workgroups select, a token each, the others
// form the values of all rows, shortlisted or not, and k_refine leaves out those that no token shortlists.  The selection
// is a chain on one compute unit per token (6 us at 16 tokens, 8 at 64) during which the rest of the chip waits; the
// stage's rows do not depend on it where nearly all of them are read anyway, or where they are few.  run_front says which
// layouts take it.  d = 2048,
// 64 tokens, 16384 rows: 23.6 us against 8.1 + 19.8 one after the other.
template <int TT, int TG, int KS, typename K, int LOADS>
__global__ __launch_bounds__(256 * TG * KS) void k_select_filter(KeysSelect ks, FilterUnits p) {
  static_assert(256 * TG * KS == kSelThreads && sizeof(KeysSelectShared<K>) <= kFtStages * ft_stage_bytes(TT), "LDS fits both");
  extern __shared__ __align__(16) unsigned char lds[];
  const int tile = (int)blockIdx.x - p.B;
  if (tile < 0) keys_select_token<K, LOADS>(ks, (int)blockIdx.x, *reinterpret_cast<KeysSelectShared<K>*>(lds));  // uniform
  else filter_units_tile<TT, TG, KS, false>(p, tile, lds);
}

// The same product for the classifier (phi = identity; the union is a small part of a long vocabulary): the candidates
// in rank order, from the union bitmap (or a list), values to h[token][rank].  Every workgroup counts the bitmap's
// bits itself and takes an equal contiguous share of the ranks - tiles of at most 64, equally long - and its stages
// run on from tile to tile: the next tile's rows are requested while the current one is finished (its sums pass
// through LDS of their own, behind barriers that do not wait for loads).  A workgroup also leaves the largest values of four
// sets of its candidates per token (maxima[token][4 workgroup + set], -inf for none): the final selection bounds the k-th
// largest logit with them instead of passing over the row for a histogram.  The sets are the waves' groups of sixteen, or,
// where short tiles fill one or two of these only, quarters or halves of them: tokens of one query share most of their
// candidates, and with fewer maxima than k everything would have to be recomputed.
// Measured at d = 2048, 64 tokens, 57600 of 256000 classes (236 MB): 65 us (3.6 TB/s); with a workgroup per tile, each locating
// its own 64 candidates first, 92.
constexpr int kFrMaxRows = 512;  // candidates per workgroup
static_assert(kFrMaxRows * 256 >= kSoftmaxRefineMaxRow, "256 workgroups hold the longest row");
constexpr int fr_stages(int TT) { return TT >= 4 ? 3 : 4; }

template <int TT, int TG, int KS>
__global__ __launch_bounds__(256 * TG * KS) void k_filter_ranks(const uint16_t* __restrict__ W, const uint16_t* __restrict__ x,
                                                          int B, int d, const int32_t* __restrict__ list,
                                                          const int32_t* __restrict__ n_dev, int n_cap,
                                                          float* __restrict__ h, long long stride_h, GatherUnion un,
                                                          float* __restrict__ xnorm, float* __restrict__ wnorm_tiles,
                                                          float* __restrict__ maxima) {
  using S = FtShape<TT, TG, KS>;
  constexpr int NW = S::NW, NT = S::NT, TTW = S::TTW, CI = S::CI, TI = S::TI, kStage = S::kStage, ST = fr_stages(TT);
  extern __shared__ __align__(16) unsigned char lds[];  // stages, then the K shares' sums [KS - 1][4 TG][TTW * 4][64]
  __shared__ int32_t rows_sh[kFrMaxRows];
  __shared__ float xsq[KS][TT][16], wsq[KS][kFtRows], wmx[4];
  double* shares = reinterpret_cast<double*>(lds + ST * kStage);
  const int tid = (int)threadIdx.x, lane = lane_id(), jl = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(wave_id());  // uniform for the matrix cores
  const int cpr = d / 8;
  int n, e0, rows;  // candidates in all, this workgroup's first rank and number
  auto share_of = [&](int total, int& r0, int& R) {
    n = __builtin_amdgcn_readfirstlane(min(total, n_cap));  // uniform, and known to be
    const int per = (n + (int)gridDim.x - 1) / (int)gridDim.x;  // <= kFrMaxRows
    r0 = e0 = (int)blockIdx.x * per;
    R = per;
  };
  if (un.bitmap != nullptr) {
    union_locate_range<NT, kUnionLocateMaxWords / NT>(un.bitmap, un.words, *reinterpret_cast<SelSharedT<NT>*>(lds), share_of,
                                                      rows_sh);
    rows = max(0, min(n - e0, (n + (int)gridDim.x - 1) / (int)gridDim.x));
    if (blockIdx.x == 0) publish_union(un, n);
    for (int i = tid; i < rows; i += NT) un.list_out[e0 + i] = rows_sh[i];
  } else {
    int r0, R;
    share_of(*n_dev, r0, R);
    rows = max(0, min(n - e0, R));
    for (int i = tid; i < rows; i += NT) rows_sh[i] = list[e0 + i];
    __syncthreads();
  }
  float* my_max = maxima + 4 * blockIdx.x;
  const int cw = w & 3, tt0 = (w >> 2) % TG * TTW, kh = (w >> 2) / TG;  // this wave's candidates, tokens, steps (uniform)
  if (rows == 0) {  // uniform over the workgroup
    if (tid == 0) wnorm_tiles[blockIdx.x] = 0.0f;
    for (int i = tid; i < 4 * B; i += NT) my_max[(size_t)(i / 4) * kFilterMaxima + i % 4] = -__builtin_inff();
    return;
  }
  const int tiles = (rows + kFtRows - 1) / kFtRows, rt = (rows + tiles - 1) / tiles;  // rows per tile
  const int nst = (cpr + kFtChunks - 1) / kFtChunks, all = tiles * nst;               // stages per tile, in all
  const int ci = (rt + 4 * NW - 1) / (4 * NW);
  const uint32_t base = lds_offset(lds);
  const int r4 = 4 * w + g, ch = jl ^ (r4 & 15);
  const char* wptr[CI];
  const char* xptr[TI];
#pragma unroll
  for (int i = 0; i < TI; ++i) xptr[i] = reinterpret_cast<const char*>(x + (size_t)min((4 * NW * i + r4) % (16 * TT), B - 1) * d);
  int req_tile = 0, req_st = 0, req_slot = 0;  // the next stage to request
  auto aim = [&]() {
    const int t0 = req_tile * rt, last = min(rows - t0, rt) - 1;
#pragma unroll
    for (int i = 0; i < CI; ++i)
      wptr[i] = reinterpret_cast<const char*>(W + (size_t)rows_sh[t0 + min(4 * NW * i + r4, last)] * d);
  };
  auto request = [&]() {
    const int at = kFtChunks * req_st + ch;
    const int off = 16 * (at < cpr ? at : 0);  // past the row's end: its first chunk, masked when it is used
    const uint32_t to = base + req_slot * kStage + 1024 * w;
    const uint32_t to_tok = base + req_slot * kStage + kFtRows * kFtRowBytes + 1024 * w % (16 * TT * kFtRowBytes);
#pragma unroll
    for (int i = 0; i < CI; ++i)
      if (i < ci) load_to_lds(wptr[i] + off, to + 1024 * NW * i);
#pragma unroll
    for (int i = 0; i < TI; ++i) load_to_lds(xptr[i] + off, to_tok + 1024 * NW * i);
    req_slot = req_slot == ST - 1 ? 0 : req_slot + 1;
    if (++req_st == nst) {
      req_st = 0;
      if (++req_tile < tiles) aim();
    }
  };
  aim();
#pragma unroll
  for (int i = 0; i < ST - 1; ++i)
    if (i < all) request();
  FtAcc<TTW> acc{};
  float vmax[TTW][4], wmax = 0.0f;
#pragma unroll
  for (int t = 0; t < TTW; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) vmax[t][r] = -__builtin_inff();
  const float up = 1.0f + (float)d * 0x1p-22f;  // more than the relative error of the norms' sums
  int slot = 0, st = 0, tile = 0;
  for (int i = 0; i < all; ++i) {
    stage_barrier_loads<CI, TI, ST>(ci, i + ST - 2 < all);
    if (i + ST - 1 < all) request();
    const int t0 = tile * rt, c = min(rows - t0, rt);  // the tile's candidates
    if (16 * cw < c) ft_stage<TT, TG, KS>(lds + slot * kStage, cw, tt0, kh, cpr - kFtChunks * st, tile == 0, acc);
    slot = slot == ST - 1 ? 0 : slot + 1;
    if (++st < nst) continue;
    // the tile is complete
    if (tile == 0 && cw == 0 && (jl >> 2) == g) {
#pragma unroll
      for (int t = 0; t < TTW; ++t) xsq[kh][tt0 + t][jl] = pick4(acc.xx[t], jl & 3);
    }
    if (tt0 == 0 && (jl >> 2) == g) wsq[kh][16 * cw + jl] = pick4(acc.ww, jl & 3);
    if (KS > 1 && kh > 0) {
#pragma unroll
      for (int t = 0; t < TTW; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          shares[((((kh - 1) * TG + tt0 / TTW) * 4 + cw) * TTW * 4 + t * 4 + r) * kWave + lane] = acc.sum[t][r];
    }
    lds_barrier();
    const int ce = 16 * cw + jl;  // this lane's candidate
    if (w < 4 && ce < c) {
      float wn2 = 0.0f;
#pragma unroll
      for (int q = 0; q < KS; ++q) wn2 += wsq[q][ce];
      wmax = fmaxf(wmax, wn2);
    }
    if (kh == 0) {
#pragma unroll
      for (int t = 0; t < TTW; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int tk = 16 * (tt0 + t) + 4 * g + r;
          double s = acc.sum[t][r];
#pragma unroll
          for (int q = 1; q < KS; ++q)
            s += shares[((((q - 1) * TG + tt0 / TTW) * 4 + cw) * TTW * 4 + t * 4 + r) * kWave + lane];
          const float v = (float)s;
          if (ce < c) {
            vmax[t][r] = fmaxf(vmax[t][r], v);
            if (tk < B) h[(size_t)tk * stride_h + e0 + t0 + ce] = v;
          }
        }
    }
    acc = FtAcc<TTW>{};
    st = 0;
    ++tile;
  }
  if (w < 4) {
    wmax = fmaxf(wmax, __shfl_xor(wmax, 1));
    wmax = fmaxf(wmax, __shfl_xor(wmax, 2));
    wmax = fmaxf(wmax, __shfl_xor(wmax, 4));
    wmax = fmaxf(wmax, __shfl_xor(wmax, 8));
    if (lane == 0) wmx[cw] = wmax;
  }
  const int groups = (rt + 15) / 16, split = groups == 1 ? 4 : (groups == 2 ? 2 : 1);  // sets of a group
  if (kh == 0 && (split == 1 || cw < groups)) {  // uniform
#pragma unroll
    for (int t = 0; t < TTW; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v = vmax[t][r];
        v = fmaxf(v, __shfl_xor(v, 1));
        v = fmaxf(v, __shfl_xor(v, 2));
        if (split < 4) v = fmaxf(v, __shfl_xor(v, 4));
        if (split < 2) v = fmaxf(v, __shfl_xor(v, 8));
        const int tk = 16 * (tt0 + t) + 4 * g + r, lanes = 16 / split;
        if (jl % lanes == 0 && tk < B) my_max[(size_t)tk * kFilterMaxima + split * cw + jl / lanes] = v;
      }
  }
  __syncthreads();
  if (tid == 0) wnorm_tiles[blockIdx.x] = sqrtf(fmaxf(fmaxf(wmx[0], wmx[1]), fmaxf(wmx[2], wmx[3])) * up) * 1.0001f;
  if (blockIdx.x == 0)
    for (int t = tid; t < B; t += NT) {
      float xn2 = 0.0f;
#pragma unroll
      for (int q = 0; q < KS; ++q) xn2 += xsq[q][t / 16][t % 16];
      xnorm[t] = sqrtf(xn2 * up) * 1.0001f;
    }
}

static int gather_mfma_tiles(int cap, int gs) { return max(1, (int)((((long long)cap << gs) + 15) / 16)); }

hipError_t launch_gather_dot_mfma(const uint16_t* W, const uint16_t* x, int B, int d, const int32_t* list, int n,
                                  const int32_t* n_dev, int n_cap, int relu, double* h, long long stride_h,
                                  const HistRefs& hr, const UnionRefs* un, int gs, hipStream_t s) {
  const int cap = n_dev ? n_cap : n;
  const GatherUnion u = make_gather_union(un, hr, B);
  if (B <= 4)
    return launch(k_gather_dot_mfma<4>, dim3(gather_mfma_tiles(cap, gs), 1), dim3(256), 0, s, W, x, B, d,
                  u.bitmap ? nullptr : list, n, n_dev, cap, relu, h, stride_h, u, gs);
  return launch(k_gather_dot_mfma<16>, dim3(gather_mfma_tiles(cap, gs), (B + 15) / 16), dim3(256), 0, s, W, x, B, d,
                u.bitmap ? nullptr : list, n, n_dev, cap, relu, h, stride_h, u, gs);
}

int filter_tiles(int n) { return max(1, (n + kFtRows - 1) / kFtRows); }
// A workgroup per compute unit while that leaves each sixteen candidates, a matrix instruction's rows.  64 of them per workgroup,
// on fewer compute units: 256000 classes of d = 2048, us per step, sixteen tokens with k' = 512 93.3 against 91.7, four 81.1
// against 80.2; 40000, eight tokens with k' = 256 49.7 against 48.6.
int filter_rank_blocks(int n_cap) { return min((n_cap + 15) / 16, 256); }
static_assert(4 * 256 <= kFilterMaxima && kFrMaxRows * 256 >= kSoftmaxRefineMaxRow, "maxima and rows per workgroup");

// Where every workgroup reads the same 256 bytes of its rows at a time, rows that are whole multiples of 4 KB apart queue in the
// memory system: all requests of a moment go to the same few channels.  With up to 32 tokens, whose stages are mostly rows, and most
// of a workgroup's units candidates, the workgroups of a die therefore start in different stages.  us per layer, not turned /
// turned, 9, 16 and 32 tokens: d = 2048, 16384 units 55.3 / 54.5, 53.2 / 50.5, 60.8 / 59.3 (65 MB in 14.8 us instead of 16.7 at 16
// tokens); d = 4096, 9216 units 65.5 / 65.1, 61.5 / 60.7, 72.8 / 71.9; d = 6144, 6144 units 68.3 / 68.2, 68.3 / 67.8, 81.6 / 80.9;
// d = 8192, 4608 units 76.6 / 77.1, 75.0 / 74.6, 90.9 / 91.0.  Rows of other lengths are spread over the channels as they are, and
// lose by it: d = 2080, 16384 units 61.7 / 62.3, 59.7 / 60.8, 69.2 / 69.8; d = 2304 63.7 / 64.2, 61.3 / 61.8, 68.7 / 69.1; d = 3936,
// 9590 units, 16 tokens 64.0 / 64.8; d = 2112, 2560, 2816 and 3072 within half a us either way.  Nor do shorter rows gain (d = 1024,
// 32 tokens 42.0 / 42.3), 64 tokens (68.8 / 69.4), workgroups with a selection beside them (8192 units, 16 tokens 35.1 / 35.9) or few
// candidates (tokens of one query 41.5 / 42.1).
hipError_t launch_filter_units(const uint16_t* W, const uint16_t* x, int B, int d, const uint32_t* bitmap,
                               const int32_t* n_dev, int n_rows, float* h, long long stride_h, float* xnorm,
                               float* wnorm_tiles, uint32_t* wnorm_max, hipStream_t s) {
  if (B < 1 || B > 64 || d % 8 != 0) return hipErrorInvalidValue;
  static std::atomic<size_t> raised_to[3] = {};
  const FilterUnits p{W, x, B, d, bitmap, n_dev, n_rows, h, stride_h, xnorm, wnorm_tiles, wnorm_max, gather_filter_error(B),
                      d % 2048 == 0 ? 1 : 0};
  auto go = [&](auto kernel, int tt, int waves, std::atomic<size_t>& raised) {
    const size_t lds = (size_t)kFtStages * ft_stage_bytes(tt);
    if (const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, raised); e != hipSuccess)
      return e;
    return launch(kernel, dim3(filter_tiles(n_rows)), dim3(64 * waves), lds, s, p);
  };
  // Two (beyond 16 tokens four) waves share a group of candidates: halves of every stage's steps and, with several
  // token tiles, halves of the tiles, so that the fp64 additions and the operand reads of a stage are short next to
  // its loads.
  if (B <= 16) return go(k_filter_units<1, 1, 2>, 1, 8, raised_to[0]);
  if (B <= 32) return go(k_filter_units<2, 2, 2>, 2, 16, raised_to[1]);
  return go(k_filter_units<4, 2, 2>, 4, 16, raised_to[2]);
}

hipError_t launch_select_filter(const KeysSelect& ks, int B, const uint16_t* W, const uint16_t* x, int d, float* h,
                                long long stride_h, float* xnorm, float* wnorm_tiles, hipStream_t s) {
  if (B < 1 || B > 64 || d % 8 != 0 || !keys_select_ok(ks) || (ks.f64 && ks.N > kSelectFilterMaxF64)) return hipErrorInvalidValue;
  const FilterUnits p{W, x, B, d, nullptr, nullptr, ks.N, h, stride_h, xnorm, wnorm_tiles, nullptr, gather_filter_error(B), 0};
  static std::atomic<size_t> raised_to[9] = {};
  auto go = [&](auto kernel, int tt, std::atomic<size_t>& raised) {
    const size_t lds = (size_t)kFtStages * ft_stage_bytes(tt);
    if (const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, raised); e != hipSuccess)
      return e;
    return launch(kernel, dim3(B + filter_tiles(ks.N)), dim3(kSelThreads), lds, s, ks, p);
  };
  if (ks.f64) {
    if (B <= 16) return go(k_select_filter<1, 1, 4, uint64_t, 8>, 1, raised_to[6]);
    if (B <= 32) return go(k_select_filter<2, 2, 2, uint64_t, 8>, 2, raised_to[7]);
    return go(k_select_filter<4, 2, 2, uint64_t, 8>, 4, raised_to[8]);
  }
  if (ks.N <= 16384) {
    if (B <= 16) return go(k_select_filter<1, 1, 4, uint32_t, 4>, 1, raised_to[0]);
    if (B <= 32) return go(k_select_filter<2, 2, 2, uint32_t, 4>, 2, raised_to[1]);
    return go(k_select_filter<4, 2, 2, uint32_t, 4>, 4, raised_to[2]);
  }
  if (B <= 16) return go(k_select_filter<1, 1, 4, uint32_t, 8>, 1, raised_to[3]);
  if (B <= 32) return go(k_select_filter<2, 2, 2, uint32_t, 8>, 2, raised_to[4]);
  return go(k_select_filter<4, 2, 2, uint32_t, 8>, 4, raised_to[5]);
}

hipError_t launch_filter_ranks(const uint16_t* W, const uint16_t* x, int B, int d, const int32_t* list,
                               const int32_t* n_dev, int n_cap, float* h, long long stride_h, const HistRefs& hr,
                               const UnionRefs* un, int n_rows, float* xnorm, float* wnorm_tiles, float* maxima,
                               hipStream_t s) {
  if (B < 1 || B > 64 || d % 8 != 0 || n_cap > kFrMaxRows * 256) return hipErrorInvalidValue;
  GatherUnion u = make_gather_union(un, hr, B);
  u.words = min(u.words, (n_rows + 31) / 32);  // the bitmap's padding words hold no bits
  if (u.bitmap == nullptr && list == nullptr) return hipErrorInvalidValue;
  static std::atomic<size_t> raised_to[3] = {};
  auto go = [&](auto kernel, int tt, int tg, std::atomic<size_t>& raised) {
    const size_t lds = (size_t)fr_stages(tt) * ft_stage_bytes(tt) + (size_t)4 * tg * (tt / tg) * 4 * kWave * sizeof(double);
    if (const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, raised); e != hipSuccess)
      return e;
    return launch(kernel, dim3(filter_rank_blocks(n_cap)), dim3(512 * tg), lds, s, W, x, B, d, list, n_dev, n_cap, h,
                  stride_h, u, xnorm, wnorm_tiles, maxima);
  };
  if (B <= 16) return go(k_filter_ranks<1, 1, 2>, 1, 1, raised_to[0]);
  if (B <= 32) return go(k_filter_ranks<2, 2, 2>, 2, 2, raised_to[1]);
  return go(k_filter_ranks<4, 2, 2>, 4, 2, raised_to[2]);
}

}  // namespace hire

#ifdef HIRE_TIMESTAMPS
extern "C" int hire_debug_timestamps_gather(unsigned long long* host64) {
  return (int)hipMemcpyFromSymbol(host64, HIP_SYMBOL(hire_ts), sizeof(hire_ts));
}
#endif
