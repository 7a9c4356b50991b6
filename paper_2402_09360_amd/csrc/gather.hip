// Exact stage of HiRE (arXiv 2402.09360, Algorithm 1 line 2 and eq. (4)):
//   gather_dot    h[b,t] = phi(<z_{U[t]}, x_b>) over the candidate rows only
//   w2_list       y_b    = sum_{j in S_b} h[b,j] v_j over the selected rows only
// Rows are unit-major, so every gathered row is one contiguous run of 2*d bytes
// read with 16-byte loads.
//
// gather_dot accumulates in fp64: a bf16*bf16 product is exact in fp32, and
// fp64 sums of such products differ between summation orders only in the last
// bits, which keeps the top-k decision that follows independent of the order.
#include "device_utils.h"
#include "hist.h"
#include "kernels.h"
#include "listed_rows.h"

namespace hire {

// One token: a wave per candidate row, the token in LDS as raw bf16.  The candidates come either as a list
// (list != nullptr, count from n_dev or n_host) or as the union bitmap, which every workgroup compacts for its
// own contiguous share of ranks (union_locate); it then also writes that share of the ascending candidate list,
// and workgroup 0 the count.
// gs > 0 (group-sparse FFN, eq. (6)): the candidates are groups of 2^gs adjacent rows; entry e of the list stands
// for rows list[e] * 2^gs + l, l < 2^gs, whose results go to h[e * 2^gs + l].  Counts and capacities stay in
// entries.
__global__ __launch_bounds__(256) void k_gather_dot(const uint16_t* __restrict__ W, const uint16_t* __restrict__ x,
                                                    int d, const int32_t* __restrict__ list, int n_host,
                                                    const int32_t* __restrict__ n_dev, int n_cap, int relu,
                                                    double* __restrict__ h, GatherUnion un, int share, int gs) {
  extern __shared__ uint4 xs[];  // [d/8] raw bf16 token, then (bitmap mode) the indices of the workgroup's ranks
  __shared__ SelSharedT<256> sh;
  const int cpr = d / 8;         // 16-byte chunks per row
  const int lane = lane_id();
  for (int i = (int)threadIdx.x; i < cpr; i += 256) xs[i] = reinterpret_cast<const uint4*>(x)[i];
  // ranks of this workgroup: a contiguous share of the capacity
  const int r0 = (int)blockIdx.x * share;
  const int gmask = (1 << gs) - 1;
  int n;
  const int32_t* rows;  // indices of ranks r0 ..
  if (un.bitmap != nullptr) {
    int32_t* mine = reinterpret_cast<int32_t*>(xs + cpr);
    n = un.words <= 4 * 64 * kLocateStepsShort ? union_locate<256, kLocateStepsShort>(un.bitmap, un.words, sh, r0, share, mine)
                                               : union_locate<256>(un.bitmap, un.words, sh, r0, share, mine);
    n = min(n, n_cap);
    if (blockIdx.x == 0) publish_union(un, n);
    for (int t = (int)threadIdx.x; t < share && r0 + t < n; t += 256) un.list_out[r0 + t] = mine[t];
    rows = mine;
  } else {
    n = n_dev ? min(*n_dev, n_cap) : n_host;
    rows = list ? list + r0 : nullptr;  // no list: entry e is row e itself
    __syncthreads();
  }
  for (int t = wave_id(); t < (share << gs) && r0 + (t >> gs) < n; t += 4) {
    const int entry = rows ? rows[t >> gs] : r0 + (t >> gs);
    const uint4* row = reinterpret_cast<const uint4*>(W + (((size_t)entry << gs) + (t & gmask)) * d);
    double acc = 0.0;
#pragma unroll 4
    for (int c = lane; c < cpr; c += kWave) {
      const uint4 wv = load_streaming(&row[c]);
      const uint32_t wd[4] = {wv.x, wv.y, wv.z, wv.w};
      const uint4 xv = xs[c];
      const uint32_t xd[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        acc += (double)(bf16_lo(wd[q]) * bf16_lo(xd[q]));
        acc += (double)(bf16_hi(wd[q]) * bf16_hi(xd[q]));
      }
    }
    double s = wave_sum(acc);
    if (relu) s = s > 0.0 ? s : 0.0;
    if (s == 0.0) s = 0.0;
    if (lane == 0) h[((size_t)r0 << gs) + t] = s;
  }
}

// ---------------------------------------------------------------------------
// Second layer, y_b = sum_e coef(b, e) * W2[row(b, e), :] over the k entries (row, coefficient) that the selection
// left for token b, plus (CommonPath, eq. (7)) sum_r fl32(hd[b, r]) * Wd[r, :] over m1 dense rows.  One kernel, no
// partial sums: a workgroup owns 8 LPR columns of one token and all of its rows, and writes y itself.  The entries
// pass through LDS in chunks; add_listed_rows (listed_rows.h) adds up a chunk.
//
// Bound: the round trips list -> rows for few tokens; for many the caches (64 tokens read 215 MB of rows that are
// 67 MB in HBM, 11 TB/s).  Narrow slices spread few tokens over the chip; wide ones read longer runs and are faster
// once 256 workgroups exist.  The dispatcher places workgroup i on die i % 8, and a die takes an eighth of the
// (slice, token) pairs, slice by slice, so that the tokens share a slice's rows in one L2 and every die has as much to do
// (whole slices per die left dies idle where slices do not come in eights: 49 tokens of d = 288, k = 1949 12.2 us, now
// 10.2; 64 of d = 640, k = 1200 15.9, now 13.7).  Measured at d = 2048, k = 819 of 16384 units: 19.8 us for
// 64 tokens (16 take k_refine_w2), against 23.7 for 256-column workgroups without
// the second batch in flight at 64.
constexpr int kW2Threads = 512;
constexpr int kW2Waves = kW2Threads / kWave;
constexpr int kW2Chunk = 1024;  // entries staged in LDS at a time

template <int LPR, int FL, bool SHORT = false>
__global__ __launch_bounds__(kW2Threads, 4) void k_w2_list(const uint16_t* __restrict__ W2, int d, int B, int k,
                                                           const uint2* __restrict__ list,
                                                           const uint16_t* __restrict__ Wd, int m1,
                                                           const double* __restrict__ hd, float* __restrict__ y) {
  constexpr int kCols = 8 * LPR;                         // columns of the workgroup
  constexpr int kStride = kW2Waves * (kWave / LPR);      // rows of the workgroup per load instruction
  static_assert((SHORT || kW2Chunk % (kStride * FL) == 0) && kCols <= kW2Threads, "whole batches per chunk, a thread per column");
  constexpr int kBatch = kStride * FL, kChunk = SHORT ? kBatch : kW2Chunk;
  constexpr int kFill = ((SHORT ? 0 : kW2Chunk) + kBatch + kW2Threads - 1) / kW2Threads;  // entries per thread
  __shared__ uint2 entries[kFill * kW2Threads];
  __shared__ float red[kW2Waves][kCols];
  const int lane = lane_id(), w = wave_id(), tid = (int)threadIdx.x;
  const int n_items = (d + kCols - 1) / kCols * B;
  const int item = (int)(blockIdx.x & 7) * ((n_items + 7) / 8) + (int)(blockIdx.x >> 3);
  if (item >= n_items) return;  // uniform: the last dies' shares may be short
  const int slice = item / B, b = item % B;
  const int sub = lane % LPR, first = w * (kWave / LPR) + lane / LPR;
  const int colc = min(slice * kCols + sub * 8, d - 8);  // d is a multiple of 8
  float acc[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) acc[q] = 0.0f;
  // adds up the n entries in LDS (behind them some row with coefficient 0, to the end of one batch more)
  auto add_chunk = [&](const uint16_t* __restrict__ M, int n) {
    add_listed_rows<LPR, FL, kW2Waves, SHORT>(M + colc, d, n, first, [&](int t) { return entries[t]; }, acc);
  };
  const uint2* mine = list + (size_t)b * k;
  for (int e0 = 0; e0 < (SHORT ? 1 : k); e0 += kChunk) {
    if (e0 > 0) __syncthreads();
#pragma unroll
    for (int u = 0; u < kFill; ++u) {
      const int i = u * kW2Threads + tid;
      const uint2 e = mine[min(e0 + i, k - 1)];
      entries[i] = make_uint2(e.x, i < kChunk && e0 + i < k ? e.y : 0u);
    }
    __syncthreads();
    add_chunk(W2, min(kChunk, k - e0));
  }
  for (int e0 = 0; e0 < (SHORT ? 0 : m1); e0 += kW2Chunk) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kFill; ++u) {
      const int i = u * kW2Threads + tid;
      const float c = (float)hd[(size_t)b * m1 + min(e0 + i, m1 - 1)];
      entries[i] = make_uint2((uint32_t)min(e0 + i, m1 - 1), i < kW2Chunk && e0 + i < m1 ? __float_as_uint(c) : 0u);
    }
    __syncthreads();
    add_chunk(Wd, min(kW2Chunk, m1 - e0));
  }
  // the lanes of a wave that hold the same columns (fixed tree), then the waves in order
  fold_lanes<LPR>(acc);
  if (lane < LPR) {
    float4* dst = reinterpret_cast<float4*>(&red[w][sub * 8]);
    dst[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
    dst[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
  }
  __syncthreads();
  if (tid < kCols && slice * kCols + tid < d) {
    float s = 0.0f;
#pragma unroll
    for (int u = 0; u < kW2Waves; ++u) s += red[u][tid];
    y[(size_t)b * d + slice * kCols + tid] = s;
  }
}

// ---------------------------------------------------------------------------
// Group sums (eq. (6)): out[b, J] = sum_{l < 2^gs} |in[b, J * 2^gs + l]|, added in index order in the type of
// the input, for J < n (n from n_dev if given).
template <typename T>
__global__ __launch_bounds__(256) void k_group_sums(const T* __restrict__ in, long long stride_in, int n_host,
                                                    const int32_t* __restrict__ n_dev, int n_cap, int gs,
                                                    T* __restrict__ out, long long stride_out) {
  const int n = n_dev ? min(*n_dev, n_cap) : n_host;
  const int J = (int)(blockIdx.x * blockDim.x + threadIdx.x), b = (int)blockIdx.y;
  if (J >= n) return;
  const T* src = in + (size_t)b * stride_in + ((size_t)J << gs);
  T sum = (T)0;
  for (int l0 = 0; l0 < (1 << gs); l0 += 4) {  // group sizes 1, 2 or a multiple of 4
    T v[4];
#pragma unroll
    for (int l = 0; l < 4; ++l) v[l] = src[min(l0 + l, (1 << gs) - 1)];
#pragma unroll
    for (int l = 0; l < 4; ++l)
      if (l0 + l < (1 << gs)) sum += v[l] < (T)0 ? -v[l] : v[l];
  }
  out[(size_t)b * stride_out + J] = sum;
}

template <typename T>
static hipError_t group_sums(const T* in, int B, long long stride_in, int n, const int32_t* n_dev, int n_cap, int gs,
                             T* out, long long stride_out, hipStream_t s) {
  const int cap = n_dev ? n_cap : n;
  return launch(k_group_sums<T>, dim3((cap + 255) / 256, B), dim3(256), 0, s, in, stride_in, n, n_dev, n_cap, gs, out,
                stride_out);
}
hipError_t launch_group_sums_f32(const float* in, int B, long long stride_in, int n, int gs, float* out,
                                 long long stride_out, hipStream_t s) {
  return group_sums<float>(in, B, stride_in, n, nullptr, n, gs, out, stride_out, s);
}
hipError_t launch_group_sums_f64(const double* in, int B, long long stride_in, int n, const int32_t* n_dev, int n_cap,
                                 int gs, double* out, long long stride_out, hipStream_t s) {
  return group_sums<double>(in, B, stride_in, n, n_dev, n_cap, gs, out, stride_out, s);
}

// Entries per workgroup: about four rows (one per wave), more once 2048 workgroups no longer cover the list.
static int gather_dot_share(int cap, int gs) { return max(max(1, 4 >> gs), (cap + 2047) / 2048); }

bool union_in_gather(int words) { return words <= kUnionLocateMaxWords; }

hipError_t launch_gather_dot(const uint16_t* W, const uint16_t* x, int d, const int32_t* list, int n,
                             const int32_t* n_dev, int n_cap, int relu, double* h, const HistRefs& hr,
                             const UnionRefs* un, int gs, hipStream_t s) {
  const int cap = n_dev ? n_cap : n;
  const GatherUnion u = make_gather_union(un, hr, 1);
  const int share = gather_dot_share(cap, gs);
  const int blocks = max(1, (cap + share - 1) / share);
  size_t lds = (size_t)d * 2;
  if (u.bitmap) lds += (size_t)share * 4;
  return launch(k_gather_dot, dim3(blocks), dim3(256), lds, s, W, x, d, u.bitmap ? nullptr : list, n, n_dev, cap, relu, h,
                u, share, gs);
}

hipError_t launch_w2_list(const uint16_t* W2, int d, int B, int k, const void* list, const uint16_t* Wd, int m1,
                          const double* hd, float* y, hipStream_t s) {
  auto items = [&](int cols) { return (d + cols - 1) / cols * B; };
  auto go = [&](auto kernel, int cols) {
    return launch(kernel, dim3((items(cols) + 7) / 8 * 8), dim3(kW2Threads), 0, s, W2, d, B, k,
                  static_cast<const uint2*>(list), Wd, m1, hd, y);
  };
  // The widest slices that still give a workgroup to (nearly) every compute unit and leave few of them out of the last
  // round of 256.  us with slices of 256 / 128 / 64 / 32 columns, units drawn at random, W2 not in the caches, * the rule:
  //   d = 2048, k = 819 of 16384:  5 tokens  9.0  7.0  6.4* 6.7    8   9.8  7.5  7.5* 7.2   12  11.1  8.6  9.5* 9.5
  //     16  12.2  9.8* 10.3 12.1   24  13.9 13.8* 14.3 17.0   33  19.9 17.3* 19.6 21.5   64  21.6* 20.8 28.5 34.7
  //   d = 800, k = 251 of 5003:    8  4.8 4.2 4.1* 4.2   33  5.1 4.9* 5.1 7.4   64  5.5* 5.6 7.7 10.6
  //   d = 4096, k = 400 of 8192:   5  6.5 5.7 5.7* 6.4   16  9.5* 9.4 11.1 14.3   33  16.6 16.0* 20.2 26.5
  //   d = 288, k = 1949 of 24000, 49 tokens  18.3 12.4 10.6* 10.5     d = 512, k = 900 of 20003, 16  9.7 7.1 6.0* 5.6
  // Of 28 shapes 22 within 4 % of the best width, 12 tokens and the last of these 7 to 10 % off; where few rows make the
  // reduction count more the rule is too narrow.  Short lists, us per step: d = 256, k = 51 of 1024, five tokens 21.1 / 21.2 / 21.3 / 21.5*;
  // d = 1024, k = 205 of 4096, 33 29.2 / 28.8 / 29.6* / 31.5, 64 31.0 / 30.4 / 31.8 / 35.1 (the rule 30.9: 256); groups of eight, k = 104, 33 39.5 / 39.5 / 40.5* /
  // 42.3, with 304 dense units 48.0 / 48.1 / 50.5* / 55.0; d = 2048, k = 256 of 16384, 33 50.8 / 50.5* / 50.5 / 53.5.
  auto fill = [&](int n) { return (double)n / ((n + 255) / 256 * 256); };
  // Lists of up to eight loads per lane, and no dense rows, have kernels that ask for no second batch: by a branch inside the kernel it
  // was slower than asking in vain (110 registers instead of 78).  us per step, two batches always / so: d = 256, k = 51 of 1024, eight
  // tokens 22.4 / 21.7, 64 25.0 / 24.2; d = 800, k = 251 of 5003, five 26.8 / 26.3, 33 32.8 / 32.6; d = 2048, k = 256 of 16384, eight 39.4 / 39.0;
  // d = 4096, k = 100 of 8192, 33 60.1 / 58.9 (59.2 with a branch around every request); groups of eight, d = 1024, 33 tokens 41.9 / 40.4.
  auto pick = [&](auto l1, auto l2, auto l4, auto l8, auto longer, int cols) {
    const int n = m1 == 0 ? (k * cols + 8 * kW2Threads - 1) / (8 * kW2Threads) : INT_MAX;  // a load: 8 columns per thread
    return n <= 1 ? go(l1, cols) : (n <= 2 ? go(l2, cols) : (n <= 4 ? go(l4, cols) : (n <= 8 ? go(l8, cols) : go(longer, cols))));
  };
  if (items(256) >= 250 && fill(items(256)) > 0.9)
    return pick(k_w2_list<32, 1, true>, k_w2_list<32, 2, true>, k_w2_list<32, 4, true>, k_w2_list<32, 8, true>, k_w2_list<32, 4>, 256);
  if (items(128) >= 200 && fill(items(128)) > 0.6)
    return pick(k_w2_list<16, 1, true>, k_w2_list<16, 2, true>, k_w2_list<16, 4, true>, k_w2_list<16, 8, true>, k_w2_list<16, 4>, 128);
  if (items(64) >= 128)
    return pick(k_w2_list<8, 1, true>, k_w2_list<8, 2, true>, k_w2_list<8, 4, true>, k_w2_list<8, 8, true>, k_w2_list<8, 8>, 64);
  return pick(k_w2_list<4, 1, true>, k_w2_list<4, 2, true>, k_w2_list<4, 4, true>, k_w2_list<4, 8, true>, k_w2_list<4, 8>, 32);
}

}  // namespace hire
