// Host-side launch interface of the HiRE kernels (internal to libhire).
// Every launcher enqueues on `stream` and returns the HIP launch status.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace hire {

// Launch and report this launch's status only.  One runtime call: the launch syntax pushes and pops its configuration
// and would need the sticky "last error" cleared before and read after, because other users of the runtime in the
// same process (PyTorch) may have left an unrelated one behind.
template <typename... Params, typename... Args>
inline hipError_t launch(void (*kernel)(Params...), dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                         Args... args) {
  return [&](Params... params) {
    void* pointers[] = {const_cast<void*>(static_cast<const void*>(&params))...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, pointers, lds, stream);
    if (e != hipSuccess) (void)hipGetLastError();  // reported to the caller, not left behind
    return e;
  }(static_cast<Params>(args)...);
}

// Dynamic LDS beyond the default limit needs the kernel's attribute raised before the launch.  `raised_to` is a
// counter of the call site's own (one per kernel instantiation): the attribute is set again only when a launch
// asks for more than any before it.  Threads that race here set the same attribute twice, which is harmless.
constexpr size_t kDefaultDynamicLds = 48 * 1024;
inline hipError_t ensure_dynamic_lds(const void* kernel, size_t lds, std::atomic<size_t>& raised_to) {
  if (lds <= kDefaultDynamicLds || raised_to.load(std::memory_order_acquire) >= lds) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e == hipSuccess) raised_to.store(lds, std::memory_order_release);
  return e;
}

// Places of the general route's histograms in the caller's workspace (any may be null: no histograms).
struct HistRefs {
  void* header;      // general_header_bytes() at a fixed place, cleared by the workspace initialisation
  void* multi_body;  // multi_body_bytes_host(B): per-token histograms of the scorer keys (long rows)
};
size_t general_header_bytes();
unsigned long long layout_signature(int scorer_kind, int B, int d, int N, int r, int k, int kprime, int ffn);
constexpr unsigned long long kSigOverlays = 1ull << 63;  // set in signatures of layouts that reuse the token regions

// ---- scorer.hip ------------------------------------------------------------
// The packed blob is rows * cols / 2 bytes of codes followed by kPackTrailerBytes: the first trailer word holds the
// largest row scale (float bits; all-zero rows left out), which the scorers turn into an upper bound
// of every key of a step; the rest is zero.
constexpr size_t kPackTrailerBytes = 64;
hipError_t launch_pack_int4(const uint16_t* w, int rows, int cols, uint32_t* q4, float* scale, hipStream_t s);
hipError_t launch_unpack_int4(const uint32_t* q4, int rows, int cols, int8_t* codes, hipStream_t s);

// x bf16, or fp32 that is rounded to it (nearest even) first, [B,d] -> xq int8 [B,d], sumabs (optional) fp32 [B] = sum |xq|;
// also clears `zero_words` 32-bit words at zero_ptr.  As a step's first kernel it checks the general header (optional)
// against the layout signature.
hipError_t launch_quantize_tokens(const void* x, bool f32, int B, int d, int8_t* xq, float* sumabs, uint32_t* zero_ptr,
                                  int zero_words, void* general_header, unsigned long long sig, hipStream_t s);

// One token (B == 1): keys[j] = phi(float(sum_i q[j,i] xq[i]) * scale[j]); acc (optional) gets the integer sums.
// With histogram places the kernel also leaves the key counts and the per-workgroup maxima for launch_mark_f32.
hipError_t launch_scorer_int4(const uint32_t* q4, const float* scale, const int8_t* xq, int B, int N, int d, int relu,
                              float* keys, int32_t* acc, const HistRefs& hr, hipStream_t s);
int scorer_int4_blocks(int N);
// The same as a step's first kernel, for rows of at most 8192 codes: quantises the token itself (x bf16 [d]),
// clears zero_words words at zero_ptr and checks the general header against the layout signature.
bool scorer_int4_fused_supported(int d);
// out[i] = bf16(in[i]), round to nearest even, i < n.
hipError_t launch_f32_to_bf16(const float* in, int n, uint16_t* out, hipStream_t s);
hipError_t launch_scorer_int4_fused(const uint32_t* q4, const float* scale, const void* x, bool x_is_f32, int N, int d,
                                    int relu, float* keys, int32_t* acc, const HistRefs& hr, uint32_t* zero_ptr,
                                    int zero_words, unsigned long long sig, hipStream_t s);
// x_is_f32: the token is fp32 [d] and is rounded to bf16 (nearest even) before it is quantised; only for rows the
// short-row kernels take (scorer_int4_fused_takes_f32(d)).
bool scorer_int4_fused_takes_f32(int d);
int scorer_int4_fused_blocks(int N, int d);  // workgroups launch_scorer_int4_fused uses
int scorer_int4_fused_maxima(int N, int d);  // maxima it leaves per token: one per workgroup, short rows one per wave
// The same on the int8 matrix cores, for batches (scorer_mfma.hip); B <= 64.  keys: [B, stride].  The tokens come as codes
// (launch_quantize_tokens), or the scorer quantises them itself (scorer_mfma_quantises) and is then, in that kernel's
// place, the step's first.
struct ScorerTokens {
  const int8_t* xq;          // [B, d] codes; or, with x:
  const void* x;             // [B, d] bf16, or
  bool f32;                  // fp32, which is rounded to bf16 (nearest even) first
  float* sumabs;             // optional [B]: sums of the codes' absolute values
  uint32_t* zero_ptr;        // words to clear
  int zero_words;
  void* header;              // general header to check against sig; optional
  unsigned long long sig;
};
bool scorer_mfma_quantises(int B, int N, int d, bool f32);
hipError_t launch_scorer_int4_mfma(const uint32_t* q4, const float* scale, const ScorerTokens& tok, int B, int N, int d,
                                   int relu, float* keys, long long stride, int32_t* acc, const HistRefs& hr, hipStream_t s);
int scorer_mfma_maxima(int N);  // maxima it leaves per token (long rows): two per wave

// t[b,:] = bf16(Z1^T x_b); also clears zero_words words at zero_ptr and, as a step's first kernel, checks the
// general header (optional) against the layout signature.
hipError_t launch_lr_project(const uint16_t* z1, const uint16_t* x, int B, int d, int r, uint16_t* t, uint32_t* zero_ptr,
                             int zero_words, void* general_header, unsigned long long sig, hipStream_t s);
// One token: keys[j] = phi(<Z2[j,:], t>) in fp64.  Batches: launch_lr_score_mfma.
// *out = an upper bound of the largest row norm of the bf16 matrix W [rows, cols] (cols a multiple of 8).
hipError_t launch_row_norm_max(const uint16_t* W, int rows, int cols, float* out, hipStream_t s);
hipError_t launch_lr_score(const uint16_t* z2, const uint16_t* t, int N, int r, int relu, double* keys, hipStream_t s);
// The same for batches on the fp64 matrix cores (gather_mfma.hip); keys [B, stride].
hipError_t launch_lr_score_mfma(const uint16_t* z2, const uint16_t* t, int B, int N, int r, int relu, double* keys,
                                long long stride, hipStream_t s);

// Clears `words` 32-bit words.
hipError_t launch_clear_words(uint32_t* p, int words, hipStream_t s);

// Plain device-to-device copy of `bytes` (multiple of 16).
hipError_t launch_plain_copy(const void* src, void* dst, size_t bytes, hipStream_t s);

// ---- select.hip ------------------------------------------------------------
struct SelectParams {
  const void* vals;         // float or double [B, stride]
  long long stride;
  int n;                    // number of entries per row when n_dev == nullptr
  const int32_t* n_dev;     // device-side count (overrides n); n_cap bounds it
  int n_cap;                // host upper bound of n (chooses the register-resident or the streaming variant)
  int k;
  int relu;                 // rank max(v, 0)
  int rank_order;           // outputs in rank order instead of ascending index
  int32_t* idx_out;         // [B,k] selected indices (through map if given), optional
  float* val_out;           // [B,k] selected values, optional
  const int32_t* map;       // optional translation of positions to indices for idx_out
  long long map_stride;     // row b uses map + b * map_stride (0: one map for all rows)
  int32_t* pos_out;         // [B,k] selected positions (no map), optional
  float* prob_out;          // [B,k] softmax over the selected values (rank order only), optional
  uint32_t* bitmap;         // optional: bit i set (atomic or) for every selected position of any row
  uint32_t* window_misses;  // optional device counter: rows whose window histogram did not give the k-th largest
  // Filter and refine (launch_softmax_refine only): vals are fp32 rows written by launch_filter_ranks, within
  // err_c |u| |x| of the logits; map lists the rows' classes.  The kernels recompute in fp64
  // (<refine_w[map[i], :], refine_x[b, :]>) what can still be among the k largest.
  const uint16_t* refine_w;  // bf16 [rows, refine_d]
  const uint16_t* refine_x;  // bf16 [B, refine_d]
  int refine_d;
  const float* xnorm;
  const float* wnorm_tiles;  // [wnorm_n]
  int wnorm_n;
  float err_c;
  const float* maxima;      // [B, kFilterMaxima], n_maxima of them used: largest values of disjoint parts of the row
  int n_maxima;
  void* refine_slots;       // softmax_refine_slot_bytes(B) of scratch
  unsigned long long* refine_keys;  // [B, refine_keys_stride] of scratch: logits of entries that do not fit the slots
  long long refine_keys_stride;
  int nonneg;               // != 0: every value is known to be >= 0 (keys and activations after a ReLU); such rows
                            // of 1025..16384 entries in index order take a leaner kernel
  // Second layer: list_out (optional) receives for every row its k << gs selected units in ascending order, as
  // (row of the weight matrix, fp32 value): what launch_w2_list reads.  gs = 0: the selected entries themselves
  // (through map) with their values.  gs > 0: the entries are groups of 2^gs units; unit l of the group at position
  // pos has the row (map[pos] << gs) + l and the value unit_h[b * unit_h_stride + (pos << gs) + l]; unit_val_out
  // (optional, [B, k << gs]) receives the values.  gs > 0 needs pos_out.
  uint2* list_out;
  int gs;
  const double* unit_h;
  long long unit_h_stride;
  float* unit_val_out;
};
hipError_t launch_select_f32(const SelectParams& p, int B, hipStream_t s);
// The k largest of every row of scores [B, N] in ascending index order, selected by many workgroups per row
// through key histograms (for long rows).  general_header: general_header_bytes() cleared by the workspace
// initialisation; body: topk_long_workspace_bytes(B, N).  N <= 16384 * 4096.
size_t topk_long_workspace_bytes(int B, int N);
hipError_t launch_topk_long(const float* scores, int B, int N, int k, int relu, int32_t* idx_out, float* val_out,
                            void* general_header, void* body, unsigned long long sig, hipStream_t s);
// The same for few entries of long rows, in either order, without histograms (topk_rows_supported): the same places.
bool topk_rows_supported(int N, int k);
hipError_t launch_topk_rows(const float* scores, int B, int N, int k, int relu, int rank_order, int32_t* idx_out,
                            float* val_out, void* general_header, void* body, unsigned long long sig, hipStream_t s);
hipError_t launch_select_f64(const SelectParams& p, int B, hipStream_t s);
// Filter and refine for the classifier (phi = identity, signed values, rank order, softmax over the k survivors): every
// entry within 2 * err_c * xnorm[b] * *wnorm_max below the k-th largest stored value is recomputed in fp64 and the k
// largest of those are returned in rank order (idx_out through map, val_out, prob_out).  Rows of at most
// kSoftmaxRefineMaxRow fp32 entries, k <= kSoftmaxRefineMaxK.
constexpr int kSoftmaxRefineMaxRow = 131072, kSoftmaxRefineMaxK = 512;
size_t softmax_refine_slot_bytes(int B);
hipError_t launch_softmax_refine(const SelectParams& p, int B, hipStream_t s);

// HiRE-Softmax for one token after launch_scorer_int4_fused on a long vocabulary (key histograms present): from the
// scorer's per-workgroup maxima (n_max of them) a lower bound of the k'-th largest key, exact logits of the keys at
// or above it (a superset of the shortlist), then Algorithm 1's shortlist, the k largest logits in rank order
// (top_idx, optional top_logit) and their softmax (top_prob); optional cand_idx (the k' shortlisted classes,
// ascending) and n_cand.  q4: the packed codes the keys were scored with, rows of sd codes (their trailer bounds the
// keys); slots: softmax_b1_slot_bytes(N) of scratch.
bool softmax_b1_supported(int N, int d, int k, int kprime);
bool softmax_b1_worthwhile(int N, int kprime, int n_max);  // enough maxima and slots for the bound to serve
size_t softmax_b1_slot_bytes(int N);
hipError_t launch_softmax_b1(const float* keys, int N, int d, int sd, int k, int kprime, int n_max, const void* q4,
                             const uint16_t* W, const uint16_t* x, const HistRefs& hr, void* slots, int32_t* top_idx,
                             float* top_prob, float* top_logit, int32_t* cand_idx, int32_t* n_cand, hipStream_t s);

// The same bound from the scorer's maxima for batches, long rows (maxima_select_supported): for every token the keys
// at or above its bound, then exactly its k' largest keys (ties to the lower index) as bits of the union bitmap
// (which must be clear).  Replaces launch_mark_f32 + launch_resolve_compact; takes no histogram and leaves none.
// slots: maxima_select_slot_bytes(B, N) of scratch.  maxima_select_worthwhile says whether the bound will serve.
bool maxima_select_supported(int N);
bool maxima_select_worthwhile(int B, int N, int kprime, int n_max);
size_t maxima_select_slot_bytes(int B, int N);
hipError_t launch_maxima_select(const float* keys, int B, int N, int sd, int kprime, int n_max, const void* q4,
                                const HistRefs& hr, void* slots, uint32_t* bitmap, hipStream_t s);

// Ascending list of the set bits of bitmap[0..words): list_out, count to count_out[0] and (optional) count_out2[0].
// Also clears zero_words words at zero_ptr (may be nullptr).
hipError_t launch_bitmap_compact(const uint32_t* bitmap, int words, int32_t* list_out, int32_t* count_out,
                                 int32_t* count_out2, uint32_t* zero_ptr, int zero_words, hipStream_t s);

// ---- batch_select.hip --------------------------------------------------------
// The selections of a batched FFN step, one workgroup per token, rows of at most 32768 units, k <= 4096.
bool batch_select_supported(int N, int k);
// The k' largest keys of every row of non-negative keys -> bits of the union bitmap (which must be clear).
struct KeysSelect {
  const void* keys;    // [B, stride] fp32, or
  bool f64;            // fp64; rows at multiples of 16 bytes
  long long stride;
  int N, kprime;
  const float* sumabs;  // fp32: sumabs[b], *smax bound token b's keys (the sums of the absolute codes, the trailer of the
  const float* smax;    // packed codes)
  uint32_t* bitmap;
  uint32_t* window_misses;
};
constexpr int kSelectFilterMaxF64 = 16384;  // rows of fp64 keys that launch_select_filter takes
hipError_t launch_keys_select(const KeysSelect& p, int B, hipStream_t s);
// The k groups of eight with the largest sums of |vals[8 i + l]| (added in index order), ties to the lower group: bits of a
// bitmap; or, of fp64 activations by candidate, the selected groups and their units.
constexpr int kGroupSelectMax = 4096;  // groups
struct GroupSelect {
  const void* vals;      // [B, stride] fp32, or
  bool f64;              // fp64; rows at multiples of 16 bytes, stride a multiple of 8
  long long stride;
  int n_cap;             // groups,
  const int32_t* n_dev;  // optional: the first *n_dev of them
  int k;
  uint32_t* bitmap;      // the selected groups' bits are added to it; or nullptr:
  const int32_t* map;    // group of position i
  int32_t* idx_out;      // optional [B, k]: groups, in the order of their positions
  uint2* list_out;       // [B, 8 k] (unit, value) for launch_w2_list
  float* val_out;        // optional [B, 8 k]
  uint32_t* window_misses;
};
hipError_t launch_group_select(const GroupSelect& p, int B, hipStream_t s);
// The k largest activations relu(<W[j, :], x_b>) of every token among the bitmap's units, ties to the lower unit, from
// the filter stage's values in unit order (launch_filter_units).
constexpr int kRefineTokenMax = 8192;  // longest token staged in LDS
struct RefineParams {
  const float* vals;        // [B, stride], 16-byte aligned rows
  long long stride;
  int B, N, k, d;
  const uint16_t* W;        // bf16 [N, d]
  const uint16_t* x;        // bf16 [B, d]
  const float* xnorm;       // [B], wnorm_tiles [wnorm_n], err_c: bounds of the values' error
  const float* wnorm_tiles;
  int wnorm_n;
  float err_c;
  int all_rows;             // != 0: vals has values of units that are no candidates, too (launch_select_filter)
  const uint32_t* bitmap;   // the candidates; they are listed as well: ascending, and their number
  int32_t* cand_out;        // optional; cand_cap entries fit
  int cand_cap;
  int32_t* n_cand_out;      // optional (with cand_out)
  double* h64;              // [B, h_stride] scratch, as many per token as there can be candidates
  long long h_stride;
  int32_t* idx_out;         // optional [B, k] ascending
  float* val_out;           // optional [B, k]
  uint2* list_out;          // [B, k] (unit, value) for launch_w2_list
  int exact_values;         // != 0: all values are rounded from fp64, not only those around the threshold
  uint32_t* window_misses;  // optional counter: tokens that the histogram and the list in LDS did not settle
};
hipError_t launch_refine(const RefineParams& p, hipStream_t s);
// The same and the second layer, y_b = sum of the selected (unit, value) pairs' rows of W2, in one kernel (list_out is not
// written); what of it refine_w2_supported says.
bool refine_w2_supported(const RefineParams& p);
hipError_t launch_refine_w2(const RefineParams& p, const uint16_t* W2, float* y, hipStream_t s);
// The activations of the listed (token, unit) pairs, rounded once from fp64: into lists [B, k] and (optional) val_out.
hipError_t launch_exact_values(uint2* lists, float* val_out, const uint16_t* W, const uint16_t* x, int B, int k, int d,
                               hipStream_t s);

// Histogram-guided top-k' of every token's keys and their union, for keys whose producer has filled the
// key histograms:
// launch_mark_f32 sets the bits of all keys above the threshold bin and lists the keys inside it;
// launch_resolve_compact ranks those, falls back to a streaming selection for tokens whose histogram did not
// answer, restores the region to all-zero and (list_out != nullptr) turns the bitmap into the ascending list.
size_t multi_body_bytes_host(int B);
int multi_hist_shift(int N, int B);  // == the producer-side bin width exactly when the producer counts the keys
bool multi_producer_counts(int N, int B);
// uint32 counters inside the general header: 0 streaming k' selections of the many-workgroup route, 1 window
// misses of single-workgroup selections, 2 stampings of the key histograms
size_t general_fallbacks_offset(int which);
hipError_t launch_mark_f32(const float* keys, int B, int N, int kprime, int slots, const HistRefs& hr, uint32_t* bitmap,
                           hipStream_t s);
hipError_t launch_resolve_compact(const float* keys, int B, int N, int kprime, const HistRefs& hr, uint32_t* bitmap,
                                  int words, int32_t* list_out, int32_t* count_out, int32_t* count_out2,
                                  uint32_t* zero_ptr, int zero_words, hipStream_t s);

// ---- gather.hip, gather_mfma.hip ---------------------------------------------
// The candidate union handed over as a bitmap: the gather kernels then compact it themselves (every workgroup for
// its own share of ranks), write the ascending list and the count, and stamp the key histograms' header on a
// fresh workspace; no compaction kernel runs in between.  Only for bitmaps of at most kUnionLocateMaxWords words
// (union_in_gather); longer ones go through launch_bitmap_compact and the list.
constexpr int kUnionLocateMaxWords = 8192;
struct UnionRefs {
  const uint32_t* bitmap;
  int words;
  int32_t* list_out;
  int32_t* count_out;
  int32_t* count_out2;  // optional
  bool stamp_keys;      // the key histograms were cleared by the kernel before: stamp their header
};
bool union_in_gather(int words);

// One token: h[t] = phi(<W[list[t], :], x>) for t < n (n from n_dev if given), fp64 accumulation.
// list == nullptr without a union bitmap: row t itself.
// gs > 0 (both gathers): list entries are groups of 2^gs adjacent rows (2^gs <= 16); entry e, row l of the group
// -> W row list[e] * 2^gs + l -> h column e * 2^gs + l.  n, n_dev and n_cap count entries.
hipError_t launch_gather_dot(const uint16_t* W, const uint16_t* x, int d, const int32_t* list, int n,
                             const int32_t* n_dev, int n_cap, int relu, double* h, const HistRefs& hr,
                             const UnionRefs* un, int gs, hipStream_t s);
// Batches, on the fp64 matrix cores: h[b*stride_h + t].  list == nullptr without a union bitmap: row t itself
// (all n rows in order).
hipError_t launch_gather_dot_mfma(const uint16_t* W, const uint16_t* x, int B, int d, const int32_t* list, int n,
                                  const int32_t* n_dev, int n_cap, int relu, double* h, long long stride_h,
                                  const HistRefs& hr, const UnionRefs* un, int gs, hipStream_t s);

// Filter stage of the exact pre-activations for batches: values within gather_filter_error(B) * |u_j| * |x_b| of
// <u_j, x_b> (bf16 matrix cores, fp32 segments of 32 or 64 products; see the kernels for what exactly is stored),
// xnorm[b] = |x_b|, wnorm_tiles = max |u_j| over the candidates of every workgroup.  Rows only (no groups).
constexpr int filter_segment_steps(int B) { return B > 32 ? 2 : 1; }  // 32-product MFMA steps per fp32 segment
inline float gather_filter_error(int B) { return (float)filter_segment_steps(B) * 0x1p-17f; }
// FFN (phi = ReLU): the candidates are the bits of the union bitmap over n_rows rows (whole 64-bit words; nullptr: rows
// below *n_dev <= n_rows), the value of unit j goes to h[b*stride_h + j], zeros where j is no candidate (also up to
// the stride, which covers n_rows).  wnorm_tiles [filter_tiles(n_rows)]; without it *wnorm_max receives the maximum
// over all as float bits, by atomics (cleared before).
int filter_tiles(int n);
hipError_t launch_filter_units(const uint16_t* W, const uint16_t* x, int B, int d, const uint32_t* bitmap,
                               const int32_t* n_dev, int n_rows, float* h, long long stride_h, float* xnorm,
                               float* wnorm_tiles, uint32_t* wnorm_max, hipStream_t s);
// launch_keys_select and, at the same time, launch_filter_units over all rows: keys and h do not overlap.
hipError_t launch_select_filter(const KeysSelect& ks, int B, const uint16_t* W, const uint16_t* x, int d, float* h,
                                long long stride_h, float* xnorm, float* wnorm_tiles, hipStream_t s);
// Classifier (phi = identity): the candidate of rank t (of un's bitmap over n_rows classes, or list with n_dev) goes to
// h[b*stride_h + t]; n_cap <= kSoftmaxRefineMaxRow.  wnorm_tiles [filter_rank_blocks(n_cap)]; maxima [B,
// kFilterMaxima], 4 filter_rank_blocks(n_cap) of them per token: the largest values of as many disjoint groups of
// candidates (-inf: of none).
constexpr int kFilterMaxima = 1024;
int filter_rank_blocks(int n_cap);
hipError_t launch_filter_ranks(const uint16_t* W, const uint16_t* x, int B, int d, const int32_t* list,
                               const int32_t* n_dev, int n_cap, float* h, long long stride_h, const HistRefs& hr,
                               const UnionRefs* un, int n_rows, float* xnorm, float* wnorm_tiles, float* maxima,
                               hipStream_t s);

// out[b*stride_out + J] = sum_{l < 2^gs} |in[b*stride_in + J*2^gs + l]| for J < n, added in index order in the
// input's type (the group activations of eq. (6)).
hipError_t launch_group_sums_f32(const float* in, int B, long long stride_in, int n, int gs, float* out,
                                 long long stride_out, hipStream_t s);
hipError_t launch_group_sums_f64(const double* in, int B, long long stride_in, int n, const int32_t* n_dev, int n_cap,
                                 int gs, double* out, long long stride_out, hipStream_t s);

// y[b,:] = sum_{e < k} coef * W2[row, :] over token b's entries (row, coefficient) of list [B, k] (SelectParams::
// list_out), plus sum_{r < m1} fl32(hd[b*m1 + r]) * Wd[r, :] (CommonPath's dense units; m1 = 0: none).  Fixed order.
hipError_t launch_w2_list(const uint16_t* W2, int d, int B, int k, const void* list, const uint16_t* Wd, int m1,
                          const double* hd, float* y, hipStream_t s);

// ---- ffn_fast.hip ----------------------------------------------------------
// FFN step of few tokens in three kernels; see the file header.  All pointers device.
constexpr int kFastTokens = 8;               // most tokens of a step that takes this route
constexpr size_t kFastRegionBytes = 256 + 2 * 8192 * 4;  // state and histograms of one token
struct FfnFastArgs {
  int B, N, d, k, kprime;
  const void* q4;
  const float* q4_scale;
  const uint16_t* w1u;
  const uint16_t* w2u;
  const uint16_t* x;
  float* y;
  int32_t* topk_idx;   // optional
  float* topk_val;     // optional
  int32_t* cand_out;   // optional: the caller's copy of the candidate list
  int32_t* n_cand;     // optional
  int32_t* scorer_acc; // optional
  // workspace
  void* fast_region;   // kFastTokens regions near the head of the workspace (cookie, anchors, histograms)
  float* keys;         // [B, key_stride], key_stride a multiple of 4
  long long key_stride;
  double* h;           // [B, ffn_fast_entries(N, gs)]: activations of the units (gs = 3: of the groups)
  float* h32;          // the same rounded to fp32
  // group-sparse step with groups of eight units (gs = 3; 0 otherwise): N, k, kprime still count units; cand_out,
  // n_cand and topk_idx are in groups, topk_val per unit
  int gs;
  float* gkeys;        // gs = 3: [B, gkey_stride], gkey_stride a multiple of 4
  long long gkey_stride;
  float* u32;          // gs = 3: [B, ffn_fast_entries(N, gs) << gs] activations of the units
  // CommonPath (eq. (7)): m1 dense units next to the sparse ones, folded into the gather and second-layer
  // launches as extra workgroups (m1 = 0: none).
  const uint16_t* dense_w1u;  // [m1, d]
  const uint16_t* dense_w2u;  // [m1, d]
  int m1;
  double* h_dense;            // [B, m1] workspace
  // several tokens: the union of their shortlists, a place for its list where the caller wants its length only, and
  // (lrq) the quantised tokens
  uint32_t* bitmap;
  int32_t* cand_scratch;
  int8_t* xq;
  // Low-rank scorer (lowrank, up to four tokens; otherwise the int4 one): keys are fp64 (keys64, [B, key_stride], rows of
  // whole 16-byte vectors), t the bf16 intermediate [B, r], norm_bounds the two row-norm bounds of
  // hire_lr_prepare; gs = 3: gkeys64 instead of gkeys, in rows of whole vectors as well.
  bool lowrank;
  const void* lr_a;
  const void* lr_b;
  int r;
  const float* norm_bounds;
  uint16_t* t;
  double* keys64;
  double* gkeys64;
  // int4 low-rank scorer (lrq, up to four tokens): lr_a / lr_b are the packed blobs of Z1 transposed and Z2 with their
  // scales, keys_t B * r + 4 floats for the intermediate; the keys are fp32 (keys); norm_bounds[0] bounds the rows of w1u
  bool lrq;
  const float* lr_a_scale;
  const float* lr_b_scale;
  float* keys_t;
  hipEvent_t* stage_events;  // optional: 4 events recorded around the kernels
  unsigned long long* scorer_clocks;  // optional, one token: start/end wall clock (100 MHz ticks) of every scorer workgroup
};
int ffn_fast_score_blocks(int N);
size_t ffn_fast_fallbacks_offset();  // two uint32 counters inside the region
// Where the region keeps its cookie (and the value that says "key histogram all zero") and its two histograms.
void ffn_fast_state_layout(size_t* cookie_off, unsigned long long* cookie, size_t* hist1_off, size_t* hist2_off,
                           size_t* hist_words);
bool ffn_fast_supported(int B, int N, int d, int k, int kprime, bool groups = false);
bool ffn_fast_group8_supported(int B, int N, int d, int k, int kprime);  // the same route for groups of eight units
int ffn_fast_entries(int N, int gs);
hipError_t launch_ffn_fast(const FfnFastArgs& a, hipStream_t s);
// ---- ffn_fast_tokens.hip: the first two kernels for two to kFastTokens tokens
bool ffn_fast_tokens_supported(int B, int d, bool groups);
hipError_t launch_fast_score_tokens(const FfnFastArgs& a, const void* x, bool lrq, hipStream_t s);
hipError_t launch_fast_gather_tokens(const FfnFastArgs& a, hipStream_t s);

// ---- ffn_shard.hip -----------------------------------------------------------
// HiRE-FFN step with Algorithm 2's sharded approximate top-k, one workgroup per shard; see the file header.
// Requires ffn_shard_supported(N, d, shards); quotas ceil(k'/shards), ceil(k/shards).  All pointers device.
constexpr int kShardMaxUnits = 1024;  // units per shard
struct FfnShardArgs {
  int N, d, B, k, kprime, shards;
  const void* q4;
  const float* q4_scale;
  const uint16_t* w1u;
  const uint16_t* w2u;
  const uint16_t* x;
  float* y;
  int32_t* topk_idx;    // optional [B, shards*ceil(k/shards)]
  float* topk_val;      // optional [B, shards*ceil(k/shards)]
  int32_t* cand;        // optional [shards, min(B*ceil(k'/shards), N/shards)]
  int32_t* n_cand;      // optional [shards]
  int32_t* scorer_acc;  // optional [B, N]
  float* partial;       // workspace: ffn_shard_partial_floats(B, d, shards) floats
};
bool ffn_shard_supported(int N, int d, int shards);
size_t ffn_shard_partial_floats(int B, int d, int shards);
hipError_t launch_ffn_shard(const FfnShardArgs& a, hipStream_t s);         // the shards' partial rows
// ---- ffn_shard_batch.hip: the same step for batches and long shards, in the unsharded step's kernels
bool ffn_shard_batch(int B, int N, int d, int shards);  // whether it is the faster one
struct FfnShardBuffers {
  int8_t* xq;            // [B, d]
  float* vals;           // [B, stride], stride a multiple of 4: keys, then the filter stage's values
  long long stride;
  uint32_t* bitmap;      // union: zero_words words, whole 64-bit ones over the units
  int zero_words;
  float* xnorm;          // [HIRE_MAX_BATCH]
  float* wnorm_tiles;    // [filter_tiles(N)]
  uint2* list;           // [B, shards ceil(k/shards)]
};
hipError_t launch_ffn_shard_batch(const FfnShardArgs& a, const FfnShardBuffers& f, hipStream_t s);
hipError_t launch_ffn_shard_reduce(const FfnShardArgs& a, hipStream_t s);  // y = their sum

}  // namespace hire
