// C ABI of libhire (declared in include/hire.h): argument validation, workspace
// carving and the kernel sequence of one HiRE-FFN / HiRE-Softmax decode step.
#include "../../include/hire.h"

#include "kernels.h"

#include <atomic>
#include <cmath>
#include <vector>

// Scratch memory of hire_ffn_step_static: one array per GPU the library runs on, held until the process ends,
// all zero when the code object is loaded (which is the state hire_workspace_init gives a workspace).  In host
// code this name only stands for the symbol; the memory is reached through the per-device address that
// hipGetSymbolAddress returns (static_scratch below), never through the name.
static __device__ __align__(256) unsigned char scratch[HIRE_STATIC_SCRATCH_BYTES];

namespace {

using namespace hire;

constexpr size_t kAlign = 256;
constexpr int kSingleWgMaxRow = 32768;  // up to this row length one workgroup per token selects the k' keys
constexpr int kMfmaMinBatch = 2;  // from this batch size on the scorer and the gather run on the matrix cores; and one token of
                                  // an FFN with more units than the route for few tokens takes, up to 32768: its kernels are
                                  // the batch's.  20000 units of d = 800 37.3 us per step, against 56.4 with selections that
                                  // stream the keys; 24000 of 1440 42.7 against 70.5, fp64 keys 50.4 against 80.8
// FFN step, rows of at most 32768 units: filter and refine from kFilterMinBatch tokens on.  Up to four tokens are one tile
// of the fp64 matrix cores (d = 512, 20003 units: 38 / 39 / 41 us for 2 / 3 / 4 tokens against 46 / 47 / 48); they take it
// where the union may have more than 16384 units, which the selection of fp64 values streams (ffn_filter; four tokens, 24000
// units: d = 288 40.4 against 63.9, d = 1440 58.9 against 73.2).  From
// kFilterValuesMinBatch on values of the filter stage may be handed out (hire_ffn_step says which).
constexpr int kFilterMinBatch = 5;
constexpr int kFilterValuesMinBatch = 16;
constexpr int kCounters = 64;     // int32 counters behind the union bitmap, cleared with it by a step's first kernel
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// The head of every workspace: the general route's header, then the state of the route for few tokens, a region per token.
// Both keep what the step before left, whichever entry point and shapes that had - with one exception: FFN layouts that
// cannot take the route for few tokens keep the first region only and put their buffers on the others, and their steps
// leave the cookie at one region (general_header_check).
size_t regions_offset() { return align_up(general_header_bytes()); }
size_t body_offset(int regions) { return regions_offset() + align_up((size_t)regions * kFastRegionBytes); }

// Bump allocator over the caller's workspace; with base == nullptr it only measures.
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base(static_cast<char*>(b)) {}
  template <typename T>
  T* take(size_t count) {
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off = align_up(off + count * sizeof(T));
    return p;
  }
};

struct StepBuffers {
  HistRefs hist;      // general route: header at offset 0; key histograms (long rows)
  void* fast_region;  // behind it: state and histograms of the three-kernel route, a region per token
  uint32_t* window_misses;  // counter inside the header
  unsigned long long sig;  // names this layout
  int8_t* xq;
  float* sumabs;     // [B] sums of the tokens' absolute int8 codes
  uint16_t* t;       // low-rank intermediate, bf16 [B, r]
  float* keys_t;     // int4 low-rank scorer: the intermediate before rounding, fp32 [B, r]
  void* keys;        // fp32 or fp64 [B, key_stride]
  long long key_stride;
  void* gkeys;       // group-sparse: summed absolute keys, same type, [B, N >> gs] ([B, gkey_stride] for 1 to 8 tokens)
  long long gkey_stride;
  double* hg;        // group-sparse: summed absolute exact activations [B, cap_u]
  uint32_t* bitmap;  // candidate union bitmap, then (after it) the counters
  int32_t* counters; // [0] = |U|
  int32_t* cand;     // U
  double* h;         // [B, cap_u]
  double* h_refine;  // filter and refine: scratch of the refining selection, in the candidates' order
  int32_t* pos;      // group-sparse: [B, k >> gs] positions inside U of every token's selected groups
  uint2* list;       // [B,k] selected units as (row, coefficient), for the second layer
  float* h32;        // few tokens: activations by unit (by group) in fp32
  float* u32;        // ... groups: the units'
  // filter and refine of the exact stage (batches): upper bounds of the tokens' norms, the fp32 stored values
  float* xnorm;      // [B]
  float* wnorm_tiles; // largest candidate row norm of every workgroup of the filter stage
  void* refine_slots; // softmax: the final selection's slots
  float* maxima;     // softmax: [B, kFilterMaxima] largest values of parts of hf's rows
  float* hf;         // [B, hf_stride]: by unit (FFN, in the keys' place) or by rank in the union (softmax)
  long long hf_stride;
  bool by_unit;      // FFN batches on rows of at most 32768 units: the selections of batch_select.hip
  bool all_rows;     // ... whose filter stage runs beside the selection of k', over all rows (filter_all_rows)
  void* sm1_slots;   // long rows: slots of the keys at or above the bound from the scorer's maxima
  bool sm1_ok;       // ... which this layout has
  bool max_ok;       // long rows: slots for the selection of k' from the scorer's maxima
  int words, cap_u, zero_words;
  size_t bytes;
};

constexpr int kSoftmaxOwnMaxRow = 65536;  // longer unions of a softmax step keep the refining selection's buffers in others' places
constexpr int kKeysInRegisters = 16384;  // rows that the route for few tokens and the selection of fp64 values hold
bool ffn_filter(const StepBuffers& s, int B) { return s.by_unit && (B >= kFilterMinBatch || s.cap_u > kKeysInRegisters); }

// Softmax step, filter and refine: for which unions (of at most cap_u classes) and k the refining selection is cheaper than
// ranking fp64 logits.  It finds its mark from the filter stage's maxima, up to four per workgroup; with few more than k of
// them much of the union lies above the mark, with fewer than k all of it, and what does not fit the slots is ranked in rounds.  The
// maxima are counted for a union of 1.5 k' too, about what tokens of one query leave, and as if every workgroup had 64 classes;
// small unions go to up to four times as many workgroups of sixteen, with more maxima, but where they are too few by this count
// fp64 is still the faster one.  Beyond 32 tokens the union is larger, and ranking dearer.  us per step, fp64 / refined, * the rule: 40000
// classes of d = 512, k' = 1536, k = 128, eight tokens 52.5 / 44.4*, fifteen 78.5 / 50.8*; k' = 256, k = 128, three (48 maxima by this count)
// 33.2* / 41.4, of one query 33.1* / 48.3, eight (128) 36.8* / 39.5, fifteen (240) 39.1* / 41.3; k' = 1024, k = 512, sixteen 58.7* / 104.6, 64 189.6 /
// 125.7*; k = 256, eight 47.5 / 49.2*, fifteen 57.0 / 55.9*; k' = 256, k = 64, 17 44.9 / 41.6*, 64 90.7 / 55.9*.  256000 classes of d = 2048, k' = 1024, k = 128,
// three 79.6* / 85.0, eight 97.5 / 89.6*, fifteen 119.3 / 102.3*; k = 256, 64 589.7 / 203.9*; k' = 1200, k = 100, 64 681 / 200*.  A few tokens with
// short lists would be faster through fp64 too: k' = 512, k = 64, three 32.9* / 36.6, eight 36.5 / 38.3*, of 256000 classes 82.0 / 84.7*; k' = 256, k = 16,
// three 31.0 / 34.6*.  The longest union is what 256 workgroups of the filter stage list in LDS.
bool softmax_filter(int B, int cap_u, int k, int kprime) {
  if (B < 3 || cap_u > kSoftmaxRefineMaxRow || k > (B < 16 ? kSoftmaxRefineMaxK / 2 : kSoftmaxRefineMaxK)) return false;
  const int blocks = min(filter_tiles(cap_u), 256), each = (kprime + kprime / 2 + blocks - 1) / blocks;
  return 2 * blocks >= k && 4 * blocks * min(4, (each + 3) / 4) >= (B > 32 ? 3 : 5) * k;
}

// Whether the filter stage reads all rows of the FFN at once with the selection of k' instead of the union's rows behind it:
// where what it reads in vain costs less than the wait that it saves, also for tokens that share most of their picks (about
// k' (1 + log2(B) / 4) rows between them; independent ones soon need nearly all).  us per step behind the selection / beside
// it, k' = N / 5, independent tokens; tokens with nine tenths in common:
//   d = 2048, N = 8192: 16 tokens 38.8 / 34.7; 36.6 / 33.5   64: 55.8 / 50.1; 50.2 / 43.6
//   d = 800, N = 5003:  16 tokens 34.7 / 30.4; 33.7 / 30.1   33: 42.7 / 36.7; 41.4 / 36.1
//   d = 4096, N = 8192: 16 tokens 57.5 / 53.7; 49.1 / 51.1 (40 MB in vain)   64: 81.1 / 75.6; 70.5 / 70.1
// With more workgroups than compute units, a token or 64 rows each, the last of them wait for a selection:
//   d = 2048, N = 16384: 16 tokens 52.9 / 50.1; 41.3 / 47.4   33: 66.0 / 62.8; 55.1 / 58.6   64: 72.4 / 68.7; 60.9 / 63.9
//   d = 1024, N = 16384: 16 tokens 38.4 / 37.2; 35.0 / 35.0   64: 53.8 / 51.0; 49.6 / 46.4
// There up to 32 tokens, where samples of one query are more likely, need half as much to be read in vain.  fp64 keys (the
// low-rank scorer) gain a microsecond or two more each: d = 800, N = 5003, 33 tokens 46.5 / 38.2, d = 2048, N = 16384, 16
// tokens 57.7 / 54.9; 45.5 / 51.5.
bool filter_all_rows(int B, int d, int N, int kprime) {
  const double shared = kprime * (1.0 + 0.25 * std::log2((double)B)), vain = N - (shared < N ? shared : N);
  return vain * 2.0 * d <= (B + filter_tiles(N) <= 256 || B > 32 ? 36.0 : 18.0) * (1 << 20);
}

// gs > 0: group-sparse FFN with groups of 2^gs units; the selections, the bitmap, the union and cap_u then count
// groups, while keys and h keep one value per unit.
StepBuffers carve(void* ws, int scorer_kind, int B, int d, int N, int r, int k, int kprime, bool ffn, int gs = 0) {
  StepBuffers s{};
  Carver c(ws);
  const int Ns = N >> gs, kps = kprime >> gs;
  s.cap_u = (int)((long long)B * kps < (long long)Ns ? B * kps : Ns);
  s.words = (Ns + 31) / 32 + 2;
  const bool fast = ffn && (gs == 3 ? ffn_fast_group8_supported(B, N, d, k, kprime)
                                    : (gs == 0 && ffn_fast_supported(B, N, d, k, kprime)));
  s.hist.header = c.take<char>(general_header_bytes());
  s.fast_region = c.take<char>((ffn && !fast ? 1 : kFastTokens) * kFastRegionBytes);
  s.sig = layout_signature(scorer_kind, B, d, N, r, k, kprime, (ffn ? 1 : 0) + 16 * gs) | (ffn && !fast ? kSigOverlays : 0);
  s.window_misses = s.hist.header ? reinterpret_cast<uint32_t*>(static_cast<char*>(s.hist.header) +
                                                                 general_fallbacks_offset(1))
                                  : nullptr;
  const bool int4_like = scorer_kind == HIRE_SCORER_INT4 || scorer_kind == HIRE_SCORER_LRQ;
  s.by_unit = ffn && (B >= kMfmaMinBatch || N > kKeysInRegisters) && gs == 0 && batch_select_supported(N, k);
  s.key_stride = s.by_unit || (fast && gs == 0) ? (N + 3) / 4 * 4 : N;  // whole 16-byte vectors
  if (int4_like && N > kSingleWgMaxRow && gs == 0) s.hist.multi_body = c.take<char>(multi_body_bytes_host(B));
  if (int4_like) {
    s.xq = c.take<int8_t>((size_t)B * (d > r ? d : r));
    s.sumabs = c.take<float>(B);
    s.keys = c.take<float>((size_t)B * s.key_stride + 4);
    s.gkey_stride = (Ns + 3) / 4 * 4;
    if (gs > 0) s.gkeys = c.take<float>((size_t)B * s.gkey_stride + 4);
    if (scorer_kind == HIRE_SCORER_LRQ) {
      s.keys_t = c.take<float>((size_t)B * r + 4);
      s.t = c.take<uint16_t>((size_t)B * r);
    }
  } else {
    s.t = c.take<uint16_t>((size_t)B * r);
    s.keys = c.take<double>((size_t)B * s.key_stride);
    s.gkey_stride = (Ns + 1) / 2 * 2;
    if (gs > 0) s.gkeys = c.take<double>((size_t)B * s.gkey_stride);
  }
  // bitmap and counters are contiguous so that one pass clears both.  counters[0] = |U|
  s.bitmap = c.take<uint32_t>((size_t)s.words + kCounters);
  s.counters = s.bitmap ? reinterpret_cast<int32_t*>(s.bitmap + s.words) : nullptr;
  s.zero_words = s.words + kCounters;
  s.cand = c.take<int32_t>(s.cap_u);
  const bool sm_filter = !ffn && gs == 0 && softmax_filter(B, s.cap_u, k, kprime);
  auto sm_buffers = [&](Carver& at) {
    s.xnorm = at.take<float>(HIRE_MAX_BATCH);
    s.maxima = at.take<float>((size_t)B * kFilterMaxima);
    s.refine_slots = at.take<char>(softmax_refine_slot_bytes(B));
  };
  const bool sm_long = sm_filter && s.cap_u > kSoftmaxOwnMaxRow;
  s.all_rows = ffn_filter(s, B) && !fast && s.key_stride <= 2 * (long long)s.cap_u &&
               (int4_like || N <= kSelectFilterMaxF64) && filter_all_rows(B, d, N, kprime);
  if (ffn_filter(s, B)) {
    s.xnorm = c.take<float>(HIRE_MAX_BATCH);
    s.wnorm_tiles = c.take<float>(filter_tiles(N));
    s.hf_stride = s.key_stride;  // rows start at multiples of 16 bytes
    s.hf = static_cast<float*>(s.keys);  // nobody reads the keys any more when the filter stage runs
  } else if (sm_filter && !sm_long) {
    sm_buffers(c);
    s.hf_stride = (s.cap_u + 3) / 4 * 4;
    s.hf = c.take<float>((size_t)B * s.hf_stride);
  }
  const size_t h_doubles = ((size_t)B * s.cap_u << gs) + 2, fast_doubles = fast ? (size_t)B * ffn_fast_entries(N, gs) : 0;
  s.h = c.take<double>(h_doubles > fast_doubles ? h_doubles : fast_doubles);
  // all_rows: the filter stage writes its values while the keys are read.  h is the selection's scratch only after that, so
  // the keys or the values go there: the fp32 keys, whose own place is too small for the scratch, or else the values
  s.h_refine = s.h;
  if (s.all_rows && int4_like) {
    s.keys = s.h;
  } else if (s.all_rows) {
    s.hf = reinterpret_cast<float*>(s.h);
    s.h_refine = static_cast<double*>(s.keys);
  }
  if (fast) {
    s.h32 = c.take<float>((size_t)B * ffn_fast_entries(N, gs));
    if (gs > 0) s.u32 = c.take<float>((size_t)B * ffn_fast_entries(N, 0));
  }
  if (gs > 0) s.hg = c.take<double>((size_t)B * s.cap_u + 2);
  s.sm1_ok = !ffn && B == 1 && gs == 0 && int4_like && N > kSingleWgMaxRow && softmax_b1_supported(N, d, 1, 1);
  s.max_ok = gs == 0 && int4_like && N > kSingleWgMaxRow && maxima_select_supported(N);
  if (s.sm1_ok || s.max_ok) s.sm1_slots = c.take<char>(maxima_select_slot_bytes(B, N));
  // Long unions ask for no more workspace than the route through fp64 logits: their fp32 logits lie in the place of the keys, which nobody
  // reads any more when the filter stage runs, and the rest (37 KB per token) where the selection of k' had its slots (64 KB), or
  // behind the fp32 logits where it has none: fp64 keys, and keys of more than 262144 classes, leave 256 KB per token there.  Shorter
  // ones have places of their own, but for the row norms, of which there may be more than there once were; with the logits in the keys' place
  // too, 35 tokens of d = 352, 48950 classes took 56.5 us per step instead of 55.6, 36 of d = 1760, 117306 classes 82.6 instead of 81.5.
  if (sm_filter) {
    Carver in_keys(s.keys), in_slots(s.sm1_slots);
    if (sm_long) {
      s.hf_stride = s.cap_u;
      s.hf = in_keys.take<float>((size_t)B * s.hf_stride);
      sm_buffers(s.max_ok ? in_slots : in_keys);
    }
    s.wnorm_tiles = in_keys.take<float>(filter_rank_blocks(s.cap_u));
  }
  if (ffn) {
    if (gs > 0) s.pos = c.take<int32_t>((size_t)B * (k >> gs));
    s.list = c.take<uint2>((size_t)B * k);
  }
  s.bytes = c.off;
  return s;
}

int check_common(int d, int N, int B, int k, int kprime, int scorer_kind, const void* q4, const float* q4_scale,
                 const void* lr_a, const void* lr_b, int r, const float* lr_a_scale, const float* lr_b_scale,
                 const void* W, const void* x) {
  if (d < 32 || d % 8 != 0 || N < 1 || B < 1 || B > HIRE_MAX_BATCH) return HIRE_EINVAL;
  if (k < 1 || k > kprime || kprime > N) return HIRE_EINVAL;
  if (!W || !x || !aligned(W, 256) || !aligned(x, 16)) return HIRE_EINVAL;
  if (scorer_kind == HIRE_SCORER_INT4) {
    if (d % 32 != 0 || !q4 || !q4_scale || !aligned(q4, 256)) return HIRE_EINVAL;
  } else if (scorer_kind == HIRE_SCORER_LRQ) {
    if (d % 32 != 0 || r < 32 || r % 32 != 0 || r > 1024 || !lr_a || !lr_b || !lr_a_scale || !lr_b_scale ||
        !aligned(lr_a, 256) || !aligned(lr_b, 256))
      return HIRE_EINVAL;
  } else if (scorer_kind == HIRE_SCORER_LOWRANK) {
    if (r < 8 || r % 8 != 0 || r > 1024 || !lr_a || !lr_b || !aligned(lr_a, 16) || !aligned(lr_b, 256))
      return HIRE_EINVAL;
  } else {
    return HIRE_EINVAL;
  }
  return HIRE_OK;
}

thread_local hipError_t g_last_hip_error = hipSuccess;

#define HIRE_TRY(expr)                 \
  do {                                 \
    const hipError_t e_ = (expr);      \
    if (e_ != hipSuccess) {            \
      g_last_hip_error = e_;           \
      return HIRE_ELAUNCH;             \
    }                                  \
  } while (0)

// Optional stage timing: when the caller has handed over events, event i is recorded on the stream in front of
// stage i and one more after the last stage.
thread_local hipEvent_t* g_stage_events = nullptr;
thread_local int g_force_generic = 0;      // testing: route every step through the general multi-kernel path
thread_local int g_force_exact_stage = 0;  // testing: batches compute every candidate's activation in fp64
thread_local unsigned long long* g_scorer_clocks = nullptr;  // measuring: where the one-token scorer leaves its clocks

#define HIRE_STAGE(i, st)                                             \
  do {                                                                \
    if (g_stage_events) HIRE_TRY(hipEventRecord(g_stage_events[i], st)); \
  } while (0)

// Steps 1-3 of a step, shared by FFN and softmax: scorer, per-token top-k', union, exact scores on the union.
struct ScorerRefs {
  int kind;
  const void* q4;
  const float* q4_scale;
  const void* lr_a;
  const void* lr_b;
  int r;
  const float* lr_a_scale;
  const float* lr_b_scale;
};
template <typename Layer>
ScorerRefs scorer_of(const Layer* L) {
  return ScorerRefs{L->scorer_kind, L->q4, L->q4_scale, L->lr_a, L->lr_b, L->r, L->lr_a_scale, L->lr_b_scale};
}

// filter: the exact stage writes the fast bf16 approximations (launch_filter_units) instead of the fp64
// activations; the caller then refines around the selection threshold.
// maxima_out (one token, int4 scorers): return after the scorer, with the number of maxima it left.
int run_front(const StepBuffers& s, const ScorerRefs& sc, const void* W, const void* x, int B, int d, int N,
              int kprime, int relu, int32_t* cand_out, int32_t* n_cand, int32_t* scorer_acc, hipStream_t st,
              int gs = 0, bool filter = false, int* maxima_out = nullptr) {
  const int scorer_kind = sc.kind, r = sc.r;
  const void* lr_a = sc.lr_a;
  const void* lr_b = sc.lr_b;
  const uint16_t* xb = static_cast<const uint16_t*>(x);
  // what the int4 scorer and its token quantisation work on: the layer's own int4 copy and the token, or
  // (int4 low-rank scorer) the int4 copy of Z2 and the r-vector t
  const bool lrq = scorer_kind == HIRE_SCORER_LRQ;
  const bool int4_like = scorer_kind == HIRE_SCORER_INT4 || lrq;
  const bool batch = B >= kMfmaMinBatch || s.by_unit;
  const void* q4 = lrq ? sc.lr_b : sc.q4;
  const float* q4_scale = lrq ? sc.lr_b_scale : sc.q4_scale;
  const uint16_t* tok = lrq ? s.t : xb;
  const int sd = lrq ? r : d;
  // what is ranked: units, or groups of 2^gs units by their summed absolute keys.  Groups of eight are summed by
  // the selection as it loads the keys; other sizes by a kernel of their own.
  const int Ns = N >> gs;
  const bool in_select = gs == 3 && Ns <= kGroupSelectMax;
  GroupSelect gsel{s.keys, !int4_like, N, Ns, nullptr, kprime >> gs, s.bitmap, nullptr, nullptr, nullptr, nullptr, s.window_misses};
  SelectParams sp{};
  sp.stride = gs == 0 ? s.key_stride : Ns;
  sp.n = Ns;
  sp.n_cap = Ns;
  sp.k = kprime >> gs;
  sp.relu = 0;  // the scorers already applied phi
  sp.nonneg = relu;  // phi = ReLU (and sums of absolute values): nothing negative is ranked
  sp.bitmap = s.bitmap;
  sp.vals = (gs > 0 && !in_select) ? s.gkeys : s.keys;
  int32_t* cand = cand_out ? cand_out : s.cand;
  // short bitmaps are compacted by the gather kernel itself; long ones by a kernel of their own
  const bool in_gather = union_in_gather(s.words);
  const bool many_wg = int4_like && N > kSingleWgMaxRow && gs == 0;  // long rows: key histograms
  UnionRefs un{s.bitmap, s.words, cand, s.counters, n_cand, many_wg};
  sp.window_misses = s.window_misses;
  KeysSelect ks{s.keys, !int4_like, s.key_stride, N, kprime, nullptr, nullptr, s.bitmap, s.window_misses};
  HIRE_STAGE(0, st);
  bool t_is_f32 = false;
  if (lrq) {
    // first product of the int4 low-rank scorer: t = bf16(float(Z1q^T xq) * s1), the r rows of Z1^T scored like
    // any int4 matrix (no phi), then rounded to the bf16 activation the second product quantises
    const HistRefs header_only{s.hist.header, nullptr};
    const uint32_t* qa = static_cast<const uint32_t*>(lr_a);
    if (!batch && scorer_int4_fused_supported(d)) {
      HIRE_TRY(launch_scorer_int4_fused(qa, sc.lr_a_scale, xb, false, r, d, 0, s.keys_t, nullptr, header_only, s.bitmap,
                                        s.zero_words, s.sig, st));
    } else if (batch) {
      ScorerTokens tk{s.xq, nullptr, false, nullptr, s.bitmap, s.zero_words, s.hist.header, s.sig};
      if (scorer_mfma_quantises(B, r, d, false)) tk.x = xb;
      else HIRE_TRY(launch_quantize_tokens(xb, false, B, d, s.xq, s.sumabs, s.bitmap, s.zero_words, s.hist.header, s.sig, st));
      HIRE_TRY(launch_scorer_int4_mfma(qa, sc.lr_a_scale, tk, B, r, d, 0, s.keys_t, r, nullptr, header_only, st));
    } else {
      HIRE_TRY(launch_quantize_tokens(xb, false, B, d, s.xq, s.sumabs, s.bitmap, s.zero_words, s.hist.header, s.sig, st));
      HIRE_TRY(launch_scorer_int4(qa, sc.lr_a_scale, s.xq, B, r, d, 0, s.keys_t, nullptr, header_only, st));
    }
    // whatever quantises the intermediate rounds it as well
    t_is_f32 = batch || (scorer_int4_fused_supported(r) && scorer_int4_fused_takes_f32(r));
    if (!t_is_f32) HIRE_TRY(launch_f32_to_bf16(s.keys_t, B * r, s.t, st));
  }
  if (int4_like) {
    // the scorer quantises the token itself
    const bool fused = !batch && scorer_int4_fused_supported(sd);
    const bool fused_batch = batch && scorer_mfma_quantises(B, N, sd, t_is_f32);
    if (!fused && !fused_batch)
      HIRE_TRY(launch_quantize_tokens(t_is_f32 ? static_cast<const void*>(s.keys_t) : tok, t_is_f32, B, sd, s.xq, s.sumabs,
                                      s.bitmap, s.zero_words, s.hist.header, s.sig, st));
    HIRE_STAGE(1, st);
    int slots;
    if (fused) {
      HIRE_TRY(launch_scorer_int4_fused(static_cast<const uint32_t*>(q4), q4_scale,
                                        t_is_f32 ? static_cast<const void*>(s.keys_t) : static_cast<const void*>(tok),
                                        t_is_f32, N, sd, relu,
                                        static_cast<float*>(s.keys), scorer_acc, s.hist, s.bitmap, s.zero_words, s.sig,
                                        st));
      slots = scorer_int4_fused_maxima(N, sd);
    } else if (batch) {
      ScorerTokens tk{s.xq, nullptr, t_is_f32, s.sumabs, s.bitmap, s.zero_words, s.hist.header, s.sig};
      if (fused_batch) tk.x = t_is_f32 ? static_cast<const void*>(s.keys_t) : static_cast<const void*>(tok);
      HIRE_TRY(launch_scorer_int4_mfma(static_cast<const uint32_t*>(q4), q4_scale, tk, B, N, sd, relu,
                                       static_cast<float*>(s.keys), s.key_stride, scorer_acc, s.hist, st));
      slots = scorer_mfma_maxima(N);
    } else {
      HIRE_TRY(launch_scorer_int4(static_cast<const uint32_t*>(q4), q4_scale, s.xq, B, N, sd, relu,
                                  static_cast<float*>(s.keys), scorer_acc, s.hist, st));
      slots = scorer_int4_blocks(N);
    }
    HIRE_STAGE(2, st);
    if (maxima_out != nullptr) {
      *maxima_out = slots;
      return fused ? HIRE_OK : HIRE_EINVAL;
    }
    if (gs > 0 && !in_select)
      HIRE_TRY(launch_group_sums_f32(static_cast<const float*>(s.keys), B, N, Ns, gs, static_cast<float*>(s.gkeys), Ns,
                                     st));
    if (many_wg && B >= 2 && s.max_ok && in_gather && maxima_select_worthwhile(B, N, kprime, slots) && !g_force_generic) {
      // long rows, batches: every token's k' largest keys from the bound that the scorer's maxima give (no key
      // histogram is filled or read, so none is stamped clean either)
      HIRE_TRY(launch_maxima_select(static_cast<const float*>(s.keys), B, N, sd, kprime, slots, q4, s.hist, s.sm1_slots,
                                    s.bitmap, st));
      HIRE_STAGE(3, st);
      un.stamp_keys = false;
    } else if (many_wg) {
      HIRE_TRY(launch_mark_f32(static_cast<const float*>(s.keys), B, N, kprime, slots, s.hist, s.bitmap, st));
      HIRE_STAGE(3, st);
      HIRE_TRY(launch_resolve_compact(static_cast<const float*>(s.keys), B, N, kprime, s.hist, s.bitmap, s.words,
                                      in_gather ? nullptr : cand, s.counters, n_cand, nullptr, 0, st));
    } else if (s.by_unit) {
      ks.sumabs = s.sumabs;
      ks.smax = reinterpret_cast<const float*>(static_cast<const char*>(q4) + (size_t)N * (sd / 2));
      if (s.all_rows && filter) {
        HIRE_TRY(launch_select_filter(ks, B, static_cast<const uint16_t*>(W), xb, d, s.hf, s.hf_stride, s.xnorm, s.wnorm_tiles,
                                      st));
        HIRE_STAGE(3, st);
        HIRE_STAGE(4, st);
        return HIRE_OK;
      }
      HIRE_TRY(launch_keys_select(ks, B, st));
      HIRE_STAGE(3, st);
    } else {
      if (in_select) HIRE_TRY(launch_group_select(gsel, B, st));
      else HIRE_TRY(launch_select_f32(sp, B, st));
      HIRE_STAGE(3, st);
      if (!in_gather) HIRE_TRY(launch_bitmap_compact(s.bitmap, s.words, cand, s.counters, n_cand, nullptr, 0, st));
    }
  } else {
    HIRE_TRY(launch_lr_project(static_cast<const uint16_t*>(lr_a), xb, B, d, r, s.t, s.bitmap, s.zero_words, s.hist.header,
                               s.sig, st));
    HIRE_STAGE(1, st);
    if (batch)
      HIRE_TRY(launch_lr_score_mfma(static_cast<const uint16_t*>(lr_b), s.t, B, N, r, relu, static_cast<double*>(s.keys),
                                    s.key_stride, st));
    else
      HIRE_TRY(launch_lr_score(static_cast<const uint16_t*>(lr_b), s.t, N, r, relu, static_cast<double*>(s.keys), st));
    HIRE_STAGE(2, st);
    if (s.all_rows && filter) {
      HIRE_TRY(launch_select_filter(ks, B, static_cast<const uint16_t*>(W), xb, d, s.hf, s.hf_stride, s.xnorm, s.wnorm_tiles,
                                    st));
      HIRE_STAGE(3, st);
      HIRE_STAGE(4, st);
      return HIRE_OK;
    }
    if (gs > 0 && !in_select)
      HIRE_TRY(launch_group_sums_f64(static_cast<const double*>(s.keys), B, N, Ns, nullptr, Ns, gs,
                                     static_cast<double*>(s.gkeys), Ns, st));
    if (s.by_unit)
      HIRE_TRY(launch_keys_select(ks, B, st));
    else if (in_select)
      HIRE_TRY(launch_group_select(gsel, B, st));
    else
      HIRE_TRY(launch_select_f64(sp, B, st));
    HIRE_STAGE(3, st);
    if (!in_gather) HIRE_TRY(launch_bitmap_compact(s.bitmap, s.words, cand, s.counters, n_cand, nullptr, 0, st));
  }
  HIRE_STAGE(4, st);
  if (filter && s.by_unit)
    HIRE_TRY(launch_filter_units(static_cast<const uint16_t*>(W), xb, B, d, s.bitmap, nullptr, N, s.hf, s.hf_stride, s.xnorm,
                                 s.wnorm_tiles, nullptr, st));
  else if (filter)
    HIRE_TRY(launch_filter_ranks(static_cast<const uint16_t*>(W), xb, B, d, cand, s.counters, s.cap_u, s.hf, s.hf_stride,
                                 s.hist, in_gather ? &un : nullptr, N, s.xnorm, s.wnorm_tiles, s.maxima, st));
  else if (batch)
    HIRE_TRY(launch_gather_dot_mfma(static_cast<const uint16_t*>(W), xb, B, d, cand, 0, s.counters, s.cap_u, relu, s.h,
                                    (long long)s.cap_u << gs, s.hist, in_gather ? &un : nullptr, gs, st));
  else
    HIRE_TRY(launch_gather_dot(static_cast<const uint16_t*>(W), xb, d, cand, 0, s.counters, s.cap_u, relu, s.h,
                               s.hist, in_gather ? &un : nullptr, gs, st));
  return HIRE_OK;
}

}  // namespace

extern "C" {

int hire_version(void) { return 100; }

const char* hire_strerror(int code) {
  switch (code) {
    case HIRE_OK: return "ok";
    case HIRE_EINVAL: return "invalid argument";
    case HIRE_ENOSPC: return "workspace too small";
    case HIRE_EUNSUPPORTED: return "unsupported combination";
    case HIRE_ELAUNCH: return "kernel launch failed";
    default: return "unknown error";
  }
}

int hire_workspace_init(void* workspace, size_t workspace_bytes, void* stream) {
  if (!workspace || workspace_bytes < kAlign || !aligned(workspace, 256)) return HIRE_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the general route's header and the head of the first region (smaller workspaces hold neither)
  const size_t state = regions_offset() + kAlign;
  HIRE_TRY(launch_clear_words(static_cast<uint32_t*>(workspace), (int)((workspace_bytes < state ? kAlign : state) / 4), st));
  return HIRE_OK;
}

int hire_debug_fast_fallbacks(const void* workspace, uint32_t* host_out2, void* stream) {
  if (!workspace || !host_out2) return HIRE_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  HIRE_TRY(hipMemcpyAsync(host_out2, static_cast<const char*>(workspace) + regions_offset() + ffn_fast_fallbacks_offset(),
                          2 * sizeof(uint32_t), hipMemcpyDeviceToHost, st));
  HIRE_TRY(hipStreamSynchronize(st));
  return HIRE_OK;
}

int hire_debug_fast_state(const void* workspace, uint32_t* host_out3, void* stream) {
  if (!workspace || !host_out3) return HIRE_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  size_t cookie_off, h1, h2, words;
  unsigned long long want = 0, cookie = 0;
  ffn_fast_state_layout(&cookie_off, &want, &h1, &h2, &words);
  const char* base = static_cast<const char*>(workspace) + regions_offset();
  std::vector<uint32_t> host(2 * words);
  HIRE_TRY(hipMemcpyAsync(&cookie, base + cookie_off, sizeof(cookie), hipMemcpyDeviceToHost, st));
  HIRE_TRY(hipMemcpyAsync(host.data(), base + h1, words * sizeof(uint32_t), hipMemcpyDeviceToHost, st));
  HIRE_TRY(hipMemcpyAsync(host.data() + words, base + h2, words * sizeof(uint32_t), hipMemcpyDeviceToHost, st));
  HIRE_TRY(hipStreamSynchronize(st));
  host_out3[0] = cookie - want < (unsigned long long)kFastTokens ? 1u : 0u;
  host_out3[1] = host_out3[2] = 0u;
  for (size_t i = 0; i < words; ++i) {
    host_out3[1] += host[i] != 0u ? 1u : 0u;
    host_out3[2] += host[words + i];
  }
  return HIRE_OK;
}

int hire_debug_general_fallbacks(const void* workspace, uint32_t* host_out3, void* stream) {
  if (!workspace || !host_out3) return HIRE_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const char* hdr = static_cast<const char*>(workspace);
  for (int i = 0; i < 3; ++i)
    HIRE_TRY(hipMemcpyAsync(host_out3 + i, hdr + general_fallbacks_offset(i), sizeof(uint32_t), hipMemcpyDeviceToHost,
                            st));
  HIRE_TRY(hipStreamSynchronize(st));
  return HIRE_OK;
}

int hire_debug_plain_copy(const void* src, void* dst, size_t bytes, void* stream) {
  if (!src || !dst || bytes == 0 || bytes % 16 != 0 || !aligned(src, 16) || !aligned(dst, 16)) return HIRE_EINVAL;
  HIRE_TRY(launch_plain_copy(src, dst, bytes, static_cast<hipStream_t>(stream)));
  return HIRE_OK;
}

int hire_lr_prepare(const hire_ffn_layer* L, float* bounds2_out, void* stream) {
  const bool lrq = L && L->scorer_kind == HIRE_SCORER_LRQ;
  if (!L || !bounds2_out || (L->scorer_kind != HIRE_SCORER_LOWRANK && !lrq) || !L->w1u || !L->lr_b || L->d_ff < 1 ||
      L->d_model < 8 || L->d_model % 8 != 0 || L->r < 8 || L->r % 8 != 0 || !aligned(L->w1u, 16) ||
      !aligned(L->lr_b, 16) || !aligned(bounds2_out, 4))
    return HIRE_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  HIRE_TRY(launch_row_norm_max(static_cast<const uint16_t*>(L->w1u), L->d_ff, L->d_model, bounds2_out, st));
  if (lrq)  // the int4 copy of Z2 bounds its own keys (largest row scale, kept behind its codes)
    HIRE_TRY(launch_clear_words(reinterpret_cast<uint32_t*>(bounds2_out + 1), 1, st));
  else
    HIRE_TRY(launch_row_norm_max(static_cast<const uint16_t*>(L->lr_b), L->d_ff, L->r, bounds2_out + 1, st));
  return HIRE_OK;
}

int hire_debug_filter_stage(const void* W, const void* x, int B, int d, int rows, const int32_t* rows_dev, float* stored,
                            float* xnorm, uint32_t* wnorm_max, float* err_c, void* stream) {
  if (!W || !x || !rows_dev || !stored || !xnorm || !wnorm_max || !err_c || B < 1 || B > HIRE_MAX_BATCH || rows < 1 ||
      d < 8 || d % 8 != 0 || !aligned(W, 16) || !aligned(x, 16))
    return HIRE_EINVAL;
  *err_c = gather_filter_error(B);
  HIRE_TRY(launch_filter_units(static_cast<const uint16_t*>(W), static_cast<const uint16_t*>(x), B, d, nullptr, rows_dev,
                               rows, stored, rows, xnorm, nullptr, wnorm_max, static_cast<hipStream_t>(stream)));
  return HIRE_OK;
}

int hire_set_scorer_clocks(void* device_buf, size_t bytes) {
  if (device_buf && (bytes < 2 * 1024 * sizeof(unsigned long long) || !aligned(device_buf, 8))) return HIRE_EINVAL;
  g_scorer_clocks = static_cast<unsigned long long*>(device_buf);
  return HIRE_OK;
}

int hire_ffn_scorer_workgroups(int d_ff) { return d_ff > 0 ? ffn_fast_score_blocks(d_ff) : 0; }

void hire_force_generic_path(int on) { g_force_generic = on; }

void hire_force_exact_stage(int on) { g_force_exact_stage = on; }

void hire_set_stage_events(void** events) { g_stage_events = reinterpret_cast<hipEvent_t*>(events); }

const char* hire_last_launch_error(void) { return hipGetErrorString(g_last_hip_error); }

size_t hire_pack_int4_bytes(int rows, int cols) {
  if (rows < 1 || cols < 32 || cols % 32 != 0) return 0;
  return (size_t)rows * (size_t)(cols / 2) + kPackTrailerBytes;
}

int hire_pack_int4(const void* w_bf16, int rows, int cols, void* q4_out, float* scale_out, void* stream) {
  if (!w_bf16 || !q4_out || !scale_out || rows < 1 || cols < 32 || cols % 32 != 0) return HIRE_EINVAL;
  if (!aligned(q4_out, 16)) return HIRE_EINVAL;
  HIRE_TRY(launch_pack_int4(static_cast<const uint16_t*>(w_bf16), rows, cols, static_cast<uint32_t*>(q4_out),
                            scale_out, static_cast<hipStream_t>(stream)));
  return HIRE_OK;
}

int hire_unpack_int4(const void* q4, int rows, int cols, int8_t* codes_out, void* stream) {
  if (!q4 || !codes_out || rows < 1 || cols < 32 || cols % 32 != 0) return HIRE_EINVAL;
  HIRE_TRY(launch_unpack_int4(static_cast<const uint32_t*>(q4), rows, cols, codes_out,
                              static_cast<hipStream_t>(stream)));
  return HIRE_OK;
}

size_t hire_ffn_workspace_bytes(const hire_ffn_layer* L, int B, int k, int kprime) {
  if (!L || L->d_model < 32 || L->d_ff < 1 || B < 1 || B > HIRE_MAX_BATCH || k < 1 || k > kprime || kprime > L->d_ff)
    return 0;
  return carve(nullptr, L->scorer_kind, B, L->d_model, L->d_ff, L->r, k, kprime, true).bytes;
}

size_t hire_softmax_workspace_bytes(const hire_softmax_layer* L, int B, int k, int kprime) {
  if (!L || L->d_model < 32 || L->vocab < 1 || B < 1 || B > HIRE_MAX_BATCH || k < 1 || k > kprime ||
      kprime > L->vocab)
    return 0;
  return carve(nullptr, L->scorer_kind, B, L->d_model, L->vocab, L->r, k, kprime, false).bytes;
}

// Long rows in index order go through the many-workgroup selection, which keeps histograms in the workspace.
// Rank order on such rows: the same selection in index order into the workspace, then the k survivors of every row
// are ranked by the single-workgroup kernel (positions there are in index order, so ties still go to the lower
// index).
static bool topk_long_route(int N, int /*flags*/) { return N > kSingleWgMaxRow; }
static size_t topk_rank_tmp_bytes(int B, int k, int flags) {
  return (flags & HIRE_ORDER_RANK) ? 2 * align_up((size_t)B * k * sizeof(int32_t)) : 0;
}

size_t hire_topk_workspace_bytes(int B, int N, int k, int flags) {
  if (B < 1 || N < 1 || k < 1 || k > N) return 0;
  if (!topk_long_route(N, flags)) return kAlign;  // LDS and registers only; a token amount keeps the pointer non-null
  // the head is that of the step workspaces, so that one initialisation routine serves all
  return body_offset(kFastTokens) + align_up(topk_long_workspace_bytes(B, N)) + topk_rank_tmp_bytes(B, k, flags);
}

int hire_ffn_step(const hire_ffn_layer* L, const void* x, int B, int k, int kprime, float* y, int32_t* topk_idx,
                  float* topk_val, int32_t* cand_idx, int32_t* n_cand, int32_t* scorer_acc, void* workspace,
                  size_t workspace_bytes, void* stream) {
  if (!L || !y || !workspace) return HIRE_EINVAL;
  const int d = L->d_model, N = L->d_ff;
  int rc = check_common(d, N, B, k, kprime, L->scorer_kind, L->q4, L->q4_scale, L->lr_a, L->lr_b, L->r, L->lr_a_scale,
                        L->lr_b_scale, L->w1u, x);
  if (rc != HIRE_OK) return rc;
  if (!L->w2u || !aligned(L->w2u, 256) || !aligned(workspace, 256) || !aligned(y, 16)) return HIRE_EINVAL;
  if (scorer_acc && L->scorer_kind != HIRE_SCORER_INT4) return HIRE_EINVAL;
  const StepBuffers s = carve(workspace, L->scorer_kind, B, d, N, L->r, k, kprime, true);
  if (workspace_bytes < s.bytes) return HIRE_ENOSPC;
  hipStream_t st = static_cast<hipStream_t>(stream);

  const bool fast_int4 = L->scorer_kind == HIRE_SCORER_INT4;
  const bool fast_lr = L->scorer_kind == HIRE_SCORER_LOWRANK && L->row_norm_bounds != nullptr;
  const bool fast_lrq = L->scorer_kind == HIRE_SCORER_LRQ && L->row_norm_bounds != nullptr && scorer_int4_fused_supported(d);
  if ((fast_int4 || fast_lr || fast_lrq) && ffn_fast_supported(B, N, d, k, kprime) && !g_force_generic &&
      !(B > 1 && g_force_exact_stage)) {
    FfnFastArgs a{};
    a.B = B; a.N = N; a.d = d; a.k = k; a.kprime = kprime;
    a.q4 = L->q4; a.q4_scale = L->q4_scale;
    a.lowrank = fast_lr;
    a.lrq = fast_lrq;
    if (fast_lr || fast_lrq) {
      a.lr_a = L->lr_a; a.lr_b = L->lr_b; a.r = L->r; a.norm_bounds = L->row_norm_bounds;
      a.t = s.t; a.keys64 = static_cast<double*>(s.keys);
      a.lr_a_scale = L->lr_a_scale; a.lr_b_scale = L->lr_b_scale; a.keys_t = s.keys_t;
    }
    a.w1u = static_cast<const uint16_t*>(L->w1u); a.w2u = static_cast<const uint16_t*>(L->w2u);
    a.x = static_cast<const uint16_t*>(x); a.y = y;
    a.topk_idx = topk_idx; a.topk_val = topk_val;
    a.cand_out = cand_idx; a.n_cand = n_cand; a.scorer_acc = scorer_acc;
    a.fast_region = s.fast_region;
    a.keys = static_cast<float*>(s.keys); a.key_stride = s.key_stride; a.h = s.h; a.h32 = s.h32;
    a.bitmap = s.bitmap; a.cand_scratch = s.cand; a.xq = s.xq;
    a.stage_events = g_stage_events;
    a.scorer_clocks = g_scorer_clocks;
    HIRE_TRY(launch_ffn_fast(a, st));
    return HIRE_OK;
  }

  // steps 1-3.  Batches: filter and refine (kFilterMinBatch).  The exact stage runs on the bf16 matrix cores and stores fp32 values
  // within a proven distance of the activations; the selection recomputes in fp64 those around every token's k-th
  // largest.  Whatever lies outside that band is on the same side of the threshold in fp64 as its stored value, so
  // the selected sets are those of the fp64 activations.
  const bool filter = ffn_filter(s, B) && !g_force_exact_stage;
  rc = run_front(s, scorer_of(L), L->w1u, x, B, d, N, kprime, 1, cand_idx, n_cand, scorer_acc, st, 0, filter);
  if (rc != HIRE_OK) return rc;
  HIRE_STAGE(5, st);

  // step 4: exact top-k over U for every token
  if (filter) {
    RefineParams rp{};
    rp.vals = s.hf;
    rp.stride = s.hf_stride;
    rp.B = B; rp.N = N; rp.k = k; rp.d = d;
    rp.W = static_cast<const uint16_t*>(L->w1u);
    rp.x = static_cast<const uint16_t*>(x);
    rp.xnorm = s.xnorm;
    rp.wnorm_tiles = s.wnorm_tiles;
    rp.wnorm_n = filter_tiles(N);
    rp.err_c = gather_filter_error(B);
    rp.bitmap = s.bitmap;
    rp.all_rows = s.all_rows ? 1 : 0;
    if (cand_idx != nullptr || n_cand != nullptr) {
      rp.cand_out = cand_idx != nullptr ? cand_idx : s.cand;
      rp.cand_cap = s.cap_u;
      rp.n_cand_out = n_cand;
    }
    rp.h64 = s.h_refine;
    rp.h_stride = s.cap_u;
    rp.idx_out = topk_idx;
    rp.val_out = topk_val;
    rp.list_out = s.list;
    // Which values are handed out.  From 16 tokens on, with unions of 1025 to 16384 units (an even number), the filter
    // stage's fp32 sums, up to 2.3 half ulps off, have been the result since that stage exists, and forming all B k of
    // them once more would cost most there (64 tokens at the ~1B shape: 215 MB of rows).  Everywhere else callers have
    // had activations formed in fp64 and rounded once: 8 tokens at the ~1B shape 57.7 us per step, against 51.6 with the
    // filter's values and 65.5 with the fp64 stage; 33 tokens of d = 800, 5003 units 47.0, 41.7 and 54.5.
    rp.exact_values = !(B >= kFilterValuesMinBatch && s.cap_u > 1024 && s.cap_u <= 16384 && s.cap_u % 2 == 0);
    rp.window_misses = s.window_misses;
    if (refine_w2_supported(rp)) {
      HIRE_TRY(launch_refine_w2(rp, static_cast<const uint16_t*>(L->w2u), y, st));
      HIRE_STAGE(6, st);
      HIRE_STAGE(7, st);
      return HIRE_OK;
    }
    HIRE_TRY(launch_refine(rp, st));
  } else {
    SelectParams sp{};
    sp.vals = s.h;
    sp.stride = s.cap_u;
    sp.n_dev = s.counters;
    sp.n_cap = s.cap_u;
    sp.k = k;
    sp.idx_out = topk_idx;
    sp.val_out = topk_val;
    sp.list_out = s.list;
    sp.map = cand_idx ? cand_idx : s.cand;
    sp.nonneg = 1;  // activations after the ReLU
    sp.window_misses = s.window_misses;
    HIRE_TRY(launch_select_f64(sp, B, st));
  }
  HIRE_STAGE(6, st);

  // step 5: second layer over each token's selected rows
  HIRE_TRY(launch_w2_list(static_cast<const uint16_t*>(L->w2u), d, B, k, s.list, nullptr, 0, nullptr, y, st));
  HIRE_STAGE(7, st);
  return HIRE_OK;
}

// Address of the calling thread's current device's copy of `scratch`, looked up once per device.
static int static_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::atomic<void*> ptr_of_device[kMaxDevices];
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    g_last_hip_error = e != hipSuccess ? e : hipErrorInvalidDevice;
    return HIRE_ELAUNCH;
  }
  void* p = ptr_of_device[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr) {
      g_last_hip_error = e != hipSuccess ? e : hipErrorInvalidSymbol;
      return HIRE_ELAUNCH;
    }
    ptr_of_device[dev].store(p, std::memory_order_release);  // threads that race here store the same address
  }
  *out = p;
  return HIRE_OK;
}

int hire_ffn_step_static(const hire_ffn_layer* L, const void* x, int B, int k, int kprime, float* y, int32_t* topk_idx,
                         float* topk_val, int32_t* cand_idx, int32_t* n_cand, int32_t* scorer_acc, void* stream) {
  const size_t need = hire_ffn_workspace_bytes(L, B, k, kprime);
  if (need == 0) return HIRE_EINVAL;
  if (need > (size_t)HIRE_STATIC_SCRATCH_BYTES) return HIRE_ENOSPC;
  void* ws = nullptr;
  if (const int rc = static_scratch(&ws); rc != HIRE_OK) return rc;
  return hire_ffn_step(L, x, B, k, kprime, y, topk_idx, topk_val, cand_idx, n_cand, scorer_acc, ws,
                       (size_t)HIRE_STATIC_SCRATCH_BYTES, stream);
}

static int group_shift(int group) {
  for (int gs = 0; gs <= 4; ++gs)
    if (group == 1 << gs) return gs;
  return -1;
}

static int check_group(const hire_ffn_layer* L, int B, int k, int kprime, int group) {
  const int gs = group_shift(group);
  if (!L || gs < 0 || L->d_ff < 1 || L->d_ff % group || k % group || kprime % group) return -1;
  if ((L->d_ff >> gs) > kSingleWgMaxRow) return -1;
  if (L->d_model < 32 || B < 1 || B > HIRE_MAX_BATCH || k < 1 || k > kprime || kprime > L->d_ff) return -1;
  return gs;
}

size_t hire_ffn_group_workspace_bytes(const hire_ffn_layer* L, int B, int k, int kprime, int group) {
  const int gs = check_group(L, B, k, kprime, group);
  if (gs < 0) return 0;
  return carve(nullptr, L->scorer_kind, B, L->d_model, L->d_ff, L->r, k, kprime, true, gs).bytes;
}

// Dense common-path units riding along with a group-sparse step (eq. (7)): the step's own launches add them to y.
struct DenseRefs {
  const uint16_t* w1u;
  const uint16_t* w2u;
  int m1;
  double* h;           // [B, m1] workspace
};

static int ffn_group_step_impl(const hire_ffn_layer* L, const void* x, int B, int k, int kprime, int group, float* y,
                               int32_t* topk_group, float* topk_val, int32_t* cand_group, int32_t* n_cand,
                               int32_t* scorer_acc, void* workspace, size_t workspace_bytes, void* stream,
                               DenseRefs* dense) {
  if (!L || !y || !workspace) return HIRE_EINVAL;
  const int d = L->d_model, N = L->d_ff;
  int rc = check_common(d, N, B, k, kprime, L->scorer_kind, L->q4, L->q4_scale, L->lr_a, L->lr_b, L->r, L->lr_a_scale,
                        L->lr_b_scale, L->w1u, x);
  if (rc != HIRE_OK) return rc;
  if (!L->w2u || !aligned(L->w2u, 256) || !aligned(workspace, 256) || !aligned(y, 16)) return HIRE_EINVAL;
  if (scorer_acc && L->scorer_kind != HIRE_SCORER_INT4) return HIRE_EINVAL;
  const int gs = group_shift(group);
  if (gs < 0 || N % group || k % group || kprime % group) return HIRE_EINVAL;
  if ((N >> gs) > kSingleWgMaxRow) return HIRE_EUNSUPPORTED;
  if (gs == 0 && dense == nullptr)  // groups of one: the plain step, which has the same workspace layout
    return hire_ffn_step(L, x, B, k, kprime, y, topk_group, topk_val, cand_group, n_cand, scorer_acc, workspace,
                         workspace_bytes, stream);
  const StepBuffers s = carve(workspace, L->scorer_kind, B, d, N, L->r, k, kprime, true, gs);
  if (workspace_bytes < s.bytes) return HIRE_ENOSPC;
  hipStream_t st = static_cast<hipStream_t>(stream);

  // few tokens, groups of eight: the three-kernel route on group activations (the low-rank scorers' kernels take up to four).
  // Five to eight tokens without dense units on up to 8192 units are faster in the longer sequence from d = 288 on, us per step for
  // five and eight, three kernels / longer sequence: d = 288, 1504 units 26.2 / 23.9, 27.9 / 24.4, 8192 units 27.3 / 27.3, 30.0 / 28.3;
  // d = 480, 2000 units 27.1 / 24.0, 28.2 / 24.6, 8192 units 26.9 / 27.8, 30.5 / 28.5; d = 512, 6000 units 28.5 / 26.9, 30.4 / 28.5;
  // d = 1024, 6000 units 31.9 / 29.2, 36.9 / 32.1; d = 3200, 4000 units 57.0 / 39.3, 61.5 / 40.6.  Up to d = 256
  // neither is the faster one throughout: d = 256, 1504 units 24.8 / 24.3, 28.0 / 24.8, 6000 units 26.3 / 26.0, 28.8 / 27.9, 8192 units
  // 26.2 / 27.9, 29.4 / 28.6; d = 64, 8192 units 25.9 / 26.9, 28.7 / 27.4.  More units, or 1600 dense ones: d = 256, 14000 units
  // 29.9 / 33.0, 33.5 / 33.8; d = 2048, 16384 units 48.5 / 51.5, 59.3 / 59.0, 8000 and dense ones 46.7 / 52.5, 56.7 / 53.7.
  const bool fast_int4 = L->scorer_kind == HIRE_SCORER_INT4 && (B <= 4 || N > 8192 || d <= 256 || (dense != nullptr && dense->m1 > 0));
  const bool fast_lr = L->scorer_kind == HIRE_SCORER_LOWRANK && L->row_norm_bounds != nullptr && B <= 4;
  const bool fast_lrq = L->scorer_kind == HIRE_SCORER_LRQ && L->row_norm_bounds != nullptr && B <= 4 &&
                        scorer_int4_fused_supported(d);
  if ((fast_int4 || fast_lr || fast_lrq) && gs == 3 && ffn_fast_group8_supported(B, N, d, k, kprime) && !g_force_generic) {
    FfnFastArgs a{};
    a.B = B; a.N = N; a.d = d; a.k = k; a.kprime = kprime;
    a.q4 = L->q4; a.q4_scale = L->q4_scale;
    a.w1u = static_cast<const uint16_t*>(L->w1u); a.w2u = static_cast<const uint16_t*>(L->w2u);
    a.x = static_cast<const uint16_t*>(x); a.y = y;
    a.topk_idx = topk_group; a.topk_val = topk_val;
    a.cand_out = cand_group; a.n_cand = n_cand; a.scorer_acc = scorer_acc;
    a.fast_region = s.fast_region;
    a.keys = static_cast<float*>(s.keys); a.key_stride = s.key_stride; a.h = s.h; a.h32 = s.h32;
    a.bitmap = s.bitmap; a.cand_scratch = s.cand;
    a.gs = 3; a.gkeys = static_cast<float*>(s.gkeys); a.gkey_stride = s.gkey_stride; a.u32 = s.u32;
    a.lowrank = fast_lr;
    a.lrq = fast_lrq;
    if (fast_lr || fast_lrq) {
      a.lr_a = L->lr_a; a.lr_b = L->lr_b; a.r = L->r; a.norm_bounds = L->row_norm_bounds;
      a.t = s.t; a.keys64 = static_cast<double*>(s.keys); a.gkeys64 = static_cast<double*>(s.gkeys);
      a.lr_a_scale = L->lr_a_scale; a.lr_b_scale = L->lr_b_scale; a.keys_t = s.keys_t;
      a.xq = s.xq;
    }
    if (dense != nullptr && dense->m1 > 0) {
      a.dense_w1u = dense->w1u; a.dense_w2u = dense->w2u; a.m1 = dense->m1; a.h_dense = dense->h;
    }
    a.stage_events = g_stage_events;
    a.scorer_clocks = g_scorer_clocks;
    HIRE_TRY(launch_ffn_fast(a, st));
    return HIRE_OK;
  }

  // scorer, group sums of its keys, top k'/g groups per token, union, exact activations of the union's units
  rc = run_front(s, scorer_of(L), L->w1u, x, B, d, N, kprime, 1, cand_group, n_cand, scorer_acc, st, gs);
  if (rc != HIRE_OK) return rc;
  const int32_t* cand = cand_group ? cand_group : s.cand;
  HIRE_STAGE(5, st);

  // exact group activations and the top k/g groups of every token
  // (groups of eight: summed by the selection as it loads h; other sizes by a kernel of their own)
  if (gs == 3 && s.cap_u <= kGroupSelectMax) {
    const GroupSelect gsel{s.h, true, (long long)s.cap_u << gs, s.cap_u, s.counters, k >> gs, nullptr, cand, topk_group, s.list,
                           topk_val, s.window_misses};
    HIRE_TRY(launch_group_select(gsel, B, st));
  } else {
    const double* ranked = s.h;
    if (gs > 0) {
      HIRE_TRY(launch_group_sums_f64(s.h, B, (long long)s.cap_u << gs, 0, s.counters, s.cap_u, gs, s.hg, s.cap_u, st));
      ranked = s.hg;
    }
    SelectParams sp{};
    sp.vals = ranked;
    sp.stride = s.cap_u;
    sp.n_dev = s.counters;
    sp.n_cap = s.cap_u;
    sp.k = k >> gs;
    sp.idx_out = topk_group;
    sp.map = cand;
    sp.list_out = s.list;
    if (gs > 0) {
      sp.pos_out = s.pos;
      sp.gs = gs;
      sp.unit_h = s.h;
      sp.unit_h_stride = (long long)s.cap_u << gs;
      sp.unit_val_out = topk_val;
    } else {
      sp.val_out = topk_val;
    }
    sp.nonneg = 1;  // activations after the ReLU, or sums of their absolute values
    sp.window_misses = s.window_misses;
    HIRE_TRY(launch_select_f64(sp, B, st));
  }
  HIRE_STAGE(6, st);

  // second layer over the units of each token's groups, and over the dense units
  if (dense != nullptr) {
    const uint16_t* xb = static_cast<const uint16_t*>(x);
    const HistRefs none{};
    if (B >= kMfmaMinBatch)
      HIRE_TRY(launch_gather_dot_mfma(dense->w1u, xb, B, d, nullptr, dense->m1, nullptr, dense->m1, 1, dense->h, dense->m1,
                                      none, nullptr, 0, st));
    else
      HIRE_TRY(launch_gather_dot(dense->w1u, xb, d, nullptr, dense->m1, nullptr, dense->m1, 1, dense->h, none, nullptr, 0,
                                 st));
    HIRE_TRY(launch_w2_list(static_cast<const uint16_t*>(L->w2u), d, B, k, s.list, dense->w2u, dense->m1, dense->h, y,
                            st));
  } else {
    HIRE_TRY(launch_w2_list(static_cast<const uint16_t*>(L->w2u), d, B, k, s.list, nullptr, 0, nullptr, y, st));
  }
  HIRE_STAGE(7, st);
  return HIRE_OK;
}

int hire_ffn_group_step(const hire_ffn_layer* L, const void* x, int B, int k, int kprime, int group, float* y,
                        int32_t* topk_group, float* topk_val, int32_t* cand_group, int32_t* n_cand,
                        int32_t* scorer_acc, void* workspace, size_t workspace_bytes, void* stream) {
  return ffn_group_step_impl(L, x, B, k, kprime, group, y, topk_group, topk_val, cand_group, n_cand, scorer_acc,
                             workspace, workspace_bytes, stream, nullptr);
}

// CommonPath: the group-sparse step's workspace, then the dense units' activations and partial rows.
struct CommonBuffers {
  size_t sparse_bytes;
  double* h;       // [B, m1]
  size_t bytes;
};
static CommonBuffers carve_common(void* ws, const hire_ffn_layer* L, int m1, int B, int k, int kprime, int gs) {
  CommonBuffers c{};
  c.sparse_bytes = align_up(carve(nullptr, L->scorer_kind, B, L->d_model, L->d_ff, L->r, k, kprime, true, gs).bytes);
  Carver cv(ws);
  cv.take<char>(c.sparse_bytes);
  c.h = cv.take<double>((size_t)B * m1 + 2);
  c.bytes = cv.off;
  return c;
}

size_t hire_ffn_commonpath_workspace_bytes(const hire_ffn_layer* L, int m1, int B, int k, int kprime, int group) {
  const int gs = check_group(L, B, k, kprime, group);
  if (gs < 0 || m1 < 0) return 0;
  return carve_common(nullptr, L, m1, B, k, kprime, gs).bytes;
}

int hire_ffn_commonpath_step(const hire_ffn_layer* L, const void* dense_w1u, const void* dense_w2u, int m1,
                             const void* x, int B, int k, int kprime, int group, float* y, int32_t* topk_group,
                             float* topk_val, int32_t* cand_group, int32_t* n_cand, int32_t* scorer_acc,
                             void* workspace, size_t workspace_bytes, void* stream) {
  if (!L || m1 < 0) return HIRE_EINVAL;
  if (m1 > 0 && (!dense_w1u || !dense_w2u || !aligned(dense_w1u, 256) || !aligned(dense_w2u, 256))) return HIRE_EINVAL;
  const int gs = group_shift(group);
  if (gs < 0) return HIRE_EINVAL;
  const size_t need = hire_ffn_commonpath_workspace_bytes(L, m1, B, k, kprime, group);
  if (need != 0 && workspace_bytes < need) return HIRE_ENOSPC;
  CommonBuffers c{};
  DenseRefs dense{};
  if (need != 0 && m1 > 0) {
    c = carve_common(workspace, L, m1, B, k, kprime, gs);
    dense = DenseRefs{static_cast<const uint16_t*>(dense_w1u), static_cast<const uint16_t*>(dense_w2u), m1, c.h};
  }
  return ffn_group_step_impl(L, x, B, k, kprime, group, y, topk_group, topk_val, cand_group, n_cand, scorer_acc,
                             workspace, workspace_bytes, stream, (need != 0 && m1 > 0) ? &dense : nullptr);
}

// The partial rows sit behind the head, so that a workspace shared with the other entry points keeps their state intact.
static size_t shard_partial_offset() { return body_offset(kFastTokens); }

static bool shard_args_ok(const hire_ffn_layer* L, int B, int k, int kprime, int shards) {
  if (!L || L->d_model < 32 || L->d_ff < 1 || B < 1 || B > HIRE_MAX_BATCH || k < 1 || k > kprime || kprime > L->d_ff)
    return false;
  return shards >= 1 && L->d_ff % shards == 0;
}

// Batches and long shards (ffn_shard_batch); behind the head as well.
static size_t carve_shard_batch(void* ws, int B, int d, int N, int k, int shards, FfnShardBuffers* out) {
  Carver c(ws);
  c.take<char>(shard_partial_offset());
  FfnShardBuffers f{};
  f.xq = c.take<int8_t>((size_t)B * d);
  f.stride = (N + 3) / 4 * 4;
  f.vals = c.take<float>((size_t)B * f.stride + 4);
  f.zero_words = (N + 63) / 64 * 2 + 2;
  f.bitmap = c.take<uint32_t>(f.zero_words);
  f.xnorm = c.take<float>(HIRE_MAX_BATCH);
  f.wnorm_tiles = c.take<float>(filter_tiles(N));
  f.list = c.take<uint2>((size_t)B * shards * ((k + shards - 1) / shards));
  if (out) *out = f;
  return c.off;
}

size_t hire_ffn_shard_workspace_bytes(const hire_ffn_layer* L, int B, int k, int kprime, int shards) {
  if (!shard_args_ok(L, B, k, kprime, shards) || !ffn_shard_supported(L->d_ff, L->d_model, shards)) return 0;
  if (ffn_shard_batch(B, L->d_ff, L->d_model, shards))
    return carve_shard_batch(nullptr, B, L->d_model, L->d_ff, k, shards, nullptr);
  return shard_partial_offset() + align_up(ffn_shard_partial_floats(B, L->d_model, shards) * sizeof(float));
}

int hire_ffn_shard_step(const hire_ffn_layer* L, const void* x, int B, int k, int kprime, int shards, float* y,
                        int32_t* topk_idx, float* topk_val, int32_t* cand_idx, int32_t* n_cand, int32_t* scorer_acc,
                        void* workspace, size_t workspace_bytes, void* stream) {
  if (!L || !y || !workspace) return HIRE_EINVAL;
  const int d = L->d_model, N = L->d_ff;
  if (L->scorer_kind != HIRE_SCORER_INT4) return HIRE_EUNSUPPORTED;
  int rc = check_common(d, N, B, k, kprime, L->scorer_kind, L->q4, L->q4_scale, L->lr_a, L->lr_b, L->r, L->lr_a_scale,
                        L->lr_b_scale, L->w1u, x);
  if (rc != HIRE_OK) return rc;
  if (!L->w2u || !aligned(L->w2u, 256) || !aligned(workspace, 256) || !aligned(y, 16)) return HIRE_EINVAL;
  if (!shard_args_ok(L, B, k, kprime, shards)) return HIRE_EINVAL;
  if (!ffn_shard_supported(N, d, shards)) return HIRE_EUNSUPPORTED;
  if (workspace_bytes < hire_ffn_shard_workspace_bytes(L, B, k, kprime, shards)) return HIRE_ENOSPC;
  FfnShardArgs a{};
  a.N = N; a.d = d; a.B = B; a.k = k; a.kprime = kprime; a.shards = shards;
  a.q4 = L->q4; a.q4_scale = L->q4_scale;
  a.w1u = static_cast<const uint16_t*>(L->w1u); a.w2u = static_cast<const uint16_t*>(L->w2u);
  a.x = static_cast<const uint16_t*>(x); a.y = y;
  a.topk_idx = topk_idx; a.topk_val = topk_val; a.cand = cand_idx; a.n_cand = n_cand; a.scorer_acc = scorer_acc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (ffn_shard_batch(B, N, d, shards)) {
    FfnShardBuffers f{};
    carve_shard_batch(workspace, B, d, N, k, shards, &f);
    HIRE_STAGE(0, st);
    HIRE_TRY(launch_ffn_shard_batch(a, f, st));
    HIRE_STAGE(1, st);
    HIRE_STAGE(2, st);
    return HIRE_OK;
  }
  a.partial = reinterpret_cast<float*>(static_cast<char*>(workspace) + shard_partial_offset());
  HIRE_STAGE(0, st);
  HIRE_TRY(launch_ffn_shard(a, st));
  HIRE_STAGE(1, st);
  HIRE_TRY(launch_ffn_shard_reduce(a, st));
  HIRE_STAGE(2, st);
  return HIRE_OK;
}

int hire_softmax_step(const hire_softmax_layer* L, const void* x, int B, int k, int kprime, int32_t* top_idx,
                      float* top_prob, float* top_logit, int32_t* cand_idx, int32_t* n_cand, int32_t* scorer_acc,
                      void* workspace, size_t workspace_bytes, void* stream) {
  if (!L || !top_idx || !top_prob || !workspace) return HIRE_EINVAL;
  const int d = L->d_model, N = L->vocab;
  int rc = check_common(d, N, B, k, kprime, L->scorer_kind, L->q4, L->q4_scale, L->lr_a, L->lr_b, L->r, L->lr_a_scale,
                        L->lr_b_scale, L->w, x);
  if (rc != HIRE_OK) return rc;
  if (k > HIRE_MAX_RANK_ORDER_K) return HIRE_EUNSUPPORTED;
  if (!aligned(workspace, 256)) return HIRE_EINVAL;
  if (scorer_acc && L->scorer_kind != HIRE_SCORER_INT4) return HIRE_EINVAL;
  const StepBuffers s = carve(workspace, L->scorer_kind, B, d, N, L->r, k, kprime, false);
  if (workspace_bytes < s.bytes) return HIRE_ENOSPC;
  hipStream_t st = static_cast<hipStream_t>(stream);

  // Batches: filter and refine as in the FFN step - fp32 logits with a proven error from the bf16 matrix cores,
  // fp64 only for the entries that can still be among the k largest.
  const bool filter = s.hf != nullptr && d % 8 == 0 && !g_force_exact_stage;
  // One token on a long vocabulary: the scorer (both int4 kinds), the exact logits of a superset of the shortlist
  // (from the scorer's maxima), and the final selections with the softmax.
  const bool lrq = L->scorer_kind == HIRE_SCORER_LRQ;
  const int sd = lrq ? L->r : d;  // codes per row of the matrix that produces the keys
  if (s.sm1_ok && scorer_int4_fused_supported(sd) && (!lrq || scorer_int4_fused_supported(d)) &&
      softmax_b1_supported(N, d, k, kprime) && softmax_b1_worthwhile(N, kprime, scorer_int4_fused_maxima(N, sd)) &&
      !g_force_generic) {
    int n_max = 0;
    rc = run_front(s, scorer_of(L), L->w, x, B, d, N, kprime, 0, cand_idx, n_cand, scorer_acc, st, 0, false, &n_max);
    if (rc != HIRE_OK) return rc;
    HIRE_STAGE(3, st);
    HIRE_STAGE(4, st);
    HIRE_TRY(launch_softmax_b1(static_cast<const float*>(s.keys), N, d, sd, k, kprime, n_max, lrq ? L->lr_b : L->q4,
                               static_cast<const uint16_t*>(L->w), static_cast<const uint16_t*>(x), s.hist,
                               s.sm1_slots, top_idx, top_prob, top_logit, cand_idx, n_cand, st));
    HIRE_STAGE(5, st);
    HIRE_STAGE(6, st);
    return HIRE_OK;
  }
  rc = run_front(s, scorer_of(L), L->w, x, B, d, N, kprime, 0, cand_idx, n_cand, scorer_acc, st, 0, filter);
  if (rc != HIRE_OK) return rc;
  HIRE_STAGE(5, st);

  SelectParams sp{};
  sp.vals = s.h;
  sp.stride = s.cap_u;
  sp.n_dev = s.counters;
  sp.n_cap = s.cap_u;
  sp.k = k;
  sp.rank_order = 1;
  sp.idx_out = top_idx;
  sp.val_out = top_logit;
  sp.prob_out = top_prob;
  sp.map = cand_idx ? cand_idx : s.cand;
  sp.window_misses = s.window_misses;
  if (filter) {
    sp.vals = s.hf;
    sp.stride = s.hf_stride;
    sp.refine_w = static_cast<const uint16_t*>(L->w);
    sp.refine_x = static_cast<const uint16_t*>(x);
    sp.refine_d = d;
    sp.xnorm = s.xnorm;
    sp.wnorm_tiles = s.wnorm_tiles;
    sp.wnorm_n = filter_rank_blocks(s.cap_u);
    sp.maxima = s.maxima;
    sp.refine_slots = s.refine_slots;
    sp.refine_keys = reinterpret_cast<unsigned long long*>(s.h);  // (no fp64 logits are formed otherwise)
    sp.refine_keys_stride = s.cap_u;
    sp.n_maxima = 4 * filter_rank_blocks(s.cap_u);
    sp.err_c = gather_filter_error(B);
    HIRE_TRY(launch_softmax_refine(sp, B, st));
  } else {
    HIRE_TRY(launch_select_f64(sp, B, st));
  }
  HIRE_STAGE(6, st);
  return HIRE_OK;
}

int topk_select(const float* scores, int B, int N, int k, int flags, int32_t* idx_out, float* val_out, void* workspace,
                size_t workspace_bytes, void* stream) {
  if (!scores || !idx_out || B < 1 || N < 1 || k < 1 || k > N) return HIRE_EINVAL;
  if ((flags & HIRE_ORDER_RANK) && k > HIRE_MAX_RANK_ORDER_K) return HIRE_EUNSUPPORTED;
  if (topk_long_route(N, flags)) {
    if (!workspace || !aligned(workspace, 256)) return HIRE_EINVAL;
    if (workspace_bytes < hire_topk_workspace_bytes(B, N, k, flags)) return HIRE_ENOSPC;
    char* base = static_cast<char*>(workspace);
    char* body = base + body_offset(kFastTokens);
    const bool rank = (flags & HIRE_ORDER_RANK) != 0;
    int32_t* idx_tmp = reinterpret_cast<int32_t*>(body + align_up(topk_long_workspace_bytes(B, N)));
    float* val_tmp = reinterpret_cast<float*>(reinterpret_cast<char*>(idx_tmp) +
                                              align_up((size_t)B * k * sizeof(int32_t)));
    hipStream_t st = static_cast<hipStream_t>(stream);
    const unsigned long long sig = layout_signature(2 /* neither scorer: a bare selection */, B, 0, N, 0, k, 0, flags);
    if (topk_rows_supported(N, k)) {
      HIRE_TRY(launch_topk_rows(scores, B, N, k, (flags & HIRE_RELU) ? 1 : 0, rank ? 1 : 0, idx_out, val_out, base, body,
                                sig, st));
      return HIRE_OK;
    }
    HIRE_TRY(launch_topk_long(scores, B, N, k, (flags & HIRE_RELU) ? 1 : 0, rank ? idx_tmp : idx_out,
                              rank ? val_tmp : val_out, base, body, sig, st));
    if (rank) {  // all k entries of the index-ordered list, in rank order
      SelectParams sp{};
      sp.vals = val_tmp;  // max(., 0) already applied where asked for
      sp.stride = k;
      sp.n = k;
      sp.n_cap = k;
      sp.k = k;
      sp.rank_order = 1;
      sp.idx_out = idx_out;
      sp.val_out = val_out;
      sp.map = idx_tmp;
      sp.map_stride = k;
      HIRE_TRY(launch_select_f32(sp, B, st));
    }
    return HIRE_OK;
  }
  SelectParams sp{};
  sp.vals = scores;
  sp.stride = N;
  sp.n = N;
  sp.n_cap = N;
  sp.k = k;
  sp.relu = (flags & HIRE_RELU) ? 1 : 0;
  sp.rank_order = (flags & HIRE_ORDER_RANK) ? 1 : 0;
  sp.idx_out = idx_out;
  sp.val_out = val_out;
  HIRE_TRY(launch_select_f32(sp, B, static_cast<hipStream_t>(stream)));
  return HIRE_OK;
}

}  // extern "C"
