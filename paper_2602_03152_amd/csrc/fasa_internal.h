// Internal declarations shared by the translation units of libfasa (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cstddef>
#include <cstdint>
#include <tuple>
#include <utility>

#include "fasa.h"

namespace fasa {

// ---------------------------------------------------------------------------------------------
// constants of the selection stage
// ---------------------------------------------------------------------------------------------
constexpr int kHistBits = 12;              // coarse bins = top 12 bits of the order-preserving key
constexpr int kHistBins = 1 << kHistBits;  // (sign, 8 exponent bits, 3 mantissa bits)
constexpr int kKeyLowBits = 32 - kHistBits;
constexpr int kHeadDim = 128;
constexpr int kMaxGroup = 8;
// Compute units the launch plans are sized for (MI355X).  A compile-time number because
// fasa_workspace_bytes() has to be a pure host function; a GPU test checks it against the device.
constexpr int kAssumedCUs = 256;

// From how many bytes on that a call reads its large inputs are read non-temporal.  A third of the last-level cache: calls of
// this size over three caches in turn (layers, say) leave nothing there for the next round, and lines that are not kept there come faster:
// 128 MiB, never the same in 2 GB, 16-byte loads, eight workgroups of 256 on a compute unit: 21.5 -> 20.0 us (6.2 -> 6.7 TB/s).  Below that what one call has
// left there may serve the next: the same with 64 MiB, 30 buffers: 11.15 -> 10.65 us, but three buffers: 9.9 where memory takes 10.65.
// The line suits three buffers in turn.  A walk over more (a model's layers) leaves the caches nothing whatever one call reads, and loses by the line what stands below it.  us,
// kept / non-temporal, 3 | 8 | 24 sets of buffers: step of 8 rows of 32768, B = 2048 (28 MB) 16.65 / 17.3 | 16.5 / 17.1 | 17.65 / 17.05; of 65536 (46 MB) 18.95 / 19.6 | 20.0 / 19.65 |
// 20.35 / 19.5; 32 rows of 16384, 256 (40 MB) 16.4 / 16.5 | 17.7 / 16.85 | 18.25 / 17.15; 64 rows (80 MB) 21.55 / 22.35 | 24.5 / 22.45 | 24.55 / 23.65; full KV of 8 rows of 8192 (34 MB)
// 9.8 / 10.0 | 10.05 / 10.4 | 10.7 / 10.5, of 16384 (67 MB) 14.0 / 14.85 | 16.1 / 15.05 | 16.2 / 15.25.  Above it: 128 rows of 16384 (160 MB) 37.4 / 34.15 | 37.3 / 34.55 | 37.4 / 36.45; full KV of 8 rows of
// 32768 (134 MB) 26.5 / 23.35 | 26.5 / 24.8 | 26.6 / 24.9.
constexpr long long kStreamBytes = 90ll << 20;

// Per-(b,h) row counters, one 128-byte line per row so that rows served by different XCDs never
// share a line.  All zero between calls: the workgroup that finishes a row resets what it used.
struct RowCtl {
  uint32_t n_sel;     // winners written so far (tokens in bins above the threshold bin)
  uint32_t n_cand;    // candidates collected from the threshold bin
  uint32_t done_sel;  // selection workgroups of this row that finished their slice
  uint32_t done_att;  // attention workgroups of this row that wrote their partial
  float bin_mu;       // adaptive histogram of the fused step: written by the scoring kernel of a call,
  float bin_inv;      // read by its selection kernel (never has to be zero)
  uint32_t list_cut;  // lists of a row (row_list.h): the key from which on the selection looked at its scores, and how it
  uint32_t list_how;  // went about it (ListSet); written only
  uint32_t pad[24];
};
static_assert(sizeof(RowCtl) == 128, "one line per row");

// Optional per-sequence lengths (DEVICE arrays of `batch` entries, or null = the uniform values of
// the shape).  With them the shape's n_ctx and budget are upper bounds that size the grids, and
// T's row pitch is min(budget, n_ctx) of the shape.
struct RaggedLens {
  const int32_t* n_ctx;
  const int32_t* budget;
};

// Paged K/V cache as the kernels see it.  table == nullptr: contiguous cache, row (b, n) at
// b * kv_stride_b + n * kv_stride_n.  Otherwise row (b, n) lives in pool block
// table[b * max_blocks + (n >> shift)] at offset (n & (page - 1)); kv_stride_b is then the stride
// between pool blocks.  Table entries are clamped into [0, n_pool): a stray entry can never become
// a stray address.
struct PageMap {
  const int32_t* table;
  int max_blocks;
  int shift;     // log2(tokens per block)
  int n_pool;    // blocks in the pool
};
constexpr PageMap kNoPaging = {nullptr, 0, 0, 0};

// pool slot (block * page + offset) of logical token n of sequence b
__device__ __forceinline__ int kv_slot(const PageMap& pm, int b, int n) {
  const int blk = min(max(pm.table[(size_t)b * pm.max_blocks + (n >> pm.shift)], 0), pm.n_pool - 1);
  return (blk << pm.shift) | (n & ((1 << pm.shift) - 1));
}
// element offset of K/V row (b, n), without the head term
__device__ __forceinline__ long long kv_row_offset(const PageMap& pm, int b, int n, long long sb,
                                                   long long sn) {
  if (pm.table == nullptr) return b * sb + (long long)n * sn;
  const int slot = kv_slot(pm, b, n);
  return (long long)(slot >> pm.shift) * sb + (long long)(slot & ((1 << pm.shift) - 1)) * sn;
}

// The two head dims that entry f of KV head h's dominant list names, as lo | hi << 8.  The list
// holds FC numbers (one word per entry) or, for FASA_PAIR_LIST, the dim pairs themselves (two
// words).  Values are clamped into the head: a stray entry can never become a stray LDS index.
__device__ __forceinline__ int list_word(int pairing, int F, int h, int f, int which) {
  return pairing == FASA_PAIR_LIST ? (h * F + f) * 2 + which : h * F + f;
}
__device__ __forceinline__ int pair_dims(int pairing, int a, int b) {
  constexpr int D = kHeadDim;
  const int i = min(max(a, 0), D / 2 - 1);
  int lo = pairing == FASA_PAIR_INTERLEAVED ? 2 * i : i;
  int hi = pairing == FASA_PAIR_INTERLEAVED ? 2 * i + 1 : i + D / 2;
  if (pairing == FASA_PAIR_LIST) {
    lo = min(max(a, 0), D - 1);
    hi = min(max(b, 0), D - 1);
  }
  return lo | (hi << 8);
}

// Workspace carve-up (all offsets 256-byte aligned).
struct WsLayout {
  size_t hist_off, ctl_off, cand_off, part_acc_off, part_ml_off, rec_off, tslot_off, total;
  int rows, max_splits;
};

struct AttendPlan {
  int count;          // tokens attended per row
  int tok_per_split;  // list entries per workgroup
  int n_splits;
};

AttendPlan plan_attend(int rows, int count, int group);   // sizes the workspace
AttendPlan plan_attend_wide(int rows, int count);         // attend_wide_kernel: no more splits than plan_attend()

// Fused selection + attention (fused.hip): tokens per workgroup and workgroups per row.
// tpb == 0: this shape takes the stand-alone kernels (everything selected, a row longer than the merge can take slices
// of, or float32 with few query heads and a large share selected).
// Candidates per row of the fused step that are handed over with a record (logits of the group's query
// heads + V row), and the bytes of workspace a row's records take (bf16).
constexpr int kFuseRich = 64;
constexpr size_t kFuseRecBytesPerRow = (size_t)kFuseRich * (kMaxGroup * 4 + kHeadDim * 2);

struct FusePlan {
  int tpb;         // kernel instance: most tokens a workgroup can hold (0: the fused step does not apply)
  int nslices;     // workgroups per row
  int slice_len;   // tokens per workgroup, <= tpb, a multiple of 16
};
// by_sequence: lengths and budgets come from device arrays (a budget may then reach its length)
FusePlan plan_fused(const fasa_shape& s, bool by_sequence);
WsLayout ws_layout(const fasa_shape& s);

// For fast_div: ceil(2^31 / d), or 0 where quotients of up to `most` would not be exact with it.  (n m / 2^31 exceeds n / d by less than
// n / 2^31, which may not reach 1 / d.)
constexpr uint32_t div_magic(int d, long long most) {
  return most * d < (1ll << 31) ? (uint32_t)(((1ll << 31) + d - 1) / d) : 0u;
}

// Bytes of K and V that a row's selected tokens take, over all rows, and those of a step: planes, scores, and the former
inline long long gather_bytes(const fasa_shape& s) {
  const long long bsel = s.budget < s.n_ctx ? s.budget : s.n_ctx, e = s.dtype == FASA_BF16 ? 2 : 4;
  return (long long)s.batch * s.n_kv_heads * bsel * 2 * s.head_dim * e;
}
inline long long step_bytes(const fasa_shape& s) {
  const long long e = s.dtype == FASA_BF16 ? 2 : 4;
  return (long long)s.batch * s.n_kv_heads * s.n_ctx * (2 * s.n_fc * e + 4) + gather_bytes(s);
}

// ---------------------------------------------------------------------------------------------
// launch helper: plain launch, or a launch bracketed by its own start/stop timestamps
// ---------------------------------------------------------------------------------------------
bool profile_on();
// Hands out a fresh event pair owned by the profiler and remembers it under `name`.
hipError_t profile_events(const char* name, hipEvent_t* start, hipEvent_t* stop);
void set_last_hip_error(hipError_t e);

template <typename... KArgs, typename... Args>
inline hipError_t launch_lds(const char* name, void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds,
                             hipStream_t stream, Args&&... args) {
  static_assert(sizeof...(KArgs) == sizeof...(Args), "kernel argument count");
  std::tuple<KArgs...> vals{static_cast<KArgs>(std::forward<Args>(args))...};
  void* ptrs[sizeof...(KArgs) ? sizeof...(KArgs) : 1];
  std::apply([&](auto&... v) { size_t i = 0; ((ptrs[i++] = (void*)&v), ...); }, vals);
  hipError_t e;
  if (profile_on()) {
    hipEvent_t a = nullptr, b = nullptr;
    e = profile_events(name, &a, &b);
    if (e == hipSuccess)
      e = hipExtLaunchKernel((const void*)kernel, grid, block, ptrs, lds, stream, a, b, 0);
  } else {
    e = hipLaunchKernel((const void*)kernel, grid, block, ptrs, lds, stream);
  }
  if (e != hipSuccess) set_last_hip_error(e);
  return e;
}
template <typename... KArgs, typename... Args>
inline hipError_t launch(const char* name, void (*kernel)(KArgs...), dim3 grid, dim3 block, hipStream_t stream, Args&&... args) {
  return launch_lds(name, kernel, grid, block, 0, stream, std::forward<Args>(args)...);
}

// ---------------------------------------------------------------------------------------------
// stage launchers (defined in pack.hip / score.hip / topk.hip / attend.hip); shapes are already
// validated when these are called
// ---------------------------------------------------------------------------------------------
hipError_t launch_pack(const fasa_shape& s, const void* K, const int32_t* fc_idx, void* Kp,
                       int n_begin, int n_end, hipStream_t st, PageMap pm = kNoPaging);
// A freshly decoded K/V row per (b, h) ([batch][n_kv_heads][head_dim]) that the scoring kernel
// appends at token n_ctx - 1 (K, V: the caches, with the shape's strides; Kp gets the dominant pairs).
// k_new == nullptr: nothing to append.  split: K is the host part of the memory-optimised variant
// ([row][n_cap][head_dim - 2 n_fc]) and receives the dims that are not dominant.
struct AppendArgs {
  const void* k_new;
  const void* v_new;
  void* K;
  void* V;
  PageMap pm;
  bool split;
};
constexpr AppendArgs kNoAppend = {nullptr, nullptr, nullptr, nullptr, {nullptr, 0, 0, 0}, false};
// Where the scoring kernel leaves the lists of a row's largest scores (row_list.h: ListRow): [row][n_cap] 8 bytes a token, and
// [row][kListLimPitch] segments; places: of a row; pitch: of a segment, where all rows have the same length and budget.
struct ListOut {
  uint2* list;
  uint2* lims;
  int places, pitch;
};
// hist == nullptr: scores only.  adaptive_ctl != nullptr (with hist): the adaptive histogram of the
// fused step (bins of lin_bin, location and scale left in the row counters) instead of the
// exponent-based one the stand-alone selection reads.
hipError_t launch_score(const fasa_shape& s, const void* q, const void* Kp, const int32_t* fc_idx,
                        float* S, uint32_t* hist, hipStream_t st, RaggedLens rl = {nullptr, nullptr},
                        AppendArgs ap = kNoAppend, RowCtl* adaptive_ctl = nullptr);
// scores and lists
hipError_t launch_score_list(const fasa_shape& s, const void* q, void* Kp, const int32_t* fc_idx, float* S,
                             const ListOut& lists, hipStream_t st, RaggedLens rl, const AppendArgs& ap);
// zeroes the histogram and the row counters (workspace initialisation)
hipError_t launch_ws_clear(const fasa_shape& s, uint32_t* hist, RowCtl* ctl, hipStream_t st);
// TopK-I of given scores in one launch (topk.hip): the set of every row to T.  quads == 0: not for this shape.
// list, lims: as ListOut; tickets [row * ticket_stride], zero.
struct TopkPlan {
  int quads;       // of places of a row's list that a selecting thread holds
};
TopkPlan plan_topk(int n_ctx, int bsel);
hipError_t launch_topk(const TopkPlan& p, int rows, int n_ctx, int n_cap, int bsel, const float* S, int32_t* T, uint2* list,
                       uint2* lims, uint32_t* tickets, int ticket_stride, hipStream_t st);
hipError_t launch_hist(const fasa_shape& s, const float* S, uint32_t* hist, hipStream_t st);
// Tslot (paged caches only, else null): receives the pool slot of every entry of T, same layout
hipError_t launch_select(const fasa_shape& s, const float* S, const uint32_t* hist, RowCtl* ctl,
                         uint2* cand, int32_t* T, hipStream_t st, RaggedLens rl = {nullptr, nullptr},
                         PageMap pm = kNoPaging, int32_t* Tslot = nullptr);
// paged caches: T holds pool slots (launch_select's Tslot), dense must be false
hipError_t launch_attend(const fasa_shape& s, bool dense, const void* q, const void* K,
                         const void* V, const int32_t* T, float* O, RowCtl* ctl, float* part_acc,
                         float* part_ml, hipStream_t st, RaggedLens rl = {nullptr, nullptr},
                         PageMap pm = kNoPaging);

// TopK-I + FAC in one kernel after a scoring pass with the adaptive histogram (launch_score with
// adaptive_ctl); p from plan_fused, p.tpb != 0.  The partial buffers are indexed with p.nslices splits
// per row.  Paged caches are gathered through the table inside the kernel.
hipError_t launch_select_attend(const fasa_shape& s, const FusePlan& p, const void* q, const void* K,
                                const void* V, const float* S, uint32_t* hist, RowCtl* ctl, uint2* cand,
                                int32_t* T, float* O, float* part_acc, float* part_ml, unsigned char* rec,
                                hipStream_t st, RaggedLens rl = {nullptr, nullptr}, PageMap pm = kNoPaging);

// The step with one workgroup selecting and attending per row (step.hip): the whole step in one launch, or (float32)
// after a scoring launch; plan_step: which of the two, if any, takes the shape.
enum StepForm { kStepNone, kStepOne, kStepRow };
constexpr int kStepMaxBudget = 1024;   // most selected tokens per row
StepForm plan_step(const fasa_shape& s, const PageMap& pm);
hipError_t launch_step(const fasa_shape& s, StepForm form, const void* q, void* K, void* V, void* Kp,
                       const int32_t* fc_idx, const void* k_new, const void* v_new, float* S, int32_t* T, float* O,
                       RowCtl* ctl, hipStream_t st, RaggedLens rl = {nullptr, nullptr}, PageMap pm = kNoPaging);

// Selection out of lists and attention by one or several workgroups per row, after a scoring launch that makes the
// lists (step.hip).  quads == 0: not for this shape.
struct ListPlan {
  int nwgs;        // workgroups per row
  int quads;       // of places of a row's list that each of a workgroup's threads holds
};
ListPlan plan_list(const fasa_shape& s, const PageMap& pm, int max_splits);
// Quads of places of a row's list that each of nt threads holds (1 - 4, 6 or 8 of them); 0: more than `most`, or than there are segments.
int list_quads(int n, int bsel, int nt, int most);
// Places of a row's list.  by_sequence: n and bsel bound the sequences' own.
int list_places(int n, int bsel, int quads, bool by_sequence);
hipError_t launch_list_step(const fasa_shape& s, const ListPlan& p, const void* q, void* K, void* V, void* Kp,
                            const int32_t* fc_idx, const void* k_new, const void* v_new, float* S, int32_t* T, float* O,
                            RowCtl* ctl, uint2* list, uint2* lims, float* part_acc, float* part_ml, hipStream_t st,
                            RaggedLens rl = {nullptr, nullptr}, PageMap pm = kNoPaging);

// memory-optimised variant (offload.hip)
hipError_t launch_offload_split(const fasa_shape& s, const void* K, const int32_t* fc_idx, void* Kp,
                                void* Knd, int n_begin, int n_end, hipStream_t st);
hipError_t launch_offload_gather(const fasa_shape& s, const void* Kp, const void* Knd, const void* Vh,
                                 const int32_t* fc_idx, const int32_t* T, void* KT, void* VT,
                                 hipStream_t st);

hipError_t launch_offload_attend(const fasa_shape& s, int max_splits, const void* q, const void* Kp, const void* Knd,
                                 const void* Vh, const int32_t* fc_idx, const int32_t* T, void* KT, void* VT, float* O,
                                 RowCtl* ctl, float* part_acc, float* part_ml, hipStream_t st);

// offline calibration (calib.hip)
// S: rows * n_cap floats, scratch: calib_scratch_bytes()
size_t calib_scratch_bytes(int rows, int n_cap);
hipError_t launch_calib(const fasa_shape& s, const void* q, const void* Kp_all, int kk, float* S, void* scratch, float* CA_sum,
                        hipStream_t st);
int calib_max_ctx();

}  // namespace fasa
