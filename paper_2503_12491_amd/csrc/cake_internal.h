// Internal declarations shared by the translation units of libcake.  Not installed.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstddef>
#include <cstdint>
#include <type_traits>

#include "cake.h"

namespace cake {

// ---- error reporting -----------------------------------------------------------------
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

#define CAKE_HIP_TRY(expr)                                                              \
  do {                                                                                  \
    hipError_t e__ = (expr);                                                            \
    if (e__ != hipSuccess)                                                              \
      return ::cake::fail(CAKE_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e__)); \
  } while (0)

#define CAKE_REQUIRE(cond, ...)                                       \
  do {                                                                \
    if (!(cond)) return ::cake::fail(CAKE_ERR_INVALID_ARG, __VA_ARGS__); \
  } while (0)

// ---- shape checks common to the entry points -------------------------------------------
int check_shape_basic(const cake_shape* s);   // batch/heads/head_dim/window/dtype/layers
int check_shape_scores(const cake_shape* s);  // + N > S_w and the kernels' supported set

inline size_t elem_bytes(int32_t dtype) { return dtype == CAKE_BF16 ? 2 : 4; }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---- workspace layout of the score pass -------------------------------------------------
// One "slice" is (layer, sequence, KV head).  Sums over a slice's keys are kept per granule of keys and
// then reduced in a fixed order; a workgroup of the two passes handles one or more whole granules.
struct ScoreLayout {
  int32_t chunk;        // alignment of key segments, a multiple of the granule
  int32_t granule;      // keys per partial sum, a power of two times the 64-key tile
  int32_t n_granules;   // granules over all N keys (pass 1)
  int32_t n_granules_p; // granules over the N_p prefix keys (pass 2)
  int64_t n_slices;     // L * B * H_kv
  int32_t rows;         // G * S_w window rows per slice
  size_t off_lse;       // f32 [n_slices][rows]            log2-domain row normaliser
  size_t off_part;      // f32 [n_slices][n_granules][rows][2]    pass-1 (reference, sum) per window row
  size_t off_hv;        // f32 [n_slices][n_granules_p][G][2]     pass-2 (entropy, variance) sums
  size_t off_raw;       // f32 [n_slices][N_p]             un-pooled indicator
  size_t total;
};
ScoreLayout score_layout(const cake_shape& s);

// cake_window_scores (or, with row_lse, cake_window_scores_lse) and cake_layer_preference with the
// preferences computed beside the pooling; rows of pref_ld preferences and hv_ld (H, V) pairs per sequence.
// `plan` (may be NULL): the plan that follows from them, made in the same launch or behind it.
// `one` (or NULL): the buffers of a call for one layer whose addresses the host knows, instead of the tables.
struct PlanArgs;
struct LayerPointers {
  const void *q, *k;
  const float* row_lse;          // NULL: the normalisers are computed
  float* indicator;
  uint32_t* flags;               // or NULL: `ticket` goes to flags[b] once sequence b's preference and (H, V) are written
  uint32_t ticket;
};
int launch_scores_and_preference(const cake_shape* shape, const cake_params* params, const void* const* q_win,
                                 const void* const* k, const int64_t* q_strides, const int64_t* k_strides,
                                 const float* const* row_lse, float* const* indicator, const LayerPointers* one, void* workspace,
                                 size_t workspace_bytes, double* pref, double* hv, int pref_ld, int hv_ld, const PlanArgs* plan, hipStream_t stream);

// ---- ragged per-launch dimensions, passed to kernels by value ----------------------------
constexpr int kMaxLaunchLayers = 32;
constexpr int kMaxLaunchEntries = 256;   // (layer, sequence) pairs per launch

struct RaggedDims {
  int32_t cur_len[kMaxLaunchEntries];
  int32_t keep[kMaxLaunchEntries];
};
struct LayerStrides {
  int64_t s[kMaxLaunchLayers][3];
};
// Kernels that read their dimensions from a plan do without those arguments: a launch copies them to device memory (the
// top-k's and the compaction's were 2.5 and 3.5 KB; 0.3 KB cost 0.8 us of host and device against none).
struct NoArgs {};
template <bool kPlanned> using DimsArg = typename std::conditional<kPlanned, NoArgs, RaggedDims>::type;
template <bool kPlanned> using StridesArg = typename std::conditional<kPlanned, NoArgs, LayerStrides>::type;
template <bool kPlanned> struct CapsArg { int32_t cur[kMaxLaunchLayers], keep[kMaxLaunchLayers]; };      // row capacities
template <> struct CapsArg<true> {};

// ---- device-resident eviction plan (cake_plan_eviction writes it, cake_evict_planned reads it) ----
// int32 budgets[L*B], keep[L*B], cur_len[L*B], cap_keep[L], cap_cur[L], copy_blocks[L*B + 1];
// then, 8-byte aligned, four tables of L device pointers: idx, k_out, v_out, ind_out.
// copy_blocks[e] = number of kCopyBlockPieces-piece blocks that the output rows of the entries
// before e (entry l*B + b) fill, each entry rounded up: the planned compaction's work list.
constexpr int kCopyBlockPieces = 1024;       // 16-byte pieces a compaction workgroup moves per step
struct PlanLayout {
  size_t off_budgets, off_keep, off_cur, off_cap_keep, off_cap_cur, off_blocks, off_tables, total;
};
inline PlanLayout plan_layout(int n_layers, int batch) {
  PlanLayout p{};
  const size_t lb = (size_t)n_layers * batch * sizeof(int32_t), l4 = (size_t)n_layers * sizeof(int32_t);
  size_t off = 0;
  p.off_budgets = off;  off += lb;
  p.off_keep = off;     off += lb;
  p.off_cur = off;      off += lb;
  p.off_cap_keep = off; off += l4;
  p.off_cap_cur = off;  off += l4;
  p.off_blocks = off;   off += lb + sizeof(int32_t);
  off = align_up(off, 8);
  p.off_tables = off;   off += 4 * (size_t)n_layers * sizeof(void*);
  p.total = align_up(off, 256);
  return p;
}
struct PlanView {               // device addresses inside a plan buffer
  const int32_t* keep;
  const int32_t* cur_len;
  const int32_t* cap_keep;
  const int32_t* cap_cur;
  const int32_t* copy_blocks;
  void* const* idx;
  void* const* k_out;
  void* const* v_out;
  void* const* ind_out;
};
inline PlanView plan_view(const void* plan, int n_layers, int batch) {
  const PlanLayout lay = plan_layout(n_layers, batch);
  const char* b = static_cast<const char*>(plan);
  void* const* t = reinterpret_cast<void* const*>(b + lay.off_tables);
  return PlanView{reinterpret_cast<const int32_t*>(b + lay.off_keep), reinterpret_cast<const int32_t*>(b + lay.off_cur),
                  reinterpret_cast<const int32_t*>(b + lay.off_cap_keep), reinterpret_cast<const int32_t*>(b + lay.off_cap_cur),
                  reinterpret_cast<const int32_t*>(b + lay.off_blocks), t, t + n_layers, t + 2 * n_layers, t + 3 * n_layers};
}
// What the host wants to know of a plan, in pinned host memory: a 32-bit ticket at offset 0, written
// last, then int32 budgets[L*B], keep[L*B], status[B] and float64 pref[B*L], hv[B*L][2].
struct PlanMirrorLayout {
  size_t off_budgets, off_keep, off_status, off_pref, off_hv, total;
};
__host__ __device__ inline PlanMirrorLayout plan_mirror_layout(int n_layers, int batch) {
  const size_t lb = (size_t)n_layers * batch;
  PlanMirrorLayout p{};
  p.off_budgets = 64;
  p.off_keep = p.off_budgets + lb * 4;
  p.off_status = p.off_keep + lb * 4;
  p.off_pref = (p.off_status + (size_t)batch * 4 + 7) / 8 * 8;
  p.off_hv = p.off_pref + lb * 8;
  p.total = p.off_hv + lb * 16;
  return p;
}
struct PlanMirror {            // device addresses of what is copied
  void* host;                  // NULL: no copy
  const int32_t *budgets, *keep, *status;
  const double *pref, *hv;     // [B, L], [B, L, 2] or NULL
  int32_t n_layers, batch;
  uint32_t ticket;
};
// top-k and compaction of all layers with the counts and output places read from a plan
// max_cur: the longest row to expect; `bounded` if no current length of the plan exceeds it; `last`: the last layer's rows,
// which are then not in the table; `mirror`: a workgroup more writes the host's copy of the plan meanwhile
int launch_topk_planned(const cake_shape* shape, const float* const* indicator, const float* last, const PlanView& plan, int64_t max_cur, bool bounded,
                        const PlanMirror& mirror, hipStream_t stream);
// cake_evict_planned; `bounded` if the plan was made with current lengths of at most seq_len - window; most_rows: see
// launch_compact_planned
int evict_planned(const cake_shape* shape, const float* const* indicator, const void* const* k_in, const void* const* v_in,
                  const int64_t* kv_strides, const uint8_t* compacted, const void* plan, size_t plan_bytes, bool bounded, const PlanMirror& mirror,
                  int64_t most_rows, void* stream);
// What a stage of the device-chained cascade (cascade_stage.hip) does to its lists.
struct StageArgs {
  PlanView plan;                      // of this stage
  void* const* held;                  // [m] the indicators before the stage
  const float* ind;                   // the new layer's
  const char *ind_old, *ind_new;      // pools the indicators are in; the lists of places have the same layout
  const int32_t* slots_old;
  int32_t* slots_new;
  int32_t* free_slots;
  int32_t m, batch, h_kv, window, prefix_rows, prefix_len;
};
// The top-k of the stage's rows and the lists after it in one launch, for rows of at most kStageMaxCur entries.  A stage of 8
// key heads with the lists in a launch of their own, and in this one, of 512 threads with eight slots throughout: 35.2 and 31.9 us at 1500 keys (16 layers, 200 rows
// kept), 55.3 and 53.1 at 8192 (32 layers, 1024), 68.0 and 67.7 at 16000 (16 layers, 1000).  Beyond, the 1024 threads the
// row takes have no registers left for the places (30000 keys: 97.8 and 99.6; 60000: 121 and 125).
constexpr int kStageMaxCur = 512 * 8 * 4 - 3;
int launch_topk_stage(const StageArgs& a, hipStream_t stream);
constexpr int kPlanMaskWords = 32;       // one bit per layer, n_layers <= 1024
// most_rows: rows that a head of a sequence keeps in all layers together at most, windows included; 0: not known
int launch_compact_planned(const cake_shape* shape, const void* const* k_in, const void* const* v_in,
                           const int64_t* kv_strides, const uint8_t* compacted, const float* const* ind_in,
                           const PlanView& plan, int64_t most_rows, hipStream_t stream);

#ifdef __HIPCC__
// The pointer, known to point to global memory (cast by way of an integer: a pair of pointer casts is folded away).  Where the
// compiler cannot see that (an address from a table, or one of two), its accesses are flat ones, which count with those of
// LDS as well: a wait for either waits for both, and independent loads come one after the other.  With global ones, a cascade of
// 32 layers of 8192 keys takes 2055 us for 2155 (runs of one side differ by 2 %), a decode step of 12 layers of 4 sequences 59.2 for
// 61.7, a pass of 1024 keys 44.2 for 44.7.
template <typename T>
__device__ __forceinline__ T* in_global(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)reinterpret_cast<uintptr_t>(p);
}

// rows that nothing on the device reads soon
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store_streaming(char* dst, const uint4& x) {
  const u32x4 v = {x.x, x.y, x.z, x.w};
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst));
}

// ---- wave-wide reductions and scans on the vector ALU ----------------------------------------------
// Six row-shift and row-broadcast steps (DPP); the lane-permute unit behind __shfl takes some ten
// times as long per step, which counts where a kernel is a chain of such steps.  After the last step
// lane 63 holds the whole wave's result.
template <typename T> struct DppWords;
template <> struct DppWords<uint32_t> { static constexpr int n = 1; };
template <> struct DppWords<float> { static constexpr int n = 1; };
template <> struct DppWords<int64_t> { static constexpr int n = 2; };
template <> struct DppWords<uint64_t> { static constexpr int n = 2; };
template <> struct DppWords<double> { static constexpr int n = 2; };
// x of the lane that step kCtrl pairs with this one; lanes without one take `none` (0 words, or with
// kSelf their own x)
template <int kCtrl, int kRowMask, bool kSelf, typename T>
__device__ __forceinline__ T dpp_step(T x) {
  constexpr int n = DppWords<T>::n;
  int w[n];
  __builtin_memcpy(w, &x, sizeof(T));
#pragma unroll
  for (int i = 0; i < n; ++i) w[i] = __builtin_amdgcn_update_dpp(kSelf ? w[i] : 0, w[i], kCtrl, kRowMask, 0xf, !kSelf);
  T y;
  __builtin_memcpy(&y, w, sizeof(T));
  return y;
}
// inclusive scan over the lanes; op's identity is 0
template <typename T, typename Op>
__device__ __forceinline__ T wave_scan(T x, Op op) {
  x = op(x, dpp_step<0x111, 0xf, false>(x));     // row_shr:1, 2, 4, 8
  x = op(x, dpp_step<0x112, 0xf, false>(x));
  x = op(x, dpp_step<0x114, 0xf, false>(x));
  x = op(x, dpp_step<0x118, 0xf, false>(x));
  x = op(x, dpp_step<0x142, 0xa, false>(x));     // row_bcast:15 into rows 1 and 3
  x = op(x, dpp_step<0x143, 0xc, false>(x));     // row_bcast:31 into rows 2 and 3
  return x;
}
template <typename T>
__device__ __forceinline__ T from_lane(T x, int lane /* the same for the wave */) {
  constexpr int n = DppWords<T>::n;
  int w[n];
  __builtin_memcpy(w, &x, sizeof(T));
#pragma unroll
  for (int i = 0; i < n; ++i) w[i] = __builtin_amdgcn_readlane(w[i], lane);
  T y;
  __builtin_memcpy(&y, w, sizeof(T));
  return y;
}
template <typename T>
__device__ __forceinline__ T wave_sum(T x) {
  return from_lane(wave_scan(x, [](T a, T b) { return a + b; }), 63);
}
__device__ __forceinline__ float wave_max(float x) {
  x = fmaxf(x, dpp_step<0x111, 0xf, true>(x));
  x = fmaxf(x, dpp_step<0x112, 0xf, true>(x));
  x = fmaxf(x, dpp_step<0x114, 0xf, true>(x));
  x = fmaxf(x, dpp_step<0x118, 0xf, true>(x));
  x = fmaxf(x, dpp_step<0x142, 0xa, true>(x));
  x = fmaxf(x, dpp_step<0x143, 0xc, true>(x));
  return from_lane(x, 63);
}
// Sum over the layers before l of keep (or of cur - keep) of sequence b, by one wave.
__device__ __forceinline__ int32_t rows_before(const StageArgs& a, int l, int b, bool dropped, int lane) {
  uint32_t t = 0;
  for (int i = lane; i < l; i += 64) {
    const int e = i * a.batch + b;
    t += (uint32_t)(dropped ? a.plan.cur_len[e] - a.plan.keep[e] : a.plan.keep[e]);
  }
  return (int32_t)wave_sum(t);
}
#endif

// Layers [l0, l0+nl) that fit one launch under the two limits above.
inline int launch_layers(int n_layers_left, int batch) {
  int by_entries = kMaxLaunchEntries / batch;
  int nl = n_layers_left < kMaxLaunchLayers ? n_layers_left : kMaxLaunchLayers;
  return nl < by_entries ? nl : by_entries;
}

}  // namespace cake
