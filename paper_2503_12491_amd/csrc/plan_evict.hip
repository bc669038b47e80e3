// cake_plan_eviction / cake_evict_planned: the allocation step and EVICT of a one-shot pass with
// no host round trip in between.
//
// Preference-prioritised allocation (Sec. 4.1 Eq. 7; Sec. 4.2 Eq. 9, Prop. 1) on the device, with
// the same integers as the host routine cake_cascade_allocate: divisor (Webster) apportionment,
// every layer first holds its S_w window tokens, the rest go one at a time to the layer with the
// largest pref/(B + 1/2) among layers below N, ties to the lower layer.  The retained prefix
// counts k = clamp(B - S_w, 0, cur_len) (Sec. 4.3 Eq. 11-12: the window tokens are kept
// structurally and count towards B) and the places of every layer's outputs in four pools are
// derived in the same launches and left in a device-resident plan, from which the top-k and the
// compaction of all layers read their counts and output addresses.
//
// One wave per sequence, every layer owned by one lane.  The award loop is entered from a state it
// passes through: for a level lambda every layer takes at once all seats whose priority is strictly
// above lambda (counted exactly, with the very division the loop compares), which is what the loop
// would have awarded before touching any seat at or below lambda.  Only fp64 divisions and
// comparisons decide, so host and device agree bit for bit whatever level the search stops at.
//
// Latency is all there is to this step: budgets, places and work list of a few sequences are one launch
// of one workgroup, the level is found by a secant search on the piecewise-linear seat count: a few counts from rounded
// quotients (0.3 us each), then as a rule one exact one (0.9) and a seat or none to award (0.5 each); with exact counts
// alone the plan of 30 layers took 7.6 us, now 5.0.  More sequences are allocated by workgroups of their own.
#include <algorithm>
#include <cmath>

#include "plan_device.h"

namespace cake {
namespace {

constexpr int kPlanMaxWaves = 16;
constexpr int kPlanOneLaunch = 12;

// The first step of a large batch alone, a workgroup of one wave per sequence.
__global__ __launch_bounds__(64) void allocate_kernel(PlanArgs a) {
  extern __shared__ __attribute__((aligned(8))) char plan_lds[];
  const int n_layers = a.n_layers;
  double* p = reinterpret_cast<double*>(plan_lds);
  if (n_layers <= 64) allocate_sequence<true>(a, blockIdx.x, threadIdx.x, nullptr, nullptr, nullptr);
  else allocate_sequence<false>(a, blockIdx.x, threadIdx.x, p, p + n_layers, reinterpret_cast<int32_t*>(p + 2 * n_layers));
}

__global__ __launch_bounds__(64 * kPlanMaxWaves) void plan_kernel(PlanArgs a) {
  extern __shared__ __attribute__((aligned(8))) char plan_lds[];
  plan_workgroup(a, plan_lds);
}

}  // namespace
}  // namespace cake

using namespace cake;

extern "C" int cake_plan_bytes(const cake_shape* shape, size_t* bytes) {
  CAKE_REQUIRE(bytes != nullptr, "bytes is NULL");
  if (int rc = check_shape_basic(shape)) return rc;
  *bytes = plan_layout(shape->n_layers, shape->batch).total;
  return CAKE_OK;
}

int cake::plan_args(const cake_shape* shape, const double* pref, int pref_ld, int64_t total_budget, const int32_t* cur_len,
                    void* pool_idx, void* pool_k, void* pool_v, void* pool_ind, void* plan, size_t plan_bytes,
                    int32_t* status, PlanArgs* out) {
  CAKE_REQUIRE(pref && pool_idx && pool_k && pool_v && pool_ind && plan && status, "a pointer argument is NULL");
  CAKE_REQUIRE(shape->seq_len > shape->window, "seq_len %d must exceed window %d", shape->seq_len, shape->window);
  CAKE_REQUIRE(total_budget >= (int64_t)shape->n_layers * shape->window,
               "total_budget %lld is below n_layers*window = %lld", (long long)total_budget,
               (long long)shape->n_layers * shape->window);
  CAKE_REQUIRE((reinterpret_cast<uintptr_t>(plan) & 7) == 0, "plan must be 8-byte aligned");
  const PlanLayout lay = plan_layout(shape->n_layers, shape->batch);
  CAKE_REQUIRE(plan_bytes >= lay.total, "plan has %zu bytes, %zu needed", plan_bytes, lay.total);
  for (void* q : {pool_idx, pool_k, pool_v, pool_ind})
    CAKE_REQUIRE((reinterpret_cast<uintptr_t>(q) & 15) == 0, "pools must be 16-byte aligned");
  char* b = static_cast<char*>(plan);
  const int L = shape->n_layers;
  PlanArgs a{};
  a.pref = pref; a.pref_ld = pref_ld;
  a.n_layers = L; a.batch = shape->batch; a.h_kv = shape->n_kv_heads; a.window = shape->window; a.seq_len = shape->seq_len;
  a.row_bytes = (int32_t)(shape->head_dim * elem_bytes(shape->dtype));
  a.total_budget = total_budget; a.cur_len = cur_len; a.cur_known = cur_len ? L * shape->batch : 0;
  a.budgets = reinterpret_cast<int32_t*>(b + lay.off_budgets);
  a.keep = reinterpret_cast<int32_t*>(b + lay.off_keep);
  a.cur = reinterpret_cast<int32_t*>(b + lay.off_cur);
  a.cap_keep = reinterpret_cast<int32_t*>(b + lay.off_cap_keep);
  a.cap_cur = reinterpret_cast<int32_t*>(b + lay.off_cap_cur);
  a.copy_blocks = reinterpret_cast<int32_t*>(b + lay.off_blocks);
  a.status = status;
  a.pool_idx = static_cast<char*>(pool_idx); a.pool_k = static_cast<char*>(pool_k);
  a.pool_v = static_cast<char*>(pool_v); a.pool_ind = static_cast<char*>(pool_ind);
  void** tables = reinterpret_cast<void**>(b + lay.off_tables);
  a.idx_tbl = tables; a.k_tbl = tables + L; a.v_tbl = tables + 2 * L; a.ind_tbl = tables + 3 * L;
  *out = a;
  return CAKE_OK;
}

int cake::launch_plan(const PlanArgs& args, hipStream_t stream) {
  PlanArgs a = args;
  const int L = a.n_layers;
  const size_t per_wave = L > 64 ? kPlanLdsPerLayer * L : 0;
  const int by_lds = per_wave ? (int)((size_t)65536 / per_wave) : kPlanMaxWaves;
  // Up to twelve sequences share the plan's workgroup (a launch less: 1, 4 and 12 sequences of 32 layers 5.9, 8.5 and
  // 16.3 us, with a launch of their own 7.7, 10.0 and 16.3), unless its LDS holds fewer; more of them would wait for
  // each other there (16, 64 and 256 sequences 20.8, 76 and 252 us against 17.5, 26 and 63; 64 of 1024 layers 3350
  // against 617).
  if (a.batch > std::min(kPlanOneLaunch, by_lds)) {
    hipLaunchKernelGGL(allocate_kernel, dim3(a.batch), dim3(64), per_wave, stream, a);
    a.allocated = true;
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(64 * kPlanMaxWaves), 0, stream, a);
  } else {
    // a wave per sequence (at least two, so that the two scans run side by side)
    const int waves = std::max(a.batch, std::min(2, by_lds));
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(64 * waves), per_wave * waves, stream, a);
  }
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}

extern "C" int cake_plan_eviction(const cake_shape* shape, const double* pref, int64_t total_budget,
                                  const int32_t* cur_len,
                                  void* pool_idx, void* pool_k, void* pool_v, void* pool_ind,
                                  void* plan, size_t plan_bytes, int32_t* status, void* stream) {
  if (int rc = check_shape_basic(shape)) return rc;
  PlanArgs a{};
  if (int rc = plan_args(shape, pref, shape->n_layers, total_budget, cur_len, pool_idx, pool_k, pool_v, pool_ind, plan, plan_bytes,
                         status, &a)) return rc;
  return launch_plan(a, static_cast<hipStream_t>(stream));
}

extern "C" int cake_plan_layout(const cake_shape* shape, size_t* offsets) {
  CAKE_REQUIRE(offsets != nullptr, "offsets is NULL");
  if (int rc = check_shape_basic(shape)) return rc;
  const PlanLayout lay = plan_layout(shape->n_layers, shape->batch);
  const size_t tbl = (size_t)shape->n_layers * sizeof(void*);
  const size_t all[10] = {lay.off_budgets, lay.off_keep, lay.off_cur, lay.off_cap_keep, lay.off_cap_cur, lay.off_blocks,
                          lay.off_tables, lay.off_tables + tbl, lay.off_tables + 2 * tbl, lay.off_tables + 3 * tbl};
  for (int i = 0; i < 10; ++i) offsets[i] = all[i];
  return CAKE_OK;
}

int cake::evict_planned(const cake_shape* shape, const float* const* indicator, const void* const* k_in, const void* const* v_in,
                        const int64_t* kv_strides, const uint8_t* compacted, const void* plan, size_t plan_bytes, bool bounded,
                        const PlanMirror& mirror, int64_t most_rows, void* stream) {
  if (int rc = check_shape_basic(shape)) return rc;
  CAKE_REQUIRE(indicator && k_in && v_in && kv_strides && plan, "a pointer argument is NULL");
  CAKE_REQUIRE((int64_t)shape->n_layers * shape->batch * shape->n_kv_heads <= 65535 * 64,
               "too many (layer, sequence, head) rows for one call");
  const int eb = (int)elem_bytes(shape->dtype);
  for (int j = 0; j < 3; ++j) {
    CAKE_REQUIRE(kv_strides[j] >= 0, "negative stride");
    CAKE_REQUIRE((kv_strides[j] * eb) % 16 == 0, "strides must be multiples of 16 bytes");
  }
  const PlanLayout lay = plan_layout(shape->n_layers, shape->batch);
  CAKE_REQUIRE(plan_bytes >= lay.total, "plan has %zu bytes, %zu needed", plan_bytes, lay.total);
  const PlanView view = plan_view(plan, shape->n_layers, shape->batch);
  hipStream_t st = static_cast<hipStream_t>(stream);
  // without a length in the shape the kernel for any length serves
  const int64_t max_cur = shape->seq_len > shape->window ? shape->seq_len - shape->window : 0x7fffffff;
  if (int rc = launch_topk_planned(shape, indicator, nullptr, view, max_cur, bounded, mirror, st)) return rc;
  return launch_compact_planned(shape, k_in, v_in, kv_strides, compacted, indicator, view, most_rows, st);
}

// The lengths are the plan's, device data that this call cannot look at: the shape's length only says which rows
// are worth a kernel of their own.
extern "C" int cake_evict_planned(const cake_shape* shape, const float* const* indicator,
                                  const void* const* k_in, const void* const* v_in, const int64_t* kv_strides,
                                  const uint8_t* compacted,
                                  const void* plan, size_t plan_bytes, void* stream) {
  return evict_planned(shape, indicator, k_in, v_in, kv_strides, compacted, plan, plan_bytes, false, PlanMirror{}, 0, stream);
}
