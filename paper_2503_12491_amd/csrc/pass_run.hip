// One-shot pass in one host call (csrc/cake_pass.h).  A pass at 8K keys is 0.3 ms of kernels; the
// launches are made back to back from here, and the host learns the plan from pinned memory as soon
// as the plan kernel has run, so that it prepares the caller's results beside the top-k and the
// compaction instead of after four copies and a stream synchronisation behind them.
#include <algorithm>
#include <chrono>

#include "cake_pass.h"
#include "plan_device.h"

namespace cake {
namespace {

constexpr int kPlaceLayers = 256;            // per launch: 2 KiB of arguments
struct PlaceArgs {
  char *idx, *k, *v, *ind;
  void** tables;                             // [4][n_layers]
  int64_t row_i, row_kv;                     // bytes of a row of all heads in the pools
  int32_t n_layers, first, count, window;
  int64_t rows_before[kPlaceLayers];
};
__global__ __launch_bounds__(kPlaceLayers) void place_outputs(PlaceArgs a) {
  const int i = threadIdx.x, l = a.first + i;
  if (i >= a.count) return;
  const int64_t before = a.rows_before[i], before_kv = before + (int64_t)l * a.window;
  a.tables[l] = a.idx + before * a.row_i;
  a.tables[a.n_layers + l] = a.k + before_kv * a.row_kv;
  a.tables[2 * a.n_layers + l] = a.v + before_kv * a.row_kv;
  a.tables[3 * a.n_layers + l] = a.ind + before * a.row_i;
}

constexpr int kWords = 448;                  // per launch: 3.5 KiB of arguments
struct WordArgs {
  uint64_t* dst;
  int32_t n;
  uint64_t w[kWords];
};
__global__ __launch_bounds__(kWords) void write_words(WordArgs a) {
  if ((int)threadIdx.x < a.n) a.dst[threadIdx.x] = a.w[threadIdx.x];
}

// Until `flag` holds the ticket.  A watched flag is seen within a microsecond; a stream that is this slow or broken is
// left to the runtime.
int wait_flag(const uint32_t* flag, uint32_t ticket, void* stream) {
  const auto arrived = [&] { return __atomic_load_n(flag, __ATOMIC_ACQUIRE) == ticket; };
  const auto t0 = std::chrono::steady_clock::now();
  for (uint32_t i = 1; !arrived(); ++i) {
    __builtin_ia32_pause();
    if ((i & 1023) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(200)) {
      if (int rc = cake_stream_wait(stream)) return rc;
      CAKE_REQUIRE(arrived(), "the plan did not arrive");
    }
  }
  return CAKE_OK;
}

}  // namespace
}  // namespace cake

using namespace cake;

extern "C" void cake_pass_mirror_layout(int32_t n_layers, int32_t batch, uint64_t* offsets) {
  const PlanMirrorLayout lay = plan_mirror_layout(n_layers, batch);
  const uint64_t all[6] = {lay.off_budgets, lay.off_keep, lay.off_status, lay.off_pref, lay.off_hv, lay.total};
  for (int i = 0; i < 6; ++i) offsets[i] = all[i];
}

extern "C" int cake_pass_launch(const cake_pass* p, int32_t parts, uint32_t ticket, void* stream) {
  CAKE_REQUIRE(p != nullptr, "pass is NULL");
  if (int rc = check_shape_basic(&p->shape)) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  PlanArgs plan{};
  if (parts & CAKE_PASS_EVICT) {
    if (int rc = plan_args(&p->shape, p->pref, p->shape.n_layers, p->total_budget, nullptr, p->pool_idx, p->pool_k,
                           p->pool_v, p->pool_ind, p->plan, p->plan_bytes, p->status, &plan)) return rc;
  }
  if (parts & CAKE_PASS_SCORES)
    if (int rc = launch_scores_and_preference(&p->shape, &p->params, p->q_win, p->k, p->q_strides, p->kv_strides, p->row_lse,
                                              p->indicator, nullptr, p->workspace, p->workspace_bytes, p->pref, p->hv,
                                              p->shape.n_layers, p->shape.n_layers, parts & CAKE_PASS_EVICT ? &plan : nullptr, st)) return rc;
  if (parts & CAKE_PASS_EVICT) {
    if (!(parts & CAKE_PASS_SCORES))
      if (int rc = launch_plan(plan, st)) return rc;
    // the plan above takes every row at its full length
    const PlanMirror mirror{ticket ? p->mirror : nullptr, plan.budgets, plan.keep, plan.status, p->pref, p->hv, p->shape.n_layers,
                            p->shape.batch, ticket};
    return evict_planned(&p->shape, p->indicator, p->k, p->v, p->kv_strides, nullptr, p->plan, p->plan_bytes, true, mirror,
                         std::min<int64_t>(p->total_budget, (int64_t)p->shape.n_layers * p->shape.seq_len), stream);
  }
  return CAKE_OK;
}

extern "C" int cake_pass_place(const cake_pass* p, const int32_t* caps, void** tables, void* stream) {
  CAKE_REQUIRE(p && caps && tables, "a pointer argument is NULL");
  if (int rc = check_shape_basic(&p->shape)) return rc;
  const cake_shape& s = p->shape;
  for (int l = 0; l < s.n_layers; ++l) CAKE_REQUIRE(caps[l] >= 0, "caps[%d] = %d is negative", l, caps[l]);
  const int64_t bh = (int64_t)s.batch * s.n_kv_heads;
  PlaceArgs a{static_cast<char*>(p->pool_idx), static_cast<char*>(p->pool_k), static_cast<char*>(p->pool_v),
              static_cast<char*>(p->pool_ind), tables, bh * 4, bh * s.head_dim * (int64_t)elem_bytes(s.dtype), s.n_layers, 0, 0,
              s.window, {}};
  int64_t rows = 0;
  for (; a.first < s.n_layers; a.first += a.count) {
    a.count = s.n_layers - a.first < kPlaceLayers ? s.n_layers - a.first : kPlaceLayers;
    for (int i = 0; i < a.count; ++i) {
      a.rows_before[i] = rows;
      rows += caps[a.first + i];
    }
    hipLaunchKernelGGL(place_outputs, dim3(1), dim3(kPlaceLayers), 0, static_cast<hipStream_t>(stream), a);
  }
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}

extern "C" int cake_stream_wait(void* stream) {
  CAKE_HIP_TRY(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
  return CAKE_OK;
}

extern "C" int cake_pass_wait_plan(const void* mirror, uint32_t ticket, void* stream) {
  CAKE_REQUIRE(mirror != nullptr && ticket != 0, "no mirror to wait on");
  return wait_flag(static_cast<const uint32_t*>(mirror), ticket, stream);
}

extern "C" int cake_session_scores(const cake_session* s, const void* q_win, const void* k, const float* row_lse, float* indicator,
                                   const int64_t* q_strides, const int64_t* kv_strides, uint32_t ticket, void* stream) {
  CAKE_REQUIRE(s && q_win && k && indicator && q_strides && kv_strides && s->mirror && ticket != 0, "a required argument is NULL");
  if (int rc = check_shape_scores(&s->shape)) return rc;
  CAKE_REQUIRE(s->shape.n_layers == 1, "the scores of one layer, not of %d", s->shape.n_layers);
  double* pref = static_cast<double*>(s->mirror);
  const int B = s->shape.batch;
  const LayerPointers one{q_win, k, row_lse, indicator, reinterpret_cast<uint32_t*>(pref + 3 * B), ticket};
  return launch_scores_and_preference(&s->shape, &s->params, nullptr, nullptr, q_strides, kv_strides, nullptr, nullptr, &one, s->workspace,
                                      s->workspace_bytes, pref, pref + B, 1, 1, nullptr, static_cast<hipStream_t>(stream));
}

extern "C" int cake_session_wait(const cake_session* s, uint32_t ticket, void* stream) {
  CAKE_REQUIRE(s && s->mirror && ticket != 0, "no mirror to wait on");
  const int B = s->shape.batch;
  const uint32_t* flags = reinterpret_cast<const uint32_t*>(static_cast<const double*>(s->mirror) + 3 * B);
  for (int b = 0; b < B; ++b)
    if (int rc = wait_flag(flags + b, ticket, stream)) return rc;
  return CAKE_OK;
}

extern "C" int cake_write_words(void* dst, const uint64_t* words, int32_t n, void* stream) {
  CAKE_REQUIRE(dst && words && n >= 0, "a pointer argument is NULL");
  WordArgs a{};
  for (int at = 0; at < n; at += kWords) {
    a.dst = static_cast<uint64_t*>(dst) + at;
    a.n = n - at < kWords ? n - at : kWords;
    for (int i = 0; i < a.n; ++i) a.w[i] = words[at + i];
    hipLaunchKernelGGL(write_words, dim3(1), dim3(kWords), 0, static_cast<hipStream_t>(stream), a);
  }
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}
