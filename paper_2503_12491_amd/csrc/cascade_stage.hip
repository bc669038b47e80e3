// A stage of Alg. 1 with nothing read back, in one host call (csrc/cake_pass.h).
//
// A stage drops a few rows of every layer seen so far.  Copying all that stays into a second set of
// caches moves the whole budget once per layer (134 MB in and out at 32 layers x 1024 rows, 55 us), so a row
// stays where it was put when its layer was admitted: a layer is a list of places in a store of B_total
// rows per head, a stage renews the lists (8 bytes a row), puts the places of the dropped rows on a
// stack per head and takes the new layer's places from it.  One gather brings the rows into the caches'
// layout when the caller asks for them.  A stage of 8K keys, d = 128, 8 heads is a chain of launches too small for the chip,
// each waiting for the one before, with some 1.7 us between two: the scores (9 + 11 us), the plan beside the pooling
// (7), the top-k with the lists (12; apart 11 + 6) and the new layer's rows (4 to 20).  Counts and addresses come from the stage
// before and from the call, so that nothing has to be written ahead of the scores.  32 stages with the gather of 55 us: 4595 us
// with copies, 2025 now.
#include <algorithm>

#include "cake_pass.h"
#include "plan_device.h"

namespace cake {
namespace {

constexpr int kThreads = 256;
constexpr int kUnroll = 2;            // 16-byte pieces a thread moves per step
constexpr int kLongGap = 8;           // dropped rows in a row that one lane lists alone

// Lists of one held (layer, sequence, head) after the stage, and the places its dropped rows leave free, where the row is too
// long for the top-k that does both.  Bound by
// the latency of its chain of loads (counts, position, entry), some 3 us a turn, so a list is shared out
// over as many workgroups (blockIdx.z) as the chip has room for: no entry needs another's.
__global__ __launch_bounds__(kThreads) void renew_lists(StageArgs a) {
  const int l = blockIdx.y, b = blockIdx.x / a.h_kv, head = blockIdx.x;
  const int lane = threadIdx.x & 63, tid = blockIdx.z * kThreads + threadIdx.x, all = gridDim.z * kThreads;
  const int e = l * a.batch + b;
  const int cur = a.plan.cur_len[e], keep = a.plan.keep[e];
  if ((int)(blockIdx.z * kThreads) > keep) return;
  const int64_t at = (int64_t)head * a.plan.cap_keep[l];
  const int32_t* idx = in_global(static_cast<const int32_t*>(a.plan.idx[l])) + at;
  float* ind_out = in_global(static_cast<float*>(a.plan.ind_out[l])) + at;
  const int64_t from = (int64_t)head * a.plan.cap_cur[l];
  const float* ind_in = in_global(static_cast<const float*>(a.held[l])) + from;
  const int32_t* old = a.slots_old + (reinterpret_cast<const char*>(ind_in) - a.ind_old) / 4;
  int32_t* renewed = a.slots_new + (reinterpret_cast<const char*>(ind_out) - a.ind_new) / 4;
  if (keep == cur) {
    for (int r = tid; r < keep; r += all) {
      ind_out[r] = ind_in[r];
      renewed[r] = old[r];
    }
    return;
  }
  // free before this stage, then what the layers before this one drop in it
  uint32_t held = 0;
  for (int i = lane; i < a.m; i += 64) held += (uint32_t)a.plan.cur_len[i * a.batch + b];
  const int32_t top = a.prefix_rows - (int32_t)wave_sum(held) + rows_before(a, l, b, true, lane);
  int32_t* freed = a.free_slots + (int64_t)head * a.prefix_rows;
  auto release = [&](int j, int r) {  // position j, with r kept positions below it
    const int to = top + j - r;
    if (to >= 0 && to < a.prefix_rows) freed[to] = old[j];
  };
  for (int r0 = tid - lane; r0 <= keep; r0 += all) {
    const int r = r0 + lane;
    int g0 = 0, g1 = 0;               // dropped positions between the kept ones r - 1 and r
    if (r <= keep) {
      const int src = r < keep ? min(max(idx[r], 0), cur - 1) : cur;
      g0 = r > 0 ? min(max(idx[r - 1], 0), cur - 1) + 1 : 0;
      g1 = src;
      if (r < keep) {
        ind_out[r] = ind_in[src];
        renewed[r] = old[src];
      }
    }
    if (g1 - g0 <= kLongGap)
      for (int j = g0; j < g1; ++j) release(j, r);
    for (uint64_t longs = __ballot(g1 - g0 > kLongGap); longs; longs &= longs - 1) {
      const int who = __builtin_ctzll(longs);
      const int s0 = __builtin_amdgcn_readlane(g0, who), s1 = __builtin_amdgcn_readlane(g1, who);
      for (int j = s0 + lane; j < s1; j += 64) release(j, r0 + who);
    }
  }
}

// Rows of the new layer into the store: the kept prefix rows to the places on top of the free stack, the
// window rows to the layer's own; and the kept rows' indicators and places into the layer's lists.  Workgroups stride over the rows, whose number only the device knows.
__global__ __launch_bounds__(kThreads) void fill_rows(StageArgs a, const char* k, const char* v, char* k_store, char* v_store,
                                                     int64_t s0, int64_t s1, int64_t s2 /* bytes */, int64_t head_rows, int32_t pieces) {
  const int head = blockIdx.y, b = head / a.h_kv, h = head % a.h_kv;
  const int e = a.m * a.batch + b;
  const int keep = a.plan.keep[e], cur = a.plan.cur_len[e];
  const int64_t total = (int64_t)(keep + a.window) * pieces;
  if ((int64_t)blockIdx.x * kThreads * kUnroll >= total) return;
  const int32_t top = a.prefix_rows - rows_before(a, a.m, b, false, threadIdx.x & 63);
  const int64_t at = (int64_t)head * a.plan.cap_keep[a.m];
  const int32_t* idx = in_global(static_cast<const int32_t*>(a.plan.idx[a.m])) + at;
  const float* ind_in = a.ind + (int64_t)head * a.plan.cap_cur[a.m];
  float* ind_out = in_global(static_cast<float*>(a.plan.ind_out[a.m])) + at;
  int32_t* slots = a.slots_new + (static_cast<const char*>(a.plan.ind_out[a.m]) - a.ind_new) / 4 + at;
  const int32_t* freed = a.free_slots + (int64_t)head * a.prefix_rows;
  const char* kin = k + b * s0 + h * s1;
  const char* vin = v + b * s0 + h * s1;
  const int64_t row_bytes = (int64_t)pieces * 16;
  char* kout = k_store + head * head_rows * row_bytes;
  char* vout = v_store + head * head_rows * row_bytes;
  for (int64_t first = (int64_t)blockIdx.x * kThreads * kUnroll; first < total; first += (int64_t)gridDim.x * kThreads * kUnroll) {
    uint4 kv[kUnroll], vv[kUnroll];
    int64_t dst[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t p = first + u * kThreads + threadIdx.x;
      dst[u] = -1;
      if (p < total) {
        const int r = (int)(p / pieces), piece = (int)(p % pieces);
        int src = cur + (r - keep), slot = a.prefix_rows + a.m * a.window + (r - keep);
        if (r < keep) {
          src = min(max(idx[r], 0), cur - 1);
          slot = min(max(freed[min(max(top - 1 - r, 0), a.prefix_rows - 1)], 0), a.prefix_rows - 1);
          if (piece == 0) {
            slots[r] = slot;
            ind_out[r] = ind_in[src];
          }
        }
        kv[u] = *reinterpret_cast<const uint4*>(kin + src * s2 + piece * 16);
        vv[u] = *reinterpret_cast<const uint4*>(vin + src * s2 + piece * 16);
        dst[u] = slot * row_bytes + piece * 16;
      }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (dst[u] >= 0) {
        store_streaming(kout + dst[u], kv[u]);
        store_streaming(vout + dst[u], vv[u]);
      }
  }
}

// Tables of the compaction that reads the store: inputs, lists of places, outputs (the plan was made with
// the store in the place of the two pools), and for each layer the row its window rows follow.
__global__ __launch_bounds__(kThreads) void gather_tables(StageArgs a, int n_layers, void* k_store, void* v_store, char* pool_k, char* pool_v,
                                                         void** tables, int32_t* window_at) {
  for (int l = threadIdx.x; l < n_layers; l += kThreads) {
    tables[l] = k_store;
    tables[n_layers + l] = v_store;
    tables[2 * n_layers + l] = a.slots_new + (static_cast<const char*>(a.plan.ind_out[l]) - a.ind_new) / 4;
    tables[3 * n_layers + l] = pool_k + (static_cast<const char*>(a.plan.k_out[l]) - static_cast<const char*>(k_store));
    tables[4 * n_layers + l] = pool_v + (static_cast<const char*>(a.plan.v_out[l]) - static_cast<const char*>(v_store));
  }
  for (int i = threadIdx.x; i < n_layers * a.batch; i += kThreads) window_at[i] = a.prefix_rows + i / a.batch * a.window;
}

StageArgs stage_args(const cake_cascade* c, int m, const float* ind) {
  const cake_shape& s = c->shape;
  const PlanView before = plan_view(c->plan[(m & 1) ^ 1], std::max(m, 1), s.batch);
  return StageArgs{plan_view(c->plan[m & 1], m + 1, s.batch), before.ind_out, ind, reinterpret_cast<const char*>(c->ind[(m & 1) ^ 1]),
                   reinterpret_cast<const char*>(c->ind[m & 1]), c->slots[(m & 1) ^ 1], c->slots[m & 1], c->free_slots, m, s.batch,
                   s.n_kv_heads, s.window, c->prefix_rows, s.seq_len - s.window};
}
int64_t store_rows(const cake_cascade* c) { return c->prefix_rows + (int64_t)c->max_layers * c->shape.window; }

}  // namespace
}  // namespace cake

using namespace cake;

extern "C" int cake_cascade_stage(const cake_cascade* c, int32_t m, const void* q_win, const void* k, const void* v, float* indicator,
                                  const int64_t* q_strides, const int64_t* kv_strides, void* stream) {
  CAKE_REQUIRE(c && q_win && k && v && indicator && q_strides && kv_strides, "a pointer argument is NULL");
  CAKE_REQUIRE(m >= 0 && m < c->max_layers, "stage %d of %d", m, c->max_layers);
  if (int rc = check_shape_scores(&c->shape)) return rc;
  cake_shape shape = c->shape;
  shape.n_layers = m + 1;
  if (int rc = check_shape_basic(&shape)) return rc;
  const int bh = shape.batch * shape.n_kv_heads, eb = (int)elem_bytes(shape.dtype);
  CAKE_REQUIRE((int64_t)shape.n_layers * bh <= 65535 * 64 && bh <= 65535, "too many (layer, sequence, head) rows for one call");
  for (int j = 0; j < 3; ++j) {
    CAKE_REQUIRE(kv_strides[j] >= 0, "negative stride");
    CAKE_REQUIRE((kv_strides[j] * eb) % 16 == 0, "strides must be multiples of 16 bytes");
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  const StageArgs a = stage_args(c, m, indicator);
  const int L = c->max_layers;
  // the rows held before the stage: what the stage before kept, and the new layer whole
  PlanArgs plan{};
  if (int rc = plan_args(&shape, c->pref, L, c->total_budget, nullptr, c->idx, c->k_store, c->v_store, c->ind[m & 1], c->plan[m & 1],
                         c->plan_bytes, c->status, &plan)) return rc;
  if (m > 0) {
    plan.cur_len = plan_view(c->plan[(m & 1) ^ 1], m, shape.batch).keep;
    plan.cur_known = m * shape.batch;
  }
  const LayerPointers one{q_win, k, nullptr, indicator, nullptr, 0};
  if (int rc = launch_scores_and_preference(&c->shape, &c->params, nullptr, nullptr, q_strides, kv_strides, nullptr, nullptr, &one,
                                            c->workspace, c->workspace_bytes, c->pref + m, c->hv + 2 * m, L, L, &plan, st)) return rc;
  if (a.prefix_len <= kStageMaxCur) {
    if (int rc = launch_topk_stage(a, st)) return rc;
  } else {
    if (int rc = launch_topk_planned(&shape, reinterpret_cast<const float* const*>(a.held), indicator, a.plan, a.prefix_len, true, PlanMirror{}, st)) return rc;
    if (m > 0) {
      const int64_t shares = std::min<int64_t>((a.prefix_len + kThreads) / kThreads, 2048 / ((int64_t)bh * m));
      hipLaunchKernelGGL(renew_lists, dim3(bh, m, (unsigned)std::max<int64_t>(shares, 1)), dim3(kThreads), 0, st, a);
    }
  }
  // as many workgroups as the most rows the layer can keep fill, up to four for each compute unit
  const int32_t pieces = shape.head_dim * eb / 16;
  const int64_t most = std::min<int64_t>(shape.seq_len, c->total_budget - (int64_t)m * shape.window);
  const int64_t steps = (most * pieces + kThreads * kUnroll - 1) / (kThreads * kUnroll);
  const unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>(steps, std::max(1024 / bh, 1)));
  hipLaunchKernelGGL(fill_rows, dim3(gx, bh), dim3(kThreads), 0, st, a, static_cast<const char*>(k), static_cast<const char*>(v),
                     static_cast<char*>(c->k_store), static_cast<char*>(c->v_store), kv_strides[0] * eb, kv_strides[1] * eb,
                     kv_strides[2] * eb, store_rows(c), pieces);
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}

extern "C" int cake_cascade_gather(const cake_cascade* c, int32_t n_layers, void* pool_k, void* pool_v, void* stream) {
  CAKE_REQUIRE(c && pool_k && pool_v, "a pointer argument is NULL");
  CAKE_REQUIRE(n_layers >= 1 && n_layers <= c->max_layers, "%d layers of %d", n_layers, c->max_layers);
  hipStream_t st = static_cast<hipStream_t>(stream);
  cake_shape shape = c->shape;
  shape.n_layers = n_layers;
  const StageArgs a = stage_args(c, n_layers - 1, nullptr);
  void** tables = c->tables;
  int32_t* window_at = reinterpret_cast<int32_t*>(tables + 5 * (size_t)c->max_layers);
  hipLaunchKernelGGL(gather_tables, dim3(1), dim3(kThreads), 0, st, a, n_layers, c->k_store, c->v_store, static_cast<char*>(pool_k),
                     static_cast<char*>(pool_v), tables, window_at);
  PlanView view = a.plan;
  view.cur_len = window_at;
  view.idx = tables + 2 * n_layers;
  view.k_out = tables + 3 * n_layers;
  view.v_out = tables + 4 * n_layers;
  const int64_t rows = store_rows(c), d = shape.head_dim;
  const int64_t strides[3] = {shape.n_kv_heads * rows * d, rows * d, d};
  return launch_compact_planned(&shape, tables, tables + n_layers, strides, nullptr, nullptr, view,
                                std::min<int64_t>(c->total_budget, (int64_t)n_layers * shape.seq_len), st);
}
