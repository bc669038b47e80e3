// Calls between libcake and this package's host module (csrc/host_module.cpp): a one-shot pass
// described once and launched with one call, and the host's wait for its plan.  Not part of the
// public ABI.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "cake.h"

#ifdef __cplusplus
extern "C" {
#endif

// Everything the launches of a one-shot pass need; pointers are device memory unless noted.
typedef struct {
  cake_shape shape;
  cake_params params;
  const void* const* q_win;        // tables, as in cake_window_scores, cake_compact_kv
  const void* const* k;
  const void* const* v;
  const float* const* row_lse;     // NULL: the normalisers are computed (cake_window_scores)
  float* const* indicator;
  int64_t q_strides[3], kv_strides[3];
  void* workspace;
  uint64_t workspace_bytes;
  double *pref, *hv;               // [B, L], [B, L, 2]
  int64_t total_budget;
  void *pool_idx, *pool_k, *pool_v, *pool_ind;
  void* plan;
  uint64_t plan_bytes;
  int32_t* status;                 // [B]
  void* mirror;                    // pinned host memory of cake_pass_mirror_layout's size, or NULL
} cake_pass;

enum { CAKE_PASS_SCORES = 1, CAKE_PASS_EVICT = 2 };

// Byte offsets of budgets, keep, status, pref and hv in a pass's mirror, then its size.
void cake_pass_mirror_layout(int32_t n_layers, int32_t batch, uint64_t* offsets /* [6] */);
// Enqueues the parts asked for.  With CAKE_PASS_EVICT and ticket != 0 the plan is also written to
// the mirror, `ticket` last.
int cake_pass_launch(const cake_pass* pass, int32_t parts, uint32_t ticket, void* stream);
// The places of the layers' outputs in the pass's pools for row capacities the host knows (the rule of
// cake_plan_eviction): four device tables [4][n_layers] of idx, K, V and indicator outputs.  The counts travel as
// kernel arguments: nothing of the caller's is read after the call, and a captured call keeps its own.
int cake_pass_place(const cake_pass* pass, const int32_t* caps /* host [n_layers] */, void** tables, void* stream);
// Returns when the mirror holds the plan of `ticket` (the launches behind it may still be running).
int cake_pass_wait_plan(const void* mirror, uint32_t ticket, void* stream);
// Returns when everything enqueued on the stream has run.
int cake_stream_wait(void* stream);

// cake_compact_kv that also carries the rows' positions in the prompt: pos_out[l][b, h, r] =
// pos_in[l][b, h, idx[r]], laid out like ind_in and ind_out; a NULL entry of the pos_in table stands for
// rows that are their own positions.
int cake_compact_kv_positions(const cake_shape* shape, const void* const* k_in, const void* const* v_in,
                              const int64_t* kv_strides, const int32_t* cur_len, const int32_t* k, const int32_t* const* idx,
                              const float* const* ind_in, void* const* k_out, void* const* v_out, float* const* ind_out,
                              const int32_t* const* pos_in, int32_t* const* pos_out, void* stream);

// Alg. 1 with the allocation on the host (CascadeSession).  The session's own arrays are host memory; what is
// indexed by layer has room for max_layers.
typedef struct {
  cake_shape shape;                // of one layer
  cake_params params;
  int32_t max_layers, track_positions;
  int64_t total_budget;
  void* workspace;                 // of cake_workspace_bytes(shape)
  uint64_t workspace_bytes;
  void* mirror;                    // pinned: double pref[B], hv[B][2], then uint32 flags[B]
  void** tables;                   // device [9 * max_layers]
  double *pref, *hv;               // [B][max_layers], [B][max_layers][2]
  int64_t* cur_len;                // [max_layers][B] prefix rows held
  int64_t *k, *v, *ind, *pos;      // addresses of the layers' rows; pos 0: row r is position r of the prompt
  int64_t *strides, *cap;          // [max_layers][3] of K and V, row capacity
  int64_t *off_kv, *off_i;         // element offsets in the slabs, -1: the caller's own tensors
  int64_t* budgets;                // [max_layers][B] of the last stage
} cake_session;
// Scores of one layer and its preferences into the mirror; the flags take `ticket`.
int cake_session_scores(const cake_session* s, const void* q_win, const void* k, const float* row_lse, float* indicator,
                        const int64_t* q_strides, const int64_t* kv_strides, uint32_t ticket, void* stream);
// Returns when the mirror holds what the scores of `ticket` wrote.
int cake_session_wait(const cake_session* s, uint32_t ticket, void* stream);
// n words to device memory, as kernel arguments: nothing of the caller's is read after the call.
int cake_write_words(void* dst, const uint64_t* words, int32_t n, void* stream);

// The buffers of an in-place decode step (cake_decode_step) at up to 32 layers, described once.
#define CAKE_DECODE_LAYERS 32
typedef struct {
  void *k_slots, *v_slots;
  float* indicator;
  int32_t *order, *state;
} cake_decode_buffers;
typedef struct {
  cake_shape shape;
  const cake_params* params;       // host memory, read at every call
  void* const* k_slots;            // tables, as in cake_decode_step
  void* const* v_slots;
  float* const* indicator;
  int32_t* const* order;
  int32_t* const* state;
  void* workspace;
  uint64_t workspace_bytes;
  int64_t rank;                    // of the new rows' tensors: 3 for one layer, 4 with the layers first
  int64_t slot_strides[CAKE_DECODE_LAYERS][3];
  int32_t cap[CAKE_DECODE_LAYERS];
  cake_decode_buffers buffers[CAKE_DECODE_LAYERS];     // what the tables hold
} cake_decode_plan;
int cake_decode_run(const cake_decode_plan* plan, const void* q_new, const int64_t* q_strides, const void* k_new,
                    const void* v_new, const int64_t* kv_new_strides, void* stream);

// Alg. 1 in stages, each enqueued by one call (csrc/cascade_stage.hip); pointers are device memory.
// Rows live in a store [B, H_kv, store_rows, d] of K and one of V: prefix rows anywhere in the first
// `prefix_rows`, the window rows of layer l at prefix_rows + l * window.
typedef struct {
  cake_shape shape;                // of one layer
  cake_params params;
  int32_t max_layers, prefix_rows; // prefix_rows >= min(total_budget, max_layers * seq_len) - window, 1 at least
  int64_t total_budget;
  void* workspace;                 // of cake_workspace_bytes(shape)
  uint64_t workspace_bytes;
  double *pref, *hv;               // [B, max_layers], [B, max_layers, 2]
  int32_t* status;                 // [B]
  void** tables;                   // 5 * max_layers words, then int32 [max_layers, B]
  void* plan[2];                   // even and odd stages, each of cake_plan_bytes at max_layers
  uint64_t plan_bytes;
  // Lists, B * H_kv * (sum over the layers of the largest count of the batch) words each: positions chosen in
  // this stage; indicators and places in the store of the rows held after even and odd stages.
  int32_t* idx;
  float* ind[2];
  int32_t* slots[2];
  int32_t* free_slots;             // [B, H_kv, prefix_rows], to begin with 0 .. prefix_rows - 1 in each row
  void *k_store, *v_store;
} cake_cascade;
// Stage `m`: score layer m, budgets of layers 0 .. m, eviction of each from the rows it holds.
int cake_cascade_stage(const cake_cascade* c, int32_t m, const void* q_win, const void* k, const void* v, float* indicator,
                       const int64_t* q_strides, const int64_t* kv_strides, void* stream);
// The caches after `n_layers` stages, layer after layer [B, H_kv, cap_l + window, d] into the two pools.
int cake_cascade_gather(const cake_cascade* c, int32_t n_layers, void* pool_k, void* pool_v, void* stream);

#ifdef __cplusplus
}
#endif
