// cake_decode_update: indicator maintenance for one generated token (implementation appendix,
// decoding branch of the listing: the new query's attention over the cached keys outside the
// window is pooled and folded into the stored eviction indicator; the layer is then evicted
// back to its fixed budget with cake_select_topk / cake_compact_kv at k = cur_len - 1).
//
// The cache of a (layer, sequence, KV head) holds cur_len scored rows followed by the S_w window
// rows, the last of which is the new token's key.  The G query heads of the group attend to all
// cur_len + S_w rows (one query row each: a matrix-vector product, done on the vector ALU, one
// row per thread); the weights on the scored rows are averaged over the group, max-pooled along
// the row axis and added to the stored indicator.  Two launches over chunks of 256 rows, so
// that a few thousand rows per head still spread over the chip: per-chunk softmax partials, then
// normaliser + weights (with the pooling halo recomputed) + update.  The keys are read twice
// rather than keeping G logits per row.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "cake_internal.h"
#include "cake_pass.h"

namespace cake {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxGroup = 8;
constexpr float kMasked = -1.0e30f;
constexpr int kMaxHalf = 64;               // widest pooling window: 2*64+1

struct DecodeArgs {
  const void* const* q_new;
  const void* const* k_cache;
  float* const* indicator;
  int64_t qs[2];             // element strides of q_new: batch, head
  int32_t batch, h_kv, group, window, pool;
  int32_t n_chunks;          // chunks of kThreads rows per slice in `part`
  float c;                   // scale * log2(e)
  float inv_g;
  float* part;               // [slice][n_chunks][kMaxGroup][2]: (reference, sum) of each chunk and head
  int32_t cap_cur[kMaxLaunchLayers];
};

template <typename T> struct Row16;      // sixteen bytes of a key row as floats
template <> struct Row16<__bf16> {
  static constexpr int kElems = 8;
  static __device__ __forceinline__ void load(const __bf16* p, float (&x)[8]) {
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = (float)v[i];
  }
};
template <> struct Row16<float> {
  static constexpr int kElems = 4;
  static __device__ __forceinline__ void load(const float* p, float (&x)[4]) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
  }
};

// t[h] = c * <q_h, k_row> for the G heads of the group; q lies in LDS as floats [G][D].
template <typename T, int D>
__device__ __forceinline__ void row_logits(const T* k_row, const float* q_lds, int group, float c, float (&t)[kMaxGroup]) {
  using R = Row16<T>;
  float acc[kMaxGroup];
#pragma unroll
  for (int h = 0; h < kMaxGroup; ++h) acc[h] = 0.f;
#pragma unroll
  for (int e0 = 0; e0 < D; e0 += R::kElems) {
    float x[R::kElems];
    R::load(k_row + e0, x);
#pragma unroll
    for (int h = 0; h < kMaxGroup; ++h) {
      if (h < group) {
#pragma unroll
        for (int i = 0; i < R::kElems; ++i) acc[h] = fmaf(x[i], q_lds[h * D + e0 + i], acc[h]);
      }
    }
  }
#pragma unroll
  for (int h = 0; h < kMaxGroup; ++h) t[h] = acc[h] * c;
}

// Kernel 1: per chunk of kThreads rows and per head, (reference, sum of 2^(t - reference)).
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void decode_partials_kernel(DecodeArgs a, RaggedDims dims, LayerStrides ks) {
  __shared__ float q_lds[kMaxGroup * D];
  __shared__ float red_m[kWaves][kMaxGroup], red_l[kWaves][kMaxGroup];

  const int chunk = blockIdx.x, ll = blockIdx.z;
  const int b = blockIdx.y / a.h_kv, g = blockIdx.y % a.h_kv;
  const int n = dims.cur_len[ll * a.batch + b] + a.window;       // rows the new query sees
  if (chunk * kThreads >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const T* q = in_global(reinterpret_cast<const T*>(a.q_new[ll])) + b * a.qs[0] + (int64_t)(g * a.group) * a.qs[1];
  const T* k = in_global(reinterpret_cast<const T*>(a.k_cache[ll])) + b * ks.s[ll][0] + g * ks.s[ll][1];
  for (int i = tid; i < a.group * D; i += kThreads) q_lds[i] = (float)q[(i / D) * a.qs[1] + (i % D)];
  __syncthreads();

  const int j = chunk * kThreads + tid;
  float m[kMaxGroup], l[kMaxGroup];
#pragma unroll
  for (int h = 0; h < kMaxGroup; ++h) { m[h] = kMasked; l[h] = 0.f; }
  if (j < n) {
    row_logits<T, D>(k + j * ks.s[ll][2], q_lds, a.group, a.c, m);
#pragma unroll
    for (int h = 0; h < kMaxGroup; ++h) l[h] = 1.f;
  }
#pragma unroll
  for (int h = 0; h < kMaxGroup; ++h) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const float om = __shfl_xor(m[h], off), ol = __shfl_xor(l[h], off);
      const float mn = fmaxf(m[h], om);
      l[h] = l[h] * exp2f(m[h] - mn) + ol * exp2f(om - mn);
      m[h] = mn;
    }
    if (lane == 0) { red_m[wave][h] = m[h]; red_l[wave][h] = l[h]; }
  }
  __syncthreads();
  if (tid < a.group) {
    float mm = kMasked, sum = 0.f;
    for (int w = 0; w < kWaves; ++w) mm = fmaxf(mm, red_m[w][tid]);
    for (int w = 0; w < kWaves; ++w) sum += red_l[w][tid] * exp2f(red_m[w][tid] - mm);
    float* o = a.part + ((((int64_t)(ll * a.batch + b) * a.h_kv + g) * a.n_chunks + chunk) * kMaxGroup + tid) * 2;
    o[0] = mm;
    o[1] = sum;
  }
}

// Kernel 2: normalisers from the chunks' pairs, then for this chunk's scored rows (and the pooling
// halo on either side) the group-mean weights, pooled and added to the stored indicator.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void decode_apply_kernel(DecodeArgs a, RaggedDims dims, LayerStrides ks) {
  __shared__ float q_lds[kMaxGroup * D];
  __shared__ float lse_lds[kMaxGroup];
  __shared__ float obs[kThreads + 2 * kMaxHalf];

  const int chunk = blockIdx.x, ll = blockIdx.z;
  const int b = blockIdx.y / a.h_kv, g = blockIdx.y % a.h_kv;
  const int cur = dims.cur_len[ll * a.batch + b];
  const int n = cur + a.window;
  if (chunk * kThreads >= cur) return;
  const int tid = threadIdx.x;
  const T* q = in_global(reinterpret_cast<const T*>(a.q_new[ll])) + b * a.qs[0] + (int64_t)(g * a.group) * a.qs[1];
  const T* k = in_global(reinterpret_cast<const T*>(a.k_cache[ll])) + b * ks.s[ll][0] + g * ks.s[ll][1];
  for (int i = tid; i < a.group * D; i += kThreads) q_lds[i] = (float)q[(i / D) * a.qs[1] + (i % D)];
  if (tid < a.group) {
    const int used = (n + kThreads - 1) / kThreads;               // chunks that hold rows
    const float* p = a.part + (((int64_t)(ll * a.batch + b) * a.h_kv + g) * a.n_chunks * kMaxGroup + tid) * 2;
    float mm = kMasked;
    for (int c = 0; c < used; ++c) mm = fmaxf(mm, p[(int64_t)c * kMaxGroup * 2]);
    float sum = 0.f;
    for (int c = 0; c < used; ++c) sum += p[(int64_t)c * kMaxGroup * 2 + 1] * exp2f(p[(int64_t)c * kMaxGroup * 2] - mm);
    lse_lds[tid] = mm + log2f(sum);
  }
  __syncthreads();

  const int half = a.pool / 2;
  const int j0 = chunk * kThreads - half;                          // first row of the halo
  for (int i = tid; i < kThreads + 2 * half; i += kThreads) {
    const int j = j0 + i;
    float w = -INFINITY;                                           // clipped edges never win the max
    if (j >= 0 && j < cur) {
      float t[kMaxGroup];
      row_logits<T, D>(k + j * ks.s[ll][2], q_lds, a.group, a.c, t);
      float s = 0.f;
#pragma unroll
      for (int h = 0; h < kMaxGroup; ++h)
        if (h < a.group) s += exp2f(t[h] - lse_lds[h]);
      w = s * a.inv_g;
    }
    obs[i] = w;
  }
  __syncthreads();
  const int j = chunk * kThreads + tid;
  if (j < cur) {
    float mx = obs[tid + half];
    for (int d = 1; d <= half; ++d) mx = fmaxf(mx, fmaxf(obs[tid + half - d], obs[tid + half + d]));
    float* ind = in_global(a.indicator[ll]) + ((int64_t)b * a.h_kv + g) * a.cap_cur[ll];
    ind[j] += mx;
  }
}


// ------------------------------------------------------------------------------------------
// In-place decode step (cake_decode_step).  The cache of a (layer, sequence, KV head) lives in
// fixed physical slots; `order` lists the slots in logical order: the cur scored rows by position,
// then the S_w window rows, oldest first.  One generated token: its key and value go to the free
// slot and are appended to the list, so the oldest window row becomes the last scored row (with
// indicator 0); the indicator is updated as in cake_decode_update; the scored row with the
// smallest indicator (the later one among equals: what top-k at k = cur under (value descending,
// position ascending) leaves out) is deleted from the list and its slot becomes the free one.
// K and V are touched at one row per head; only the 4-byte list entries and indicators move.
// ------------------------------------------------------------------------------------------
typedef cake_decode_buffers StepBuffers;
struct StepBase {
  const void* q_new; const void* k_new; const void* v_new;
  int64_t qs[3], ns[3];             // element strides of q_new / k_new, v_new: layer, batch, head
  int32_t batch, h_kv, group, window, pool, n_chunks, rows_max;
  float c, inv_g;
  float* logits;      // [slice][group][rows_max], rows_max a multiple of 4
  float* part;        // [slice][n_chunks][kMaxGroup][2], chunks of the rows a workgroup of the first kernel takes
  float* amin;        // [slice][n_chunks][2]: (value, logical index as float bits)
};
// Arguments of a call for any number of layers: the buffers behind device tables.
struct StepArgs : StepBase {
  void* const* k_slots; void* const* v_slots;
  float* const* indicator; int32_t* const* order; int32_t* const* state;
  int64_t ss[kMaxLaunchLayers][3];  // element strides of every layer's slots: batch, head, slot
  int32_t cap[kMaxLaunchLayers];
  __device__ __forceinline__ StepBuffers buffers(int ll) const {
    return StepBuffers{in_global(k_slots[ll]), in_global(v_slots[ll]), in_global(indicator[ll]), in_global(order[ll]), in_global(state[ll])};
  }
};
// Arguments of a call for one layer whose buffers the host knows: a quarter of a kilobyte and no table
// to look through.  A kernel this short notices every load that waits for another, and each further
// line of its arguments.
struct StepOneArgs : StepBase {
  StepBuffers one;
  int64_t ss[1][3];
  int32_t cap[1];
  __device__ __forceinline__ StepBuffers buffers(int) const { return one; }
};

// Logits of sixteen cached rows against the G new query rows on the matrix core: rows on the M side,
// query heads on the N side (columns at or above G are zero).  Lane (i, kg) = (lane & 15, lane >> 4)
// supplies row i's and head i's elements of piece kg, 16 bytes of every 64, so that a load instruction
// covers a run of 64 bytes of each row; lane (h, kg) ends with head h's logits of rows 4*kg .. 4*kg + 3.
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <typename T, int D> struct RowDots;
template <int D> struct RowDots<__bf16, D> {
  typedef __bf16 frag __attribute__((ext_vector_type(8)));
  typedef __bf16 loose __attribute__((ext_vector_type(8), aligned(2)));
  static constexpr int kSteps = D / 32;
  static constexpr int kBlocks = 4;                     // sixteen-row blocks loaded before the first is used: 64 registers
  static __device__ __forceinline__ f32x4 run(const frag (&k)[kSteps], const frag (&q)[kSteps]) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kSteps; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[s], q[s], acc, 0, 0, 0);
    return acc;
  }
};
template <int D> struct RowDots<float, D> {
  typedef float frag __attribute__((ext_vector_type(4)));
  typedef float loose __attribute__((ext_vector_type(4), aligned(4)));
  static constexpr int kSteps = D / 16;
  static constexpr int kBlocks = 2;
  static __device__ __forceinline__ f32x4 run(const frag (&k)[kSteps], const frag (&q)[kSteps]) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(k[s][i], q[s][i], acc, 0, 0, 0);
    return acc;
  }
};

// v_exp_f32, which returns 0 below 2^-126: for the terms of a sum that is at least 1
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// What all forms of the step share, so that a head's result depends on neither the other layers nor the other sequences of the
// call: the (reference, sum) pairs of 64 rows each, in the rows' order, as one pair (runs of 256 rows);
template <int kPairs>
__device__ __forceinline__ float2 merge_pairs(const float (&m)[kPairs], const float (&l)[kPairs]) {
  float mm = kMasked, sum = 0.f;
#pragma unroll
  for (int i = 0; i < kPairs; ++i) mm = fmaxf(mm, m[i]);
#pragma unroll
  for (int i = 0; i < kPairs; ++i) sum = fmaf(l[i], fast_exp2(m[i] - mm), sum);
  return make_float2(mm, sum);
}

// the normaliser, log2 of the sum that the lanes' pairs stand for;
__device__ __forceinline__ float wave_normaliser(float2 x) {
  const float m = wave_max(x.x), e = fast_exp2(x.x - m);
  // (which of the sum's products are rounded is written out: it must not hang on the kernel)
  float l = fmaf(x.y, e, dpp_step<0x111, 0xf, false>(x.y * e));
  l += dpp_step<0x112, 0xf, false>(l);
  l += dpp_step<0x114, 0xf, false>(l);
  l += dpp_step<0x118, 0xf, false>(l);
  l += dpp_step<0x142, 0xa, false>(l);
  l += dpp_step<0x143, 0xc, false>(l);
  return m + log2f(from_lane(l, 63));
}

// and the sum of a row's weights over the heads.  Weights below 2^-126 too: they order rows whose indicators are still 0.  Beside
// a sum from 2^-90 on the up to eight terms that came out as 0 are less than half its last place, so the sum is the
// same to the bit; taking exp2f for all terms cost up to 7 % of a step (32 heads of 6000 rows and 8 queries 26.1 -> 28.1 us a
// layer, so 26.3).
template <int kGroup>
__device__ __forceinline__ float weight_sum(const float (&t)[kGroup], const float* lse, int group) {
  float s = 0.f;
#pragma unroll
  for (int h = 0; h < kGroup; ++h)
    if (h < group) s += fast_exp2(t[h] - lse[h]);
  if (s < 0x1p-90f) {
    s = 0.f;
#pragma unroll
    for (int h = 0; h < kGroup; ++h)
      if (h < group) s += exp2f(t[h] - lse[h]);
  }
  return s;
}

template <typename T, int D> using StepFrags = typename RowDots<T, D>::frag[RowDots<T, D>::kSteps];
// The new query rows of a group as operands: head li's piece kg of every step.
template <typename T, int D>
__device__ __forceinline__ void load_queries(StepFrags<T, D>& qf, const T* q, int li, int kg, int group) {
  using Dots = RowDots<T, D>;
  constexpr int kElems = 16 / (int)sizeof(T);
#pragma unroll
  for (int s = 0; s < Dots::kSteps; ++s) {
    qf[s] = *reinterpret_cast<const typename Dots::loose*>(q + s * 4 * kElems + kg * kElems);     // q_new may start at any element
    if (li >= group)
#pragma unroll
      for (int i = 0; i < kElems; ++i) qf[s][i] = (T)0.f;
  }
}

// A wave's 64 rows from row0 on, whose slots lane li knows (16 apart): logits of head li, four rows at a time, to `keep`; returns
// the rows' (reference, sum) of head li.
template <typename T, int D, typename Keep>
__device__ __forceinline__ float2 wave_rows(const StepFrags<T, D>& qf, const int32_t (&slot)[4], const T* ks,
                                            const T* kn, int64_t tok, int row0, int n, float c, int li, int kg, Keep keep) {
  using Dots = RowDots<T, D>;
  typedef typename Dots::frag frag;
  constexpr int kElems = 16 / (int)sizeof(T);
  float m = kMasked, l = 0.f;                             // of head li over the lane's rows
  float t[64 / 16][4];
#pragma unroll
  for (int r0 = 0; r0 < 4; r0 += Dots::kBlocks) {
    frag kf[Dots::kBlocks][Dots::kSteps];
#pragma unroll
    for (int r = 0; r < Dots::kBlocks; ++r) {
      const int j = row0 + (r0 + r) * 16 + li;
      // the generated token's row comes from the caller; rows past the end repeat it
      const T* row = j < n - 1 ? ks + slot[r0 + r] * tok : kn;
#pragma unroll
      for (int s = 0; s < Dots::kSteps; ++s) kf[r][s] = *reinterpret_cast<const frag*>(row + s * 4 * kElems + kg * kElems);
    }
#pragma unroll
    for (int r = 0; r < Dots::kBlocks; ++r) {
      const f32x4 acc = Dots::run(kf[r], qf);
      const int j0 = row0 + (r0 + r) * 16 + kg * 4;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        t[r0 + r][v] = j0 + v < n ? acc[v] * c : kMasked;
        m = fmaxf(m, t[r0 + r][v]);
      }
      keep(j0, make_float4(acc[0] * c, acc[1] * c, acc[2] * c, acc[3] * c));
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v) l += fast_exp2(t[r][v] - m);
  if (m == kMasked) l = 0.f;                              // none of the lane's rows exists
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    const float om = __shfl_xor(m, off), ol = __shfl_xor(l, off), mn = fmaxf(m, om);
    l = l * fast_exp2(m - mn) + ol * fast_exp2(om - mn);
    m = mn;
  }
  return make_float2(m, l);
}

// The generated token's key and value into the free slot.
template <typename T, int D>
__device__ __forceinline__ void store_new_row(const void* v_new, int64_t v_at, const T* kn, T* ks, T* vs, int64_t to, int tid, int threads) {
  constexpr int kElems = 16 / (int)sizeof(T), kPieces = D / kElems;
  const T* vn = reinterpret_cast<const T*>(v_new) + v_at;
  for (int i = tid; i < 2 * kPieces; i += threads) {
    const int e = (i % kPieces) * kElems;
    const T* src = i < kPieces ? kn : vn;
    T* dst = (i < kPieces ? ks : vs) + to;
    *reinterpret_cast<uint4*>(dst + e) = *reinterpret_cast<const uint4*>(src + e);
  }
}

// Step kernel 1, one workgroup per 64 rows a wave of a slice: the new row goes to its slot; logits of the G
// heads for every listed row (kept for what follows) and the chunk's (reference, sum) pairs.
// Bound by the key bytes: four 16-byte loads per row and lane, all of a wave's 64 rows in flight; the
// one-row-per-thread form on the vector ALU read its queries from LDS once per row and head and reached
// 1.1 TB/s (12 layers x 4 sequences x 8 heads of 2K rows: 179 us; now 50, 4.2 TB/s, or 39 where the keys still lie in the
// last-level cache from the token before; one layer of 1K rows per head 18 -> 6 us).  A compute unit gets some 35 bytes a nanosecond,
// so four waves of one stay for 2 us where the rows would fit compute units of their own: small calls run one-wave workgroups
// (4 layers of 2 heads, 12 queries and 335 rows at once in fp32: 14.7 -> 12.5 us, with the loads of the second kernel that no longer
// wait for the state).  Layers of 8 heads called one by one gain nothing from that: the two kernels take 4.6 and 5.0 us a layer, and
// the host as long to launch them, which is what step_whole_kernel spares short lists.
template <typename T, int D, int kStepWaves, typename Args>
__global__ __launch_bounds__(64 * kStepWaves, 4) void step_logits_kernel(Args a) {
  using Dots = RowDots<T, D>;
  typedef typename Dots::frag frag;
  constexpr int kElems = 16 / (int)sizeof(T), kRows = 64 * kStepWaves;
  __shared__ float red_m[kStepWaves][kMaxGroup], red_l[kStepWaves][kMaxGroup];
  const int chunk = blockIdx.x, ll = blockIdx.z;
  const int b = blockIdx.y / a.h_kv, g = blockIdx.y % a.h_kv;
  const int64_t head = (int64_t)b * a.h_kv + g, slice = (int64_t)ll * a.batch * a.h_kv + head;
  const StepBuffers buf = a.buffers(ll);
  const int32_t* st = buf.state + head * 4;
  const int cur = st[0], free_slot = st[1];
  const int n = cur + 1 + a.window;                       // rows the new query sees
  const int cap = a.cap[ll];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, kg = lane >> 4;
  const T* q = reinterpret_cast<const T*>(a.q_new) + ll * a.qs[0] + b * a.qs[1] + (int64_t)(g * a.group + min(li, a.group - 1)) * a.qs[2];
  const T* kn = reinterpret_cast<const T*>(a.k_new) + ll * a.ns[0] + b * a.ns[1] + g * a.ns[2];
  T* ks = reinterpret_cast<T*>(buf.k_slots) + b * a.ss[ll][0] + g * a.ss[ll][1];
  const int32_t* order = buf.order + head * (cap + a.window + 1);
  const int64_t tok = a.ss[ll][2];
  float* lg = a.logits + slice * a.group * a.rows_max;

  // layers of different lengths share a grid: most of the shorter ones' workgroups have no rows
  if (!std::is_same<Args, StepOneArgs>::value && chunk * kRows >= n) return;
  // list entries of the lane's rows: for one layer loaded beside the state that says how many there are
  int32_t slot[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) slot[r] = order[min(chunk * kRows + wave * 64 + r * 16 + li, cap + a.window)];
  frag qf[Dots::kSteps];
  load_queries<T, D>(qf, q, li, kg, a.group);
  if (chunk * kRows >= n) return;
  const float2 own = wave_rows<T, D>(qf, slot, ks, kn, tok, chunk * kRows + wave * 64, n, a.c, li, kg, [&](int j0, const float4& x) {
    if (li < a.group && j0 < n) *reinterpret_cast<float4*>(lg + (int64_t)li * a.rows_max + j0) = x;
  });
  if (lane < a.group) { red_m[wave][lane] = own.x; red_l[wave][lane] = own.y; }
  if (chunk == (n - 1) / kRows)
    store_new_row<T, D>(a.v_new, ll * a.ns[0] + b * a.ns[1] + g * a.ns[2], kn, ks, reinterpret_cast<T*>(buf.v_slots) + b * a.ss[ll][0] + g * a.ss[ll][1],
                        free_slot * tok, tid, kRows);
  __syncthreads();
  if (tid < a.group) {
    float rm[kStepWaves], rl[kStepWaves];
#pragma unroll
    for (int w = 0; w < kStepWaves; ++w) { rm[w] = red_m[w][tid]; rl[w] = red_l[w][tid]; }
    *reinterpret_cast<float2*>(a.part + ((slice * a.n_chunks + chunk) * kMaxGroup + tid) * 2) = merge_pairs(rm, rl);
  }
}

// Step kernel 2, one workgroup per slice with all of its rows in registers: normalisers from the chunks'
// pairs, pooled group-mean weights added to the indicator of the cur + 1 scored rows, the smallest
// updated indicator (the later row among equals), and the list and the indicator written back closed
// over it; its slot becomes the free one.
// A chain of latencies (arguments, state, rows, four barriers): everything the rows need is loaded
// before the first of them waits.  One launch for what two kernels of 256-row chunks and a serial
// search of their candidates did: 6 + 4 -> 5.4 us for one layer of 1K rows per head, 26 + 14 -> 11 us for
// 384 heads of 2K.  Letting the last chunk of a slice do this work inside the
// first kernel (a ticket per slice) was slower, 21 us against 14 for both: making the chunks' logits
// visible across the dies costs more than the launch.
constexpr int kStepSmallRows = 4096;       // one-wave workgroups in the first kernel: rows per slice at most
constexpr int kFinishThreads = 1024, kFinishRows = 8 * kFinishThreads;
// kSmall: the first kernel's workgroups took 64 rows each, of kStepSmallRows at most.  (One kernel that merged the pairs of
// either had registers of the four-head form spilled: 384 heads of 2K rows 11.1 -> 12.5 us.)
template <int kGroup, bool kSmall, typename Args>
__global__ __launch_bounds__(kFinishThreads, kGroup <= 4 ? 8 : 4) void step_finish_kernel(Args a) {     // <= 64 registers: two workgroups per compute unit
  constexpr int kFinishWaves = kFinishThreads / 64, kPer = (kSmall ? kStepSmallRows : kFinishRows) / kFinishThreads;
  __shared__ float obs[kFinishRows + 2 * kMaxHalf];      // group-mean weights between two clipped edges
  __shared__ float lse[kMaxGroup];
  __shared__ uint64_t cand[kFinishWaves];
  const int ll = blockIdx.y, b = blockIdx.x / a.h_kv, g = blockIdx.x % a.h_kv;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int head = b * a.h_kv + g, slice = ll * a.batch * a.h_kv + head;
  const StepBuffers buf = a.buffers(ll);
  int32_t* st = buf.state + (int64_t)head * 4;
  const int cur = st[0], free_slot = st[1];
  const int cur1 = cur + 1, n = cur1 + a.window, cap = a.cap[ll], half = a.pool / 2;
  int32_t* order = buf.order + (int64_t)head * (cap + a.window + 1);
  float* ind = buf.indicator + (int64_t)head * (cap + 1);
  const float* lg = a.logits + (int64_t)slice * a.group * a.rows_max;
  const int group = a.group;
  // A layer alone is loaded up to what its buffers hold: no load waits for the state to say how much of it is in use.
  constexpr bool kOne = std::is_same<Args, StepOneArgs>::value;
  int32_t slot[kPer];
  float val[kPer], t[kPer][kGroup];
  const int last = kOne ? cap + a.window : n - 1;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int j = i * kFinishThreads + tid;
    if (i * kFinishThreads <= last) {
      slot[i] = order[min(j, last)];
      val[i] = ind[min(j, kOne ? cap : cur)];
#pragma unroll
      for (int h = 0; h < kGroup; ++h) t[i][h] = lg[min(h, group - 1) * a.rows_max + min(j, last)];
    }
  }
  if (wave < group) {
    const float* p = a.part + ((int64_t)slice * a.n_chunks * kMaxGroup + wave) * 2;
    static_assert(kFinishRows / kThreads <= 64 && kMaxGroup <= kFinishWaves, "a lane per 256 rows and a wave per head");
    constexpr int kChunkRows = kSmall ? 64 : kThreads;
    auto pair = [&](int chunk) {            // (masked where the chunk has no rows)
      float2 x = make_float2(kMasked, 0.f);
      if (kOne) x = *reinterpret_cast<const float2*>(p + min(chunk, a.n_chunks - 1) * kMaxGroup * 2);
      else if (chunk * kChunkRows < n) x = *reinterpret_cast<const float2*>(p + chunk * kMaxGroup * 2);
      if (chunk * kChunkRows >= n) x = make_float2(kMasked, 0.f);
      return x;
    };
    float2 x;
    if constexpr (kSmall) {                 // pairs of 64 rows: four are what a workgroup of 256 rows writes
      float rm[kWaves], rl[kWaves];
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float2 y = pair(lane * kWaves + w);
        rm[w] = y.x;
        rl[w] = y.y;
      }
      x = merge_pairs(rm, rl);
    } else {
      x = pair(lane);
    }
    const float norm = wave_normaliser(x);
    if (lane == 0) lse[wave] = norm;
  }
  for (int i = tid; i < half; i += kFinishThreads) obs[i] = obs[half + cur1 + i] = -INFINITY;      // clipped edges never win the max
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int j = i * kFinishThreads + tid;
    if (i * kFinishThreads < cur1 && j < cur1) {
      obs[half + j] = weight_sum(t[i], lse, group) * a.inv_g;
    }
  }
  __syncthreads();
  uint64_t best = 0;                                     // largest complement of (order-preserving key of the value, complement of the index)
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int j = i * kFinishThreads + tid;
    if (i * kFinishThreads < cur1 && j < cur1) {
      float mx = obs[half + j];
      for (int d = 1; d <= half; ++d) mx = fmaxf(mx, fmaxf(obs[half + j - d], obs[half + j + d]));
      val[i] = (j < cur ? val[i] : 0.f) + mx;            // the row that has just left the window starts at 0
      const uint32_t u = __float_as_uint(val[i] + 0.f), key = u & 0x80000000u ? ~u : u | 0x80000000u;
      best = max(best, (uint64_t)~key << 32 | (uint32_t)j);
    }
  }
  best = wave_scan(best, [](uint64_t x, uint64_t y) { return max(x, y); });
  if (lane == 63) cand[wave] = best;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kFinishWaves; ++w) best = max(best, cand[w]);
  const int e = (int)(uint32_t)best;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int j = i * kFinishThreads + tid;
    if (i * kFinishThreads >= n || j >= n) continue;
    if (j == n - 1) slot[i] = free_slot;
    if (j > e) order[j - 1] = slot[i];
    if (j < cur1 && j != e) ind[j - (j > e ? 1 : 0)] = val[i];
    if (j == e) {
      st[1] = slot[i];
      st[2] = e;              // logical index of the evicted scored row (for inspection)
    }
    // the entries past the closed list and indicator keep what stood there
    if (j == n - 1) order[j] = free_slot;
    if (j == cur) ind[j] = val[i];
  }
}

// Both steps of a head of few rows in one launch: a workgroup with a wave per 64 rows, logits and pairs in LDS; the same sums in the
// same order as by the two kernels.  Bound by the chain state, list, keys, then by the one compute unit that takes in the head's
// keys, some 35 bytes a nanosecond; but nothing goes through memory and waits for a second launch, which the host has to
// make as well.  Heads of at most kStepWholeBytes of keys take it (all layers of a call, so that the longest decides).  Us of two launches and of
// one, 8 layers of 8 heads called one by one: 100 to 350 rows of 128 in bf16 86 and 62, 470 86 and 68, 700 85 and 88, 980 86 and
// 108; 220 rows in fp32 88 and 71, 470 87 and 102; 980 rows of 64 with 8 queries 86 and 79.  384 heads at once: up to 470 rows 21.8 and
// 18.3, 980 30.2 and 29.3; 8 heads at once: 220 rows 10.5 and 7.2, 470 10.7 and 8.9, 980 10.5 and 13.8.
constexpr int kStepOneThreads = 1024;
constexpr int64_t kStepWholeBytes = 128 << 10;
template <typename T, int D, int kGroup, typename Args>
__global__ __launch_bounds__(kStepOneThreads) void step_whole_kernel(Args a) {
  using Dots = RowDots<T, D>;
  constexpr int kLd = kStepOneThreads + 4;               // logits of a head: the heads' rows start in banks of their own
  __shared__ __attribute__((aligned(16))) float lg[kGroup * kLd];
  __shared__ float2 red[kStepOneThreads / 64][kMaxGroup];
  __shared__ float obs[kStepOneThreads + 2 * kMaxHalf];
  __shared__ float lse[kMaxGroup];
  __shared__ uint64_t cand[kStepOneThreads / 64];
  const int ll = blockIdx.y, b = blockIdx.x / a.h_kv, g = blockIdx.x % a.h_kv;
  const int threads = blockDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, kg = lane >> 4;
  const int64_t head = blockIdx.x;
  const StepBuffers buf = a.buffers(ll);
  int32_t* st = buf.state + head * 4;
  const int cur = st[0], free_slot = st[1], cur1 = cur + 1, n = cur1 + a.window, cap = a.cap[ll], half = a.pool / 2;
  int32_t* order = buf.order + head * (cap + a.window + 1);
  float* ind = buf.indicator + head * (cap + 1);
  const T* q = reinterpret_cast<const T*>(a.q_new) + ll * a.qs[0] + b * a.qs[1] + (int64_t)(g * a.group + min(li, a.group - 1)) * a.qs[2];
  const T* kn = reinterpret_cast<const T*>(a.k_new) + ll * a.ns[0] + b * a.ns[1] + g * a.ns[2];
  T* ks = reinterpret_cast<T*>(buf.k_slots) + b * a.ss[ll][0] + g * a.ss[ll][1];
  const int64_t tok = a.ss[ll][2];
  // loaded up to what the buffers hold: no load waits for the state to say how much of it is in use
  int32_t rows[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) rows[r] = order[min(wave * 64 + r * 16 + li, cap + a.window)];
  StepFrags<T, D> qf;
  load_queries<T, D>(qf, q, li, kg, a.group);
  int32_t slot = order[min(tid, cap + a.window)], last_free = free_slot;
  float val = ind[min(tid, cap)];
  if (wave * 64 < n) {
    const float2 own = wave_rows<T, D>(qf, rows, ks, kn, tok, wave * 64, n, a.c, li, kg, [&](int j0, const float4& x) {
      if (li < a.group) *reinterpret_cast<float4*>(lg + li * kLd + j0) = x;
    });
    if (lane < a.group) red[wave][lane] = own;
  }
  if (wave == 0)
    store_new_row<T, D>(a.v_new, ll * a.ns[0] + b * a.ns[1] + g * a.ns[2], kn, ks, reinterpret_cast<T*>(buf.v_slots) + b * a.ss[ll][0] + g * a.ss[ll][1],
                        free_slot * tok, lane, 64);
  asm volatile("" : "+v"(slot), "+v"(val), "+v"(last_free));       // have arrived: other waves write their places behind the barriers
  __syncthreads();
  for (int h = wave; h < a.group; h += threads >> 6) {   // a lane per 256 rows, as in step_finish_kernel
    float rm[kWaves], rl[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int chunk = lane * kWaves + w;
      const float2 y = chunk * 64 < n ? red[chunk][h] : make_float2(kMasked, 0.f);
      rm[w] = y.x;
      rl[w] = y.y;
    }
    const float norm = wave_normaliser(merge_pairs(rm, rl));
    if (lane == 0) lse[h] = norm;
  }
  for (int i = tid; i < half; i += threads) obs[i] = obs[half + cur1 + i] = -INFINITY;      // clipped edges never win the max
  float t[kGroup];
#pragma unroll
  for (int h = 0; h < kGroup; ++h) t[h] = lg[min(h, a.group - 1) * kLd + tid];
  __syncthreads();
  if (tid < cur1) obs[half + tid] = weight_sum(t, lse, a.group) * a.inv_g;
  __syncthreads();
  uint64_t best = 0;                                     // as in step_finish_kernel, from here on
  if (tid < cur1) {
    float mx = obs[half + tid];
    for (int d = 1; d <= half; ++d) mx = fmaxf(mx, fmaxf(obs[half + tid - d], obs[half + tid + d]));
    val = (tid < cur ? val : 0.f) + mx;
    const uint32_t u = __float_as_uint(val + 0.f), key = u & 0x80000000u ? ~u : u | 0x80000000u;
    best = (uint64_t)~key << 32 | (uint32_t)tid;
  }
  best = wave_scan(best, [](uint64_t x, uint64_t y) { return max(x, y); });
  if (lane == 63) cand[wave] = best;
  __syncthreads();
  for (int w = 0; w < threads >> 6; ++w) best = max(best, cand[w]);
  const int e = (int)(uint32_t)best;
  if (tid >= n) return;
  if (tid == n - 1) slot = last_free;
  if (tid > e) order[tid - 1] = slot;
  if (tid < cur1 && tid != e) ind[tid - (tid > e ? 1 : 0)] = val;
  if (tid == e) {
    st[1] = slot;
    st[2] = e;
  }
  if (tid == n - 1) order[tid] = last_free;
  if (tid == cur) ind[tid] = val;
}

// Caches of more rows than one workgroup holds: two more kernels.
// Step kernel 2: normalisers, pooled group-mean weights added to the indicator of the cur + 1
// scored rows, and this chunk's candidate for eviction: the smallest updated indicator, the later
// row among equals.  Sums as in step_finish_kernel, so that a head of up to 8192 rows comes out the same in a call that also
// holds longer ones; a lane per pair instead of a thread per head over all of them: a step of 8 heads of 9000
// rows 28.2 -> 19.0 us, of 30000 68.5 -> 35.4.
__global__ __launch_bounds__(kThreads) void step_apply_kernel(StepArgs a) {
  __shared__ float lse_lds[kMaxGroup];
  __shared__ float obs[kThreads + 2 * kMaxHalf];
  __shared__ float cand_v[kWaves];
  __shared__ int cand_j[kWaves];
  const int chunk = blockIdx.x, ll = blockIdx.z;
  const int b = blockIdx.y / a.h_kv, g = blockIdx.y % a.h_kv;
  const int64_t slice = ((int64_t)ll * a.batch + b) * a.h_kv + g;
  const int32_t* st = in_global(a.state[ll]) + ((int64_t)b * a.h_kv + g) * 4;
  const int cur1 = st[0] + 1;                              // scored rows, the newcomer included
  const int n = cur1 + a.window;
  if (chunk * kThreads >= cur1) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int used = (n + kThreads - 1) / kThreads;
  for (int h = wave; h < a.group; h += kWaves) {           // a lane per 256 rows and, of more than 16384, those 64 chunks further as well
    const float* p = a.part + (slice * a.n_chunks * kMaxGroup + h) * 2;
    float2 x = make_float2(kMasked, 0.f);
    for (int c = lane; c < used; c += 64) {
      const float2 y = *reinterpret_cast<const float2*>(p + (int64_t)c * kMaxGroup * 2);
      x = c == lane ? y : merge_pairs({x.x, y.x}, {x.y, y.y});
    }
    const float norm = wave_normaliser(x);
    if (lane == 0) lse_lds[h] = norm;
  }
  __syncthreads();
  const int half = a.pool / 2;
  const int j0 = chunk * kThreads - half;
  const float* lg = a.logits + slice * a.group * a.rows_max;
  for (int i = tid; i < kThreads + 2 * half; i += kThreads) {
    const int j = j0 + i;
    float w = -INFINITY;                                   // clipped edges never win the max
    if (j >= 0 && j < cur1) {
      float t[kMaxGroup];
#pragma unroll
      for (int h = 0; h < kMaxGroup; ++h) t[h] = h < a.group ? lg[(int64_t)h * a.rows_max + j] : 0.f;
      w = weight_sum(t, lse_lds, a.group) * a.inv_g;
    }
    obs[i] = w;
  }
  __syncthreads();
  const int j = chunk * kThreads + tid;
  float val = INFINITY;
  int best = -1;
  if (j < cur1) {
    float mx = obs[tid + half];
    for (int d = 1; d <= half; ++d) mx = fmaxf(mx, fmaxf(obs[tid + half - d], obs[tid + half + d]));
    float* ind = in_global(a.indicator[ll]) + ((int64_t)b * a.h_kv + g) * (a.cap[ll] + 1);
    val = (j < cur1 - 1 ? ind[j] : 0.f) + mx;               // the row that has just left the window starts at 0
    ind[j] = val;
    best = j;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const float ov = __shfl_xor(val, off);
    const int oj = __shfl_xor(best, off);
    if (ov < val || (ov == val && oj > best)) { val = ov; best = oj; }
  }
  if (lane == 0) { cand_v[wave] = val; cand_j[wave] = best; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kWaves; ++w)
      if (cand_v[w] < val || (cand_v[w] == val && cand_j[w] > best)) { val = cand_v[w]; best = cand_j[w]; }
    float* o = a.amin + (slice * a.n_chunks + chunk) * 2;
    o[0] = val;
    o[1] = __int_as_float(best);
  }
}

// Step kernel 3: the row to evict over all chunks; it is deleted from the list and from the
// indicator (the later entries move down by one), its slot becomes the free one.
__global__ __launch_bounds__(kThreads) void step_evict_kernel(StepArgs a) {
  __shared__ int evict_lds;
  const int ll = blockIdx.y;
  const int b = blockIdx.x / a.h_kv, g = blockIdx.x % a.h_kv;
  const int64_t slice = ((int64_t)ll * a.batch + b) * a.h_kv + g;
  int32_t* st = in_global(a.state[ll]) + ((int64_t)b * a.h_kv + g) * 4;
  const int cur = st[0], cur1 = cur + 1, n = cur1 + a.window;
  const int cap = a.cap[ll];
  const int tid = threadIdx.x;
  int32_t* order = in_global(a.order[ll]) + ((int64_t)b * a.h_kv + g) * (cap + a.window + 1);
  float* ind = in_global(a.indicator[ll]) + ((int64_t)b * a.h_kv + g) * (cap + 1);
  if (tid == 0) {
    const int used = (cur1 + kThreads - 1) / kThreads;
    const float* p = a.amin + slice * a.n_chunks * 2;
    float val = p[0];
    int best = __float_as_int(p[1]);
    for (int c = 1; c < used; ++c) {
      const float v = p[2 * c];
      const int jj = __float_as_int(p[2 * c + 1]);
      if (v < val || (v == val && jj > best)) { val = v; best = jj; }
    }
    evict_lds = best;
  }
  __syncthreads();
  const int e = evict_lds;
  const int freed = order[e];
  if (tid == 0) order[n - 1] = st[1];                      // the generated token's slot ends the list
  __syncthreads();
  for (int base = e; base < n - 1; base += kThreads) {     // entries base+1.. move to base..: read all, then write
    const int jj = base + tid;
    const bool live = jj < n - 1;
    const int32_t o = live ? order[jj + 1] : 0;
    const float x = (live && jj + 1 < cur1) ? ind[jj + 1] : 0.f;
    __syncthreads();
    if (live) order[jj] = o;
    if (live && jj + 1 < cur1) ind[jj] = x;
    __syncthreads();
  }
  if (tid == 0) {
    st[1] = freed;
    st[2] = e;          // logical index of the evicted scored row (for inspection)
  }
}

}  // namespace
}  // namespace cake

using namespace cake;

namespace {

// Scratch of the entry point that may not take a workspace from its caller: the chunks'
// (reference, sum) pairs.  Every GPU the library runs on holds its own copy of this array until
// the process ends.  In host code the array's name is only a handle: its device address is
// looked up once per device and only that address is ever handed to a kernel.
constexpr size_t kStaticScratchBytes = size_t(1) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device.
int static_scratch(void** out) {
  int dev = -1;
  CAKE_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(CAKE_ERR_UNSUPPORTED, "device ordinal %d outside [0, %d)", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    CAKE_HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (ptr == nullptr) return fail(CAKE_ERR_HIP, "hipGetSymbolAddress returned a null address");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return CAKE_OK;
}

// Bytes of (reference, sum) pairs a call with this shape writes.
size_t decode_part_bytes(const cake_shape& shape) {
  const size_t n_chunks = ((size_t)shape.seq_len + kThreads - 1) / kThreads;
  return sizeof(float) * (size_t)shape.n_layers * shape.batch * shape.n_kv_heads * n_chunks * kMaxGroup * 2;
}

// Argument checks and the two launches; `part` is device memory of at least decode_part_bytes.
int decode_update_impl(const cake_shape* shape, const cake_params* params,
                       const void* const* q_new, const int64_t* q_strides,
                       const void* const* k_cache, const int64_t* k_strides,
                       const int32_t* cur_len, float* const* indicator,
                       float* part, void* stream) {
  if (int rc = check_shape_scores(shape)) return rc;
  CAKE_REQUIRE(params != nullptr, "params is NULL");
  CAKE_REQUIRE(q_new && k_cache && indicator && q_strides && k_strides && cur_len, "a pointer argument is NULL");
  CAKE_REQUIRE(params->pool_kernel >= 1 && params->pool_kernel % 2 == 1 && params->pool_kernel <= 129,
               "pool_kernel %d must be odd and within [1, 129]", params->pool_kernel);
  CAKE_REQUIRE(std::isfinite(params->scale) && params->scale >= 0.f, "scale must be finite and >= 0");
  const int B = shape->batch, L = shape->n_layers;
  const int G = shape->n_q_heads / shape->n_kv_heads;
  const int n_p = shape->seq_len - shape->window;
  const size_t eb = elem_bytes(shape->dtype);
  CAKE_REQUIRE(q_strides[0] >= 0 && q_strides[1] >= shape->head_dim && (q_strides[0] * eb) % 16 == 0 &&
                   (q_strides[1] * eb) % 16 == 0, "q_new strides must be multiples of 16 bytes, head stride >= head_dim");
  for (int i = 0; i < L * 3; ++i)
    CAKE_REQUIRE(k_strides[i] >= 0 && (k_strides[i] * eb) % 16 == 0, "k_cache strides must be non-negative multiples of 16 bytes");
  for (int i = 0; i < L * B; ++i)
    CAKE_REQUIRE(cur_len[i] >= 0 && cur_len[i] <= n_p, "cur_len[%d] = %d outside [0, seq_len - window = %d]", i, cur_len[i], n_p);
  const int n_chunks = (shape->seq_len + kThreads - 1) / kThreads;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const double scale = params->scale > 0.f ? (double)params->scale : 1.0 / std::sqrt((double)shape->head_dim);
  for (int l0 = 0; l0 < L;) {
    const int nl = launch_layers(L - l0, B);
    DecodeArgs a{};
    RaggedDims dims{};
    LayerStrides ks{};
    a.q_new = q_new + l0; a.k_cache = k_cache + l0; a.indicator = indicator + l0;
    a.qs[0] = q_strides[0]; a.qs[1] = q_strides[1];
    a.batch = B; a.h_kv = shape->n_kv_heads; a.group = G; a.window = shape->window; a.pool = params->pool_kernel;
    a.n_chunks = n_chunks;
    a.c = (float)(scale * 1.4426950408889634);
    a.inv_g = 1.0f / (float)G;
    a.part = part + (int64_t)l0 * B * shape->n_kv_heads * n_chunks * kMaxGroup * 2;
    int max_cur = 0;
    for (int ll = 0; ll < nl; ++ll) {
      int cc = 0;
      for (int b = 0; b < B; ++b) {
        dims.cur_len[ll * B + b] = cur_len[(l0 + ll) * B + b];
        cc = std::max(cc, cur_len[(l0 + ll) * B + b]);
      }
      a.cap_cur[ll] = cc;
      max_cur = std::max(max_cur, cc);
      for (int i = 0; i < 3; ++i) ks.s[ll][i] = k_strides[(l0 + ll) * 3 + i];
    }
    const int used = (max_cur + shape->window + kThreads - 1) / kThreads;
    dim3 grid(used, B * shape->n_kv_heads, nl), block(kThreads);
#define CAKE_DECODE(T, D)                                                                        \
  do {                                                                                           \
    hipLaunchKernelGGL((decode_partials_kernel<T, D>), grid, block, 0, st, a, dims, ks);         \
    hipLaunchKernelGGL((decode_apply_kernel<T, D>), grid, block, 0, st, a, dims, ks);            \
  } while (0)
    const bool bf = shape->dtype == CAKE_BF16;
    if (bf && shape->head_dim == 128) CAKE_DECODE(__bf16, 128);
    else if (bf && shape->head_dim == 64) CAKE_DECODE(__bf16, 64);
    else if (!bf && shape->head_dim == 128) CAKE_DECODE(float, 128);
    else if (!bf && shape->head_dim == 64) CAKE_DECODE(float, 64);
    else return fail(CAKE_ERR_UNSUPPORTED, "no decode kernel for this shape");
#undef CAKE_DECODE
    l0 += nl;
  }
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}

}  // namespace

extern "C" int cake_decode_update(const cake_shape* shape, const cake_params* params,
                                  const void* const* q_new, const int64_t* q_strides,
                                  const void* const* k_cache, const int64_t* k_strides,
                                  const int32_t* cur_len, float* const* indicator,
                                  void* workspace, size_t workspace_bytes, void* stream) {
  if (int rc = check_shape_scores(shape)) return rc;
  CAKE_REQUIRE(params != nullptr, "params is NULL");
  CAKE_REQUIRE(q_new && k_cache && indicator && q_strides && k_strides && cur_len, "a pointer argument is NULL");
  const ScoreLayout lay = score_layout(*shape);
  if (workspace == nullptr || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
    return fail(CAKE_ERR_WORKSPACE, "workspace is NULL or not 256-byte aligned");
  if (workspace_bytes < lay.total)
    return fail(CAKE_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes, lay.total);
  // the chunks' (reference, sum) pairs live where the score pass keeps its own partial pairs
  const size_t part_bytes = decode_part_bytes(*shape);
  if (lay.off_part + part_bytes > lay.total)
    return fail(CAKE_ERR_WORKSPACE, "workspace layout leaves %zu bytes for the decode partials, %zu needed",
                lay.total - lay.off_part, part_bytes);
  return decode_update_impl(shape, params, q_new, q_strides, k_cache, k_strides, cur_len, indicator,
                            reinterpret_cast<float*>(static_cast<char*>(workspace) + lay.off_part), stream);
}

extern "C" int cake_decode_update_static(const cake_shape* shape, const cake_params* params,
                                         const void* const* q_new, const int64_t* q_strides,
                                         const void* const* k_cache, const int64_t* k_strides,
                                         const int32_t* cur_len, float* const* indicator, void* stream) {
  if (int rc = check_shape_scores(shape)) return rc;
  CAKE_REQUIRE(params != nullptr, "params is NULL");
  CAKE_REQUIRE(q_new && k_cache && indicator && q_strides && k_strides && cur_len, "a pointer argument is NULL");
  const size_t part_bytes = decode_part_bytes(*shape);
  if (part_bytes > kStaticScratchBytes)
    return fail(CAKE_ERR_UNSUPPORTED,
                "cake_decode_update_static: n_layers*batch*n_kv_heads*ceil(seq_len/%d) = %zu chunk entries need %zu bytes, "
                "the built-in scratch holds %zu (use cake_decode_update with a workspace)",
                kThreads, part_bytes / (sizeof(float) * kMaxGroup * 2), part_bytes, kStaticScratchBytes);
  void* ptr = nullptr;
  if (int rc = static_scratch(&ptr)) return rc;
  return decode_update_impl(shape, params, q_new, q_strides, k_cache, k_strides, cur_len, indicator,
                            static_cast<float*>(ptr), stream);
}

extern "C" int cake_decode_step_workspace_bytes(const cake_shape* shape, size_t* bytes) {
  CAKE_REQUIRE(bytes != nullptr, "bytes is NULL");
  if (int rc = check_shape_scores(shape)) return rc;
  const size_t slices = (size_t)shape->n_layers * shape->batch * shape->n_kv_heads;
  const size_t n_chunks = ((size_t)shape->seq_len + kThreads - 1) / kThreads;
  *bytes = align_up(sizeof(float) * slices * align_up(shape->seq_len, 4) * kMaxGroup, 256) +
           align_up(sizeof(float) * slices * n_chunks * (kThreads / 64) * kMaxGroup * 2, 256) + align_up(sizeof(float) * slices * n_chunks * 2, 256);
  return CAKE_OK;
}

namespace {
// buffers: the tables' contents [n_layers] on the host, or NULL
int decode_step_impl(const cake_shape* shape, const cake_params* params,
                     const void* q_new, const int64_t* q_strides,
                     const void* k_new, const void* v_new, const int64_t* kv_new_strides,
                     void* const* k_slots, void* const* v_slots, const int64_t* slot_strides,
                     float* const* indicator, int32_t* const* order, int32_t* const* state,
                     const int32_t* cap, void* workspace, size_t workspace_bytes, const StepBuffers* buffers, void* stream) {
  if (int rc = check_shape_scores(shape)) return rc;
  CAKE_REQUIRE(params != nullptr, "params is NULL");
  CAKE_REQUIRE(q_new && k_new && v_new && k_slots && v_slots && indicator && order && state && q_strides && kv_new_strides &&
                   slot_strides && cap, "a pointer argument is NULL");
  CAKE_REQUIRE(params->pool_kernel >= 1 && params->pool_kernel % 2 == 1 && params->pool_kernel <= 129,
               "pool_kernel %d must be odd and within [1, 129]", params->pool_kernel);
  CAKE_REQUIRE(std::isfinite(params->scale) && params->scale >= 0.f, "scale must be finite and >= 0");
  const int B = shape->batch, L = shape->n_layers, G = shape->n_q_heads / shape->n_kv_heads;
  CAKE_REQUIRE(L <= kMaxLaunchLayers, "at most %d layers per cake_decode_step call", kMaxLaunchLayers);
  const size_t eb = elem_bytes(shape->dtype);
  for (int i = 0; i < 3; ++i) {
    CAKE_REQUIRE(q_strides[i] >= 0 && kv_new_strides[i] >= 0, "negative stride");
    CAKE_REQUIRE((q_strides[i] * eb) % 16 == 0 && (kv_new_strides[i] * eb) % 16 == 0, "strides must be multiples of 16 bytes");
  }
  for (int i = 0; i < 3 * L; ++i) {
    CAKE_REQUIRE(slot_strides[i] >= 0, "negative stride");
    CAKE_REQUIRE((slot_strides[i] * eb) % 16 == 0, "strides must be multiples of 16 bytes");
  }
  for (int l = 0; l < L; ++l)
    CAKE_REQUIRE(cap[l] >= 0 && cap[l] + shape->window + 1 <= shape->seq_len,
                 "cap[%d] = %d: cap + window + 1 must not exceed shape.seq_len = %d", l, cap[l], shape->seq_len);
  size_t need = 0;
  if (int rc = cake_decode_step_workspace_bytes(shape, &need)) return rc;
  if (workspace == nullptr || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
    return fail(CAKE_ERR_WORKSPACE, "workspace is NULL or not 256-byte aligned");
  if (workspace_bytes < need) return fail(CAKE_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes, need);

  StepArgs a{};
  a.q_new = q_new; a.k_new = k_new; a.v_new = v_new;
  a.k_slots = k_slots; a.v_slots = v_slots; a.indicator = indicator; a.order = order; a.state = state;
  for (int i = 0; i < 3; ++i) { a.qs[i] = q_strides[i]; a.ns[i] = kv_new_strides[i]; }
  for (int l = 0; l < L; ++l)
    for (int i = 0; i < 3; ++i) a.ss[l][i] = slot_strides[l * 3 + i];
  a.batch = B; a.h_kv = shape->n_kv_heads; a.group = G; a.window = shape->window; a.pool = params->pool_kernel;
  a.rows_max = (int32_t)align_up(shape->seq_len, 4);
  a.n_chunks = (shape->seq_len + kThreads - 1) / kThreads;
  const double scale = params->scale > 0.f ? (double)params->scale : 1.0 / std::sqrt((double)shape->head_dim);
  a.c = (float)(scale * 1.4426950408889634);
  a.inv_g = 1.0f / (float)G;
  const size_t slices = (size_t)L * B * shape->n_kv_heads;
  char* ws = static_cast<char*>(workspace);
  a.logits = reinterpret_cast<float*>(ws);
  ws += align_up(sizeof(float) * slices * a.rows_max * kMaxGroup, 256);
  a.part = reinterpret_cast<float*>(ws);
  ws += align_up(sizeof(float) * slices * a.n_chunks * (kThreads / 64) * kMaxGroup * 2, 256);
  a.amin = reinterpret_cast<float*>(ws);
  int cap_max = 0;
  for (int l = 0; l < L; ++l) { a.cap[l] = cap[l]; cap_max = std::max(cap_max, cap[l]); }
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int rows = cap_max + shape->window + 1;
  const dim3 grid((rows + kThreads - 1) / kThreads, B * shape->n_kv_heads, L), block(kThreads);
  // Where workgroups of 256 rows leave compute units idle, four of 64 rows in the place of each.
  const bool small = (int64_t)grid.x * grid.y * L <= 256 && rows <= kStepSmallRows;
  const dim3 logits_grid(small ? (rows + 63) / 64 : grid.x, grid.y, L), logits_block(small ? 64 : kThreads);
  if (small) a.n_chunks *= kThreads / 64;
  const dim3 slices_grid(B * shape->n_kv_heads, L);
  const bool bf = shape->dtype == CAKE_BF16;
  const bool whole = (int64_t)rows * shape->head_dim * eb <= kStepWholeBytes && rows <= kStepOneThreads;
  auto launch = [&](const auto& args) -> int {
    using Args = std::decay_t<decltype(args)>;
    if (whole) {
#define CAKE_WHOLE(T, D) (G <= 4 ? step_whole_kernel<T, D, 4, Args> : step_whole_kernel<T, D, kMaxGroup, Args>)
      const auto one = bf ? (shape->head_dim == 128 ? CAKE_WHOLE(__bf16, 128) : CAKE_WHOLE(__bf16, 64))
                          : (shape->head_dim == 128 ? CAKE_WHOLE(float, 128) : CAKE_WHOLE(float, 64));
#undef CAKE_WHOLE
      hipLaunchKernelGGL(one, slices_grid, dim3((rows + 63) / 64 * 64), 0, st, args);
      return CAKE_OK;
    }
#define CAKE_STEP(T, D)                                                                                               \
  (small ? step_logits_kernel<T, D, 1, Args> : step_logits_kernel<T, D, kThreads / 64, Args>)
    const auto logits = bf ? (shape->head_dim == 128 ? CAKE_STEP(__bf16, 128) : CAKE_STEP(__bf16, 64))
                           : (shape->head_dim == 128 ? CAKE_STEP(float, 128) : CAKE_STEP(float, 64));
#undef CAKE_STEP
    hipLaunchKernelGGL(logits, logits_grid, logits_block, 0, st, args);
    if (rows > kFinishRows) return CAKE_OK;
    const auto finish = G <= 4 ? (small ? step_finish_kernel<4, true, Args> : step_finish_kernel<4, false, Args>)
                               : (small ? step_finish_kernel<kMaxGroup, true, Args> : step_finish_kernel<kMaxGroup, false, Args>);
    hipLaunchKernelGGL(finish, slices_grid, dim3(kFinishThreads), 0, st, args);
    return CAKE_OK;
  };
  if (L == 1 && buffers != nullptr && rows <= kFinishRows) {
    StepOneArgs one{};
    static_cast<StepBase&>(one) = a;
    one.one = buffers[0];
    std::copy(a.ss[0], a.ss[0] + 3, one.ss[0]);
    one.cap[0] = a.cap[0];
    if (int rc = launch(one)) return rc;
  } else {
    if (int rc = launch(a)) return rc;
    if (rows > kFinishRows) {       // more than a workgroup's registers hold
      hipLaunchKernelGGL(step_apply_kernel, grid, block, 0, st, a);
      hipLaunchKernelGGL(step_evict_kernel, slices_grid, block, 0, st, a);
    }
  }
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}
}  // namespace

extern "C" int cake_decode_step(const cake_shape* shape, const cake_params* params,
                                const void* q_new, const int64_t* q_strides,
                                const void* k_new, const void* v_new, const int64_t* kv_new_strides,
                                void* const* k_slots, void* const* v_slots, const int64_t* slot_strides,
                                float* const* indicator, int32_t* const* order, int32_t* const* state,
                                const int32_t* cap, void* workspace, size_t workspace_bytes, void* stream) {
  return decode_step_impl(shape, params, q_new, q_strides, k_new, v_new, kv_new_strides, k_slots, v_slots, slot_strides,
                          indicator, order, state, cap, workspace, workspace_bytes, nullptr, stream);
}

extern "C" int cake_decode_run(const cake_decode_plan* p, const void* q_new, const int64_t* q_strides, const void* k_new,
                               const void* v_new, const int64_t* kv_new_strides, void* stream) {
  CAKE_REQUIRE(p != nullptr, "plan is NULL");
  return decode_step_impl(&p->shape, p->params, q_new, q_strides, k_new, v_new, kv_new_strides, p->k_slots, p->v_slots,
                          &p->slot_strides[0][0], p->indicator, p->order, p->state, p->cap, p->workspace, p->workspace_bytes,
                          p->buffers, stream);
}
