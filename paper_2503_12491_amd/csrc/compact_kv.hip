// cake_compact_kv: EVICT's gather (Sec. 4.3 Eq. 12, K_hat = K[D,:], V_hat = V[D,:]; Alg. 1
// cache and indicator update).  Pure data movement: every output row is one contiguous run
// of head_dim elements, copied as 16-byte pieces with consecutive lanes on consecutive pieces,
// so a 256-byte bf16 row is one coalesced access of 16 lanes.
#include <algorithm>
#include <cstdint>

#include "cake_internal.h"
#include "cake_pass.h"

namespace cake {
namespace {

constexpr int kThreads = 256;
constexpr int kUnroll = 4;   // pieces per thread

template <bool kPlanned>
struct CompactArgs {
  const void* const* k_in;
  const void* const* v_in;
  const int32_t* const* idx;
  const float* const* ind_in;
  void* const* k_out;
  void* const* v_out;
  float* const* ind_out;
  const int32_t* const* pos_in;          // prompt positions of the rows that come in; NULL entry: row r is position r
  int32_t* const* pos_out;               // NULL: not carried along
  int32_t batch, h_kv, window, pieces;   // pieces: 16-byte pieces per row
  int32_t elem_bytes;
  CapsArg<kPlanned> cap;
};

// The same dimensions when they live in device memory (an eviction plan); the strides are then
// the same for every layer.
struct CompactPlan {
  const int32_t* cur_len;     // [L*B]
  const int32_t* keep;        // [L*B]
  const int32_t* cap_cur;     // [L]
  const int32_t* cap_keep;    // [L]
  const int32_t* copy_blocks; // [L*B + 1] running block counts (the work list)
  int32_t n_entries;          // L*B
  int64_t s[3];               // strides of the layers that come as the caller laid them out
  // Bit l set: layer l's K and V are themselves outputs of an earlier planned compaction,
  // contiguous [B, H_kv, cap_cur[l] + S_w, d]; their strides follow from the plan.
  uint32_t compacted[kPlanMaskWords];
};
static_assert(kThreads * kUnroll == kCopyBlockPieces, "a workgroup step is one block of the plan's work list");
constexpr int kListLds = 4096;       // work-list entries searched from LDS (longer lists are searched in memory)
constexpr int kListWave = 64;        // entries that a wave holds, one a lane
constexpr int kHostWaves = 3;        // waves a SIMD, at most, where the counts come from the host

// A table's address, the same in all lanes: in scalar registers, where it takes no vector ones.
template <typename T>
__device__ __forceinline__ T* uniform_global(T* p) {
  const uint64_t x = reinterpret_cast<uintptr_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x), hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
  return in_global(reinterpret_cast<T*>((uint64_t)hi << 32 | lo));
}

// A workgroup moves kThreads*kUnroll pieces of one (layer, sequence, head) slice per step.
// Launches that know the row counts on the host give every slice the blocks it needs.  Planned
// launches (counts known only on the device) run a fixed number of workgroups that stride over
// the plan's work list, the blocks of all (layer, sequence) entries in one sequence, head by
// blockIdx.y: the entry of a block is found by counting, in a wave's lanes, the running counts not above it, or
// in a long list by bisection.
//
// Large calls are bound by the bytes of the rows (5 TB/s), small ones by the chain of loads that leads to them: list, counts and
// addresses, index, row.  A block's index loads go out together and its row loads behind them, without a branch about either (in
// branches each of the four waited for the rows of the one before), the indicator's entries beside the rows instead of behind
// their stores; the work list of a small plan is searched without LDS and its barrier, and a call that knows how long the list can
// be brings no more workgroups.  Us of the kernel before that and now, with inputs in the caches and flushed out of them: planned, 2 layers of
// 1024 keys 5.9, 4.8 (7.0, 4.9); 2 of 4000 8.0, 4.9 (11.1, 6.8); 8 of 2000 11.4, 7.6 (13.0, 9.7); 32 of 8192, 1024 rows kept, 57.6, 50.2
// (85.1, 84.2).  Counts from the host: 4 layers of 4000 keys, 400 rows kept, 7.0, 5.3 (10.4, 8.4); 32 of 32768, 1048 rows, 48.4, 47.8 (87.8, 84.9).
// Addresses lie in scalar registers and offsets are made where they are used: 61 and 44 vector registers (with both in vector registers 72 and 88, and the
// index loads one by one behind a test for an empty list).  More waves do not copy faster: the gathers of three sessions (21 layers of 3782
// keys of 4 fp32 heads, 19 of 3119 and 16 of 6007 keys of 8 bf16 heads) take 2.61 ms at 8 waves a SIMD, 2.51 at 5, 2.49 at 4, 2.45 at 3 (before,
// with 88 registers and 5 waves, 2.58; before the grouped loads, with 8, 2.82), the eviction of 32 layers of 32768 keys 47.8, 47.0, 46.8 and
// 47.3 us; of the planned form 5 to 7 waves make no difference.
template <bool kPlanned>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, kPlanned ? 8 : kHostWaves))) void compact_kernel(CompactArgs<kPlanned> a, DimsArg<kPlanned> dims, StridesArg<kPlanned> st,
                                                          typename std::conditional<kPlanned, CompactPlan, NoArgs>::type plan) {
  __shared__ int32_t list[kPlanned ? kListLds + 1 : 1];
  const int32_t* blocks = nullptr;
  int32_t n_blocks = 0, begins = 0;
  if constexpr (kPlanned) {
    blocks = plan.copy_blocks;
    if (plan.n_entries <= kListWave) {
      const int e = threadIdx.x & 63;
      begins = e < plan.n_entries ? plan.copy_blocks[e] : 0x7fffffff;
    } else if (plan.n_entries <= kListLds) {
      for (int i = threadIdx.x; i <= plan.n_entries; i += kThreads) list[i] = plan.copy_blocks[i];
      __syncthreads();
      blocks = list;
    }
    n_blocks = blocks[plan.n_entries];
  }
  auto step = [&](int32_t blk) {
  int ll, b, h;
  int64_t first;
  if constexpr (kPlanned) {
    int lo = 0, hi = plan.n_entries;          // largest e with blocks[e] <= blk (entries without blocks share a count)
    if (hi <= kListWave) {
      lo = __popcll(__ballot(begins <= blk)) - 1;                 // the counts ascend, from 0
    } else {
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (blocks[mid] <= blk) lo = mid; else hi = mid;
      }
      lo = __builtin_amdgcn_readfirstlane(lo);
    }
    ll = lo / a.batch; b = lo % a.batch; h = blockIdx.y;
    first = (int64_t)(blk - blocks[lo]) * (kThreads * kUnroll);
  } else {
    ll = blockIdx.z; b = blockIdx.y / a.h_kv; h = blockIdx.y % a.h_kv;
    first = (int64_t)blockIdx.x * (kThreads * kUnroll);
  }
  int cur, keep, cap_cur, cap_keep;
  int64_t s0, s1, s2;
  if constexpr (kPlanned) {
    cur = plan.cur_len[ll * a.batch + b];
    keep = plan.keep[ll * a.batch + b];
    cap_cur = plan.cap_cur[ll];
    cap_keep = plan.cap_keep[ll];
    s0 = plan.s[0]; s1 = plan.s[1]; s2 = plan.s[2];
    if (plan.compacted[ll >> 5] >> (ll & 31) & 1u) {
      s2 = (int64_t)a.pieces * 16 / a.elem_bytes;
      s1 = (int64_t)(cap_cur + a.window) * s2;
      s0 = (int64_t)a.h_kv * s1;
    }
  } else {
    cur = dims.cur_len[ll * a.batch + b];
    keep = dims.keep[ll * a.batch + b];
    cap_cur = a.cap.cur[ll];
    cap_keep = a.cap.keep[ll];
    s0 = st.s[ll][0]; s1 = st.s[ll][1]; s2 = st.s[ll][2];
  }
  const int rows_out = keep + a.window;
  const int64_t total = (int64_t)rows_out * a.pieces;

  const int64_t in_off = (b * s0 + h * s1) * a.elem_bytes;
  const int64_t in_row = s2 * a.elem_bytes;
  const int64_t out_row = (int64_t)a.pieces * 16;
  const int64_t out_off = ((int64_t)b * a.h_kv + h) * (cap_keep + a.window) * out_row;
  const char* kin = uniform_global(static_cast<const char*>(a.k_in[ll])) + in_off;
  const char* vin = uniform_global(static_cast<const char*>(a.v_in[ll])) + in_off;
  char* kout = uniform_global(static_cast<char*>(a.k_out[ll])) + out_off;
  char* vout = uniform_global(static_cast<char*>(a.v_out[ll])) + out_off;
  const int32_t* idx = uniform_global(a.idx[ll]) + ((int64_t)b * a.h_kv + h) * cap_keep;

  if (first >= total) return;
  // Indicator entries of the retained prefix rows and, where the caller tracks them, their positions in
  // the prompt: composing the positions here takes the kernel no measurable time, a gather of its own
  // per layer and stage took a session of 16 layers of 6K keys two launches each.  A row split between two blocks is
  // written by the block that holds its piece 0.
  const bool entries = a.ind_in != nullptr, positions = a.pos_out != nullptr;
  const int64_t head = (int64_t)b * a.h_kv + h;
  const float* iin = nullptr;
  float* iout = nullptr;
  const int32_t* pin = nullptr;
  int32_t* pout = nullptr;
  if (entries) {
    iin = uniform_global(a.ind_in[ll]) + head * cap_cur;
    iout = uniform_global(a.ind_out[ll]) + head * cap_keep;
    if (positions) {
      if (a.pos_in[ll] != nullptr) pin = uniform_global(a.pos_in[ll]) + head * cap_cur;
      pout = uniform_global(a.pos_out[ll]) + head * cap_keep;
    }
  }
  const int64_t row0 = first / a.pieces;                               // of the block's first piece
  const uint32_t piece0 = (uint32_t)(first - row0 * a.pieces), pieces = (uint32_t)a.pieces;
  uint32_t tid = threadIdx.x;
  if (kPlanned) asm volatile("" : "+v"(tid));                            // what follows from it is made anew each turn, not kept in registers
  const int r_first = (int)row0 + (piece0 > 0 ? 1 : 0);                 // rows that begin in the block
  const int r_end = (int)min((first + kThreads * kUnroll + a.pieces - 1) / a.pieces, (int64_t)keep);
  const uint32_t here = (uint32_t)min(total - first, (int64_t)(kThreads * kUnroll));      // pieces of the block
  // The row that the list has at place r, or any where there is no list.  Pieces past the end repeat the last one, and every thread
  // reads an entry: with no branch about them the loads of a block are in flight together, the indexes first and then the rows.
  const int32_t* list_of_rows = keep > 0 ? idx : reinterpret_cast<const int32_t*>(kin);
  auto chosen = [&](int r) { return min(max(list_of_rows[max(min(r, keep - 1), 0)], 0), max(cur - 1, 0)); };
  const int own = r_first + (int)tid;
  const int own_src = chosen(own);
  int64_t src[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const uint32_t q = piece0 + min(u * kThreads + tid, here - 1), down = q / pieces, piece = q - down * pieces;
    const int r = (int)row0 + (int)down;
    // selected prefix rows first, then the window rows that follow the cur prefix rows
    const int from = chosen(r);
    src[u] = (int64_t)(r < keep ? from : cur + (r - keep)) * in_row + piece * 16;
  }
  const float own_ind = (entries && keep > 0 ? iin : reinterpret_cast<const float*>(kin))[own_src];
  int own_pos = own_src;
  if (pin != nullptr && keep > 0) own_pos = pin[own_src];
  uint4 kv[kUnroll], vv[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    kv[u] = *reinterpret_cast<const uint4*>(kin + src[u]);
    vv[u] = *reinterpret_cast<const uint4*>(vin + src[u]);
  }
  if (entries && own < r_end) {
    iout[own] = own_ind;
    if (pout != nullptr) pout[own] = own_pos;
  }
  // Streaming stores: the compacted rows are not read again by this pass, and plain stores were
  // measured to cost twice their bytes in memory writes (the rows pass through the cache first).
  char* kto = kout + first * 16;
  char* vto = vout + first * 16;
#pragma unroll
  for (int u = 0; u < kUnroll; ++u)
    if (u * kThreads + tid < here) {
      store_streaming(kto + (u * kThreads + tid) * 16, kv[u]);
      store_streaming(vto + (u * kThreads + tid) * 16, vv[u]);
    }
  if (entries)                                                        // a block of more rows than threads: rows of fewer than five pieces
    for (int r = own + kThreads; r < r_end; r += kThreads) {
      const int from = chosen(r);
      iout[r] = iin[from];
      if (pout != nullptr) pout[r] = pin != nullptr ? pin[from] : from;
    }
  };
  if constexpr (kPlanned) {
    for (int32_t blk = blockIdx.x; blk < n_blocks; blk += gridDim.x) step(blk);
  } else {
    step(blockIdx.x);                        // no loop: one of a single turn kept the offsets of its parts in 14 registers
  }
}

}  // namespace
}  // namespace cake

int cake::launch_compact_planned(const cake_shape* shape, const void* const* k_in, const void* const* v_in,
                                 const int64_t* kv_strides, const uint8_t* compacted, const float* const* ind_in,
                                 const PlanView& plan, int64_t most_rows, hipStream_t stream) {
  const int eb = (int)elem_bytes(shape->dtype);
  CompactArgs<true> a{};
  a.k_in = k_in; a.v_in = v_in;
  a.idx = reinterpret_cast<const int32_t* const*>(plan.idx);
  a.ind_in = ind_in;
  a.k_out = plan.k_out; a.v_out = plan.v_out;
  a.ind_out = ind_in ? reinterpret_cast<float* const*>(plan.ind_out) : nullptr;
  a.batch = shape->batch; a.h_kv = shape->n_kv_heads; a.window = shape->window;
  a.pieces = shape->head_dim * eb / 16;
  a.elem_bytes = eb;
  CompactPlan cp{plan.cur_len, plan.keep, plan.cap_cur, plan.cap_keep, plan.copy_blocks, shape->n_layers * shape->batch,
                 {kv_strides[0], kv_strides[1], kv_strides[2]}, {}};
  if (compacted != nullptr)
    for (int l = 0; l < shape->n_layers; ++l)
      if (compacted[l]) cp.compacted[l >> 5] |= 1u << (l & 31);
  // 8192 workgroups in all (a few rounds of what the chip holds at once), striding over the work list, or as many as the list
  // can be long
  const int64_t entries = (int64_t)shape->n_layers * shape->batch;
  const int64_t longest = most_rows > 0 ? most_rows * shape->batch * a.pieces / kCopyBlockPieces + entries : INT32_MAX;
  const unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>(8192 / shape->n_kv_heads, longest));
  hipLaunchKernelGGL(compact_kernel<true>, dim3(gx, shape->n_kv_heads), dim3(kThreads), 0,
                     stream, a, NoArgs{}, NoArgs{}, cp);
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}

using namespace cake;

extern "C" int cake_compact_kv(const cake_shape* shape,
                               const void* const* k_in, const void* const* v_in, const int64_t* kv_strides,
                               const int32_t* cur_len, const int32_t* k, const int32_t* const* idx,
                               const float* const* ind_in,
                               void* const* k_out, void* const* v_out, float* const* ind_out,
                               void* stream) {
  return cake_compact_kv_positions(shape, k_in, v_in, kv_strides, cur_len, k, idx, ind_in, k_out, v_out, ind_out, nullptr, nullptr,
                                   stream);
}

extern "C" int cake_compact_kv_positions(const cake_shape* shape,
                                         const void* const* k_in, const void* const* v_in, const int64_t* kv_strides,
                                         const int32_t* cur_len, const int32_t* k, const int32_t* const* idx,
                                         const float* const* ind_in,
                                         void* const* k_out, void* const* v_out, float* const* ind_out,
                                         const int32_t* const* pos_in, int32_t* const* pos_out, void* stream) {
  if (int rc = check_shape_basic(shape)) return rc;
  CAKE_REQUIRE(k_in && v_in && kv_strides && cur_len && k && idx && k_out && v_out, "a required pointer is NULL");
  CAKE_REQUIRE((ind_in == nullptr) == (ind_out == nullptr), "ind_in and ind_out must both be given or both be NULL");
  CAKE_REQUIRE((pos_in == nullptr) == (pos_out == nullptr) && (pos_out == nullptr || ind_out != nullptr),
               "pos_in and pos_out must both be given, beside the indicators, or both be NULL");
  const int B = shape->batch, L = shape->n_layers;
  const int eb = (int)elem_bytes(shape->dtype);
  for (int i = 0; i < L * B; ++i) {
    CAKE_REQUIRE(cur_len[i] >= 0, "cur_len[%d] = %d is negative", i, cur_len[i]);
    CAKE_REQUIRE(k[i] >= 0 && k[i] <= cur_len[i], "k[%d] = %d outside [0, cur_len = %d]", i, k[i], cur_len[i]);
    CAKE_REQUIRE(k[i] == 0 || cur_len[i] > 0, "k > 0 with an empty prefix");
  }
  for (int l = 0; l < L; ++l)
    for (int j = 0; j < 3; ++j) {
      CAKE_REQUIRE(kv_strides[l * 3 + j] >= 0, "negative stride");
      CAKE_REQUIRE((kv_strides[l * 3 + j] * eb) % 16 == 0, "strides must be multiples of 16 bytes");
    }
  hipStream_t st = static_cast<hipStream_t>(stream);
  for (int l0 = 0; l0 < L;) {
    const int nl = launch_layers(L - l0, B);
    CompactArgs<false> a{};
    RaggedDims dims{};
    LayerStrides ls{};
    a.k_in = k_in + l0; a.v_in = v_in + l0; a.idx = idx + l0;
    a.ind_in = ind_in ? ind_in + l0 : nullptr;
    a.k_out = k_out + l0; a.v_out = v_out + l0;
    a.ind_out = ind_out ? ind_out + l0 : nullptr;
    a.pos_in = pos_in ? pos_in + l0 : nullptr;
    a.pos_out = pos_out ? pos_out + l0 : nullptr;
    a.batch = B; a.h_kv = shape->n_kv_heads; a.window = shape->window;
    a.pieces = shape->head_dim * eb / 16;
    a.elem_bytes = eb;
    int max_rows = 0;
    for (int ll = 0; ll < nl; ++ll) {
      int cc = 0, ck = 0;
      for (int b = 0; b < B; ++b) {
        const int i = (l0 + ll) * B + b;
        dims.cur_len[ll * B + b] = cur_len[i];
        dims.keep[ll * B + b] = k[i];
        cc = std::max(cc, cur_len[i]);
        ck = std::max(ck, k[i]);
      }
      a.cap.cur[ll] = cc;
      a.cap.keep[ll] = ck;
      max_rows = std::max(max_rows, ck + shape->window);
      for (int j = 0; j < 3; ++j) ls.s[ll][j] = kv_strides[(l0 + ll) * 3 + j];
    }
    const int64_t pieces_total = (int64_t)max_rows * a.pieces;
    const unsigned gx = (unsigned)((pieces_total + kThreads * kUnroll - 1) / (kThreads * kUnroll));
    hipLaunchKernelGGL(compact_kernel<false>, dim3(gx, B * shape->n_kv_heads, nl), dim3(kThreads), 0, st, a, dims, ls, NoArgs{});
    l0 += nl;
  }
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}
