// cake_select_topk: per-head top-k of the eviction indicator (Sec. 4.3 Eq. 12).
//
// One workgroup per (layer, sequence, KV head) row, on order-preserving 32-bit keys.  A row of up to
// 65536 entries is read once into registers, a longer one in two sweeps: the first counts its leading
// digits, the second keeps the entries at or above the digit that holds the k-th largest (a few
// thousand of 128K) as an ordered list in LDS, which then takes the row's place.
//
// The k-th largest key is found by counting the keys over 2048 equal intervals of their range, then
// over the interval that holds it, until at most kFewKeys are left, which are ranked against each
// other.  One round and the ranking do for nearly every row: the intervals come from the row's own
// smallest and largest key, so they part the entries far better than leading key bits would (a pooled
// indicator spans some 25 binary exponents).  The ordered output writes, in ascending position, every
// entry above the threshold and the first `need` entries equal to it: the total order (value
// descending, position ascending).
//
// What bounds it is latency, a chain of barriers and LDS round trips: 992 entries 19 -> 5.0 us, 1024
// rows of 4061 89 -> 13 us, 256 rows of 32736 38 -> 21 us and of 131008 106 -> 71 us (where reading the
// row twice at the 35 bytes/ns a compute unit gets is most of it), against four sweeps of the row with a
// one-wave search of every histogram.
#include <algorithm>
#include <type_traits>

#include "cake_internal.h"

namespace cake {
namespace {

constexpr int kBins = 2048;
constexpr int kCopies = 2;          // histogram copies, chosen by lane: fewer lanes meet on one LDS address
constexpr int kFewKeys = 128;       // keys ranked by comparison with each other
constexpr int kMaxWaves = 16;

template <bool kPlanned>
struct TopkArgs {
  const float* const* indicator;
  const float* last;          // of the last layer; NULL: in the table as well
  int32_t* const* idx;
  int32_t batch, h_kv;
  CapsArg<kPlanned> cap;
};
// The same dimensions when they live in device memory (an eviction plan).
struct TopkPlan {
  const int32_t* cur_len;     // [L*B]
  const int32_t* keep;        // [L*B]
  const int32_t* cap_cur;     // [L]
  const int32_t* cap_keep;    // [L]
  int32_t n_layers;
  PlanMirror mirror;          // where its host is not NULL, row n_layers of the grid writes it
  int32_t served_slots;       // the kernel for any length leaves rows of up to so many slots to the register kernel launched before it
};

// Larger float <=> larger key.  -0 is folded onto +0 first so that they compare equal.  Key 0 stands for
// an absent entry: the one NaN whose key it would be (all bits set) shares key 1 with its neighbour.
__device__ __forceinline__ uint32_t order_key(float x) {
  uint32_t u = __float_as_uint(x + 0.0f);
  return (u & 0x80000000u) ? max(~u, 1u) : (u | 0x80000000u);
}

// LDS of one workgroup's selection.
struct SelectLds {
  uint32_t hist[kBins * kCopies];               // [interval][copy]
  uint32_t few[kFewKeys];
  int32_t few_pos[kFewKeys];
  uint32_t wave_a[kMaxWaves], wave_b[kMaxWaves], wave_sel[2][kMaxWaves];
  uint32_t bin, above, count, n_few, thr;
  int32_t last;
};

// A row seen as slots of four entries whose addresses are 16-byte aligned: slot s holds
// positions 4s - pad .. 4s - pad + 3, pad in 0..3 chosen from the row's address.  Positions
// outside [0, cur) are absent: key 0, below every key of a number.  Slots full_lo .. full_hi exist
// whole; the first and the last may not, their keys are made from single entries.
struct Row {
  const float* base;
  int cur, pad, n_slots, full_lo, full_hi;
  __device__ __forceinline__ void init(const float* row, int cur_) {
    base = row;
    cur = cur_;
    pad = (int)((reinterpret_cast<uintptr_t>(row) >> 2) & 3);
    n_slots = (cur + pad + 3) >> 2;
    full_lo = pad ? 1 : 0;
    full_hi = ((cur + pad) >> 2) - 1;
  }
  // Keys of the slots slot(0), slot(1), .., the first n_u of them (the others' are 0).  The loads are
  // unconditional (a slot that does not exist whole repeats one that does), so that all of them are
  // in flight before the first is waited for.
  template <int kSlots, typename Slot>
  __device__ __forceinline__ void load(int n_u, Slot slot, uint32_t (&key)[kSlots][4]) const {
    float4 x[kSlots];
    if (full_lo <= full_hi) {
#pragma unroll
      for (int u = 0; u < kSlots; ++u)
        if (u < n_u) x[u] = *reinterpret_cast<const float4*>(base + (4 * min(max(slot(u), full_lo), full_hi) - pad));
    }
    uint32_t first[4], last[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int p = j - pad, q = 4 * (n_slots - 1) - pad + j;
      const float f = base[min(max(p, 0), cur - 1)], l = base[min(max(q, 0), cur - 1)];
      first[j] = p >= 0 && p < cur ? order_key(f) : 0u;
      last[j] = q >= 0 && q < cur ? order_key(l) : 0u;
    }
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      const int s = slot(u);
      const bool whole = u < n_u && s >= full_lo && s <= full_hi;
      key[u][0] = whole ? order_key(x[u].x) : 0u;
      key[u][1] = whole ? order_key(x[u].y) : 0u;
      key[u][2] = whole ? order_key(x[u].z) : 0u;
      key[u][3] = whole ? order_key(x[u].w) : 0u;
      if (u < n_u && !whole && s == n_slots - 1) { key[u][0] = last[0]; key[u][1] = last[1]; key[u][2] = last[2]; key[u][3] = last[3]; }
      if (u < n_u && !whole && s == 0) { key[u][0] = first[0]; key[u][1] = first[1]; key[u][2] = first[2]; key[u][3] = first[3]; }
    }
  }
};

// What was computed from the keys so far is not kept for later: an interval or a ballot is cheaper
// made again than held in registers across a barrier (without this the kernels spill).
template <int kSlots>
__device__ __forceinline__ void forget(uint32_t (&key)[kSlots][4]) {
#pragma unroll
  for (int u = 0; u < kSlots; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(key[u][j]));
}

// The interval of the finished histogram that holds the need-th key from the top: s.bin, the keys above
// it, its own.  Thread t owns the kPer intervals below kBins - kPer*t; a scan over the threads counts
// from the top down.
template <int kThreads>
__device__ __forceinline__ void find_interval(uint32_t need, SelectLds& s) {
  constexpr int kWaves = kThreads / 64, kPer = kBins / kThreads;
  static_assert(kCopies == 2, "the copies of an interval are read as one 8-byte word");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int top = kBins - 1 - kPer * tid;
  uint32_t c[kPer], sum = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint2 x = *reinterpret_cast<const uint2*>(&s.hist[(top - j) * kCopies]);
    c[j] = x.x + x.y;
    sum += c[j];
  }
  uint32_t incl = wave_scan(sum, [](uint32_t a, uint32_t b) { return a + b; });
  if (lane == 63) s.wave_a[wave] = incl;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w)
    if (w < wave) incl += s.wave_a[w];
  uint32_t above = incl - sum;
  if (above < need && need <= incl) {          // exactly one thread
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      if (above < need && need <= above + c[j]) { s.bin = top - j; s.above = above; s.count = c[j]; }
      above += c[j];
    }
  }
  __syncthreads();
}

struct LeaveOut {
  __device__ __forceinline__ void operator()(uint32_t, int, int) const {}
  __device__ __forceinline__ void operator()(int) const {}
};

// The keys that satisfy `pick`, in order: store(rank, u, j); the others: other(how many picked ones come before, u, j); ahead
// of group u's: begin(u).  Wave w holds a contiguous run of groups,
// group u of it in the lanes' slots u.  `before` counts the keys of earlier calls; a call alternates
// between two sets of wave totals, so that one barrier per call is enough.
template <int kThreads, int kSlots, typename Pick, typename Store, typename Other = LeaveOut, typename Begin = LeaveOut>
__device__ __forceinline__ void write_picked(uint32_t (&key)[kSlots][4], int n_u, Pick pick, uint32_t (&wave_sel)[kMaxWaves],
                                             uint32_t& before, Store store, Other other = LeaveOut{}, Begin begin = LeaveOut{}) {
  constexpr int kWaves = kThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t n = 0;
#pragma unroll
  for (int u = 0; u < kSlots; ++u)
    if (u < n_u)
#pragma unroll
      for (int j = 0; j < 4; ++j) n += __popcll(__ballot(pick(key[u][j], u, j)));
  if (lane == 0) wave_sel[wave] = n;
  __syncthreads();
  n = before;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t c = wave_sel[w];
    before += c;
    if (w < wave) n += c;
  }
  forget(key);
#pragma unroll
  for (int u = 0; u < kSlots; ++u) {
    if (u >= n_u) continue;
    begin(u);
    uint32_t rank = n;
    bool p[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      p[j] = pick(key[u][j], u, j);
      const uint64_t ballot = __ballot(p[j]);
      rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, rank));
      n += __popcll(ballot);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (p[j]) store(rank, u, j);
      else other(rank, u, j);
      rank += p[j] ? 1u : 0u;
    }
  }
}

// Threshold of the k largest of the workgroup's keys under (key descending, position ascending): every
// key above `thr`, and those equal to it at positions up to `last`.  Each thread brings kSlots groups of
// four keys, of which the first n_u (the same for the whole workgroup) are filled; absent entries are 0.
// They share the lowest interval with the smallest keys, where they change nothing: at least k real
// keys lie at or above every threshold.
template <int kThreads, int kSlots, typename Position>
__device__ __forceinline__ void find_threshold(uint32_t (&key)[kSlots][4], int n_u, uint32_t k, Position position, SelectLds& s,
                                               uint32_t& thr, int& last) {
  constexpr int kWaves = kThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, copy = lane & (kCopies - 1);
  uint32_t kmax = 0, kmin1 = 0xffffffffu;        // kmin1: smallest key minus one (an absent 0 wraps to the top)
#pragma unroll
  for (int u = 0; u < kSlots; ++u)
    if (u < n_u)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        kmax = max(kmax, key[u][j]);
        kmin1 = min(kmin1, key[u][j] - 1u);
      }
  auto umax = [](uint32_t a, uint32_t b) { return max(a, b); };
  kmax = wave_scan(kmax, umax);
  kmin1 = ~wave_scan(~kmin1, umax);
  if (lane == 63) { s.wave_a[wave] = kmax; s.wave_b[wave] = kmin1; }
  if (tid == 0) s.n_few = 0;
  if (tid < kFewKeys) s.few[tid] = 0u;           // equal to no key and above none
  for (int i = tid; i < kBins * kCopies / 4; i += kThreads) reinterpret_cast<uint4*>(s.hist)[i] = uint4{0, 0, 0, 0};
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) { kmax = max(kmax, s.wave_a[w]); kmin1 = min(kmin1, s.wave_b[w]); }
  forget(key);
  uint32_t lo = kmin1 + 1u, need = k;            // the interval at hand starts at lo
  int bits = 32 - __clz((int)(kmax - lo));       // and is 2^bits wide (bits = 32: all there is)
  // Neighbouring entries of a pooled indicator are mostly equal: a slot whose four entries fall
  // into one interval takes one update instead of four.
  auto count_slot = [&](const uint32_t (&d)[4], bool all) {
    if (d[0] == d[1] && d[1] == d[2] && d[2] == d[3]) {
      if (all || d[0] < kBins) atomicAdd(&s.hist[d[0] * kCopies + copy], 4u);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (all || d[j] < kBins) atomicAdd(&s.hist[d[j] * kCopies + copy], 1u);
    }
  };
  int shift = max(bits - 11, 0);
#pragma unroll
  for (int u = 0; u < kSlots; ++u)
    if (u < n_u) {                               // first round: every key lies in [lo, lo + 2^bits) or is absent
      uint32_t d[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) d[j] = (max(key[u][j], lo) - lo) >> shift;
      count_slot(d, true);
    }
  for (;;) {
    __syncthreads();
    find_interval<kThreads>(need, s);
    forget(key);
    lo += s.bin << shift;
    need -= s.above;
    bits = shift;
    if (bits == 0 || s.count <= kFewKeys) break;
    for (int i = tid; i < kBins * kCopies / 4; i += kThreads) reinterpret_cast<uint4*>(s.hist)[i] = uint4{0, 0, 0, 0};
    __syncthreads();
    shift = max(bits - 11, 0);
#pragma unroll
    for (int u = 0; u < kSlots; ++u)
      if (u < n_u) {
        uint32_t d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t v = key[u][j] - lo;
          // (an interval that holds the largest key may reach past 2^32, to where an absent key's difference wraps)
          d[j] = v >> bits == 0 && key[u][j] != 0u ? v >> shift : kBins;
        }
        count_slot(d, false);
      }
  }
  if (s.count <= kFewKeys) {
    const uint32_t width_1 = (bits < 32 ? 1u << bits : 0u) - 1u;
#pragma unroll
    for (int u = 0; u < kSlots; ++u)
      if (u < n_u)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (key[u][j] - lo <= width_1 && key[u][j] != 0u) {
            const uint32_t i = atomicAdd(&s.n_few, 1u);
            s.few[i] = key[u][j];
            s.few_pos[i] = position(u, j);
          }
    __syncthreads();
    const int n = (int)s.n_few;
    if (tid < n) {
      const uint32_t x = s.few[tid];
      const int px = s.few_pos[tid];
      uint32_t gt = 0, eq_before = 0;
      for (int i = 0; i < n; i += 8) {
        uint32_t y[8];
        int p[8];
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          const uint4 a = *reinterpret_cast<const uint4*>(&s.few[i + 4 * v]);
          const int4 b = *reinterpret_cast<const int4*>(&s.few_pos[i + 4 * v]);
          y[4 * v] = a.x; y[4 * v + 1] = a.y; y[4 * v + 2] = a.z; y[4 * v + 3] = a.w;
          p[4 * v] = b.x; p[4 * v + 1] = b.y; p[4 * v + 2] = b.z; p[4 * v + 3] = b.w;
        }
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          gt += y[v] > x ? 1u : 0u;
          eq_before += y[v] == x && p[v] < px ? 1u : 0u;
        }
      }
      if (gt + eq_before + 1 == need) { s.thr = x; s.last = px; }
    }
    __syncthreads();
    thr = s.thr;
    last = s.last;
    return;
  }
  // The key is known to the last bit and more entries equal it than are ranked: the need-th of them in order.
  thr = lo;
  uint32_t before = 0;
  write_picked<kThreads, kSlots>(key, n_u, [&](uint32_t x, int, int) { return x == lo; }, s.wave_sel[0], before,
                                 [&](uint32_t rank, int u, int j) { if (rank + 1 == need) s.last = position(u, j); });
  __syncthreads();
  last = s.last;
}

// The host's copy of the plan, by the last row's first workgroup of a launch: plain stores over the bus, then one flag
// once they are all out, so that a host that watches the flag knows the plan while the top-k and the compaction are
// still running.  The plan's own kernel would wait for the bus before the top-k may begin (1.5 us).
template <int kThreads>
__device__ __forceinline__ void write_mirror(const PlanMirror& a) {
  if (blockIdx.x > 0) return;
  const PlanMirrorLayout lay = plan_mirror_layout(a.n_layers, a.batch);
  char* h = static_cast<char*>(a.host);
  const int n = a.n_layers * a.batch, tid = threadIdx.x;
  for (int i = tid; i < n; i += kThreads) {
    reinterpret_cast<int32_t*>(h + lay.off_budgets)[i] = a.budgets[i];
    reinterpret_cast<int32_t*>(h + lay.off_keep)[i] = a.keep[i];
    reinterpret_cast<double*>(h + lay.off_pref)[i] = a.pref[i];
    if (a.hv != nullptr) {
      reinterpret_cast<double*>(h + lay.off_hv)[2 * i] = a.hv[2 * i];
      reinterpret_cast<double*>(h + lay.off_hv)[2 * i + 1] = a.hv[2 * i + 1];
    }
  }
  for (int b = tid; b < a.batch; b += kThreads) reinterpret_cast<int32_t*>(h + lay.off_status)[b] = a.status[b];
  __threadfence_system();
  __syncthreads();
  if (tid == 0) __hip_atomic_store(reinterpret_cast<uint32_t*>(h), a.ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A workgroup's row and output.
struct RowTask {
  Row row;
  int32_t* out;
  int keep;
};
template <bool kPlanned>
using PlanArg = typename std::conditional<kPlanned, TopkPlan, NoArgs>::type;
template <bool kPlanned>
__device__ __forceinline__ RowTask row_task(const TopkArgs<kPlanned>& a, const DimsArg<kPlanned>& dims, const PlanArg<kPlanned>& plan) {
  const int ll = blockIdx.y;                           // layer within this launch
  const int b = blockIdx.x / a.h_kv, h = blockIdx.x % a.h_kv;
  const int e = ll * a.batch + b;
  int cur, cap_cur, cap_keep;
  RowTask t;
  const float* indicator;
  if constexpr (kPlanned) {
    cur = plan.cur_len[e];
    cap_cur = plan.cap_cur[ll];
    cap_keep = plan.cap_keep[ll];
    t.keep = plan.keep[e];
    indicator = a.last != nullptr && ll == plan.n_layers - 1 ? a.last : a.indicator[ll];
  } else {
    cur = dims.cur_len[e];
    cap_cur = a.cap.cur[ll];
    cap_keep = a.cap.keep[ll];
    t.keep = dims.keep[e];
    indicator = a.indicator[ll];
  }
  t.row.init(in_global(indicator) + ((int64_t)b * a.h_kv + h) * cap_cur, cur);
  t.out = in_global(a.idx[ll]) + ((int64_t)b * a.h_kv + h) * cap_keep;
  return t;
}

// Rows that fit the workgroup's registers: kThreads * kSlots * 4 entries, up to three of them absent.
template <bool kPlanned, int kThreads, int kSlots>
__global__ __launch_bounds__(kThreads) void select_topk_kernel(TopkArgs<kPlanned> a, DimsArg<kPlanned> dims, PlanArg<kPlanned> plan) {
  __shared__ __attribute__((aligned(16))) SelectLds lds;
  if constexpr (kPlanned)
    if ((int)blockIdx.y == plan.n_layers) return write_mirror<kThreads>(plan.mirror);
  const RowTask t = row_task<kPlanned>(a, dims, plan);
  if (t.keep <= 0) return;
  if (kPlanned && t.row.n_slots > kThreads * kSlots) return;       // a plan's row longer than the caller's shape says: the next launch's
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (t.keep >= t.row.cur) {                           // everything stays
    for (int i = tid; i < t.row.cur; i += kThreads) t.out[i] = i;
    return;
  }
  // slots are dealt to the waves in runs of 64*n_u, so that short rows keep every wave busy
  const int n_u = (t.row.n_slots + kThreads - 1) / kThreads;
  const int s0 = wave * 64 * n_u + lane;
  uint32_t key[kSlots][4];
  t.row.load(n_u, [&](int u) { return s0 + 64 * u; }, key);
  auto position = [&](int u, int j) { return 4 * (s0 + 64 * u) - t.row.pad + j; };
  uint32_t thr, before = 0;
  int last;
  find_threshold<kThreads, kSlots>(key, n_u, (uint32_t)t.keep, position, lds, thr, last);
  write_picked<kThreads, kSlots>(key, n_u, [&](uint32_t x, int u, int j) { return x > thr - (position(u, j) <= last ? 1u : 0u); },
                                 lds.wave_sel[1], before, [&](uint32_t rank, int u, int j) { t.out[rank] = position(u, j); });
}

// The same for a stage of the cascade (cascade_stage.hip), one workgroup per (layer, sequence, head): the list of a layer held
// before is renewed where the places of its rows are known anyway, with the number of kept rows before each.  The kept
// rows' indicators and places go to the new lists, the places of the dropped ones to the head's free stack.  Of the new layer,
// whose rows get their places afterwards, the kept positions are written.
template <int kThreads, int kSlots>
__global__ __launch_bounds__(kThreads) void select_stage_kernel(StageArgs a) {
  __shared__ __attribute__((aligned(16))) SelectLds lds;
  const int l = blockIdx.y, head = blockIdx.x, b = head / a.h_kv, e = l * a.batch + b;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cur = a.plan.cur_len[e], keep = a.plan.keep[e];
  const bool held = l < a.m;
  const int64_t at = (int64_t)head * a.plan.cap_keep[l];
  int32_t* idx = in_global(static_cast<int32_t*>(a.plan.idx[l])) + at;
  float* ind_out = in_global(static_cast<float*>(a.plan.ind_out[l])) + at;
  const float* ind_in = in_global(held ? static_cast<const float*>(a.held[l]) : a.ind) + (int64_t)head * a.plan.cap_cur[l];
  const int32_t* old = a.slots_old + (reinterpret_cast<const char*>(ind_in) - a.ind_old) / 4;
  int32_t* renewed = a.slots_new + (reinterpret_cast<const char*>(ind_out) - a.ind_new) / 4;
  int32_t* freed = a.free_slots + (int64_t)head * a.prefix_rows;
  // counts of the layers before, for the places the dropped ones go to (more than 64 layers: added up below)
  const int le = min(lane, max(a.m - 1, 0)) * a.batch + b;
  const int32_t cur_le = a.plan.cur_len[le], keep_le = a.plan.keep[le];
  int top = 0;
  auto stack_height = [&] {
    if (!held || keep >= cur) return;
    uint32_t t = (lane < l ? (uint32_t)(cur_le - keep_le) : 0u) - (lane < a.m ? (uint32_t)cur_le : 0u);
    for (int i = lane + 64; i < a.m; i += 64) {
      const int32_t c = a.plan.cur_len[i * a.batch + b];
      t += (i < l ? (uint32_t)(c - a.plan.keep[i * a.batch + b]) : 0u) - (uint32_t)c;
    }
    top = a.prefix_rows + (int32_t)wave_sum(t);
  };
  auto stays = [&](int r, int p, float value, int32_t place) {
    if (held) {
      ind_out[r] = value;
      renewed[r] = place;
    } else {
      idx[r] = p;
    }
  };
  auto goes = [&](int r, int p, int32_t place) {
    const int to = top + p - r;
    if (held && to >= 0 && to < a.prefix_rows) freed[to] = place;
  };
  if (keep >= cur || keep <= 0) {
    stack_height();
    constexpr int kCopied = 8;                         // a thread's, in flight together
    for (int p0 = tid; p0 < cur; p0 += kThreads * kCopied) {
      float x[kCopied];
      int32_t o[kCopied];
#pragma unroll
      for (int i = 0; i < kCopied; ++i) {
        const int p = min(p0 + i * kThreads, cur - 1);
        x[i] = held ? ind_in[p] : 0.f;
        o[i] = held ? old[p] : 0;
      }
#pragma unroll
      for (int i = 0; i < kCopied; ++i) {
        const int p = p0 + i * kThreads;
        if (p < cur && keep > 0) stays(p, p, x[i], o[i]);
        else if (p < cur) goes(0, p, o[i]);
      }
    }
    return;
  }
  Row row;
  row.init(ind_in, cur);
  const int n_u = (row.n_slots + kThreads - 1) / kThreads;
  const int s0 = wave * 64 * n_u + lane;
  uint32_t key[kSlots][4];
  row.load(n_u, [&](int u) { return s0 + 64 * u; }, key);
  auto position = [&](int u, int j) { return 4 * (s0 + 64 * u) - row.pad + j; };
  // values and places of the group at hand and the next one's: the first ones arrive while the threshold is found
  float value[2][4];
  int32_t place[2][4];
  auto fetch = [&](int u) {
    if (!held) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int p = min(max(position(u, j), 0), cur - 1);
      value[u & 1][j] = ind_in[p];
      place[u & 1][j] = old[p];
    }
  };
  fetch(0);
  uint32_t thr, before = 0;
  int last;
  find_threshold<kThreads, kSlots>(key, n_u, (uint32_t)keep, position, lds, thr, last);
  stack_height();
  write_picked<kThreads, kSlots>(key, n_u, [&](uint32_t x, int u, int j) { return x > thr - (position(u, j) <= last ? 1u : 0u); },
                                 lds.wave_sel[1], before,
                                 [&](uint32_t rank, int u, int j) { stays(rank, position(u, j), value[u & 1][j], place[u & 1][j]); },
                                 [&](uint32_t rank, int u, int j) { if (key[u][j] != 0u) goes(rank, position(u, j), place[u & 1][j]); },
                                 [&](int u) { if (u + 1 < kSlots && u + 1 < n_u) fetch(u + 1); });
}

// Longer rows.
constexpr int kLongThreads = 1024;
constexpr int kLongSlots = 4;                          // 16-byte loads in flight per thread
constexpr int kListSlots = 4;                          // the list has as many keys as four slots of four per thread hold, less what
constexpr int kListKeys = 14336;                       // 160 KiB of LDS cannot: 112 KiB of keys and positions
static_assert(kListKeys <= kLongThreads * kListSlots * 4 && kListKeys % 4 == 0, "the list is re-read in slots of four");
struct LongLds {
  SelectLds sel;
  alignas(16) uint32_t key[kListKeys];                 // read in 16-byte pieces
  int32_t pos[kListKeys];
};
static_assert(offsetof(LongLds, key) % 16 == 0 && sizeof(LongLds) <= 160 * 1024, "aligned pieces, a compute unit's LDS");
static_assert(offsetof(SelectLds, hist) % 16 == 0 && offsetof(SelectLds, few) % 16 == 0 && offsetof(SelectLds, few_pos) % 16 == 0,
              "read in 16-byte pieces from a 16-byte aligned block");

template <bool kPlanned>
__global__ __launch_bounds__(kLongThreads) void select_topk_long_kernel(TopkArgs<kPlanned> a, DimsArg<kPlanned> dims, PlanArg<kPlanned> plan) {
  extern __shared__ __attribute__((aligned(16))) char long_lds[];
  LongLds& lds = *reinterpret_cast<LongLds*>(long_lds);
  SelectLds& s = lds.sel;
  if constexpr (kPlanned)
    if ((int)blockIdx.y == plan.n_layers) return write_mirror<kLongThreads>(plan.mirror);
  const RowTask t = row_task<kPlanned>(a, dims, plan);
  if (t.keep <= 0) return;
  const Row& row = t.row;
  if constexpr (kPlanned)
    if (row.n_slots <= plan.served_slots) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, copy = lane & (kCopies - 1);
  if (t.keep >= row.cur) {
    for (int i = tid; i < row.cur; i += kLongThreads) t.out[i] = i;
    return;
  }
  // Digits of 11, 11 and 10 bits from the top, one sweep of the row each, until the entries of the
  // digit that holds the k-th largest fit the list (the first sweep nearly always does it) or the key
  // is known to the last bit.  Where those above it fit as well, the list takes the row's place.
  // Too many entries of one digit are mostly one value (an indicator that is 0 nearly everywhere): the second
  // sweep looks whether they are, and then knows the key.
  uint32_t prefix = 0, mask = 0, need = (uint32_t)t.keep;
  bool fits = false, all_fit = false, one_value = false;
  uint32_t ones = 0, zeros = 0;                          // bits set, and not set, in some entry of the digit at hand
  auto count_digits = [&](auto first, int shift, uint32_t digit_mask) {
    for (int s0 = tid; s0 < row.n_slots; s0 += kLongThreads * kLongSlots) {
      uint32_t key[kLongSlots][4];
      row.load(kLongSlots, [&](int u) { return s0 + u * kLongThreads; }, key);
#pragma unroll
      for (int u = 0; u < kLongSlots; ++u) {
        uint32_t d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool in = key[u][j] != 0u && (first || (key[u][j] & mask) == prefix);
          d[j] = in ? key[u][j] >> shift & digit_mask : kBins;
          if (!first && in) { ones |= key[u][j]; zeros |= ~key[u][j]; }
        }
        if (d[0] == d[1] && d[1] == d[2] && d[2] == d[3]) {
          if (d[0] < kBins) atomicAdd(&s.hist[d[0] * kCopies + copy], 4u);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (d[j] < kBins) atomicAdd(&s.hist[d[j] * kCopies + copy], 1u);
        }
      }
    }
  };
  for (int pass = 0; pass < 3 && !fits && !one_value; ++pass) {
    const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
    const uint32_t digit_mask = pass == 2 ? 1023u : 2047u;
    for (int i = tid; i < kBins * kCopies / 4; i += kLongThreads) reinterpret_cast<uint4*>(s.hist)[i] = uint4{0, 0, 0, 0};
    __syncthreads();
    if (pass == 0) {
      count_digits(std::true_type{}, shift, digit_mask);
    } else {
      ones = zeros = 0;
      count_digits(std::false_type{}, shift, digit_mask);
      auto bits_or = [](uint32_t a, uint32_t b) { return a | b; };
      ones = wave_scan(ones, bits_or);
      zeros = wave_scan(zeros, bits_or);
      if (lane == 63) { s.few[2 * wave] = ones; s.few[2 * wave + 1] = zeros; }
    }
    __syncthreads();
    find_interval<kLongThreads>(need, s);
    if (pass == 1) {
      ones = zeros = 0;
#pragma unroll
      for (int w = 0; w < kMaxWaves; ++w) { ones |= s.few[2 * w]; zeros |= s.few[2 * w + 1]; }
      one_value = (ones & zeros) == 0u;
    }
    prefix |= s.bin << shift;
    need -= s.above;
    mask |= digit_mask << shift;
    fits = s.count <= (uint32_t)kListKeys;
    all_fit = (uint32_t)t.keep - need + s.count <= (uint32_t)kListKeys;
    if (one_value) prefix = ones;
  }
  // Ordered sweep of the row from slot `from` on, `before` entries picked ahead of it; returns the number of entries picked.
  auto sweep = [&](auto pick, auto store, int from = 0, uint32_t before = 0) {
    int parity = 0;
    for (int t0 = from; t0 < row.n_slots; t0 += kLongThreads * kLongSlots, parity ^= 1) {
      uint32_t key[kLongSlots][4];
      auto slot = [&](int u) { return t0 + wave * 64 * kLongSlots + u * 64 + lane; };
      row.load(kLongSlots, slot, key);
      auto position = [&](int u, int j) { return 4 * slot(u) - row.pad + j; };
      write_picked<kLongThreads, kLongSlots>(key, kLongSlots, [&](uint32_t x, int u, int j) { return pick(x, position(u, j)); },
                                             s.wave_sel[parity], before,
                                             [&](uint32_t rank, int u, int j) { store(rank, key[u][j], position(u, j)); });
    }
    __syncthreads();
    return before;
  };
  uint32_t thr = prefix;
  int last = 0;
  if (fits) {
    auto to_list = [&](uint32_t rank, uint32_t x, int pos) {
      if (rank < (uint32_t)kListKeys) { lds.key[rank] = x; lds.pos[rank] = pos; }
    };
    const uint32_t found = all_fit ? sweep([&](uint32_t x, int) { return x >= prefix && x != 0u; }, to_list)
                                   : sweep([&](uint32_t x, int) { return (x & mask) == prefix && x != 0u; }, to_list);
    const int n = min((int)found, kListKeys), n_u = (n + 4 * kLongThreads - 1) / (4 * kLongThreads);
    const int i0 = 4 * (wave * 64 * n_u + lane);
    uint32_t key[kListSlots][4];
#pragma unroll
    for (int u = 0; u < kListSlots; ++u) {
      key[u][0] = key[u][1] = key[u][2] = key[u][3] = 0u;
      const int i = i0 + 256 * u;
      if (u < n_u && i < n) {
        const uint4 x = *reinterpret_cast<const uint4*>(&lds.key[i]);
        key[u][0] = x.x;
        key[u][1] = i + 1 < n ? x.y : 0u;
        key[u][2] = i + 2 < n ? x.z : 0u;
        key[u][3] = i + 3 < n ? x.w : 0u;
      }
    }
    auto position = [&](int u, int j) { return lds.pos[min(i0 + 256 * u + j, kListKeys - 1)]; };
    find_threshold<kLongThreads, kListSlots>(key, n_u, all_fit ? (uint32_t)t.keep : need, position, s, thr, last);
    if (all_fit) {
      uint32_t before = 0;
      write_picked<kLongThreads, kListSlots>(key, n_u,
                                             [&](uint32_t x, int u, int j) { return x > thr || (x == thr && position(u, j) <= last); },
                                             s.wave_sel[1], before, [&](uint32_t rank, int u, int j) { t.out[rank] = position(u, j); });
      return;
    }
  } else {
    // The key is known: every entry above it and the first `need` equal to it, in one ordered sweep; behind the last of
    // those that are equal only the ones above count.  Counts of a step travel as two halves of a word, at most 16 waves
    // * 1024 entries each.  With two sweeps here and all three digits counted 8 rows of 131008 equal entries took 116 us, now
    // 52, and rows of zeros with every 200th entry above them 124, now 77 (four sweeps: 80 and 89).
    static_assert(kMaxWaves * 64 * kLongSlots * 4 < 1 << 16, "two counts of a step in one word");
    uint32_t above = 0, equal = 0;                       // in the row before this step
    int t0 = 0, parity = 0;
    for (; equal < need && t0 < row.n_slots; t0 += kLongThreads * kLongSlots, parity ^= 1) {
      uint32_t key[kLongSlots][4];
      auto slot = [&](int u) { return t0 + wave * 64 * kLongSlots + u * 64 + lane; };
      row.load(kLongSlots, slot, key);
      uint32_t n = 0;
#pragma unroll
      for (int u = 0; u < kLongSlots; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) n += __popcll(__ballot(key[u][j] > thr)) + (__popcll(__ballot(key[u][j] == thr)) << 16);
      if (lane == 0) s.wave_sel[parity][wave] = n;
      __syncthreads();
      uint32_t g = above, e = equal;                     // before the wave's entries
#pragma unroll
      for (int w = 0; w < kMaxWaves; ++w) {
        const uint32_t c = s.wave_sel[parity][w];
        above += c & 0xffffu;
        equal += c >> 16;
        if (w < wave) { g += c & 0xffffu; e += c >> 16; }
      }
#pragma unroll
      for (int u = 0; u < kLongSlots; ++u) {
        uint32_t rank_g = g, rank_e = e;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint64_t bg = __ballot(key[u][j] > thr), be = __ballot(key[u][j] == thr);
          rank_g = __builtin_amdgcn_mbcnt_hi((uint32_t)(bg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bg, rank_g));
          rank_e = __builtin_amdgcn_mbcnt_hi((uint32_t)(be >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)be, rank_e));
          g += __popcll(bg);
          e += __popcll(be);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool is_above = key[u][j] > thr, is_equal = key[u][j] == thr;
          if (is_above || (is_equal && rank_e < need)) t.out[rank_g + min(rank_e, need)] = 4 * slot(u) - row.pad + j;
          rank_g += is_above ? 1u : 0u;
          rank_e += is_equal ? 1u : 0u;
        }
      }
    }
    __syncthreads();                                     // the counts of the last step have been read
    if (above + need < (uint32_t)t.keep)
      sweep([&](uint32_t x, int) { return x > thr; }, [&](uint32_t rank, uint32_t, int pos) { t.out[rank] = pos; }, t0, above + need);
    return;
  }
  sweep([&](uint32_t x, int pos) { return x > thr - (pos <= last ? 1u : 0u); }, [&](uint32_t rank, uint32_t, int pos) { t.out[rank] = pos; });
}

// The kernel for rows of up to `most` entries, with as few slots a thread as hold them (a slot that no row has costs its tests:
// 992 entries 5.9 us with four of 256 threads, 5.0 with one; 8160 in 256 rows of a pass 13.5 with eight of 512, 12.2 with four).
// More threads leave a thread less to do in a row, but idle at its barriers, and fewer rows share a compute unit.  Us at 8, 256
// and 1024 rows:
//   entries   256 threads          512                 1024
//    1000     4.8   5.1   7.6      4.8   5.2  11.8     5.5   5.9  24.2
//    2000     5.6   6.2   9.9      4.8   5.3  11.9     5.4   6.1  24.9
//    4000     7.4   8.5  13.8      5.9   6.8  13.3     5.8   6.6  23.4
//    6000     9.7  10.0            7.4   7.9           7.7   8.1
//    8100    11.4  11.8  19.9      8.5   9.1  19.2     8.0   8.5  29.8
//   16300                         12.0  15.5          10.3  13.0
// In a pass, where workgroups beside the rows write the plan's copy, 1024 threads are not the faster at 256 rows: 5000, 6000, 8100, 9000
// and 16300 entries 9.0, 9.4, 11.0, 13.0 and 15.4 us with 512 threads, 12.2, 12.7, 13.2, 15.0 and 17.5 with 1024; at 128 rows of
// 9000 and 16000 entries 12.0 and 14.8, 10.6 and 12.4.  (1024 threads with two slots would save half a microsecond at 8 rows of
// 8100: not built.)
// Where `most` is only what the caller's shape suggests (!bounded: the lengths are device data), rows that do not fit it are
// left out by that kernel and served by the one for any length, launched behind it.
template <bool kPlanned>
int launch_topk(dim3 grid, int64_t most, bool bounded, const TopkArgs<kPlanned>& a, const DimsArg<kPlanned>& dims, PlanArg<kPlanned> plan,
                hipStream_t stream) {
  const int64_t need = most + 3;                       // up to three absent entries in front
  int32_t served_slots = 0;
#define CAKE_TOPK(T, S)                                                                                    \
  do {                                                                                                     \
    hipLaunchKernelGGL((select_topk_kernel<kPlanned, T, S>), grid, dim3(T), 0, stream, a, dims, plan);     \
    served_slots = T * S;                                                                                  \
  } while (0)
  int64_t rows = (int64_t)grid.x * grid.y;
  if constexpr (kPlanned) rows = (int64_t)grid.x * plan.n_layers;      // not the workgroups that write the plan's copy
  if (need <= 256 * 1 * 4) CAKE_TOPK(256, 1);
  else if (need <= 256 * 2 * 4 && rows > 256) CAKE_TOPK(256, 2);
  else if (need <= 512 * 1 * 4) CAKE_TOPK(512, 1);
  else if (need <= 512 * 2 * 4) CAKE_TOPK(512, 2);
  else if (need <= 512 * 3 * 4) CAKE_TOPK(512, 3);
  else if (need <= 512 * 4 * 4) CAKE_TOPK(512, 4);
  else if (need <= 1024 * 4 * 4 && rows <= 128) CAKE_TOPK(1024, 4);
  else if (need <= 512 * 8 * 4) CAKE_TOPK(512, 8);
  else if (need <= 1024 * 8 * 4) CAKE_TOPK(1024, 8);
  else if (need <= 1024 * 16 * 4) CAKE_TOPK(1024, 16);
  if (served_slots == 0 || !bounded) {
    auto kern = select_topk_long_kernel<kPlanned>;
    CAKE_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)sizeof(LongLds)));
    if constexpr (kPlanned) {
      plan.served_slots = served_slots;
      grid.y = plan.n_layers + (served_slots == 0 && plan.mirror.host != nullptr ? 1 : 0);     // the copy is made once
    }
    hipLaunchKernelGGL(kern, grid, dim3(kLongThreads), sizeof(LongLds), stream, a, dims, plan);
  }
#undef CAKE_TOPK
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}

}  // namespace
}  // namespace cake

int cake::launch_topk_planned(const cake_shape* shape, const float* const* indicator, const float* last, const PlanView& plan, int64_t max_cur,
                              bool bounded, const PlanMirror& mirror, hipStream_t stream) {
  TopkArgs<true> a{};
  a.indicator = indicator;
  a.last = last;
  a.idx = reinterpret_cast<int32_t* const*>(plan.idx);
  a.batch = shape->batch;
  a.h_kv = shape->n_kv_heads;
  const TopkPlan tp{plan.cur_len, plan.keep, plan.cap_cur, plan.cap_keep, shape->n_layers, mirror, 0};
  return launch_topk<true>(dim3(shape->batch * shape->n_kv_heads, shape->n_layers + (mirror.host != nullptr ? 1 : 0)), max_cur, bounded, a, NoArgs{}, tp, stream);
}

// As many threads as leave a row the fewest slots each, while a row has a compute unit to itself: averages over the stages of
// 32 layers of 8 heads (256 rows in the last), us with 256, 512 and 1024 threads: 1000 keys 6.8, 6.7, 7.4; 2000 7.6, 6.7, 7.5;
// 4000 10.7, 8.3, 7.9; 6000 14.4, 11.3, 10.4; 8192 (512 threads with eight slots 13.2) 12.4, 11.3 for the last two; 15000 (16
// layers) 17.6, 14.7.  With more rows than compute units, in a 33rd stage, with 512 and 1024 threads: 3000 keys 9.9, 12.3; 6000
// 12.6, 15.6; 15000 19.9, 21.9.  64 layers of 8192 keys on average: 12.1, 13.4.
int cake::launch_topk_stage(const StageArgs& a, hipStream_t stream) {
  const dim3 grid(a.batch * a.h_kv, a.m + 1);
  const int need = a.prefix_len + 3;
  const bool few = (int64_t)grid.x * grid.y <= 256;
  auto run = [&](auto kern, int threads) { hipLaunchKernelGGL(kern, grid, dim3(threads), 0, stream, a); };
  if (need <= 256 * 1 * 4) run(select_stage_kernel<256, 1>, 256);
  else if (need <= 512 * 1 * 4) run(select_stage_kernel<512, 1>, 512);
  else if (need <= 1024 * 1 * 4 && few) run(select_stage_kernel<1024, 1>, 1024);
  else if (need <= 512 * 2 * 4) run(select_stage_kernel<512, 2>, 512);
  else if (need <= 1024 * 2 * 4 && few) run(select_stage_kernel<1024, 2>, 1024);
  else if (need <= 512 * 4 * 4) run(select_stage_kernel<512, 4>, 512);
  else if (few) run(select_stage_kernel<1024, 4>, 1024);
  else run(select_stage_kernel<512, 8>, 512);
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}

using namespace cake;

extern "C" int cake_select_topk(const cake_shape* shape, const float* const* indicator,
                                const int32_t* cur_len, const int32_t* k, int32_t* const* idx,
                                void* workspace, size_t workspace_bytes, void* stream) {
  (void)workspace; (void)workspace_bytes;
  if (int rc = check_shape_basic(shape)) return rc;
  CAKE_REQUIRE(indicator && idx && cur_len && k, "indicator, idx, cur_len or k is NULL");
  const int B = shape->batch, L = shape->n_layers;
  for (int i = 0; i < L * B; ++i) {
    CAKE_REQUIRE(cur_len[i] >= 0, "cur_len[%d] = %d is negative", i, cur_len[i]);
    CAKE_REQUIRE(k[i] >= 0 && k[i] <= cur_len[i], "k[%d] = %d outside [0, cur_len = %d]", i, k[i], cur_len[i]);
  }
  CAKE_REQUIRE((int64_t)B * shape->n_kv_heads <= 0x7fffffff, "too many rows");
  hipStream_t st = static_cast<hipStream_t>(stream);
  for (int l0 = 0; l0 < L;) {
    const int nl = launch_layers(L - l0, B);
    TopkArgs<false> a{};
    RaggedDims dims{};
    a.indicator = indicator + l0;
    a.idx = idx + l0;
    a.batch = B;
    a.h_kv = shape->n_kv_heads;
    int most = 0, rows = 0;
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
      most = std::max(most, cc);
      rows = std::max(rows, ck);
    }
    if (rows > 0)
      if (int rc = launch_topk<false>(dim3(B * shape->n_kv_heads, nl), most, true, a, dims, NoArgs{}, st)) return rc;
    l0 += nl;
  }
  return CAKE_OK;
}
