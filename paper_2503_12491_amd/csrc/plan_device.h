// The allocation step of an eviction plan on the device (plan_evict.hip): one workgroup, in a launch of its own or beside
// other work that the step does not depend on.
#pragma once

#include "cake_internal.h"

#ifdef __HIPCC__
namespace cake {

constexpr int kPlanMaxLayers = 1024;

// p/(s + 1/2) > lam, decided exactly as the fp64 division and comparison would.  The rounded
// quotient lies within one part in 2^52 of p/x, so away from a narrow band around p = lam*x a
// multiplication settles it; inside the band the division itself is done.
__device__ __forceinline__ bool seat_above(double p, double lam, int64_t s) {
  const double x = (double)s + 0.5;
  const double t = lam * x;
  if (!(lam > 0x1p-900 && t < 0x1p900)) return p / x > lam;     // products near the ends of the range: no shortcut
  if (p > t * (1.0 + 0x1p-50)) return true;
  if (p < t * (1.0 - 0x1p-50)) return false;
  return p / x > lam;
}

// 1/x to some 50 bits.
__device__ __forceinline__ double approx_rcp(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return r * (2.0 - x * r);
}

// Number of seat counts s in [window, n-1] with p/(s + 1/2) > lam.  The quotient never increases
// with s, so the count is fixed by the last s that passes; it is searched from a closed-form guess with
// the exact predicate.  The guess is a seat off at most, unless the quotients are subnormal: they are then rounded so
// coarsely that it can be off by a large share of n, and what is left after four tries is halved.
__device__ int64_t seats_above(double p, double lam, int window, int n) {
  if (!seat_above(p, lam, window)) return 0;
  int64_t lo = window, hi = n - 1, s = hi;        // above lam at lo, not above it beyond hi
  if (lam > 0.0) {
    const double guess = floor(p / lam - 0.5);
    s = guess >= (double)hi ? hi : guess <= (double)lo ? lo : (int64_t)guess;
  }
  for (int tries = 1; lo < hi; ++tries) {
    const bool above = seat_above(p, lam, s);
    if (above) lo = s; else hi = s - 1;
    s = tries >= 4 ? lo + (hi - lo + 1) / 2 : above ? lo + 1 : hi;
  }
  return lo - window + 1;
}

// The largest value, of several equal ones the lowest layer; the wave's answer in every lane.
__device__ __forceinline__ void wave_argmax(double& best, int& best_l) {
  auto step = [&](double ob, uint32_t ol) {
    if (ob > best || (ob == best && (int)ol < best_l)) { best = ob; best_l = (int)ol; }
  };
  step(dpp_step<0x111, 0xf, true>(best), dpp_step<0x111, 0xf, true>((uint32_t)best_l));
  step(dpp_step<0x112, 0xf, true>(best), dpp_step<0x112, 0xf, true>((uint32_t)best_l));
  step(dpp_step<0x114, 0xf, true>(best), dpp_step<0x114, 0xf, true>((uint32_t)best_l));
  step(dpp_step<0x118, 0xf, true>(best), dpp_step<0x118, 0xf, true>((uint32_t)best_l));
  step(dpp_step<0x142, 0xa, true>(best), dpp_step<0x142, 0xa, true>((uint32_t)best_l));
  step(dpp_step<0x143, 0xc, true>(best), dpp_step<0x143, 0xc, true>((uint32_t)best_l));
  best = from_lane(best, 63);
  best_l = (int)from_lane((uint32_t)best_l, 63);
}

struct PlanArgs {
  const double* pref;         // [B] rows of pref_ld
  int32_t pref_ld, n_layers, batch, h_kv, window, seq_len, row_bytes;
  int64_t total_budget;
  const int32_t* cur_len;     // of the first cur_known of the [L*B] entries; the others': seq_len - window
  int32_t cur_known;
  int32_t *budgets, *keep, *cur, *cap_keep, *cap_cur, *copy_blocks, *status;
  char *pool_idx, *pool_k, *pool_v, *pool_ind;
  void **idx_tbl, **k_tbl, **v_tbl, **ind_tbl;
  bool allocated;             // budgets, keep and cur are there already (allocate_kernel)
};

constexpr size_t kPlanLdsPerLayer = 2 * sizeof(double) + sizeof(int32_t);     // p, prio, bud of one layer of one sequence

// A value per layer, entry l only ever touched by lane l mod 64 (so that nothing here synchronises): a
// register where every lane owns one layer at most, the wave's own LDS array otherwise.
template <bool kOne, typename T>
struct PerLayer {
  T one;
  T* many;
  __device__ __forceinline__ explicit PerLayer(T* lds) : one(T(0)), many(lds) {}
  __device__ __forceinline__ T& operator[](int l) { return kOne ? one : many[l]; }
};

// budgets, keep, cur_out of sequence b by one wave.
// status[b] = 1 if a preference of the sequence is NaN, negative or infinite (the budgets are then
// those of equal preferences, so that everything downstream stays in bounds), else 0.
template <bool kOne>
__device__ void allocate_sequence(const PlanArgs& a, int b, int lane, double* p_lds, double* prio_lds, int32_t* bud_lds) {
  const int n_layers = a.n_layers, window = a.window, seq_len = a.seq_len;
  PerLayer<kOne, double> p(p_lds), prio(prio_lds);
  PerLayer<kOne, int32_t> bud(bud_lds);
  bool bad = false, any_pos = false;
  for (int l = lane; l < n_layers; l += 64) {
    const double x = a.pref[(int64_t)b * a.pref_ld + l];
    p[l] = x;
    bad = bad || !(x >= 0.0) || isinf(x);
    any_pos = any_pos || x != 0.0;
  }
  bad = __any(bad);
  any_pos = __any(any_pos);
  if (lane == 0) a.status[b] = bad ? 1 : 0;
  if (!any_pos || bad)                            // all-zero preferences count as equal ones
    for (int l = lane; l < n_layers; l += 64) p[l] = 1.0;

  if ((int64_t)n_layers * seq_len <= a.total_budget) {   // every layer fits whole: nothing to evict
    for (int l = lane; l < n_layers; l += 64) bud[l] = seq_len;
  } else {
    const int64_t r_total = a.total_budget - (int64_t)n_layers * window;
    const int64_t most = seq_len - window;          // seats of a full layer
    // Seats above a level; bud receives every layer's count.
    auto taken_above = [&](double lam) {
      int64_t t = 0;
      for (int l = lane; l < n_layers; l += 64) {
        const int64_t s = seats_above(p[l], lam, window, seq_len);
        bud[l] = (int32_t)s;
        t += s;
      }
      return wave_sum(t);
    };
    // Any level with at most r_total seats above it is a state of the award loop; the search stops as
    // soon as the seats left for the loop are few.
    constexpr int kFew = 6;
    double hi = 0.0, lo = 0.0, sum_p = 0.0;
    int64_t positive = 0;                           // layers whose every seat lies above 0 (no quotient underflows)
    bool tiny = false;
    for (int l = lane; l < n_layers; l += 64) {
      hi = fmax(hi, p[l] / (window + 0.5));
      sum_p += p[l];
      positive += p[l] > 1e-290 ? 1 : 0;
      tiny = tiny || (p[l] > 0.0 && !(p[l] > 1e-290));
    }
    hi = from_lane(wave_scan(hi, [](double x, double y) { return fmax(x, y); }), 63);      // nothing lies above this
    sum_p = wave_sum(sum_p);
    int64_t at_hi = 0;
    double counted = -1.0;                          // the level whose counts bud holds
    if ((__any(tiny) ? taken_above(lo) : wave_sum(positive) * most) <= r_total) {
      hi = lo;
    } else {
      // Without floors and caps the budgets are pref/lambda - 1/2 and sum to the total at
      // lambda = sum(pref)/(total + L/2).  From there a secant step: the layers that are neither at
      // their floor nor full hold p/lambda - window seats each (give or take one), so the level that
      // leaves `margin` seats to the award loop follows from their sum.  A step that would leave
      // the bracket is replaced by its middle.
      double lam = sum_p / ((double)a.total_budget + 0.5 * n_layers);
      // First with seats counted from rounded quotients, a third of the time of an exact count: wherever this ends, what
      // follows counts exactly.  Of a step only the layers count that are neither at their floor nor full.
      double below = lo, over = hi;
      for (int it = 0; it < 8; ++it) {
        if (!(lam > below && lam < over)) lam = 0.5 * (below + over);
        if (!(lam > below && lam < over)) break;
        const double inv = approx_rcp(lam);
        double t = 0.0, active_p = 0.0;
        for (int l = lane; l < n_layers; l += 64) {
          const double s = fmin(fmax(ceil(p[l] * inv - 0.5) - window, 0.0), (double)most);
          t += s;
          if (s > 0.0 && s < (double)most) active_p += p[l];
        }
        t = wave_sum(t);
        const double left = (double)r_total - t;
        if (left >= 0.0 && left <= 1.0) break;
        if (left >= 0.0) over = lam;
        else below = lam;
        active_p = wave_sum(active_p);
        // sum over the active layers of p/lam is to grow by the seats that are left
        const double seats = active_p * inv + left - 0.5;
        lam = active_p > 0.0 && seats > 0.0 ? active_p * approx_rcp(seats) : 0.5 * (below + over);
      }
      double margin = 3.0;
      for (int it = 0; it < 96 && r_total - at_hi > kFew; ++it) {
        if (!(lam > lo && lam < hi)) {
          lam = 0.5 * (lo + hi);
          if (!(lam > lo && lam < hi)) break;
        }
        // tied priorities: no level parts them, and what is left is at most a seat or two per layer
        if (hi - lo <= hi * 0x1p-40 && r_total - at_hi <= 2 * (int64_t)n_layers) break;
        const int64_t t = taken_above(lam);
        counted = lam;
        if (t <= r_total) {
          hi = lam;
          at_hi = t;
          if (r_total - at_hi <= kFew) break;
        } else { lo = lam; margin += (double)min(t - r_total, (int64_t)n_layers) + 1.0; }
        double active_p = 0.0;
        int64_t active_full = 0;                    // active layers in the low word, full ones above
        for (int l = lane; l < n_layers; l += 64) {
          const int64_t s = bud[l];
          if (s > 0 && s < most) { active_p += p[l]; active_full += 1; }
          else if (s == most) active_full += (int64_t)1 << 32;
        }
        active_p = wave_sum(active_p);
        active_full = wave_sum(active_full);
        const int64_t n_active = active_full & 0xffffffff, n_full = active_full >> 32;
        const double seats = (double)(r_total - n_full * most) - margin + (double)(n_active * window);
        // (a search that has not ended by then halves the bracket at every other step)
        lam = n_active > 0 && seats > 0.0 && (it < 6 || (it & 1) == 0) ? active_p / seats : 0.5 * (lo + hi);
      }
    }
    if (counted != hi) (void)taken_above(hi);
    int64_t taken = 0;
    for (int l = lane; l < n_layers; l += 64) {
      taken += bud[l];
      bud[l] += window;
      prio[l] = bud[l] < seq_len ? p[l] / ((double)bud[l] + 0.5) : -1.0;
    }
    int64_t remaining = r_total - wave_sum(taken);
    // Award what is left one seat at a time: largest pref/(B + 1/2), ties to the lower layer.
    double own = -2.0;                              // the lane's best layer
    int own_l = kPlanMaxLayers;
    auto pick = [&]() {
      own = -2.0;
      own_l = kPlanMaxLayers;
      for (int l = lane; l < n_layers; l += 64)
        if (prio[l] > own) { own = prio[l]; own_l = l; }         // first maximum within the lane's layers
    };
    pick();
    while (remaining > 0) {
      double best = own;
      int best_l = own_l;
      wave_argmax(best, best_l);
      if (best < 0.0) break;
      int64_t take = 1;
      if ((best_l & 63) == lane) {
        // A layer of zero preference keeps the priority 0 until it is full, and the lowest such
        // layer wins every tie: it takes all it can hold at once.
        if (best == 0.0) take = min(remaining, (int64_t)(seq_len - bud[best_l]));
        bud[best_l] += (int32_t)take;
        prio[best_l] = bud[best_l] < seq_len ? p[best_l] / ((double)bud[best_l] + 0.5) : -1.0;
        pick();
      }
      remaining -= best == 0.0 ? from_lane(take, best_l & 63) : 1;
    }
  }
  for (int l = lane; l < n_layers; l += 64) {
    const int64_t e = (int64_t)l * a.batch + b;
    const int cur = e < a.cur_known ? a.cur_len[e] : seq_len - window;
    a.budgets[e] = bud[l];
    a.keep[e] = min(max(bud[l] - window, 0), cur);
    a.cur[e] = cur;
  }
}

// The whole plan in one workgroup: budgets and keep counts (a wave per sequence), row capacities of
// every layer (the largest count over the batch), the places of the layers' outputs, one after the
// other, in the four pools, and the compaction's work list.
// kAtMost64: no plan of more layers than that gets here (the code for them is nearly half of the kernel).
template <bool kAtMost64 = false>
__device__ __forceinline__ void plan_workgroup(const PlanArgs& a, char* plan_lds /* kPlanLdsPerLayer bytes per wave and layer beyond 64 layers */) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n_waves = blockDim.x >> 6;
  const int n_layers = a.n_layers, batch = a.batch;
  if (!a.allocated) {
    double* p = reinterpret_cast<double*>(plan_lds) + (size_t)wave * 2 * n_layers;
    int32_t* bud = reinterpret_cast<int32_t*>(plan_lds + (size_t)n_waves * n_layers * 2 * sizeof(double)) + (size_t)wave * n_layers;
    for (int b = wave; b < batch; b += n_waves) {
      if (kAtMost64 || n_layers <= 64) allocate_sequence<true>(a, b, lane, nullptr, nullptr, nullptr);
      else allocate_sequence<false>(a, b, lane, p, p + n_layers, bud);
    }
  }
  __threadfence_block();
  __syncthreads();
  if (a.allocated) {                       // many sequences: a wave per layer
    for (int l = wave; l < n_layers; l += n_waves) {
      uint32_t ck = 0, cc = 0;             // counts are not negative
      for (int b = lane; b < batch; b += 64) {
        ck = max(ck, (uint32_t)a.keep[(int64_t)l * batch + b]);
        cc = max(cc, (uint32_t)a.cur[(int64_t)l * batch + b]);
      }
      auto umax = [](uint32_t x, uint32_t y) { return max(x, y); };
      ck = wave_scan(ck, umax);
      cc = wave_scan(cc, umax);
      if (lane == 63) { a.cap_keep[l] = (int32_t)ck; a.cap_cur[l] = (int32_t)cc; }
    }
  } else {
    for (int l = tid; l < n_layers; l += blockDim.x) {
      int ck = 0, cc = 0;
      for (int b = 0; b < batch; ++b) {
        ck = max(ck, a.keep[(int64_t)l * batch + b]);
        cc = max(cc, a.cur[(int64_t)l * batch + b]);
      }
      a.cap_keep[l] = ck;
      a.cap_cur[l] = cc;
    }
  }
  __threadfence_block();
  __syncthreads();
  // Running sums over the layers (output places, wave 0) and over the (layer, sequence) entries (the
  // work list, the last wave): every lane sums a run of consecutive items, a wave scan gives the
  // runs' starts.
  auto scan = [&](int64_t own) {           // exclusive prefix sum over the lanes
    return wave_scan(own, [](int64_t x, int64_t y) { return x + y; }) - own;
  };
  if (wave == 0) {
    const int64_t bh = (int64_t)batch * a.h_kv;
    const int per = (n_layers + 63) / 64;
    const int l0 = min(lane * per, n_layers), l1 = min(l0 + per, n_layers);
    int64_t rows = 0;
    for (int l = l0; l < l1; ++l) rows += a.cap_keep[l];
    int64_t before = scan(rows);            // rows of capacity in the layers before l0
    for (int l = l0; l < l1; ++l) {
      const int64_t off_i = bh * before, off_kv = bh * (before + (int64_t)l * a.window) * a.row_bytes;
      a.idx_tbl[l] = a.pool_idx + off_i * 4;
      a.ind_tbl[l] = a.pool_ind + off_i * 4;
      a.k_tbl[l] = a.pool_k + off_kv;
      a.v_tbl[l] = a.pool_v + off_kv;
      before += a.cap_keep[l];
    }
  }
  if (wave == n_waves - 1) {
    const int64_t n = (int64_t)n_layers * batch, pieces = a.row_bytes / 16;
    const int64_t per = (n + 63) / 64;
    const int64_t e0 = min(lane * per, n), e1 = min(e0 + per, n);
    auto blocks_of = [&](int64_t e) { return ((a.keep[e] + a.window) * pieces + kCopyBlockPieces - 1) / kCopyBlockPieces; };
    int64_t own = 0;
    for (int64_t e = e0; e < e1; ++e) own += blocks_of(e);
    int64_t before = scan(own);
    for (int64_t e = e0; e < e1; ++e) {
      a.copy_blocks[e] = (int32_t)before;
      before += blocks_of(e);
    }
    if (lane == 63) a.copy_blocks[n] = (int32_t)before;     // the last lane's run ends the list
  }
}

// The arguments of cake_plan_eviction (with rows of pref_ld preferences per sequence), checked.
int plan_args(const cake_shape* shape, const double* pref, int pref_ld, int64_t total_budget, const int32_t* cur_len,
              void* pool_idx, void* pool_k, void* pool_v, void* pool_ind, void* plan, size_t plan_bytes,
              int32_t* status, PlanArgs* out);
int launch_plan(const PlanArgs& args, hipStream_t stream);

}  // namespace cake
#endif
