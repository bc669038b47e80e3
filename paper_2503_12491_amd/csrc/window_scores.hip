// cake_window_scores / cake_layer_preference: observation-window attention statistics.
//
// Sec. 2 (attention weights), Sec. 4.1 (recent-window submatrix A[-S_w:, :-S_w]),
// Sec. 3 Eq. 4-5 (dispersion, shift), Sec. 4.3 Eq. 11 (Mean + gamma*Var indicator).
//
// A "slice" is one (layer, sequence, KV head).  Its G*S_w window rows (G query heads of the
// group, S_w rows each) attend to the slice's N keys.  The softmax normaliser of a row needs
// every key, the column statistics need the normalised weights, so the keys are visited twice:
//
//   pass 1  logits via MFMA (keys on the M side, window rows on the N side, so that each lane
//           owns ONE window row per 32-row block and keeps a running (reference, sum) pair for
//           it with no cross-lane traffic); partial pairs per granule of keys      -> workspace
//   combine partial pairs -> log2-domain normaliser per window row                  -> workspace
//   pass 2  logits again (window rows on the M side, keys on the N side, so that each lane owns
//           ONE key column and the Mean/Var over the S_w rows are in-register sums); weights
//           p = exp2(t), t = logit*scale*log2(e) - lse2; per column sum p, sum p^2; entropy
//           sum p*t; group mean of I_q through LDS                      -> un-pooled indicator
//           (software-pipelined for bf16 at S_w = 64: the MFMAs of one 32-key sub-tile are
//           interleaved with the statistics of the previous one)
//   pool    stride-1 max-pool over prefix positions                              -> indicator
//   pref    fixed-order fp64 reduction of the per-granule entropy/variance sums    -> P_l, H_l, V_l
//
// One workgroup = G wavefronts = one or more granules of keys of one slice; wave w serves query head
// g*G + w (packed kernels: several slices a workgroup; large launches of some group sizes: scores_stream.hip; all to the same
// bits).  K tiles of 64 keys go from global memory straight into LDS (global_load_lds, 16
// bytes per lane), double-buffered so that tile t+1 is in flight while tile t is consumed, and
// are shared by the G waves.  Rows are stored unpadded with their 16-byte pieces XOR-swizzled by
// the row index so that the MFMA operand reads spread over the banks.
// With the row normalisers supplied by the caller (cake_window_scores_lse) pass 1 and the
// combine give way to a kernel that converts them to the log2 domain.
// Everything is deterministic: no float atomics, fixed reduction orders.
#include "plan_device.h"
#include "score_device.h"

namespace cake {
namespace {

// Transfer of keys [t0, t0+64) of one slice into an LDS tile.  The tile is moved as 1 KiB
// groups, one wave-wide instruction each, group i by wave i mod G.  Lane j of a group fills LDS
// bytes [16 j, 16 j + 16) of that group and fetches the piece of the key row that the swizzle
// assigns to that place: group i holds rows i*kRows + lr (lr = j / kPieces), and since kRows is a
// power of two the swizzle splits into a per-lane part (slot ^ lr) and a per-group part
// (i*kRows mod kPieces) that is XORed in with one instruction.  The per-lane offsets are computed
// once per kernel; per transfer there remain a scalar base, one XOR and one add, and no branch.
// Rows past the last key are clamped to it (their logits are masked later), so every access
// stays inside the slice.
template <typename T, int D>
struct TileMover {
  using TL = Tile<T, D>;
  static constexpr int kRows = 1024 / TL::kRowBytes;                           // key rows per group
  uint32_t row_off, piece_off;              // per-lane: lr * token stride; (slot ^ lr) * 16
  const char* kbase;
  int64_t tok_bytes;
  int last_key, wave, n_waves, lane;

  __device__ __forceinline__ void init(const char* kbase_, int64_t tok_bytes_, int last_key_, int wave_, int n_waves_,
                                       int lane_) {
    kbase = kbase_; tok_bytes = tok_bytes_; last_key = last_key_; wave = wave_; n_waves = n_waves_; lane = lane_;
    const int lr = lane / TL::kPieces, slot = lane % TL::kPieces;
    row_off = (uint32_t)(lr * tok_bytes);
    piece_off = (uint32_t)((slot ^ lr) << 4);
  }
  __device__ __forceinline__ void issue(char* tile, int t0) const {
    if (t0 + kTileKeys - 1 <= last_key) {       // whole tile inside the slice
      const char* base = kbase + (int64_t)t0 * tok_bytes;
      for (int i = wave; i < TL::kGroups; i += n_waves) {
        const uint32_t group_bits = (uint32_t)(((i * kRows) & (TL::kPieces - 1)) << 4);
        const char* src = base + (int64_t)i * kRows * tok_bytes + (row_off + (piece_off ^ group_bits));
        __builtin_amdgcn_global_load_lds((global_cptr)src, (lds_ptr)(tile + i * 1024), 16, 0, kStreamPolicy);
      }
    } else {
      for (int i = wave; i < TL::kGroups; i += n_waves) {
        const int off = i * 1024 + lane * 16;
        const int r = off / TL::kRowBytes, slot = (off % TL::kRowBytes) >> 4;
        const int q = slot ^ (r & (TL::kPieces - 1));
        const char* src = kbase + (int64_t)min(t0 + r, last_key) * tok_bytes + q * 16;
        __builtin_amdgcn_global_load_lds((global_cptr)src, (lds_ptr)(tile + i * 1024), 16, 0, kStreamPolicy);
      }
    }
  }
};

// All of this wave's outstanding vector-memory operations (the tile transfers) have landed.
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

template <typename T, int D, int MB>
__device__ __forceinline__ void load_q(typename Frag<T>::type (&qf)[MB][D / Frag<T>::kElems], const T* q,
                                       int64_t tok_stride, int c32, int hh) {
  using F = Frag<T>;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int s = 0; s < D / F::kElems; ++s) qf[mb][s] = F::load_global(q + (int64_t)(mb * 32 + c32) * tok_stride, s, hh);
}

// ------------------------------------------------------------------------------------------
// Pass 1: per window row, (reference, sum of 2^(t - reference)) over one chunk of keys.
// ------------------------------------------------------------------------------------------
// Logits of sub-tile `sub` of `tile` (32 keys) against the wave's window rows.
// acc[nb][v]: key = kb + 8*(v/4) + 4*hh + (v%4), window row = nb*32 + c32.
template <typename T, int D, int MB>
__device__ __forceinline__ void pass1_logits(const char* tile, int sub,
                                             const typename Frag<T>::type (&qf)[MB][D / Frag<T>::kElems],
                                             f32x16 (&acc)[MB], int c32, int hh) {
  using F = Frag<T>;
  using TL = Tile<T, D>;
  constexpr int kSteps = D / F::kElems;
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const typename F::type kf = F::template load_lds<TL>(tile, sub * 32 + c32, s, hh);
#pragma unroll
    for (int nb = 0; nb < MB; ++nb) {
      if (s == 0) {
        f32x16 zero;
#pragma unroll
        for (int v = 0; v < 16; ++v) zero[v] = 0.f;
        acc[nb] = F::mfma(kf, qf[nb][s], zero);
      } else {
        acc[nb] = F::mfma(kf, qf[nb][s], acc[nb]);
      }
    }
  }
}

// The finished logits of a sub-tile (first key kb) folded into the rows' running
// (reference, sum) pairs.  Key j is visible to window row r iff j <= n_p + r (and j < n);
// kTail: some key of the sub-tile may be hidden or lie past the end.
template <int MB, bool kTail>
__device__ __forceinline__ void pass1_sums(const f32x16 (&acc)[MB], int kb, float (&mref)[MB], float (&lsum)[MB],
                                           float cv, int n, int n_p, int c32, int hh) {
#pragma unroll
  for (int nb = 0; nb < MB; ++nb) {
    const int last = min(n_p + nb * 32 + c32, n - 1) - kb - 4 * hh;
    auto hidden = [&](int v) { return kTail && 8 * (v / 4) + (v % 4) > last; };
    float bsum[2];                        // two chains: consecutive additions do not wait on each other
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float e = hidden(v) ? 0.f : fast_exp2(fmaf(acc[nb][v], cv, -mref[nb]));
      if (v < 2) bsum[v] = e;
      else bsum[v & 1] += e;
    }
    add_block_sum<kTail>(acc[nb], bsum[0] + bsum[1], mref[nb], lsum[nb], cv, last);
  }
}

// Packed kernels (kSlices > 1): as many slices share a workgroup, G waves each, every slice with tile buffers of its own.  A
// workgroup's waves are dealt over the compute unit's four SIMDs in turn, so that a group of 5 or 6 heads alone leaves two waves on
// one SIMD and one on the others, and the barriers make every wave wait for the doubled SIMD; three slices of 5 waves (or two of
// 6) fill the SIMDs almost evenly.  Slices past the last one (the final workgroup) repeat the last slice's work and store nothing.
struct WaveRole {
  int slice, w;      // the wave's slice and its head within the group
  int sub;           // the slice's place in the workgroup
  bool live;         // false: a repeat of the last slice, stores nothing
};
template <int kSlices>
__device__ __forceinline__ WaveRole wave_role(const ScoreArgs& a) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);       // wave index, known uniform
  if (kSlices == 1) return WaveRole{(int)blockIdx.y, w, 0, true};
  const int sub = w / a.group, slice = blockIdx.y * kSlices + sub;
  return WaveRole{min(slice, a.n_slices - 1), w - sub * a.group, sub, slice < a.n_slices};
}

template <typename T, int D, int MB, int kSlices = 1>
__global__ __launch_bounds__(kSlices > 1 ? 1024 : 512) void scores_pass1(ScoreArgs a) {
  using F = Frag<T>;
  using TL = Tile<T, D>;
  constexpr int kSteps = D / F::kElems;
  // double buffer: tile t+1 is in flight while tile t is consumed (rings of three and four tiles
  // measured no faster, with waits for the oldest tile alone as well)
  __shared__ __attribute__((aligned(1024))) char all_tiles[kSlices * 2 * TL::kBytes];

  const WaveRole role = wave_role<kSlices>(a);
  const int slice = role.slice, w = role.w;
  int l, b, g;
  slice_coords(a, slice, l, b, g);
  char* tiles = all_tiles + role.sub * (2 * TL::kBytes);
  const int lane = threadIdx.x & 63, c32 = lane & 31, hh = lane >> 5;
  const int n_waves = a.group;
  constexpr int s_w = MB * 32;
  const T* q = in_global(reinterpret_cast<const T*>(a.q_win ? a.q_win[l] : a.one.q)) + b * a.qs[0] + (int64_t)(g * a.group + w) * a.qs[1];
  const int64_t tok_bytes = a.ks[2] * (int64_t)sizeof(T);
  // address of key 0 of the slice (keys below key_lo are not behind the pointer and never touched)
  const char* kbase = reinterpret_cast<const char*>(in_global(reinterpret_cast<const T*>(a.k ? a.k[l] : a.one.k)) + b * a.ks[0] + (int64_t)g * a.ks[1]) -
                      (int64_t)a.key_lo * tok_bytes;

  const int key0 = a.key0 + blockIdx.x * a.wg_keys;
  const int key_end = min(key0 + a.wg_keys, min(a.n, a.key_hi));
  const int n_tiles = (key_end - key0 + kTileKeys - 1) / kTileKeys;
  TileMover<T, D> mover;
  mover.init(kbase, tok_bytes, min(a.n, a.key_hi) - 1, w, n_waves, lane);
  mover.issue(tiles, key0);

  typename F::type qf[MB][kSteps];
  load_q<T, D, MB>(qf, q, a.qs[2], c32, hh);
  float mref[MB], lsum[MB];
#pragma unroll
  for (int nb = 0; nb < MB; ++nb) { mref[nb] = 0.f; lsum[nb] = 0.f; }
  float cv = a.c;
  asm volatile("" : "+v"(cv));     // a vector register: a scalar operand halves the issue rate of the multiply

  // The MFMAs of a 32-key sub-tile, then the exponentials and sums of its logits.  An explicit
  // software pipeline over two accumulator sets (each k-step's MFMAs followed by a share of the
  // previous sub-tile's vector work, as in pass 2) measured 10 % slower here: it costs a wave
  // per SIMD in registers, and under the chip's power limit overlapping the two pipes buys no time.
  f32x16 acc[MB];
  // The (reference, sum) pairs of a finished granule: the two lane halves of each window row merged.
  float* out = a.part + ((int64_t)slice * a.n_granules * a.group + w) * s_w * 2;
  const int granule_shift = __builtin_ctz(a.granule), granule_tiles = a.granule / kTileKeys;      // powers of two
  auto finish = [&](int t) {
    if (((t + 1) & (granule_tiles - 1)) != 0 && t + 1 != n_tiles) return;
    float* o = out + (int64_t)((key0 + t * kTileKeys) >> granule_shift) * (a.group * s_w) * 2;
#pragma unroll
    for (int nb = 0; nb < MB; ++nb) {
      const float2 pair = merge_halves(mref[nb], lsum[nb]);
      if (hh == 0 && role.live) *reinterpret_cast<float2*>(o + (nb * 32 + c32) * 2) = pair;
      mref[nb] = 0.f;
      lsum[nb] = 0.f;
    }
  };
  auto tail_of = [&](int kb) { return kb + 31 > a.n_p; };      // some key of the sub-tile may be hidden or past the end

  // Stage t consumes buffer t mod 2 (known at compile time: the operand reads then address LDS
  // with immediate offsets) and refills the other one, which stage t-1 consumed.
  auto stage = [&](auto slot_c, int t) {
    constexpr int kSlot = decltype(slot_c)::value;
    const char* cur = tiles + kSlot * TL::kBytes;
    char* nxt = tiles + (kSlot ^ 1) * TL::kBytes;
    wait_vmem();
    __syncthreads();                 // tile t complete in `cur`; everyone is done reading `nxt`
    const int t0 = key0 + t * kTileKeys;
    if (t + 1 < n_tiles) mover.issue(nxt, t0 + kTileKeys);
#pragma unroll
    for (int sub = 0; sub < kTileKeys / 32; ++sub) {
      const int kb = t0 + sub * 32;
      if (kb >= key_end) break;
      pass1_logits<T, D, MB>(cur, sub, qf, acc, c32, hh);
      if (tail_of(kb))
        pass1_sums<MB, true>(acc, kb, mref, lsum, cv, a.n, a.n_p, c32, hh);
      else
        pass1_sums<MB, false>(acc, kb, mref, lsum, cv, a.n, a.n_p, c32, hh);
    }
  };
  for (int t = 0; t < n_tiles; t += 2) {
    stage(std::integral_constant<int, 0>{}, t);
    finish(t);
    if (t + 1 < n_tiles) {
      stage(std::integral_constant<int, 1>{}, t + 1);
      finish(t + 1);
    }
  }
}

// Combine the granules' pairs of a window row into lse2 = log2 sum_j 2^(t_j).  Four chains share
// a row: each folds every fourth granule into a running (reference, sum) pair in one sweep, the four
// pairs are merged in a fixed order, so that the result does not depend on how the chains are dealt to lanes: kChains
// of a lane's own (4, 2 or 1), merged by then into one pair; `partner` folds into it, in place, the pairs of the other lanes of the
// row, the pair of the earlier chains first.  p: the row's first pair; chain0: the lane's first chain; all of a row's lanes get the result.
// Bound by latency: a chain of loads, then of fp64 additions.  With four lanes a row and 16 rows a turn, pass 2 of one layer of
// 8192 keys waited 5.6 us for its first tile (8 x 4 heads of 128; 16.5 us in all, now 12.6).
constexpr int kCombineAhead = 8;          // pairs in flight per chain
template <int kChains>
struct RowPairs {
  float2 x[kChains][kCombineAhead];
  // the pairs of granules from `first` on; past the last one it is repeated, until drop_absent
  __device__ __forceinline__ void load(const float* p, int rows_per_slice, int n_granules, int first, int chain0) {
#pragma unroll
    for (int u = 0; u < kCombineAhead; ++u)
#pragma unroll
      for (int c = 0; c < kChains; ++c) {
        const int g = min(first + 4 * u + chain0 + c, n_granules - 1);
        x[c][u] = *reinterpret_cast<const float2*>(p + (int64_t)g * rows_per_slice * 2);
      }
  }
  // Separate from the loads, so that no masks are held while they are under way.
  __device__ __forceinline__ void drop_absent(int left /* granules from the lane's first chain's first pair on */) {
    asm volatile("" : "+v"(left));
#pragma unroll
    for (int u = 0; u < kCombineAhead; ++u)
#pragma unroll
      for (int c = 0; c < kChains; ++c)
        if (4 * u + c >= left) x[c][u] = make_float2(kMasked, 0.f);
  }
};
template <int kChains, typename Partner>
__device__ __forceinline__ float combine_row(RowPairs<kChains>& pairs, const float* p, int rows_per_slice, int n_granules, int chain0, Partner partner) {
  float m[4];
  double s[4];
#pragma unroll
  for (int c = 0; c < kChains; ++c) { m[c] = kMasked; s[c] = 0.0; }
  for (int first = 0;;) {
    pairs.drop_absent(n_granules - first - chain0);
    // The references of a sweep are one and the same (0) in most layers: every factor below is 1 then.  The test is the
    // wave's, its branch parts no lanes.
    const float ref = pairs.x[0][0].x;
    uint32_t other = 0;                   // bits in which some reference differs
    auto compare = [&](float r) { other |= r == kMasked ? 0u : __float_as_uint(r) ^ __float_as_uint(ref); };
#pragma unroll
    for (int c = 0; c < kChains; ++c) {
      compare(m[c]);
#pragma unroll
      for (int u = 0; u < kCombineAhead; ++u) {
        compare(pairs.x[c][u].x);
        asm volatile("" : "+v"(other));   // one after the other: the masks of all at once fill the scalar registers
      }
    }
    if (__all(other == 0)) {
#pragma unroll
      for (int u = 0; u < kCombineAhead; ++u)
#pragma unroll
        for (int c = 0; c < kChains; ++c) s[c] += (double)pairs.x[c][u].y;
#pragma unroll
      for (int c = 0; c < kChains; ++c) m[c] = ref;
    } else {
#pragma unroll
      for (int c = 0; c < kChains; ++c) {
        float top = m[c];
#pragma unroll
        for (int u = 0; u < kCombineAhead; ++u) top = fmaxf(top, pairs.x[c][u].x);
        s[c] *= (double)fast_exp2(m[c] - top);
        m[c] = top;
#pragma unroll
        for (int u = 0; u < kCombineAhead; ++u) s[c] += (double)pairs.x[c][u].y * (double)fast_exp2(pairs.x[c][u].x - top);
      }
    }
    first += 4 * kCombineAhead;
    if (first >= n_granules) break;
    pairs.load(p, rows_per_slice, n_granules, first, chain0);
  }
  auto merge = [](float& m0, double& s0, float m1, double s1) {
    const float mm = fmaxf(m0, m1);
    s0 = s0 * (double)fast_exp2(m0 - mm) + s1 * (double)fast_exp2(m1 - mm);
    m0 = mm;
  };
  if (kChains == 4) merge(m[2], s[2], m[3], s[3]);
  if (kChains >= 2) merge(m[0], s[0], m[1], s[1]);
  if (kChains == 4) merge(m[0], s[0], m[2], s[2]);
  else partner(m[0], s[0], merge);
  // log2 of the sum from its exponent and mantissa: the instruction's error is that of a value below 1; rounded once
  return (float)((double)m[0] + (double)__builtin_amdgcn_frexp_exp(s[0]) + (double)__builtin_amdgcn_logf((float)__builtin_amdgcn_frexp_mant(s[0])));
}
// The other chains of a row in neighbouring lanes, one chain each: lanes 4i .. 4i + 3.
__device__ __forceinline__ auto quad_partner(int chain) {
  return [chain](float& m, double& s, auto merge) {
    auto with = [&](float om, double os, bool upper) {     // the lower lane's pair first: the same order in both partners
      float a = upper ? om : m, b = upper ? m : om;
      double x = upper ? os : s, y = upper ? s : os;
      merge(a, x, b, y);
      m = a;
      s = x;
    };
    with(dpp_step<0xB1, 0xf, true>(m), dpp_step<0xB1, 0xf, true>(s), chain & 1);      // quad_perm [1, 0, 3, 2]
    with(dpp_step<0x4E, 0xf, true>(m), dpp_step<0x4E, 0xf, true>(s), chain & 2);      // quad_perm [2, 3, 0, 1]
  };
}

// Two chains each in lanes i and i + 32.
__device__ __forceinline__ auto half_partner() {
  return [](float& m, double& s, auto merge) {
    uint32_t w[3];
    __builtin_memcpy(w, &m, 4);
    __builtin_memcpy(w + 1, &s, 8);
    uint32_t lower[3], upper[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const auto r = __builtin_amdgcn_permlane32_swap(w[i], w[i], false, false);
      lower[i] = r[0];
      upper[i] = r[1];
    }
    float om;
    double os;
    __builtin_memcpy(&m, lower, 4);
    __builtin_memcpy(&s, lower + 1, 8);
    __builtin_memcpy(&om, upper, 4);
    __builtin_memcpy(&os, upper + 1, 8);
    merge(m, s, om, os);
  };
}

__global__ __launch_bounds__(256) void scores_combine(ScoreArgs a, int rows_per_slice, int64_t total_rows) {
  const int64_t i = min(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2, total_rows - 1);
  const int part = threadIdx.x & 3;
  const int64_t slice = i / rows_per_slice;
  const int row = (int)(i % rows_per_slice);
  const float* p = a.part + (slice * a.n_granules * rows_per_slice + row) * 2;
  RowPairs<1> pairs;
  pairs.load(p, rows_per_slice, a.n_granules, 0, part);
  const float lse = combine_row(pairs, p, rows_per_slice, a.n_granules, part, quad_partner(part));
  if (part == 0) a.lse[i] = lse;
}

// Row normalisers handed over by the caller (natural log, [B, H_q, S_w] per layer) -> log2 domain
// in the workspace layout, which is the same order: slice (l, b, g), then head within the group, row.
__global__ void scores_import_lse(ScoreArgs a, const float* const* row_lse, int64_t per_layer, int64_t total) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  a.lse[i] = in_global(row_lse ? row_lse[i / per_layer] : a.one.row_lse)[i % per_layer] * 1.4426950408889634f;
}

// ------------------------------------------------------------------------------------------
// Pass 2: normalised weights on the prefix columns; column Mean/Var, entropy, group mean.
// ------------------------------------------------------------------------------------------
// One period of pass 2.  kMfma: the MFMAs of sub-tile `sub` of `tile` accumulate into `dst`,
// starting from `init`, which holds -lse2/c of the lane's window rows, so that the accumulator
// times c is already the log2 of the weight.  kValu: the finished accumulators in `src` are
// turned into weights and column sums; with both, the vector work is dealt out over the MFMA
// steps and a scheduling barrier per step pins the interleaving.
// src[mb][v]: window row mb*32 + 8*(v/4) + 4*hh + (v%4) of the key column this lane owns.
// kTail: the column may lie at or beyond the end of the chunk (col_valid false): its weights are
// forced to zero.  kPivot: the sums are taken about the weight of window row 0 (Var and Mean*Var
// indicators: sum p^2 - (sum p)^2/S_w would cancel in fp32 where the weights barely move).
template <typename T, int D, int MB, bool kMfma, bool kValu, bool kTail, bool kPivot>
__device__ __forceinline__ void pass2_period(const char* tile, int sub,
                                             const typename Frag<T>::type (&qf)[MB][D / Frag<T>::kElems],
                                             const f32x16 (&init)[MB], f32x16 (&dst)[MB], const f32x16 (&src)[MB],
                                             float cv, bool col_valid, float (&entv)[2], ColSums& out,
                                             int c32, int hh) {
  using F = Frag<T>;
  using TL = Tile<T, D>;
  constexpr int kSteps = D / F::kElems;
  constexpr int kGroups = 4 * MB;      // groups of four logits per lane in a sub-tile
  constexpr int kAhead = 2;            // operand reads in flight ahead of their MFMA step
  float spv[2] = {0.f, 0.f}, sp2v[2] = {0.f, 0.f};
  float pivot = 0.f;
  auto logit = [&](int mb, int v) { return (kTail && !col_valid) ? -1.0e30f : src[mb][v]; };
  if (kValu && kPivot) {
    // the weight of window row 0 lives in the lower lane half (mb 0, v 0); both halves take it
    const float p0 = fast_exp2(logit(0, 0) * cv);
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(p0), __float_as_uint(p0), false, false);
    pivot = __uint_as_float(r[0]);
  }
  typename F::type kf[kSteps];
  if (kMfma) {
#pragma unroll
    for (int s = 0; s < kAhead && s < kSteps; ++s) kf[s] = F::template load_lds<TL>(tile, sub * 32 + c32, s, hh);
  }
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    if (kMfma) {
      if (s + kAhead < kSteps) kf[s + kAhead] = F::template load_lds<TL>(tile, sub * 32 + c32, s + kAhead, hh);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) dst[mb] = F::mfma(qf[mb][s], kf[s], s == 0 ? init[mb] : dst[mb]);
    }
    if (kValu) {
#pragma unroll
      for (int gi = 0; gi < kGroups; ++gi) {
        if (gi * kSteps / kGroups != s) continue;
        const int mb = gi / 4, v4 = (gi % 4) * 4;
        float x[4], p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = logit(mb, v4 + i);
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = fast_exp2(x[i] * cv);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float pd = kPivot ? p[i] - pivot : p[i];
          spv[i & 1] += pd;
          sp2v[i & 1] = fmaf(pd, pd, sp2v[i & 1]);
          entv[i & 1] = fmaf(p[i], x[i], entv[i & 1]);      // sum p * log2(p) / c
        }
        // keep the accumulation in this step (it would otherwise be sunk to the end of the period)
        asm volatile("" : "+v"(spv[0]), "+v"(spv[1]), "+v"(sp2v[0]), "+v"(sp2v[1]), "+v"(entv[0]), "+v"(entv[1]));
      }
    }
    if (kMfma && kValu) __builtin_amdgcn_sched_barrier(0);
  }
  if (kValu) {
    out.sp = spv[0] + spv[1];
    out.sp2 = sp2v[0] + sp2v[1];
    out.pivot = pivot;
  }
}

// Pass 2 comes with and without the code to combine the pairs of pass 1 by itself (kCombine).  The software-pipelined form has
// it for a workgroup per compute unit only (its registers are full): 8192 keys of one layer, 8 x 4 heads, scores of 64 rows
// 32.4 -> 29.7 us with it, 512 workgroups of 8 layers of 1000 keys 32.9 -> 33.9.
template <typename T, int MB> constexpr bool kPipelinedForm = sizeof(T) == 2 && MB == 2;

template <typename T, int D, int MB, bool kPivot, bool kCombine, int kSlices = 1>
__global__ __launch_bounds__(kSlices > 1 ? 1024 : 512) void scores_pass2(ScoreArgs a) {
  using F = Frag<T>;
  using TL = Tile<T, D>;
  constexpr int kSteps = D / F::kElems;
  // double buffer: tile t+1 is in flight while tile t is consumed (deeper rings measured no faster)
  __shared__ __attribute__((aligned(1024))) char all_tiles[kSlices * 2 * TL::kBytes];
  // I_q of the G heads for two tiles in turn: the flush of one tile reads one buffer in the
  // stage in which the other is written, and a barrier separates the stages
  __shared__ float iq_lds[2][kSlices > 1 ? 16 : 8][kTileKeys];

  const WaveRole role = wave_role<kSlices>(a);
  const int slice = role.slice, w = role.w;
  int l, b, g;
  slice_coords(a, slice, l, b, g);
  char* tiles = all_tiles + role.sub * (2 * TL::kBytes);
  auto iq_row = [&](int buf, int wave) { return iq_lds[buf][role.sub * a.group + wave]; };
  const int lane = threadIdx.x & 63, c32 = lane & 31, hh = lane >> 5;
  const int n_waves = a.group;
  constexpr int s_w = MB * 32;
  const T* q = in_global(reinterpret_cast<const T*>(a.q_win ? a.q_win[l] : a.one.q)) + b * a.qs[0] + (int64_t)(g * a.group + w) * a.qs[1];
  const int64_t tok_bytes = a.ks[2] * (int64_t)sizeof(T);
  // address of key 0 of the slice (keys below key_lo are not behind the pointer and never touched)
  const char* kbase = reinterpret_cast<const char*>(in_global(reinterpret_cast<const T*>(a.k ? a.k[l] : a.one.k)) + b * a.ks[0] + (int64_t)g * a.ks[1]) -
                      (int64_t)a.key_lo * tok_bytes;

  const int key0 = a.key0 + blockIdx.x * a.wg_keys;
  const int key_end = min(key0 + a.wg_keys, min(a.n_p, a.key_hi));
  const int n_tiles = (key_end - key0 + kTileKeys - 1) / kTileKeys;
  TileMover<T, D> mover;
  mover.init(kbase, tok_bytes, min(a.n, a.key_hi) - 1, w, n_waves, lane);
  // Few workgroups: each wave combines its own rows' pairs beside the first tile's transfer, which spares the launch
  // in between; their loads go out ahead of everything else.
  constexpr int kChains = s_w / 16;        // 32 rows: two lanes each
  const int chain0 = MB == 1 ? 2 * hh : 0;
  const float* row_pairs = a.part + ((int64_t)slice * a.n_granules * (a.group * s_w) + w * s_w + (lane & (s_w - 1))) * 2;
  RowPairs<kChains> pairs;
  if (kCombine) pairs.load(row_pairs, a.group * s_w, a.n_granules, 0, chain0);
  mover.issue(tiles, key0);

  typename F::type qf[MB][kSteps];
  load_q<T, D, MB>(qf, q, a.qs[2], c32, hh);
  // -lse2/c of the lane's window rows, in the accumulator layout: the MFMA chain of a sub-tile
  // starts from it, so its result times c is the log2 of the normalised weight.
  f32x16 init[MB];
  const float neg_inv_c = -1.0f / a.c;
  auto row_of = [&](int mb, int v) { return mb * 32 + 8 * (v / 4) + 4 * hh + (v % 4); };
  auto load_init = [&](const float* lse) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) init[mb][v] = lse[row_of(mb, v)] * neg_inv_c;
  };
  if (kCombine) {
    float* mine = iq_row(0, w);            // the wave's I_q row serves until its first tile is done
    mine[lane & (s_w - 1)] = combine_row(pairs, row_pairs, a.group * s_w, a.n_granules, chain0, half_partner());
    load_init(mine);
  } else {
    load_init(a.lse + (int64_t)slice * (a.group * s_w) + w * s_w);
  }
  float cv = a.c;
  asm volatile("" : "+v"(cv));     // a vector register: a scalar operand halves the issue rate of the multiply

  float entv[2] = {0.f, 0.f};      // sum p * log2(p) / c over this lane's logits, two chains
  float var_acc = 0.f;
  float* raw = a.raw + (int64_t)slice * a.n_p;
  // Two accumulator sets (logits of even / odd sub-tiles) let one sub-tile's MFMAs overlap the
  // previous one's statistics.  Measured, this pays for bf16 with two row blocks per wave
  // (S_w = 64); with one row block the periods are too short and the plain order is faster, and
  // the fp32 kernels hold twice the query registers (128 of them at two row blocks of 128) and would spill.  Those run
  // the two phases of a sub-tile one after the other on a single set.
  constexpr bool kPipelined = kPipelinedForm<T, MB>;
  f32x16 acc_a[MB], acc_b[MB];
  ColSums cs0{}, cs1{};

  // Group mean of the G heads' I_q for the 64 keys of tile t, one key per lane; the waves take
  // the tiles in turn.
  auto flush = [&](int t) {
    if (t % n_waves != w) return;
    const int key = key0 + t * kTileKeys + lane;
    float s = 0.f;
    for (int ww = 0; ww < a.group; ++ww) s += iq_row(t & 1, ww)[lane];
    if (key < key_end && role.live) raw[key] = s * a.inv_g;
  };
  // Entropy and variance sums of the granule that ends with tile t.
  const int granule_shift = __builtin_ctz(a.granule), granule_tiles = a.granule / kTileKeys;      // powers of two
  auto finish = [&](int t) {
    const float ent = wave_sum((entv[0] + entv[1]) * cv), var = wave_sum(var_acc);
    const int64_t granule = (key0 + t * kTileKeys) >> granule_shift;
    if (lane == 0 && role.live)
      *reinterpret_cast<float2*>(a.hv + (((int64_t)slice * a.n_granules_p + granule) * a.group + w) * 2) = make_float2(ent, var);
    entv[0] = entv[1] = var_acc = 0.f;
  };
  // Tile t: its first sub-tile's MFMAs run beside the statistics of tile t-1's second sub-tile,
  // its second sub-tile's MFMAs beside the statistics of its first.  Only the last tile of a
  // chunk can hold columns at or beyond key_end.
  // Stage t consumes buffer t mod 2 (known at compile time: the operand reads then address LDS
  // with immediate offsets) and refills the other one, which stage t-1 consumed.
  constexpr int kFlushLag = kPipelined ? 2 : 1;     // stages between a tile's MFMAs and the flush of its I_q
  auto stage = [&](auto slot_c, int t, auto tail_c) {
    constexpr int kSlot = decltype(slot_c)::value;
    constexpr bool kTail = decltype(tail_c)::value;
    const char* cur = tiles + kSlot * TL::kBytes;
    char* nxt = tiles + (kSlot ^ 1) * TL::kBytes;
    wait_vmem();
    __syncthreads();       // tile t complete in `cur`; every wave is done with `nxt` and with the I_q buffer written next
    const int t0 = key0 + t * kTileKeys;
    if (t + 1 < n_tiles) mover.issue(nxt, t0 + kTileKeys);
    if (t >= kFlushLag) flush(t - kFlushLag);
    const bool v0 = t0 + c32 < key_end, v1 = t0 + 32 + c32 < key_end;
    if (kPipelined) {
      if (t == 0) {
        pass2_period<T, D, MB, true, false, false, kPivot>(cur, 0, qf, init, acc_a, acc_b, cv, true, entv, cs1, c32, hh);
      } else {
        // statistics of tile t-1's second sub-tile: never a tail, tile t-1 is not the last
        pass2_period<T, D, MB, true, true, false, kPivot>(cur, 0, qf, init, acc_a, acc_b, cv, true, entv, cs1, c32, hh);
        iq_row((t - 1) & 1, w)[lane] = pass2_tile_stats<kPivot>(cs0, cs1, a, hh, var_acc);
        if (kSlot == 0 && (t & (granule_tiles - 1)) == 0) finish(t - 1);      // granules of S_w = 64 are an even number of tiles
      }
      pass2_period<T, D, MB, true, true, kTail, kPivot>(cur, 1, qf, init, acc_b, acc_a, cv, v0, entv, cs0, c32, hh);
    } else {
      pass2_period<T, D, MB, true, false, false, kPivot>(cur, 0, qf, init, acc_a, acc_a, cv, true, entv, cs0, c32, hh);
      pass2_period<T, D, MB, false, true, kTail, kPivot>(cur, 0, qf, init, acc_a, acc_a, cv, v0, entv, cs0, c32, hh);
      pass2_period<T, D, MB, true, false, false, kPivot>(cur, 1, qf, init, acc_a, acc_a, cv, true, entv, cs1, c32, hh);
      pass2_period<T, D, MB, false, true, kTail, kPivot>(cur, 1, qf, init, acc_a, acc_a, cv, v1, entv, cs1, c32, hh);
      iq_row(t & 1, w)[lane] = pass2_tile_stats<kPivot>(cs0, cs1, a, hh, var_acc);
      if (((t + 1) & (granule_tiles - 1)) == 0 || t + 1 == n_tiles) finish(t);
    }
  };
  const bool last_partial = (key_end - key0) % kTileKeys != 0;
  auto stage_at = [&](auto slot_c, int t) {
    if (t + 1 == n_tiles && last_partial) stage(slot_c, t, std::true_type{});
    else stage(slot_c, t, std::false_type{});
  };
  const int loop_tiles = kPipelined ? granule_tiles : n_tiles;
  for (int t0 = 0; t0 < n_tiles; t0 += loop_tiles) {
    const int t1 = min(t0 + loop_tiles, n_tiles);
    for (int t = t0; t < t1; t += 2) {
      stage_at(std::integral_constant<int, 0>{}, t);
      if (t + 1 < t1) stage_at(std::integral_constant<int, 1>{}, t + 1);
    }
  }
  if (kPipelined) {    // drain: statistics of the last sub-tile, then of the last tile
    const bool v1 = key0 + (n_tiles - 1) * kTileKeys + 32 + c32 < key_end;
    if (last_partial)
      pass2_period<T, D, MB, false, true, true, kPivot>(tiles, 0, qf, init, acc_a, acc_b, cv, v1, entv, cs1, c32, hh);
    else
      pass2_period<T, D, MB, false, true, false, kPivot>(tiles, 0, qf, init, acc_a, acc_b, cv, true, entv, cs1, c32, hh);
    iq_row((n_tiles - 1) & 1, w)[lane] = pass2_tile_stats<kPivot>(cs0, cs1, a, hh, var_acc);
    finish(n_tiles - 1);
  }
  __syncthreads();
  if (kFlushLag == 2 && n_tiles >= 2) flush(n_tiles - 2);
  flush(n_tiles - 1);
}

// Eq. 6 per (layer, sequence): fixed-order fp64 reduction of the chunk sums, then the powers, by one
// workgroup of kPrefThreads.  Bound by latency: at 128K keys a layer has 2048 pairs, eight loads per
// thread (with one wave of 64 threads the 32 dependent rounds took 17 us).
struct PrefArgs {
  const float* hv;             // the score pass's partial sums
  int32_t n_layers, batch, h_kv, group, n_granules_p;
  double inv_tau1, inv_tau2;
  double* pref;                // [B] rows of pref_ld
  double* hv_out;              // [B, n_layers, 2] or NULL
  int32_t pref_ld, hv_ld;
  uint32_t* flags;             // of a layer alone, or NULL (LayerPointers)
  uint32_t ticket;
};
constexpr int kPrefThreads = 256;

// What becomes of an entry's sums.
__device__ __forceinline__ void store_preference(const PrefArgs& a, int entry, double e, double v) {
  const int l = entry / a.batch, b = entry % a.batch;
  const double heads = (double)(a.h_kv * a.group);
  // Both are non-negative by definition; with nearly one-hot attention the fp32 sums can come
  // out a rounding error below zero, which the fractional powers below would turn into NaN.
  const double h_l = fmax(-0.6931471805599453 * e / heads, 0.0);   // sum p*log2 p -> -sum p ln p
  const double v_l = fmax(v / heads, 0.0);
  // (a power costs half a microsecond of a chain that the plan waits for, and the usual one is the first)
  const double h_pow = a.inv_tau1 == 1.0 ? h_l : pow(h_l, a.inv_tau1), v_pow = a.inv_tau2 == 1.0 ? v_l : pow(v_l, a.inv_tau2);
  a.pref[(int64_t)b * a.pref_ld + l] = h_pow * v_pow;
  if (a.hv_out) {
    a.hv_out[((int64_t)b * a.hv_ld + l) * 2 + 0] = h_l;
    a.hv_out[((int64_t)b * a.hv_ld + l) * 2 + 1] = v_l;
  }
  if (a.flags) {                // a host that watches the flag finds the preference in its memory
    __threadfence_system();
    __hip_atomic_store(a.flags + b, a.ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

__device__ __forceinline__ void preference_of(const PrefArgs& a, int entry) {
  __shared__ double red[2][kPrefThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int count = a.h_kv * a.n_granules_p * a.group;
  const float2* base = reinterpret_cast<const float2*>(a.hv) + (int64_t)entry * count;
  double e = 0.0, v = 0.0;
  for (int i = tid; i < count; i += kPrefThreads) {
    const float2 x = base[i];
    e += (double)x.x;
    v += (double)x.y;
  }
  e = wave_sum(e);
  v = wave_sum(v);
  if (lane == 0) { red[0][tid >> 6] = e; red[1][tid >> 6] = v; }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int w = 1; w < kPrefThreads / 64; ++w) { e += red[0][w]; v += red[1][w]; }
    store_preference(a, entry, e, v);
  }
}

// The same sums by one wave, which does the four waves' parts side by side.
__device__ __forceinline__ void preference_of_wave(const PrefArgs& a, int entry, int lane) {
  constexpr int kParts = kPrefThreads / 64;
  const int count = a.h_kv * a.n_granules_p * a.group;
  const float2* base = reinterpret_cast<const float2*>(a.hv) + (int64_t)entry * count;
  double e[kParts] = {}, v[kParts] = {};
  constexpr int kAhead = 4;                 // loads of a part in flight
  for (int i0 = lane; i0 - lane < count; i0 += kAhead * kPrefThreads) {
    float2 x[kAhead][kParts];
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
#pragma unroll
      for (int w = 0; w < kParts; ++w) x[u][w] = base[min(i0 + u * kPrefThreads + 64 * w, count - 1)];
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
#pragma unroll
      for (int w = 0; w < kParts; ++w)
        if (i0 + u * kPrefThreads + 64 * w < count) {
          e[w] += (double)x[u][w].x;
          v[w] += (double)x[u][w].y;
        }
  }
#pragma unroll
  for (int w = 0; w < kParts; ++w) {
    e[w] = wave_sum(e[w]);
    v[w] = wave_sum(v[w]);
  }
#pragma unroll
  for (int w = 1; w < kParts; ++w) { e[0] += e[w]; v[0] += v[w]; }
  if (lane == 0) store_preference(a, entry, e[0], v[0]);
}

__global__ __launch_bounds__(kPrefThreads) void layer_preference_kernel(PrefArgs a) { preference_of(a, blockIdx.x); }

// Stride-1 max-pool over the prefix positions, edges clipped (Sec. 4.3 pooling layer).
// A workgroup stages kPoolSpan consecutive positions plus the halo in LDS with coalesced loads,
// so that every un-pooled value is read from memory once.
constexpr int kPoolSpan = 2048;
constexpr int kPoolMaxHalf = 64;        // widest supported pooling window: 2*64+1
constexpr int kPoolQuadHalf = 4;        // widest half window of the four-outputs-per-lane path

// Four consecutive outputs from the twelve staged values around them (w[4..7] are the outputs' own
// positions).
template <int kHalf>
__device__ __forceinline__ float4 pool_quad(const float (&w)[12]) {
  float o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float m = w[4 + k];
#pragma unroll
    for (int d = 1; d <= kHalf; ++d) m = fmaxf(m, fmaxf(w[4 + k - d], w[4 + k + d]));
    o[k] = m;
  }
  return make_float4(o[0], o[1], o[2], o[3]);
}

// Span blockIdx.x of one slice.
__device__ __forceinline__ void pool_span(const ScoreArgs& a, int slice) {
  // position j0 + i of the span sits at win[kPoolMaxHalf + i]
  __shared__ __attribute__((aligned(16))) float win[kPoolSpan + 2 * kPoolMaxHalf];
  int l, b, g;
  slice_coords(a, slice, l, b, g);
  const int half = a.pool / 2;
  const int j0 = blockIdx.x * kPoolSpan;
  const int span = min(kPoolSpan, a.n_p - j0);
  const float* raw = a.raw + (int64_t)slice * a.n_p;
  float* out = in_global(a.indicator ? a.indicator[l] : a.one.indicator) + ((int64_t)b * a.h_kv + g) * a.n_p;
  // Rows of a multiple of four positions at 16-byte aligned addresses, windows of at most nine:
  // 16-byte loads and stores, four outputs per lane from three 16-byte LDS reads.
  const bool quads = a.n_p % 4 == 0 && half <= kPoolQuadHalf &&
                     ((reinterpret_cast<uintptr_t>(raw) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
  if (quads) {
    const float4* raw4 = reinterpret_cast<const float4*>(raw + j0);
    for (int q = threadIdx.x; q < span / 4; q += 256)
      *reinterpret_cast<float4*>(&win[kPoolMaxHalf + 4 * q]) = raw4[q];
    if (threadIdx.x < 8) {            // four positions on either side; clipped edges never win the max
      const int i = threadIdx.x < 4 ? (int)threadIdx.x - 4 : span + (int)threadIdx.x - 4;
      const int j = j0 + i;
      win[kPoolMaxHalf + i] = (j >= 0 && j < a.n_p) ? raw[j] : -INFINITY;
    }
    __syncthreads();
    float4* out4 = reinterpret_cast<float4*>(out + j0);
    for (int q = threadIdx.x; q < span / 4; q += 256) {
      float w[12];
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        const float4 x = *reinterpret_cast<const float4*>(&win[kPoolMaxHalf + 4 * q - 4 + 4 * v]);
        w[4 * v] = x.x; w[4 * v + 1] = x.y; w[4 * v + 2] = x.z; w[4 * v + 3] = x.w;
      }
      float4 r;
      switch (half) {
        case 0: r = pool_quad<0>(w); break;
        case 1: r = pool_quad<1>(w); break;
        case 2: r = pool_quad<2>(w); break;
        case 3: r = pool_quad<3>(w); break;
        default: r = pool_quad<4>(w); break;
      }
      out4[q] = r;
    }
    return;
  }
  for (int i = (int)threadIdx.x - half; i < span + half; i += 256) {
    const int j = j0 + i;
    win[kPoolMaxHalf + i] = (j >= 0 && j < a.n_p) ? raw[j] : -INFINITY;     // clipped edges never win the max
  }
  __syncthreads();
  for (int i = threadIdx.x; i < span; i += 256) {
    float m = win[kPoolMaxHalf + i];
    for (int k = 1; k <= half; ++k) m = fmaxf(m, fmaxf(win[kPoolMaxHalf + i - k], win[kPoolMaxHalf + i + k]));
    out[j0 + i] = m;
  }
}

// With kPref the first `pref_rows` rows of the grid compute the layer preferences beside the pooling
// (both follow pass 2 and neither reads the other): a launch and its latency less.
template <bool kPref>
__global__ __launch_bounds__(256) void pool_indicator(ScoreArgs a, PrefArgs pa, int pref_rows) {
  static_assert(kPrefThreads == 256, "the preference shares the pooling's workgroups");
  if (kPref && (int)blockIdx.y < pref_rows) {
    const int entry = blockIdx.y * gridDim.x + blockIdx.x;
    if (entry < pa.n_layers * pa.batch) preference_of(pa, entry);
    return;
  }
  pool_span(a, blockIdx.y - (kPref ? pref_rows : 0));
}

// Pooling, and in the first workgroup the preferences of a few (layer, sequence) entries, a wave each, and the plan
// that follows from them.
constexpr int kPoolPlanEntries = 4;
__global__ __launch_bounds__(256) void pool_and_plan(ScoreArgs a, PrefArgs pa, PlanArgs plan) {
  static_assert(kPoolPlanEntries == 256 / 64, "a wave per entry");
  if (blockIdx.y > 0) {
    pool_span(a, blockIdx.y - 1);
    return;
  }
  if (blockIdx.x > 0) return;
  for (int entry = threadIdx.x >> 6; entry < pa.n_layers * pa.batch; entry += kPoolPlanEntries) preference_of_wave(pa, entry, threadIdx.x & 63);
  __threadfence_block();
  __syncthreads();
  plan_workgroup<true>(plan, nullptr);
}

// Optional event timing of the four kernels (diagnostics).  Process-wide and not thread-safe:
// one set of five events per profiled call, the last kProfileSets calls are kept.
constexpr int kProfileSets = 64;
struct Profile {
  bool enabled = false, created = false;
  int64_t calls = 0;                       // profiled calls since cake_profile_enable(1)
  hipEvent_t ev[kProfileSets][5] = {};
};
Profile g_profile;

inline void mark(int i, hipStream_t stream) {
  if (g_profile.enabled && g_profile.created) (void)hipEventRecord(g_profile.ev[g_profile.calls % kProfileSets][i], stream);
}

// Which parts of the score stage a call runs: everything on a resident layer, or one of the
// four steps of the segment-wise form (keys handed over a range at a time).
enum ScoreParts { kPartsAll, kPartsPass1Segment, kPartsCombine, kPartsPass2Segment, kPartsPool };

template <typename T, int D, int MB, bool kPivot>
int launch_scores(const ScoreArgs& a_in, int64_t n_slices, const float* const* row_lse, ScoreParts parts, const PrefArgs* pref,
                  const PlanArgs* plan, hipStream_t stream) {
  ScoreArgs a = a_in;
  const dim3 block(64 * a.group);
  const unsigned gy = (unsigned)n_slices;
  // Keys per workgroup: the chunk's granules, or a half or quarter of them where that shortens the rounds of workgroups
  // over the chip.  A workgroup's prologue (its queries, the first tile's way from memory) counts as a tile of keys.  A
  // compute unit holds as many workgroups as LDS and the registers of the pass allow; those of five and more heads of 64
  // window rows count as all it holds, and in fp32, whose products keep a matrix core busy with one wave, those of three and
  // more heads (of 32 rows of 64: six).  A single layer's 8K keys take 256 workgroups of one granule instead of 64 of four
  // (pass 1 20 -> 10 us, pass 2 24 -> 10.7 us).  Cutting until there were 2048 workgroups, whatever the chip holds, was up
  // to 36 % slower than whole chunks (16 layers of 6007 keys, 4 heads of 64 in fp32: 156 us against 115, by this rule 116; 8
  // layers of 4093, 4 x 8 heads of 128 in bf16, 64 rows: 72 against 66, now 61); whole chunks alone are slower where they
  // leave a round half empty (8 layers of 40000, 4 x 5 heads of 128, 64 rows: 405 us against 359).
  // Sums are kept per granule, whoever computes it.
  auto set_span = [&](int pass, int lo, int hi) -> unsigned {
    constexpr bool kF32 = sizeof(T) == 4, kSmall = D == 64, kWide = MB == 2;
    constexpr int kWaves1 = kF32 ? (kWide ? (kSmall ? 3 : 2) : (kSmall ? 5 : 4)) : (kWide ? (kSmall ? 4 : 3) : (kSmall ? 6 : 5));
    constexpr int kWaves2 = kWide ? 2 : kF32 ? (kSmall ? 4 : 3) : (kSmall ? 5 : 4);      // waves per SIMD
    constexpr int kLds = 2 * Tile<T, D>::kBytes + (int)sizeof(float) * 2 * 8 * kTileKeys;
    const int by_waves = 4 * (pass == 1 ? kWaves1 : kWaves2) / a.group;
    const bool alone = a.group > (kF32 ? (kSmall && !kWide ? 5 : 2) : kWide ? 4 : 8);
    const int64_t slots = 256 * (alone ? 1 : std::max(1, std::min(160 * 1024 / kLds, by_waves)));
    int64_t least = INT64_MAX;
    int best = 1;
    for (int per = a.chunk / a.granule; per >= 1; per >>= 1) {
      const int keys = per * a.granule, rest = (hi - lo) % keys;
      const int64_t whole = (int64_t)gy * ((hi - lo) / keys), all = whole + (rest > 0 ? gy : 0);
      // The shorter workgroups at the slices' ends run beside the last round or as a round of their own; where one fills a
      // compute unit they take a place in the order of dispatch like any other.
      const int64_t rounds = ((alone ? all : whole) + slots - 1) / slots;
      const int64_t cost = rounds * (keys + kTileKeys) + (all > rounds * slots ? rest + kTileKeys : 0);
      if (cost < least) { least = cost; best = per; }
    }
    a.key0 = lo;
    a.wg_keys = best * a.granule;
    return (unsigned)((hi - lo + a.wg_keys - 1) / a.wg_keys);
  };
  // The form of a launch and its keys per workgroup (per wave where waves stream): the cheapest by form_rates where the group
  // has more than one.  Launches of few granules take a wave per head: their granules on compute units of their own are done
  // sooner than packed ones (8 x 8192 keys, 5 heads of 128: pass 1 16.0 -> 12.4 us, pass 2 27 -> 17.6; 16384 keys 37 -> 27
  // and 50 -> 35), pass 2 may combine the pairs by itself, and of fewer granules than a quarter of the streaming waves streaming never was the fastest.
  enum Form { kPerHead, kPacked, kStreaming };
  struct Launch {
    Form form;
    unsigned gx;
    int key0, wg_keys;
  };
  const int pack = a.group == 5 ? 3 : 2;          // slices of a packed workgroup
  auto choose = [&](int pass, int lo, int hi) -> Launch {
    const FormRates rates = sizeof(T) == 2 ? form_rates(pass, D, MB, a.group) : FormRates{};
    const int64_t granules = ((int64_t)hi - lo + a.granule - 1) / a.granule;
    if (rates.per_head[0] == 0 || a.granule < rates.least_granule || n_slices * granules <= 512) {
      const unsigned gx = set_span(pass, lo, hi);
      return Launch{kPerHead, gx, a.key0, a.wg_keys};
    }
    int64_t least = INT64_MAX;
    Launch best{};
    auto consider = [&](Form form, int64_t per, int64_t gx, int64_t rows, const int* rate, int places, int prologue) {
      const int64_t slots = 256 * places, whole = gx * rows / slots, left = gx * rows % slots;
      const int64_t cost = (per * a.granule + prologue) * (whole * rate[places - 1] + (left ? rate[(left + 255) / 256 - 1] : 0));
      if (cost >= least) return;
      least = cost;
      best = Launch{form, (unsigned)gx, lo, (int)(per * a.granule)};
    };
    for (int per = a.chunk / a.granule; per >= 1; per >>= 1) {
      const int64_t gx = (granules + per - 1) / per;
      consider(kPerHead, per, gx, n_slices, rates.per_head, rates.per_head[3] ? 4 : 3, kFormPrologue);
      if (rates.packed) consider(kPacked, per, gx, (n_slices + pack - 1) / pack, &rates.packed, 1, kFormPrologue);
    }
    const int waves = stream_waves(pass, D, MB, a.group);
    if (waves > 0)
      for (int64_t per = 1; per <= granules && per * a.granule <= 4096; ++per)
        consider(kStreaming, per, (granules + waves * per - 1) / (waves * per), n_slices, rates.stream, 8 / waves, kStreamPrologue);
    return best;
  };
  // packed3, packed2: kernels of three and two slices a workgroup.
  auto run = [&](const Launch& launch, auto per_head, auto packed3, auto packed2) {
    a.key0 = launch.key0;
    a.wg_keys = launch.wg_keys;
    if (launch.form == kPacked)
      hipLaunchKernelGGL(pack == 3 ? packed3 : packed2, dim3(launch.gx, (gy + pack - 1) / pack), dim3(64 * a.group * pack), 0, stream, a);
    else
      hipLaunchKernelGGL(per_head, dim3(launch.gx, gy), block, 0, stream, a);
  };
  constexpr bool kPacks = sizeof(T) == 2 && MB == 1;      // (where no rates pack, the kernel of one slice stands in for the others)
  auto run_pass1 = [&](const Launch& launch) -> int {
    if (launch.form == kStreaming) {
      a.key0 = launch.key0;
      a.wg_keys = launch.wg_keys;
      return launch_stream_pass1(a, D, MB, launch.gx, stream);
    }
    run(launch, scores_pass1<T, D, MB, 1>, scores_pass1<T, D, MB, 1>, scores_pass1<T, D, MB, kPacks ? 2 : 1>);
    return CAKE_OK;
  };
  auto run_pass2 = [&](const Launch& launch, bool combine) -> int {
    if (launch.form == kStreaming) {
      a.key0 = launch.key0;
      a.wg_keys = launch.wg_keys;
      return launch_stream_pass2(a, D, MB, kPivot, launch.gx, stream);
    }
    run(launch, combine ? scores_pass2<T, D, MB, kPivot, true, 1> : scores_pass2<T, D, MB, kPivot, false, 1>,
        scores_pass2<T, D, MB, kPivot, false, kPacks ? 3 : 1>, scores_pass2<T, D, MB, kPivot, false, kPacks ? 2 : 1>);
    return CAKE_OK;
  };
  const int rows = a.group * MB * 32;
  const int64_t total_rows = n_slices * rows;
  if (parts != kPartsAll) {
    // the keys of this launch: those of [key_lo, key_hi) (pass 2: below n_p as well)
    const int hi1 = min(a.n, a.key_hi), hi2 = min(a.n_p, a.key_hi);
    if (parts == kPartsPass1Segment) {
      if (int rc = run_pass1(choose(1, a.key_lo, hi1))) return rc;
    } else if (parts == kPartsCombine)
      hipLaunchKernelGGL(scores_combine, dim3((unsigned)((total_rows * 4 + 255) / 256)), dim3(256), 0, stream, a, rows, total_rows);
    else if (parts == kPartsPass2Segment && hi2 > a.key_lo) {
      if (int rc = run_pass2(choose(2, a.key_lo, hi2), false)) return rc;
    } else if (parts == kPartsPool)
      hipLaunchKernelGGL(pool_indicator<false>, dim3((a.n_p + kPoolSpan - 1) / kPoolSpan, (unsigned)n_slices), dim3(256), 0,
                         stream, a, PrefArgs{}, 0);
    CAKE_HIP_TRY(hipGetLastError());
    return CAKE_OK;
  }
  mark(0, stream);
  const Launch second = choose(2, 0, a.n_p);
  bool combine = false;
  if (row_lse == nullptr && a.one.row_lse == nullptr) {
    if (int rc = run_pass1(choose(1, 0, a.n))) return rc;
    mark(1, stream);
    // every workgroup of pass 2 reads its slice's pairs where it combines them itself: at most 16 MB in all
    const int64_t workgroups = (int64_t)gy * second.gx;
    combine = second.form == kPerHead && workgroups * rows * a.n_granules * 8 <= 16 << 20 && (!kPipelinedForm<T, MB> || workgroups <= 256);
    if (!combine)
      hipLaunchKernelGGL(scores_combine, dim3((unsigned)((total_rows * 4 + 255) / 256)), dim3(256), 0, stream, a, rows, total_rows);
  } else {
    const int64_t per_layer = (int64_t)a.batch * a.h_kv * rows;
    hipLaunchKernelGGL(scores_import_lse, dim3((unsigned)((total_rows + 255) / 256)), dim3(256), 0, stream, a, row_lse,
                       per_layer, total_rows);
    mark(1, stream);
  }
  mark(2, stream);
  if (int rc = run_pass2(second, combine)) return rc;
  mark(3, stream);
  const unsigned spans = (a.n_p + kPoolSpan - 1) / kPoolSpan;
  const unsigned pref_rows = pref ? (pref->n_layers * pref->batch + spans - 1) / spans : 0;
  // The plan of a few preferences beside the pooling, by the workgroup that computes them: two launches and what they wait
  // for less (a stage of a cascade of 8192 keys, 8 heads: 16.8 -> 10.3 us behind pass 2).  Each round of kPoolPlanEntries costs it 2 us.
  const bool with_plan = plan && pref && pref->n_layers * pref->batch <= 2 * kPoolPlanEntries && plan->batch <= kPoolPlanEntries &&
                         plan->n_layers <= 64 && n_slices < 65535;
  if (with_plan) {
    hipLaunchKernelGGL(pool_and_plan, dim3(spans, (unsigned)n_slices + 1), dim3(256), 0, stream, a, *pref, *plan);
  } else if (pref && n_slices + pref_rows <= 65535) {
    hipLaunchKernelGGL(pool_indicator<true>, dim3(spans, (unsigned)n_slices + pref_rows), dim3(256), 0, stream, a, *pref, (int)pref_rows);
  } else {
    hipLaunchKernelGGL(pool_indicator<false>, dim3(spans, (unsigned)n_slices), dim3(256), 0, stream, a, PrefArgs{}, 0);
    if (pref) hipLaunchKernelGGL(layer_preference_kernel, dim3(pref->n_layers * pref->batch), dim3(kPrefThreads), 0, stream, *pref);
  }
  mark(4, stream);             // a plan in a launch of its own is no part of the pooling
  if (g_profile.enabled && g_profile.created) g_profile.calls += 1;
  if (plan && !with_plan)
    if (int rc = launch_plan(*plan, stream)) return rc;
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}

}  // namespace
}  // namespace cake

using namespace cake;

extern "C" int cake_profile_enable(int enable) {
  if (enable && !g_profile.created) {
    for (auto& set : g_profile.ev)
      for (auto& e : set) CAKE_HIP_TRY(hipEventCreate(&e));
    g_profile.created = true;
  }
  if (!enable && g_profile.created) {
    for (auto& set : g_profile.ev)
      for (auto& e : set) (void)hipEventDestroy(e);
    g_profile.created = false;
  }
  g_profile.calls = 0;
  g_profile.enabled = enable != 0;
  return CAKE_OK;
}

extern "C" int cake_profile_read(float* ms) {
  CAKE_REQUIRE(ms != nullptr, "ms is NULL");
  CAKE_REQUIRE(g_profile.enabled && g_profile.calls > 0, "no profiled cake_window_scores call to read");
  const int64_t n = g_profile.calls < kProfileSets ? g_profile.calls : kProfileSets;
  double sum[4] = {0, 0, 0, 0};
  for (int64_t c = g_profile.calls - n; c < g_profile.calls; ++c) {
    hipEvent_t* ev = g_profile.ev[c % kProfileSets];
    CAKE_HIP_TRY(hipEventSynchronize(ev[4]));
    for (int i = 0; i < 4; ++i) {
      float x = 0.f;
      CAKE_HIP_TRY(hipEventElapsedTime(&x, ev[i], ev[i + 1]));
      sum[i] += x;
    }
  }
  for (int i = 0; i < 4; ++i) ms[i] = (float)(sum[i] / (double)n);
  return CAKE_OK;
}

namespace {
int window_scores_impl(const cake_shape* shape, const cake_params* params,
                       const void* const* q_win, const void* const* k,
                       const int64_t* q_strides, const int64_t* k_strides,
                       const float* const* row_lse, float* const* indicator,
                       void* workspace, size_t workspace_bytes, void* stream,
                       ScoreParts parts = kPartsAll, int key_begin = 0, int key_count = 0, const PrefArgs* pref = nullptr,
                       const PlanArgs* plan = nullptr, const LayerPointers* one = nullptr) {
  if (int rc = check_shape_scores(shape)) return rc;
  CAKE_REQUIRE(params != nullptr, "params is NULL");
  // what the parts of this call touch: the two finishing steps read neither queries nor keys,
  // and only the resident form and the pooling step write the indicator
  const bool reads_keys = parts == kPartsAll || parts == kPartsPass1Segment || parts == kPartsPass2Segment;
  const bool writes_indicator = parts == kPartsAll || parts == kPartsPool;
  if (reads_keys) {
    CAKE_REQUIRE((q_win && k) || one, "q_win or k table is NULL");
    CAKE_REQUIRE(q_strides && k_strides, "q_strides or k_strides is NULL");
  }
  CAKE_REQUIRE(!writes_indicator || indicator || one, "indicator table is NULL");
  CAKE_REQUIRE(params->pool_kernel >= 1 && params->pool_kernel % 2 == 1 && params->pool_kernel <= 2 * kPoolMaxHalf + 1,
               "pool_kernel %d must be odd and within [1, %d]", params->pool_kernel, 2 * kPoolMaxHalf + 1);
  CAKE_REQUIRE(params->indicator_mode >= CAKE_IND_MEAN_PLUS_VAR && params->indicator_mode <= CAKE_IND_CUMULATIVE,
               "indicator_mode %d is not a cake_indicator", params->indicator_mode);
  CAKE_REQUIRE(params->var_correction == 0 || params->var_correction == 1, "var_correction %d must be 0 or 1", params->var_correction);
  CAKE_REQUIRE(std::isfinite(params->gamma) && std::isfinite(params->scale) && params->scale >= 0.f, "gamma/scale must be finite, scale >= 0");
  const size_t eb = elem_bytes(shape->dtype);
  if (reads_keys) {
    for (int i = 0; i < 3; ++i) {
      CAKE_REQUIRE(q_strides[i] >= 0 && k_strides[i] >= 0, "negative stride");
      CAKE_REQUIRE((q_strides[i] * eb) % 16 == 0 && (k_strides[i] * eb) % 16 == 0, "strides must be multiples of 16 bytes");
    }
    CAKE_REQUIRE(q_strides[2] >= shape->head_dim && k_strides[2] >= shape->head_dim, "token stride below head_dim");
    CAKE_REQUIRE(k_strides[2] * (int64_t)eb <= (int64_t)1 << 27, "key token stride above 128 MiB");
  }
  const ScoreLayout lay = score_layout(*shape);
  if (workspace == nullptr || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
    return fail(CAKE_ERR_WORKSPACE, "workspace is NULL or not 256-byte aligned");
  if (workspace_bytes < lay.total)
    return fail(CAKE_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes, lay.total);
  if (lay.n_slices > 65535) return fail(CAKE_ERR_UNSUPPORTED, "layers*batch*kv_heads = %lld exceeds 65535 per call", (long long)lay.n_slices);

  ScoreArgs a{};
  a.q_win = q_win; a.k = k; a.indicator = indicator;
  if (one) a.one = *one;
  if (reads_keys)
    for (int i = 0; i < 3; ++i) { a.qs[i] = q_strides[i]; a.ks[i] = k_strides[i]; }
  a.batch = shape->batch; a.h_kv = shape->n_kv_heads; a.group = shape->n_q_heads / shape->n_kv_heads;
  a.n = shape->seq_len; a.n_p = shape->seq_len - shape->window;
  a.chunk = lay.chunk; a.granule = lay.granule; a.n_granules = lay.n_granules; a.n_granules_p = lay.n_granules_p; a.pool = params->pool_kernel;
  a.key_lo = 0; a.key_hi = a.n;
  a.n_slices = (int32_t)lay.n_slices;
  if (parts == kPartsPass1Segment || parts == kPartsPass2Segment) {
    CAKE_REQUIRE(key_begin >= 0 && key_count > 0 && (int64_t)key_begin + key_count <= a.n,
                 "segment [%d, %d + %d) outside [0, seq_len = %d)", key_begin, key_begin, key_count, a.n);
    CAKE_REQUIRE(key_begin % a.chunk == 0, "key_begin %d is not a multiple of the chunk of %d keys", key_begin, a.chunk);
    CAKE_REQUIRE((key_begin + key_count) % a.chunk == 0 || key_begin + key_count == a.n,
                 "a segment must end on a multiple of the chunk of %d keys or at seq_len", a.chunk);
    a.key_lo = key_begin; a.key_hi = key_begin + key_count;
  }
  const int mode = params->indicator_mode;     // Eq. 11; Mean, Var, Mean*Var of the indicator ablation; the window's column sum
  a.w_mean = (mode == CAKE_IND_MEAN_PLUS_VAR || mode == CAKE_IND_MEAN) ? 1.f
             : mode == CAKE_IND_CUMULATIVE ? (float)shape->window : 0.f;     // Sec. 5.5: column sum = S_w * Mean
  a.w_var = mode == CAKE_IND_MEAN_PLUS_VAR ? params->gamma : mode == CAKE_IND_VAR ? 1.f : 0.f;
  a.w_prod = mode == CAKE_IND_MEAN_TIMES_VAR ? 1.f : 0.f;
  const double scale = params->scale > 0.f ? (double)params->scale : 1.0 / std::sqrt((double)shape->head_dim);
  a.c = (float)(scale * 1.4426950408889634);
  a.inv_sw = 1.0f / (float)shape->window;
  a.inv_swc = 1.0f / (float)(shape->window - params->var_correction);
  a.inv_g = 1.0f / (float)a.group;
  char* ws = static_cast<char*>(workspace);
  a.lse = reinterpret_cast<float*>(ws + lay.off_lse);
  a.part = reinterpret_cast<float*>(ws + lay.off_part);
  a.hv = reinterpret_cast<float*>(ws + lay.off_hv);
  a.raw = reinterpret_cast<float*>(ws + lay.off_raw);
  hipStream_t st = static_cast<hipStream_t>(stream);

  // Var and Mean*Var score a token by the variance alone or by a product with it: those take the
  // pivoted column sums.  Eq. 11's sum and the plain mean do not need them.
  const bool pivot = mode == CAKE_IND_VAR || mode == CAKE_IND_MEAN_TIMES_VAR;
#define CAKE_DISPATCH(T, D, MB)                                                         \
  return pivot ? launch_scores<T, D, MB, true>(a, lay.n_slices, row_lse, parts, pref, plan, st)     \
               : launch_scores<T, D, MB, false>(a, lay.n_slices, row_lse, parts, pref, plan, st)
  const bool bf = shape->dtype == CAKE_BF16;
  const int d = shape->head_dim, mb = shape->window / 32;
  if (bf && d == 128 && mb == 1) CAKE_DISPATCH(__bf16, 128, 1);
  if (bf && d == 128 && mb == 2) CAKE_DISPATCH(__bf16, 128, 2);
  if (bf && d == 64 && mb == 1) CAKE_DISPATCH(__bf16, 64, 1);
  if (bf && d == 64 && mb == 2) CAKE_DISPATCH(__bf16, 64, 2);
  if (!bf && d == 128 && mb == 1) CAKE_DISPATCH(float, 128, 1);
  if (!bf && d == 128 && mb == 2) CAKE_DISPATCH(float, 128, 2);
  if (!bf && d == 64 && mb == 1) CAKE_DISPATCH(float, 64, 1);
  if (!bf && d == 64 && mb == 2) CAKE_DISPATCH(float, 64, 2);
#undef CAKE_DISPATCH
  return fail(CAKE_ERR_UNSUPPORTED, "no score kernel for this shape");
}
}  // namespace

extern "C" int cake_window_scores(const cake_shape* shape, const cake_params* params,
                                  const void* const* q_win, const void* const* k,
                                  const int64_t* q_strides, const int64_t* k_strides,
                                  float* const* indicator,
                                  void* workspace, size_t workspace_bytes, void* stream) {
  return window_scores_impl(shape, params, q_win, k, q_strides, k_strides, nullptr, indicator, workspace,
                            workspace_bytes, stream);
}

extern "C" int cake_window_scores_lse(const cake_shape* shape, const cake_params* params,
                                      const void* const* q_win, const void* const* k,
                                      const int64_t* q_strides, const int64_t* k_strides,
                                      const float* const* row_lse, float* const* indicator,
                                      void* workspace, size_t workspace_bytes, void* stream) {
  CAKE_REQUIRE(row_lse != nullptr, "row_lse table is NULL");
  return window_scores_impl(shape, params, q_win, k, q_strides, k_strides, row_lse, indicator, workspace,
                            workspace_bytes, stream);
}

extern "C" int cake_scores_chunk_keys(const cake_shape* shape, int32_t* chunk) {
  CAKE_REQUIRE(chunk != nullptr, "chunk is NULL");
  if (int rc = check_shape_scores(shape)) return rc;
  *chunk = score_layout(*shape).chunk;
  return CAKE_OK;
}

extern "C" int cake_window_scores_segment(const cake_shape* shape, const cake_params* params, int32_t pass,
                                          int32_t key_begin, int32_t key_count,
                                          const void* const* q_win, const void* const* k_segment,
                                          const int64_t* q_strides, const int64_t* k_strides,
                                          void* workspace, size_t workspace_bytes, void* stream) {
  CAKE_REQUIRE(pass == 1 || pass == 2, "pass %d must be 1 or 2", pass);
  return window_scores_impl(shape, params, q_win, k_segment, q_strides, k_strides, nullptr, nullptr, workspace,
                            workspace_bytes, stream, pass == 1 ? kPartsPass1Segment : kPartsPass2Segment, key_begin, key_count);
}

extern "C" int cake_window_scores_finish(const cake_shape* shape, const cake_params* params, int32_t pass,
                                         float* const* indicator, void* workspace, size_t workspace_bytes, void* stream) {
  CAKE_REQUIRE(pass == 1 || pass == 2, "pass %d must be 1 or 2", pass);
  return window_scores_impl(shape, params, nullptr, nullptr, nullptr, nullptr, nullptr, indicator, workspace,
                            workspace_bytes, stream, pass == 1 ? kPartsCombine : kPartsPool);
}

namespace {
int preference_args(const cake_shape* shape, const cake_params* params, const void* workspace, size_t workspace_bytes,
                    double* pref, double* hv, PrefArgs* out) {
  if (int rc = check_shape_scores(shape)) return rc;
  CAKE_REQUIRE(params != nullptr && pref != nullptr, "params or pref is NULL");
  CAKE_REQUIRE(params->tau1 > 0.f && params->tau2 > 0.f && std::isfinite(params->tau1) && std::isfinite(params->tau2),
               "tau1 and tau2 must be positive and finite");
  const ScoreLayout lay = score_layout(*shape);
  if (workspace == nullptr || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
    return fail(CAKE_ERR_WORKSPACE, "workspace is NULL or not 256-byte aligned");
  if (workspace_bytes < lay.total)
    return fail(CAKE_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes, lay.total);
  *out = PrefArgs{reinterpret_cast<const float*>(static_cast<const char*>(workspace) + lay.off_hv), shape->n_layers, shape->batch,
                  shape->n_kv_heads, shape->n_q_heads / shape->n_kv_heads, lay.n_granules_p, 1.0 / (double)params->tau1,
                  1.0 / (double)params->tau2, pref, hv, shape->n_layers, shape->n_layers, nullptr, 0};
  return CAKE_OK;
}
}  // namespace

extern "C" int cake_layer_preference(const cake_shape* shape, const cake_params* params,
                                     const void* workspace, size_t workspace_bytes,
                                     double* pref, double* hv, void* stream) {
  PrefArgs a{};
  if (int rc = preference_args(shape, params, workspace, workspace_bytes, pref, hv, &a)) return rc;
  hipLaunchKernelGGL(layer_preference_kernel, dim3(shape->n_layers * shape->batch), dim3(kPrefThreads), 0,
                     static_cast<hipStream_t>(stream), a);
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}

int cake::launch_scores_and_preference(const cake_shape* shape, const cake_params* params, const void* const* q_win,
                                       const void* const* k, const int64_t* q_strides, const int64_t* k_strides,
                                       const float* const* row_lse, float* const* indicator, const LayerPointers* one,
                                       void* workspace, size_t workspace_bytes, double* pref, double* hv, int pref_ld, int hv_ld, const PlanArgs* plan,
                                       hipStream_t stream) {
  PrefArgs a{};
  if (int rc = preference_args(shape, params, workspace, workspace_bytes, pref, hv, &a)) return rc;
  a.pref_ld = pref_ld;
  a.hv_ld = hv_ld;
  if (one) { a.flags = one->flags; a.ticket = one->ticket; }
  return window_scores_impl(shape, params, q_win, k, q_strides, k_strides, row_lse, indicator, workspace, workspace_bytes,
                            stream, kPartsAll, 0, 0, &a, plan, one);
}
