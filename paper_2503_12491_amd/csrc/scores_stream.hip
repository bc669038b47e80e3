// The two score passes for launches that fill the chip (bf16): a wave holds the window rows of all heads of a group and
// streams keys of its own, 32 at a time.  The same products and sums in the same order as in window_scores.hip, where a wave
// holds one head and the waves of a group share their keys: the same bits.
//
// What bounds them, by counter at 5 heads of 128 and 8 to 64 layers of 4 x 8 x 32768 keys, where both run at a clock of 1.4 GHz that the
// chip's power sets: pass 1 reads K at 5.2 to 5.6 TB/s, what a copy reaches, its waves wait for transfers and LDS 31 % of their time and a SIMD has a
// product or a vector instruction in flight 65 % of its cycles; pass 2 is busy so 83 % of them (vector instructions 72 %, products 37 %, two
// thirds of these at the same time) and reads 4.0 to 4.3 TB/s; its waves wait 18 % of their time, among other things once a sub-tile for all its key fragments.
// A wave per head adds to that what the workgroup's barriers cost where its waves are not a multiple of the four SIMDs;
// here no wave waits for another one, the group's mean is a sum in a register, and any number of heads loads the SIMDs
// evenly.  At 2 waves a SIMD and 256 registers, 128 of them hold queries; the rest of a larger group is read from LDS (all of 5
// heads of 128 in registers would spill nine).  Which launches take them: form_rates.
//
// A step is one row block's products (8 of 32x32x16 at d = 128) beside the sums or statistics of the block before, dealt out over
// the products, so that two accumulator sets take turns.
#include "score_device.h"

namespace cake {
namespace {

constexpr int kSubKeys = 32;         // keys of a transfer, one MFMA sub-tile

// A wave's ring of two transfers in LDS.  The transfers are written in assembly because the compiler takes any read of LDS for
// one of a transfer in flight and waits for all of them; here a read waits for its own tile alone, and the one behind it stays under way.
// Their place in LDS is an operand in m0: the compiler writes the register and knows it (the no-op keeps its write apart from its use).
// Same layout and swizzle as the tiles of window_scores.hip.
template <int D>
struct KeyRing {
  using TL = Tile<__bf16, D>;
  static constexpr int kBytes = kSubKeys * TL::kRowBytes, kGroups = kBytes / 1024, kRows = 1024 / TL::kRowBytes;
  uint32_t row_off, piece_off, lds;
  const char* kbase;
  int64_t tok_bytes;
  int last_key, lane;

  __device__ __forceinline__ void init(char* tiles, const char* kbase_, int64_t tok_bytes_, int last_key_, int lane_) {
    kbase = kbase_; tok_bytes = tok_bytes_; last_key = last_key_; lane = lane_;
    lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)tiles);
    const int lr = lane / TL::kPieces, slot = lane % TL::kPieces;
    row_off = (uint32_t)(lr * tok_bytes);
    piece_off = (uint32_t)((slot ^ lr) << 4);
  }
  __device__ __forceinline__ void issue(int slot_of_ring, int t0) const {
    const uint32_t to = lds + slot_of_ring * kBytes;
    if (t0 + kSubKeys - 1 <= last_key) {
      const char* base = kbase + (int64_t)t0 * tok_bytes;
      uint32_t piece_off = this->piece_off;
      asm volatile("" : "+v"(piece_off));        // likewise the pieces' offsets below
#pragma unroll
      for (int i = 0; i < kGroups; ++i) {
        const uint32_t off = row_off + (piece_off ^ (uint32_t)(((i * kRows) & (TL::kPieces - 1)) << 4));
        asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :: "{m0}"(to + i * 1024), "v"(off), "s"(base + (int64_t)i * kRows * tok_bytes) : "memory");
      }
    } else {                                     // rows past the last key are clamped to it
      int lane = this->lane;
      asm volatile("" : "+v"(lane));
#pragma unroll 1
      for (int i = 0; i < kGroups; ++i) {
        const int off = i * 1024 + lane * 16, r = off / TL::kRowBytes, q = ((off % TL::kRowBytes) >> 4) ^ (r & (TL::kPieces - 1));
        const char* src = kbase + (int64_t)min(t0 + r, last_key) * tok_bytes + q * 16;
        asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" :: "{m0}"(to + i * 1024), "v"(src) : "memory");
      }
    }
  }
  // Until the transfer of sub-tile t has landed; `more`: that of t + 1 is under way behind it.
  __device__ __forceinline__ void wait(bool more) const {
    if (more) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kGroups) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
};

template <int D> using KeyFrags = bf16x8[D / 16];

// first: the lane's piece of step 0 in the tile; the others differ from it in the bits of the step.
template <int D>
__device__ __forceinline__ void read_keys(KeyFrags<D>& kf, const char* tile, uint32_t first) {
  asm volatile("" : "+v"(first));      // the other addresses are made anew: held over the loop they take a register each
#pragma unroll
  for (int s = 0; s < D / 16; ++s) kf[s] = *reinterpret_cast<const bf16x8*>(tile + (first ^ (uint32_t)(s << 5)));
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the tile's place may be written again
}

// The wave's keys: whole granules of one slice.
struct WaveSpan {
  int slice, l, b, g, key0, key_end, n_sub;
};
__device__ __forceinline__ WaveSpan wave_span(const ScoreArgs& a, int w, int n_waves, int end) {
  WaveSpan s;
  s.slice = blockIdx.y;
  slice_coords(a, s.slice, s.l, s.b, s.g);
  const int64_t at = a.key0 + ((int64_t)blockIdx.x * n_waves + w) * a.wg_keys;      // behind a layer of nearly 2^31 keys: beyond an int
  s.key0 = (int)min(at, (int64_t)end);
  s.key_end = (int)min(at + a.wg_keys, (int64_t)end);
  s.n_sub = (s.key_end - s.key0 + kSubKeys - 1) / kSubKeys;
  return s;
}
__device__ __forceinline__ const char* key_base(const ScoreArgs& a, const WaveSpan& s) {
  return reinterpret_cast<const char*>(in_global(reinterpret_cast<const __bf16*>(a.k ? a.k[s.l] : a.one.k)) + s.b * a.ks[0] + (int64_t)s.g * a.ks[1]) -
         (int64_t)a.key_lo * a.ks[2] * 2;
}

// The window rows of a group: row blocks [0, kHeld) in registers, the others behind them in LDS, laid out like a tile of keys,
// from where they are read two steps ahead of their products.
template <int D, int MB, int G, int kHeld, int kWaves>
struct Queries {
  static constexpr int kBlocks = G * MB, kSteps = D / 16, kAhead = 2;
  using TL = Tile<__bf16, D>;
  static constexpr int kLdsBytes = (kBlocks - kHeld) * 32 * TL::kRowBytes;
  static_assert(kHeld > 0, "block 0's fragments are not read ahead");
  KeyFrags<D> held[kHeld];
  KeyFrags<D> read;
  const char* lds;
  uint32_t first;              // see read_keys

  static __device__ __forceinline__ const __bf16* row(const ScoreArgs& a, const WaveSpan& s, int r) {      // r: head * S_w + window row
    const __bf16* q = in_global(reinterpret_cast<const __bf16*>(a.q_win ? a.q_win[s.l] : a.one.q)) + s.b * a.qs[0] + (int64_t)s.g * G * a.qs[1];
    return q + (int64_t)(r / (MB * 32)) * a.qs[1] + (int64_t)(r % (MB * 32)) * a.qs[2];
  }
  // by the whole workgroup, a barrier follows
  static __device__ __forceinline__ void fill(const ScoreArgs& a, const WaveSpan& s, char* lds) {
    for (int i = threadIdx.x; i < kLdsBytes / 16; i += 64 * kWaves) {
      const int r = i / TL::kPieces, q = i % TL::kPieces;
      *reinterpret_cast<bf16x8*>(lds + TL::offset(r, q)) = *reinterpret_cast<const bf16x8*>(row(a, s, kHeld * 32 + r) + q * 8);
    }
  }
  __device__ __forceinline__ void load(const ScoreArgs& a, const WaveSpan& s, const char* lds_, int c32, int hh) {
    lds = lds_;
    first = TL::offset(c32, hh);
#pragma unroll
    for (int nb = 0; nb < kHeld; ++nb)
#pragma unroll
      for (int st = 0; st < kSteps; ++st) held[nb][st] = Frag<__bf16>::load_global(row(a, s, nb * 32 + c32), st, hh);
  }
  // Before step s of block nb's products, and what the next block needs.
  __device__ __forceinline__ void ahead(int nb, int s) {
    const int next = (nb + 1) % kBlocks;
    if (nb >= kHeld && s + kAhead < kSteps) fetch(nb, s + kAhead);
    if (next >= kHeld && s >= kSteps - kAhead) fetch(next, s + kAhead - kSteps);
  }
  __device__ __forceinline__ void fetch(int nb, int s) {
    uint32_t at = first;
    asm volatile("" : "+v"(at));
    read[s] = *reinterpret_cast<const bf16x8*>(lds + (nb - kHeld) * 32 * TL::kRowBytes + (at ^ (uint32_t)(s << 5)));
  }
  __device__ __forceinline__ bf16x8 frag(int nb, int s) const { return nb < kHeld ? held[nb][s] : read[s]; }
};

// Logits of a row block whose vector work lies beside step s of the products of the next one: none beside the last step, so
// that what follows from the block is known when that product has been issued.
template <int kSteps> struct Share {
  static constexpr int begin(int s) { return s == 0 ? 0 : end(s - 1); }
  static constexpr int end(int s) { return kSteps == 8 ? (s < 2 ? 3 * (s + 1) : s < 7 ? 6 + 2 * (s - 1) : 16) : (s < 3 ? 6 + 5 * s : 16); }
};

// ---- pass 1 ----
// The products of row block nb beside the sums of the block before it.
template <int D, bool kMfma, bool kValu, typename Q>
__device__ __forceinline__ void period1(Q& q, int nb, const KeyFrags<D>& kf, f32x16& dst, const f32x16& src, float& mref, float& lsum, float cv) {
  constexpr int kSteps = D / 16;
  float bsum[2];
  bool redo = false;
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    if (kValu && s == kSteps - 1) {
      bsum[0] += bsum[1];
      redo = block_sum_outside(lsum + bsum[0]);
      if (kMfma) __builtin_amdgcn_sched_barrier(0);
    }
    if (kMfma) {
      q.ahead(nb, s);
      if (s == 0) {
        f32x16 zero;
#pragma unroll
        for (int v = 0; v < 16; ++v) zero[v] = 0.f;
        dst = Frag<__bf16>::mfma(kf[s], q.frag(nb, s), zero);
      } else {
        dst = Frag<__bf16>::mfma(kf[s], q.frag(nb, s), dst);
      }
    }
    if (kValu) {
#pragma unroll
      for (int v = Share<kSteps>::begin(s); v < Share<kSteps>::end(s); ++v) {
        const float e = fast_exp2(fmaf(src[v], cv, -mref));
        if (v < 2) bsum[v] = e;
        else bsum[v & 1] += e;
      }
      asm volatile("" : "+v"(bsum[0]), "+v"(bsum[1]));
    }
    if (kMfma && kValu) __builtin_amdgcn_sched_barrier(0);
  }
  if (kValu) {
    if (__ballot(redo)) add_block_sum<false>(src, bsum[0], mref, lsum, cv, 0);
    else lsum += bsum[0];
  }
}

template <int D, int MB, int G, int kHeld, int kWaves>
__global__ __launch_bounds__(64 * kWaves, 2) void stream_pass1(ScoreArgs a) {
  constexpr int kBlocks = G * MB;
  using Ring = KeyRing<D>;
  using Q = Queries<D, MB, G, kHeld, kWaves>;
  __shared__ __attribute__((aligned(1024))) char rings[kWaves * 2 * Ring::kBytes + Q::kLdsBytes];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, c32 = lane & 31, hh = lane >> 5;
  const WaveSpan sp = wave_span(a, w, kWaves, min(a.n, a.key_hi));
  char* tiles = rings + w * (2 * Ring::kBytes);
  Ring ring;
  ring.init(tiles, key_base(a, sp), a.ks[2] * 2, min(a.n, a.key_hi) - 1, lane);
  if (sp.n_sub > 0) ring.issue(0, sp.key0);
  if (sp.n_sub > 1) ring.issue(1, sp.key0 + kSubKeys);
  Q q;
  if (kHeld < kBlocks) {
    Q::fill(a, sp, rings + kWaves * 2 * Ring::kBytes);
    __syncthreads();
  }
  if (sp.n_sub <= 0) return;
  q.load(a, sp, rings + kWaves * 2 * Ring::kBytes, c32, hh);
  float mref[kBlocks], lsum[kBlocks];
#pragma unroll
  for (int nb = 0; nb < kBlocks; ++nb) { mref[nb] = 0.f; lsum[nb] = 0.f; }
  float cv = a.c;
  asm volatile("" : "+v"(cv));     // a vector register: a scalar operand halves the issue rate of the multiply

  const int granule_shift = __builtin_ctz(a.granule), granule_subs = a.granule / kSubKeys;
  float* out = a.part + (int64_t)sp.slice * a.n_granules * (kBlocks * 32) * 2;
  auto finish = [&](int t) {         // the granule that ends with sub-tile t
    float* o = out + (int64_t)((sp.key0 + t * kSubKeys) >> granule_shift) * (kBlocks * 32) * 2;
#pragma unroll
    for (int nb = 0; nb < kBlocks; ++nb) {
      const float2 pair = merge_halves(mref[nb], lsum[nb]);
      if (hh == 0) *reinterpret_cast<float2*>(o + (nb * 32 + c32) * 2) = pair;
      mref[nb] = 0.f;
      lsum[nb] = 0.f;
    }
  };
  KeyFrags<D> kf;
  const uint32_t first_piece = Tile<__bf16, D>::offset(c32, hh);
  auto fetch = [&](int slot, int t) {
    ring.wait(t + 1 < sp.n_sub);
    read_keys<D>(kf, tiles + slot * Ring::kBytes, first_piece);
    if (t + 2 < sp.n_sub) ring.issue(slot, sp.key0 + (t + 2) * kSubKeys);
  };
  // Sub-tiles all of whose keys every row sees, in pairs.  To begin with the pending block holds weights of 0.
  const int plain = max(0, min(sp.n_sub, (a.n_p + 1 - sp.key0) / kSubKeys)) & ~1;
  f32x16 acc[2];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[1][v] = -INFINITY;
  for (int t = 0; t < plain; t += 2) {
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      fetch(sub, t + sub);
#pragma unroll
      for (int nb = 0; nb < kBlocks; ++nb) {
        const int i = sub * kBlocks + nb, before = (nb + kBlocks - 1) % kBlocks;
        period1<D, true, true>(q, nb, kf, acc[i & 1], acc[(i & 1) ^ 1], mref[before], lsum[before], cv);
        if (i == 0 && t > 0 && (t & (granule_subs - 1)) == 0) finish(t - 1);
      }
    }
  }
  if (plain > 0) {
    period1<D, false, true>(q, 0, kf, acc[0], acc[1], mref[kBlocks - 1], lsum[kBlocks - 1], cv);
    if ((plain & (granule_subs - 1)) == 0 || plain == sp.n_sub) finish(plain - 1);
  }
#pragma unroll 1
  for (int t = plain; t < sp.n_sub; ++t) {
    fetch(t & 1, t);
    const int kb = sp.key0 + t * kSubKeys;
#pragma unroll
    for (int nb = 0; nb < kBlocks; ++nb) {
      period1<D, true, false>(q, nb, kf, acc[0], acc[1], mref[nb], lsum[nb], cv);
      const int last = min(a.n_p + nb % MB * 32 + c32, a.n - 1) - kb - 4 * hh;
      auto hidden = [&](int v) { return 8 * (v / 4) + (v % 4) > last; };
      float bsum[2];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float e = hidden(v) ? 0.f : fast_exp2(fmaf(acc[0][v], cv, -mref[nb]));
        if (v < 2) bsum[v] = e;
        else bsum[v & 1] += e;
      }
      add_block_sum<true>(acc[0], bsum[0] + bsum[1], mref[nb], lsum[nb], cv, last);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (((t + 1) & (granule_subs - 1)) == 0 || t + 1 == sp.n_sub) finish(t);
  }
}

// ---- pass 2 ----
// Column sums of a head over a sub-tile, still split over the two lane halves.
struct HeadSums {
  float sp[2], sp2[2], pivot;      // as in ColSums, in two chains
};
// The products of row block nb, which start from the normalisers in `dst`, beside the statistics of the block before it, whose
// registers take the normalisers of the block after it (next: their LDS row).
template <int D, bool kMfma, bool kValu, bool kTail, bool kPivot, typename Q>
__device__ __forceinline__ void period2(Q& q, int nb, const KeyFrags<D>& kf, f32x16& dst, f32x16& src, const float* next, bool first_block,
                                        float cv, bool col_valid, HeadSums& hs, float (&entv)[2], int hh) {
  constexpr int kSteps = D / 16;
  auto logit = [&](int v) { return (kTail && !col_valid) ? -1.0e30f : src[v]; };
  if (kValu && kPivot && first_block) {
    // the weight of window row 0 lives in the lower lane half (v 0); both halves take it
    const float p0 = fast_exp2(logit(0) * cv);
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(p0), __float_as_uint(p0), false, false);
    hs.pivot = __uint_as_float(r[0]);
  }
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    if (kMfma) {
      q.ahead(nb, s);
      dst = Frag<__bf16>::mfma(q.frag(nb, s), kf[s], dst);
    }
    if (kValu) {
      constexpr int kMost = kSteps == 8 ? 3 : 6;
      const int v0 = Share<kSteps>::begin(s), v1 = Share<kSteps>::end(s);
      float x[kMost], p[kMost];
#pragma unroll
      for (int v = v0; v < v1; ++v) x[v - v0] = logit(v);
#pragma unroll
      for (int v = v0; v < v1; ++v) p[v - v0] = fast_exp2(x[v - v0] * cv);
#pragma unroll
      for (int v = v0; v < v1; ++v) {
        const float pd = kPivot ? p[v - v0] - hs.pivot : p[v - v0];
        if (first_block && v < 2) {
          hs.sp[v & 1] = pd;
          hs.sp2[v & 1] = pd * pd;
        } else {
          hs.sp[v & 1] += pd;
          hs.sp2[v & 1] = fmaf(pd, pd, hs.sp2[v & 1]);
        }
        entv[v & 1] = fmaf(p[v - v0], x[v - v0], entv[v & 1]);      // sum p * log2(p) / c
      }
      asm volatile("" : "+v"(hs.sp[0]), "+v"(hs.sp[1]), "+v"(hs.sp2[0]), "+v"(hs.sp2[1]), "+v"(entv[0]), "+v"(entv[1]));
      if (kMfma) {
#pragma unroll
        for (int j = v0 / 4; j < v1 / 4; ++j) {
          const f32x4 x4 = *reinterpret_cast<const f32x4*>(next + 8 * j + 4 * hh);
#pragma unroll
          for (int i = 0; i < 4; ++i) src[4 * j + i] = x4[i];
        }
      }
    }
    if (kMfma && kValu) __builtin_amdgcn_sched_barrier(0);
  }
}

template <int D, int MB, int G, int kHeld, int kWaves, bool kPivot>
__global__ __launch_bounds__(64 * kWaves, 2) void stream_pass2(ScoreArgs a) {
  constexpr int kBlocks = G * MB, kRowsAll = kBlocks * 32;
  using Ring = KeyRing<D>;
  using Q = Queries<D, MB, G, kHeld, kWaves>;
  __shared__ __attribute__((aligned(1024))) char rings[kWaves * 2 * Ring::kBytes + Q::kLdsBytes];
  __shared__ __attribute__((aligned(16))) float starts[kRowsAll];
  __shared__ float lower_lds[kWaves][G][64];     // of a tile's first sub-tile: no registers left for them
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, c32 = lane & 31, hh = lane >> 5;
  const WaveSpan sp = wave_span(a, w, kWaves, min(a.n_p, a.key_hi));
  char* tiles = rings + w * (2 * Ring::kBytes);
  Ring ring;
  ring.init(tiles, key_base(a, sp), a.ks[2] * 2, min(a.n, a.key_hi) - 1, lane);
  const int n_tiles = (sp.key_end - sp.key0 + kTileKeys - 1) / kTileKeys, n_sub = 2 * n_tiles;      // whole tiles: columns past the end are masked
  if (sp.n_sub > 0) {
    ring.issue(0, sp.key0);
    ring.issue(1, sp.key0 + kSubKeys);
  }
  Q q;
  // -lse2/c of the window rows: the products start from them, so that a sum times c is the log2 of a weight
  const float neg_inv_c = -1.0f / a.c;
  for (int i = threadIdx.x; i < kRowsAll; i += 64 * kWaves) starts[i] = a.lse[(int64_t)sp.slice * kRowsAll + i] * neg_inv_c;
  if (kHeld < kBlocks) Q::fill(a, sp, rings + kWaves * 2 * Ring::kBytes);
  __syncthreads();
  if (sp.n_sub <= 0) return;
  q.load(a, sp, rings + kWaves * 2 * Ring::kBytes, c32, hh);
  float cv = a.c;
  asm volatile("" : "+v"(cv));     // a vector register: a scalar operand halves the issue rate of the multiply

  float entv[G][2], var_acc[G];
#pragma unroll
  for (int h = 0; h < G; ++h) entv[h][0] = entv[h][1] = var_acc[h] = 0.f;
  HeadSums hs{};
  float* lower = &lower_lds[w][0][lane];
  float iq = 0.f;
  float* raw = a.raw + (int64_t)sp.slice * a.n_p;
  const int granule_shift = __builtin_ctz(a.granule), granule_tiles = a.granule / kTileKeys;
  auto finish = [&](int t) {         // the granule that ends with tile t; -1: what the block before the first one left
    if (t >= 0) {
      const int64_t granule = (sp.key0 + t * kTileKeys) >> granule_shift;
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float ent = wave_sum((entv[h][0] + entv[h][1]) * cv), var = wave_sum(var_acc[h]);
        if (lane == 0) *reinterpret_cast<float2*>(a.hv + (((int64_t)sp.slice * a.n_granules_p + granule) * G + h) * 2) = make_float2(ent, var);
      }
    }
#pragma unroll
    for (int h = 0; h < G; ++h) entv[h][0] = entv[h][1] = var_acc[h] = 0.f;
  };
  KeyFrags<D> kf;
  const uint32_t first_piece = Tile<__bf16, D>::offset(c32, hh);
  auto fetch = [&](int slot, int t) {
    ring.wait(t + 1 < n_sub);
    read_keys<D>(kf, tiles + slot * Ring::kBytes, first_piece);
    if (t + 2 < n_sub) ring.issue(slot, sp.key0 + (t + 2) * kSubKeys);
  };
  // What follows from the statistics of row block nb of sub-tile `sub` of tile t.  A sub-tile's columns are in both lane halves:
  // the lower one keeps the sums of p, the upper those of p^2 (kPivot: the indicator and the variance, for which the pivot is at
  // hand), and with the second sub-tile's lane L gets both of key L of the tile.
  auto column_done = [&](int t, int sub, int nb) {
    const int h = nb / MB;
    if (nb % MB != MB - 1) return;
    auto swap = [](float x, float y) {
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
      return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1]));
    };
    const float2 parts = swap(hs.sp[0] + hs.sp[1], hs.sp2[0] + hs.sp2[1]);
    float mine = parts.x + parts.y;
    if (kPivot) {
      const float2 sums = swap(mine, mine);
      float var = 0.f;
      const float x = column_indicator<true>(sums.x, sums.y, hs.pivot, a, var);
      mine = hh ? var : x;
    }
    if (sub == 0) {
      lower[h * 64] = mine;
    } else {
      const float2 own = swap(lower[h * 64], mine);
      float x = own.x;
      if (kPivot) var_acc[h] += own.y;
      else x = column_indicator<false>(own.x, own.y, 0.f, a, var_acc[h]);
      iq = h == 0 ? x : iq + x;
      if (h == G - 1) {
        const int key = sp.key0 + t * kTileKeys + lane;
        if (t >= 0 && key < sp.key_end) raw[key] = iq * a.inv_g;
      }
    }
  };
  auto load_start = [&](f32x16& x, int nb) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4 x4 = *reinterpret_cast<const f32x4*>(starts + nb * 32 + 8 * j + 4 * hh);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[4 * j + i] = x4[i];
    }
  };
  const int whole = (sp.key_end - sp.key0) / kTileKeys;
  f32x16 acc[2];
  // To begin with the pending block is one of tile -1 with weights of 0.
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[1][v] = -1.0e30f;
#pragma unroll
  for (int h = 0; h < G; ++h) lower[h * 64] = 0.f;
  load_start(acc[0], 0);
  for (int t = 0; t < whole; ++t) {
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      fetch(sub, 2 * t + sub);
#pragma unroll
      for (int nb = 0; nb < kBlocks; ++nb) {
        const int i = sub * kBlocks + nb, before = (nb + kBlocks - 1) % kBlocks, after = (nb + 1) % kBlocks;
        period2<D, true, true, false, kPivot>(q, nb, kf, acc[i & 1], acc[(i & 1) ^ 1], starts + after * 32, before % MB == 0, cv, true, hs,
                                              entv[before / MB], hh);
        column_done(i == 0 ? t - 1 : t, nb == 0 ? sub ^ 1 : sub, before);
        if (i == 0 && (t & (granule_tiles - 1)) == 0) finish(t - 1);
      }
    }
  }
  if (whole > 0) {
    period2<D, false, true, false, kPivot>(q, 0, kf, acc[0], acc[1], starts, (kBlocks - 1) % MB == 0, cv, true, hs, entv[G - 1], hh);
    column_done(whole - 1, 1, kBlocks - 1);
    if ((whole & (granule_tiles - 1)) == 0 || whole == n_tiles) finish(whole - 1);
  }
  if (whole < n_tiles) {
#pragma unroll 1
    for (int sub = 0; sub < 2; ++sub) {
      fetch(sub, 2 * whole + sub);
      const bool valid = sp.key0 + whole * kTileKeys + sub * kSubKeys + c32 < sp.key_end;
#pragma unroll
      for (int nb = 0; nb < kBlocks; ++nb) {
        load_start(acc[0], nb);
        __builtin_amdgcn_sched_barrier(0);
        period2<D, true, false, false, kPivot>(q, nb, kf, acc[0], acc[1], starts, false, cv, true, hs, entv[nb / MB], hh);
        period2<D, false, true, true, kPivot>(q, nb, kf, acc[1], acc[0], starts, nb % MB == 0, cv, valid, hs, entv[nb / MB], hh);
        column_done(whole, sub, nb);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    finish(whole);
  }
}


template <int D, int MB, int G>
constexpr int held_blocks() { return G * MB < 512 / D ? G * MB : 512 / D; }      // row blocks in 128 registers

// The kernel of the group's size, where stream_waves says that there is one: no second list of sizes.
template <int kPass, int D, int MB, bool kPivot, int G = 1>
int run_group(const ScoreArgs& a, unsigned gx, hipStream_t stream) {
  if constexpr (G > kStreamMaxGroup) {
    return fail(CAKE_ERR_UNSUPPORTED, "no streaming score kernel for groups of %d", a.group);
  } else {
    if (a.group != G) return run_group<kPass, D, MB, kPivot, G + 1>(a, gx, stream);
    constexpr int W = stream_waves(kPass, D, MB, G), H = held_blocks<D, MB, G>();
    if constexpr (W == 0) {
      return fail(CAKE_ERR_UNSUPPORTED, "no streaming kernel of pass %d for groups of %d, %d rows of %d", kPass, G, MB * 32, D);
    } else {
      if constexpr (kPass == 1) hipLaunchKernelGGL((stream_pass1<D, MB, G, H, W>), dim3(gx, a.n_slices), dim3(64 * W), 0, stream, a);
      else hipLaunchKernelGGL((stream_pass2<D, MB, G, H, W, kPivot>), dim3(gx, a.n_slices), dim3(64 * W), 0, stream, a);
      return CAKE_OK;
    }
  }
}
template <int kPass, bool kPivot>
int run_rows(const ScoreArgs& a, int head_dim, int mb, unsigned gx, hipStream_t stream) {
  if (head_dim == 128) return mb == 1 ? run_group<kPass, 128, 1, kPivot>(a, gx, stream) : run_group<kPass, 128, 2, kPivot>(a, gx, stream);
  return mb == 1 ? run_group<kPass, 64, 1, kPivot>(a, gx, stream) : run_group<kPass, 64, 2, kPivot>(a, gx, stream);
}

}  // namespace

int launch_stream_pass1(const ScoreArgs& a, int head_dim, int mb, unsigned gx, hipStream_t stream) {
  return run_rows<1, false>(a, head_dim, mb, gx, stream);
}
int launch_stream_pass2(const ScoreArgs& a, int head_dim, int mb, bool pivot, unsigned gx, hipStream_t stream) {
  return pivot ? run_rows<2, true>(a, head_dim, mb, gx, stream) : run_rows<2, false>(a, head_dim, mb, gx, stream);
}

}  // namespace cake
