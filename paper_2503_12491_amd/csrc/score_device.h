// What the kernels of the score passes share: operand fragments, arguments, key tiles (window_scores.hip, scores_stream.hip).
#pragma once

#include <cmath>
#include <type_traits>

#include "cake_internal.h"

#ifdef __HIPCC__
namespace cake {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const void* global_cptr;
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int kTileKeys = 64;        // keys staged per LDS tile (two 32-key MFMA sub-tiles)
constexpr float kMasked = -1.0e30f;  // stands for -inf without producing NaN in differences

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }  // v_exp_f32

template <typename T, int D>
struct Tile {
  static constexpr int kRowBytes = D * (int)sizeof(T);
  static constexpr int kPieces = kRowBytes / 16;         // 16-byte pieces per key row (power of two)
  static constexpr int kBytes = kTileKeys * kRowBytes;
  static constexpr int kGroups = kBytes / 1024;          // one wave-wide 1 KiB transfer each
  // LDS byte offset of piece q of row r: pieces are permuted within the row by r.
  static __device__ __forceinline__ int offset(int r, int q) { return r * kRowBytes + ((q ^ (r & (kPieces - 1))) << 4); }
};

// MFMA operand fragments.  For both the A and the B operand of the 32x32 instructions lane
// (c32, hh) supplies, for its row/column c32, a group of consecutive reduction elements chosen
// by hh; A and B use the same element order, so the dot products come out complete.
template <typename T> struct Frag;
template <> struct Frag<__bf16> {
  using type = bf16x8;
  static constexpr int kElems = 16;  // reduction elements per MFMA
  static __device__ __forceinline__ type load_global(const __bf16* row, int step, int hh) {
    return *reinterpret_cast<const bf16x8*>(row + step * 16 + hh * 8);
  }
  template <typename TL>
  static __device__ __forceinline__ type load_lds(const char* tile, int r, int step, int hh) {
    return *reinterpret_cast<const bf16x8*>(tile + TL::offset(r, 2 * step + hh));
  }
  static __device__ __forceinline__ f32x16 mfma(type a, type b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
// Four 32x32x2 products in a row: a lane's share of eight reduction elements is one 16-byte piece, read at once.  (With a
// 4-byte read per product the addresses of all pieces took 16 to 32 registers: 900 bytes a lane were spilled at two row blocks
// of 128, and one row block ran two waves per SIMD instead of three.  8 layers of 6000 keys, 8 x 4 heads, 64 rows of 128:
// pass 1 322 -> 217 us, pass 2 446 -> 223; 32 rows of 64: 69 -> 61 and 74 -> 68; one layer of 1024 keys, 8 x 4 heads, 32 rows of
// 128: 17 -> 11 and 19 -> 13.)
template <> struct Frag<float> {
  using type = f32x4;
  typedef float loose __attribute__((ext_vector_type(4), aligned(4)));
  static constexpr int kElems = 8;
  static __device__ __forceinline__ type load_global(const float* row, int step, int hh) {
    return *reinterpret_cast<const loose*>(row + step * 8 + hh * 4);
  }
  template <typename TL>
  static __device__ __forceinline__ type load_lds(const char* tile, int r, int step, int hh) {
    return *reinterpret_cast<const f32x4*>(tile + TL::offset(r, 2 * step + hh));
  }
  static __device__ __forceinline__ f32x16 mfma(type a, type b, f32x16 c) {
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], c, 0, 0, 0);
    return c;
  }
};

struct ScoreArgs {
  const void* const* q_win;
  const void* const* k;
  float* const* indicator;
  LayerPointers one;         // one layer's, where there are no tables
  int64_t qs[3], ks[3];      // element strides: batch, head, token
  int32_t batch, h_kv, group, n, n_p, chunk, wg_keys, granule, n_granules, n_granules_p, pool;   // wg_keys: keys per workgroup, granules each
  int32_t key_lo, key_hi;    // keys [key_lo, key_hi) are behind the k pointers (row 0 = key key_lo); the whole layer: 0, n
  int32_t key0;              // first key of the first workgroup of a launch
  int32_t n_slices;
  float c;                   // scale * log2(e): logits are handled in the log2 domain
  float inv_sw, inv_swc, inv_g;
  float w_mean, w_var, w_prod;   // I_q = w_mean*Mean + w_var*Var + w_prod*Mean*Var (Eq. 11 and the ablation's variants)
  float* lse;                // [slice][G*S_w]
  float* part;               // [slice][n_granules][G*S_w][2]
  float* hv;                 // [slice][n_granules_p][G][2]
  float* raw;                // [slice][n_p]
};

// Cache-policy bits of the tile transfers: non-temporal.  Every key byte is used once per pass
// and the whole K of a pass is far larger than the caches, so the tiles should not displace the
// small arrays that are reused (partial sums, normalisers, the un-pooled indicator); measured
// 5-12 % faster on the 32K-context shapes, neutral at 128K.
constexpr int kStreamPolicy = 2;

__device__ __forceinline__ void slice_coords(const ScoreArgs& a, int slice, int& l, int& b, int& g) {
  g = slice % a.h_kv;
  b = (slice / a.h_kv) % a.batch;
  l = slice / (a.h_kv * a.batch);
}

// A row starts from reference 0 and keeps it while its sum stays within 2^-24 .. 2^24, as it does in most
// layers.  Outside (a logit outran the reference, all of them lie far below it, inf or NaN) the block is redone with
// a reference of its own.  The bounds are narrow because an exponent is rounded at its distance from the
// reference: with 2^-60 .. 2^100 rows whose largest logit exceeds some 35 (log2 units) got normalisers up to a quarter
// further off than with references of their own from the first block on (2.85e-6 rms against 2.40e-6 at 72; 2.22e-6
// with these bounds, which nowhere between logits of 2 and 92 are worse).
constexpr uint32_t kSumLow = (127u - 24u) << 23, kSumHigh = (127u + 24u) << 23;      // the two bounds as float bits
__device__ __forceinline__ bool block_sum_outside(float sum) { return __float_as_uint(sum) - kSumLow > kSumHigh - kSumLow; }
// kTail: keys of the block from position `last` + 1 on (counted as the lane's registers hold them) are hidden from the row.  (As a
// callable argument the test for them cost pass 1 ten registers and a wave a SIMD, also where nothing is hidden.)
template <bool kTail>
__device__ __forceinline__ void add_block_sum(const f32x16& acc, float block, float& mref, float& lsum, float cv, int last) {
  auto hidden = [&](int v) { return kTail && 8 * (v / 4) + (v % 4) > last; };
  float sum = lsum + block;
  if (block_sum_outside(sum)) {
    float rmax = kMasked;
#pragma unroll
    for (int v = 0; v < 16; ++v) rmax = fmaxf(rmax, hidden(v) ? kMasked : acc[v] * cv);
    if (rmax > kMasked) {               // (no key of the block is visible: nothing to refer to)
      // the earlier terms, a half wave's share of a granule, are at most 2^10: some of them are as large as their
      // sum by that, which the block's own largest logit need not be
      if (lsum != 0.f) rmax = fmaxf(rmax, mref + (float)(__builtin_amdgcn_frexp_expf(lsum) - 10));
      sum = lsum == 0.f ? 0.f : lsum * fast_exp2(mref - rmax);      // (0 * 2^(mref - rmax) would be NaN from 2^128 on)
      mref = rmax;
#pragma unroll
      for (int v = 0; v < 16; ++v) sum += hidden(v) ? 0.f : fast_exp2(fmaf(acc[v], cv, -rmax));      // not from the rounded products
    } else {
      sum = lsum;
    }
  }
  lsum = sum;
}
// The (reference, sum) pair of a row at the end of a granule: the two lane halves' merged, the lower half's first.
__device__ __forceinline__ float2 merge_halves(float mref, float lsum) {
  // (a half that has seen no key is masked: its reference 0 may lie far above the row's logits)
  const uint32_t ref = __float_as_uint(lsum == 0.f ? kMasked : mref);
  const auto rm = __builtin_amdgcn_permlane32_swap(ref, ref, false, false);
  const auto rl = __builtin_amdgcn_permlane32_swap(__float_as_uint(lsum), __float_as_uint(lsum), false, false);
  const float m0 = __uint_as_float(rm[0]), m1 = __uint_as_float(rm[1]), m = fmaxf(m0, m1);
  return make_float2(m, __uint_as_float(rl[0]) * fast_exp2(m0 - m) + __uint_as_float(rl[1]) * fast_exp2(m1 - m));
}

// Column sums of one finished sub-tile, still split over the two lane halves.
struct ColSums {
  float sp, sp2;     // sum of (p - pivot), sum of (p - pivot)^2 over this half's window rows
  float pivot;       // 0 unless the pivoted form is used
};

// I_q and variance of a column from its sums over the window rows.
template <bool kPivot>
__device__ __forceinline__ float column_indicator(float sp, float sp2, float pivot, const ScoreArgs& a, float& var_acc) {
  const float dmean = sp * a.inv_sw;                               // mean of (p - pivot)
  const float var = fmaxf((sp2 - sp * dmean) * a.inv_swc, 0.f);    // the variance does not see the pivot
  const float mean = kPivot ? dmean + pivot : dmean;
  var_acc += var;
  return fmaf(a.w_prod * mean, var, fmaf(a.w_var, var, a.w_mean * mean));
}

// Statistics of the 64 key columns of one tile from the half sums of its two sub-tiles.  One
// swap of lane halves per quantity leaves lanes 0-31 with the complete sums of sub-tile 0's
// columns and lanes 32-63 with those of sub-tile 1's: lane L ends up owning key L of the tile.
template <bool kPivot>
__device__ __forceinline__ float pass2_tile_stats(const ColSums& s0, const ColSums& s1, const ScoreArgs& a, int hh, float& var_acc) {
  auto r1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(s0.sp), __float_as_uint(s1.sp), false, false);
  auto r2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(s0.sp2), __float_as_uint(s1.sp2), false, false);
  const float sp = __uint_as_float(r1[0]) + __uint_as_float(r1[1]);
  const float sp2 = __uint_as_float(r2[0]) + __uint_as_float(r2[1]);
  return column_indicator<kPivot>(sp, sp2, hh ? s1.pivot : s0.pivot, a, var_acc);
}

// Three forms of a pass over bf16 keys, to the same bits: a wave per head of a group, the group a workgroup; slices packed three
// (groups of 5) or two (of 6) to a workgroup, which loads the four SIMDs of a compute unit evenly; waves that stream keys of their
// own through all heads (scores_stream.hip), which do that too, without barriers, but take whole granules of keys each: 2048 waves
// fill the chip.  Groups of other sizes load the SIMDs evenly with a wave per head and have no other form, but in pass 2 of
// 4 heads of 128 and of two sizes of 64 rows streaming may be the faster; pass 1 was slower so (4 heads of 128, 12 to 33 million
// keys, 0.98-1.11 of a wave per head; 64 rows of 128, 4 heads, 2450 us for 2187).  Pass 2 of 4 heads streams granules of 1024 keys
// and more only: there, over 4 to 33 million keys, 0.94-1.005 of a wave per head (256 x 32768: 442 -> 426 us), 0.975-1.07 in
// granules of 256 (976 x 4128: 221 -> 232).
//
// Waves of a streaming workgroup, 0 where there is no such kernel.
constexpr int stream_waves(int pass, int head_dim, int mb, int group) {
  if (head_dim == 128 && mb == 1) return group == 5 || (group == 4 && pass == 2) ? 4 : group == 6 ? 8 : 0;
  if (head_dim == 64 && mb == 1) return group == 5 || group == 6 ? 4 : 0;
  if (pass == 2 && head_dim == 128) return group == 3 ? 8 : 0;
  if (pass == 2 && head_dim == 64) return group == 4 ? 4 : 0;
  return 0;
}
// What a launch takes: nanoseconds per key of a workgroup (streaming: of a wave) in a round that has up to 1, 2, 3 or (4 heads) 4
// workgroups a compute unit (packed: one; streaming: as many as make 4 or 8 waves); 0: no such kernel.  Fitted, to 6-13 %, to launches of each form
// with all its spans over 140 thousand to 8.4 million keys (a call's slices together) in layers of 1100 to 131072.  The shape of it: a key
// costs by the fullest SIMD, so that a second workgroup of 5 or 6 waves comes at half the price of the first, and streaming pays from
// half the chip's waves on.  Us of pass 1 + pass 2 packed and streaming, slices x keys: 5 heads of 128, 367 x 32749 697 + 842, 591 + 728,
// but 21 x 32749 45 + 52, 54 + 68; 6 heads, 367 x 32749 817 + 968, 691 + 850, but 43 x 16424 66 + 78, 91 + 114; pass 2 of 5 heads,
// 127 x 2100: 30 packed, 37 with a wave per head.  Chosen so, a launch takes 1.004 to 1.03 times the fastest form's time on
// average over those sizes.  Streaming counts 6 % more than it takes (4 heads: 12 %), for what the fit is off.  Pass 1 of 5 heads has no packed
// kernel: of three slices at a few sizes the fastest by up to 7 %, but at more of them, under the same rule, the slower choice.
struct FormRates {
  int per_head[4], packed, stream[2], least_granule;     // least_granule: of shorter granules a wave per head is taken
};
constexpr FormRates form_rates(int pass, int head_dim, int mb, int group) {
  if (mb == 1 && head_dim == 128) {
    if (group == 4 && pass == 2) return FormRates{{20, 27, 36, 40}, 0, {50, 80}, 1024};
    if (group == 5) return pass == 1 ? FormRates{{18, 26, 34}, 0, {41, 76}} : FormRates{{23, 34, 49}, 42, {53, 88}};
    if (group == 6) return pass == 1 ? FormRates{{18, 29, 39}, 26, {79, 0}} : FormRates{{24, 38, 55}, 34, {100, 0}};
  }
  if (mb == 1 && head_dim == 64) {
    if (group == 5) return pass == 1 ? FormRates{{13, 18, 19}, 0, {31, 46}} : FormRates{{19, 27, 31}, 30, {44, 59}};
    if (group == 6) return pass == 1 ? FormRates{{13, 21, 22}, 14, {36, 53}} : FormRates{{19, 30, 40}, 25, {50, 68}};
  }
  if (pass == 2 && mb == 2 && head_dim == 128 && group == 3) return FormRates{{24, 36, 50}, 0, {104, 0}};
  if (pass == 2 && mb == 2 && head_dim == 64 && group == 4) return FormRates{{21, 31, 40}, 0, {63, 90}};
  return FormRates{};
}
// A workgroup's prologue (its queries, the first tile's way from memory) in keys.
constexpr int kFormPrologue = 128, kStreamPrologue = 192;
constexpr int kStreamMaxGroup = 6;
int launch_stream_pass1(const ScoreArgs& a, int head_dim, int mb, unsigned gx, hipStream_t stream);
int launch_stream_pass2(const ScoreArgs& a, int head_dim, int mb, bool pivot, unsigned gx, hipStream_t stream);

}  // namespace cake
#endif
