// cake_quantize_kv: b-bit storage of the retained cache (appendix "Comparison and compatibility
// with quantization methods": eviction combined with a key-per-channel / value-per-token
// quantiser).  Asymmetric uniform quantisation over groups of 32: the keys of a head per channel
// over 32 consecutive retained tokens, the values per token over 32 consecutive channels;
// zero = group minimum, scale = (max - min) / (2^b - 1), code = round-half-even((x - zero) / scale).
// The window rows are not touched: they stay in the compacted arrays as they are.
//
// Two wavefronts per (layer, sequence, head, group of 32 tokens), one for the keys and one for the
// values, no LDS and no barrier: a lane owns one 16-byte piece of a row (the same channels in every
// row it loads), so the keys' per-channel extremes are element-wise over the lane's rows plus a few
// cross-lane steps, the values' per-token extremes are over the lanes of one row that share a
// 32-channel group, and every lane packs and stores the codes of its own pieces.
//
// 10 layers x 8 heads of 6144 rows, bf16 to 4 bits (346 MB): 82.4 -> 75.6 us, 4.6 TB/s, where a plain copy of 1 GiB
// reaches 5.1.  It was bound by vector instructions: every 16-bit piece that held a value near a tie was coded a
// second time with divisions, and the extremes went through LDS permutes.  Keeping the plain product and
// redoing the pieces with ties in a loop behind the others took 108.7 us.
#include <algorithm>
#include <type_traits>

#include "cake_internal.h"

namespace cake {
namespace {

constexpr int kThreads = 256;
constexpr int kGroupsPerBlock = kThreads / 64 / 2;     // a wavefront for the keys and one for the values of each token group
constexpr int kGroup = 32;       // tokens per key group, channels per value group

struct QuantArgs {
  const void* const* k_hat;
  const void* const* v_hat;
  uint8_t* const* k_codes; float* const* k_scale; float* const* k_zero;
  uint8_t* const* v_codes; float* const* v_scale; float* const* v_zero;
  int32_t batch, h_kv, n_entries;
  int32_t cap[kMaxLaunchLayers];
  int32_t keep[kMaxLaunchEntries];                 // [layer of the launch][sequence]
  // workgroups before those of entry e: a workgroup serves kGroupsPerBlock consecutive token groups of
  // one (layer, sequence), so the grid holds no workgroup without rows however uneven the layers' counts are
  int32_t first_block[kMaxLaunchEntries + 1];
};

typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));      // one store; the arrays promise no more than a float's alignment

// The code of x in a group with minimum lo and step sc is round-half-even of the fp32 quotient
// (x - lo) / sc, clamped to [0, levels], 0 in a constant group.
//
// Codes of the N values of one piece, packed low channel first; inv is step_inverse(sc).  The quotient comes from
// a product and two residual corrections: after the first it is within an ulp, and with inv the rounded
// reciprocal the second makes it the correctly rounded one (Markstein, "Computation of elementary functions on
// the IBM RISC System/6000", 1990).  Exactness matters at the ties k + 1/2, which 16-bit inputs meet all the
// time: redoing a piece with the division wherever a plain product came close to one happened in most of
// them and bounded the kernel.  Adding 3 * 2^22 rounds the quotient, half to even, into the low bits of the sum,
// from where one alignbit per value packs it; it is in [0, levels] without a clamp.  Returns whether a sum is
// not, as for a value that is not a number: then the piece has to be coded with the division.
template <int kBits, int N, typename Lo, typename Sc, typename Inv>
__device__ __forceinline__ bool encode_piece(const float (&x)[N], Lo lo, Sc sc, Inv inv, uint64_t& packed) {
  constexpr uint32_t kMost = 0x4b400000u + (1u << kBits) - 1;      // bits of 3 * 2^22 + levels
  constexpr int kWords = (N * kBits + 31) / 32, kPerWord = N / kWords;
  uint32_t word[kWords] = {}, top = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float d = x[i] - lo(i), q0 = d * inv(i), q1 = fmaf(fmaf(-q0, sc(i), d), inv(i), q0);
    const float y = fmaf(fmaf(-q1, sc(i), d), inv(i), q1) + 0x1.8p23f;
    top = max(top, __float_as_uint(y));
    word[i / kPerWord] = __builtin_amdgcn_alignbit(__float_as_uint(y), word[i / kPerWord], kBits);
  }
  packed = word[0] >> (32 - kPerWord * kBits);
  if (kWords == 2) packed |= (uint64_t)word[kWords - 1] << 32;
  return top > kMost;
}
// The same with the division.
template <int kBits, int N, typename Lo, typename Sc>
__device__ __forceinline__ uint64_t encode_by_division(const float (&x)[N], Lo lo, Sc sc) {
  constexpr float levels = (float)((1 << kBits) - 1);
  uint64_t packed = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float c = sc(i) > 0.f ? rintf((x[i] - lo(i)) / sc(i)) : 0.f;
    packed |= (uint64_t)(uint32_t)__builtin_amdgcn_fmed3f(c, 0.f, levels) << (i * kBits);
  }
  return packed;
}
// 1 / sc, rounded: v_rcp_f32 is within an ulp and one Newton step rounds it, but for a mantissa of all ones
// (Markstein's exception).  There, and at magnitudes where a residual may underflow, not a number, which
// sends the group to the division.  0 for a constant group, whose codes are 0.
__device__ __forceinline__ float step_inverse(float sc) {
  const float r = __builtin_amdgcn_rcpf(sc), inv = fmaf(fmaf(-sc, r, 1.f), r, r);
  const uint32_t u = __float_as_uint(sc);
  const bool plain = sc > 0x1p-60f && sc < 0x1p60f && (u & 0x7fffffu) != 0x7fffffu;
  return sc > 0.f ? (plain ? inv : __uint_as_float(0x7fc00000u)) : 0.f;
}

// Smallest and largest over the lanes kFrom, 2 kFrom, .. (below kTo) apart, in all of them, on the vector ALU (a
// permute through LDS for each of the up to 128 steps of a tile kept the LDS pipe busy).
template <int kOff, typename Op>
__device__ __forceinline__ float with_partner(float x, Op op) {
  if constexpr (kOff == 1) return op(x, dpp_step<0xB1, 0xf, false>(x));            // quad_perm [1, 0, 3, 2]
  else if constexpr (kOff == 2) return op(x, dpp_step<0x4E, 0xf, false>(x));       // quad_perm [2, 3, 0, 1]
  else if constexpr (kOff == 4) return op(x, dpp_step<0x141, 0xf, false>(x));      // row_half_mirror: the other quad, whose lanes agree by now
  else if constexpr (kOff == 8) return op(x, dpp_step<0x128, 0xf, false>(x));      // row_ror:8
  else {
    const uint32_t u = __float_as_uint(x);
    const auto r = kOff == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false) : __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
}
template <int kFrom, int kTo>
__device__ __forceinline__ void extremes(float& lo, float& hi) {
  if constexpr (kFrom < kTo) {
    lo = with_partner<kFrom>(lo, [](float a, float b) { return fminf(a, b); });
    hi = with_partner<kFrom>(hi, [](float a, float b) { return fmaxf(a, b); });
    extremes<2 * kFrom, kTo>(lo, hi);
  }
}

// Memory known to be the card's: a pointer read from a table would otherwise be accessed by flat
// instructions, which occupy the LDS path too.
#define CAKE_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ CAKE_GLOBAL T* in_memory(T* p) { return (CAKE_GLOBAL T*)p; }

// The low `bytes` bytes of `packed` (1, 2, 4 or 8; dst is aligned to that size).
__device__ __forceinline__ void store_codes(uint8_t* dst, uint64_t packed, int bytes) {
  if (bytes == 8) *in_memory(reinterpret_cast<uint64_t*>(dst)) = packed;
  else if (bytes == 4) *in_memory(reinterpret_cast<uint32_t*>(dst)) = (uint32_t)packed;
  else if (bytes == 2) *in_memory(reinterpret_cast<uint16_t*>(dst)) = (uint16_t)packed;
  else *in_memory(dst) = (uint8_t)packed;
}

template <typename T, int D, int kBits>
__global__ __launch_bounds__(kThreads) void quantize_kernel(QuantArgs a, LayerStrides st) {
  constexpr int kPer16 = 16 / (int)sizeof(T);        // elements per 16-byte piece
  constexpr int kPieces = D / kPer16;                // pieces per row = lanes per row
  constexpr int kRowsPerLoad = 64 / kPieces;         // rows a wave-wide load covers
  constexpr int kLoads = kGroup / kRowsPerLoad;      // loads per lane and tile
  constexpr int kVLanes = kGroup / kPer16;           // lanes of a row that share a value group
  constexpr int kVGroups = D / kGroup;
  static_assert(64 % kPieces == 0 && kGroup % kRowsPerLoad == 0 && kPieces % kVLanes == 0, "tile does not divide over a wavefront");

  const int lane = threadIdx.x & 63;
  int e = 0;
  for (int hi = a.n_entries; hi - e > 1;) {          // first_block[e] <= blockIdx.x < first_block[e + 1]
    const int mid = (e + hi) >> 1;
    if (a.first_block[mid] <= (int)blockIdx.x) e = mid; else hi = mid;
  }
  const int ll = e / a.batch, b = e % a.batch, h = blockIdx.y;
  const int wave = threadIdx.x >> 6;
  const bool keys = (wave & 1) == 0;                  // even wavefronts take the keys, odd ones the values
  const int tg = ((int)blockIdx.x - a.first_block[e]) * kGroupsPerBlock + (wave >> 1);
  const int keep = a.keep[e];
  const int r0 = tg * kGroup;
  if (r0 >= keep) return;                            // the whole wavefront: there is no barrier below
  const int rows = min(kGroup, keep - r0);
  const int cap = a.cap[ll];
  const int q = lane % kPieces, rg = lane / kPieces;
  constexpr float levels = (float)((1 << kBits) - 1);
  constexpr int code_bytes = kPer16 * kBits / 8;     // of one piece
  constexpr int row_bytes = D * kBits / 8;
  const int64_t head = (int64_t)b * a.h_kv + h;
  const int64_t in_off = b * st.s[ll][0] + h * st.s[ll][1] + (int64_t)r0 * st.s[ll][2] + q * kPer16;
  const int64_t tok = st.s[ll][2];
  const T* src = reinterpret_cast<const T*>(keys ? a.k_hat[ll] : a.v_hat[ll]) + in_off;

  // rows past the end repeat the last one
  auto load_piece = [&](int m) { return *in_memory(reinterpret_cast<const u32x4*>(src + (int64_t)min(m * kRowsPerLoad + rg, rows - 1) * tok)); };
  auto values = [](const u32x4& piece, float (&x)[kPer16]) {
#pragma unroll
    for (int i = 0; i < kPer16; ++i) {
      if constexpr (sizeof(T) == 2) x[i] = __uint_as_float(i & 1 ? piece[i / 2] & 0xffff0000u : piece[i / 2] << 16);
      else x[i] = __uint_as_float(piece[i]);
    }
  };

  u32x4 raw[kLoads];
#pragma unroll
  for (int m = 0; m < kLoads; ++m) raw[m] = load_piece(m);
  // Pieces that need the division are coded again behind the others, one copy of it for all of them.
  uint32_t redo = 0;

  // ---- keys: per channel over the tile's tokens -------------------------------------------
  if (keys) {
    float lo[kPer16], hi[kPer16], sc[kPer16], inv[kPer16], x[kPer16];
    values(raw[0], lo);
    values(raw[0], hi);
#pragma unroll
    for (int m = 1; m < kLoads; ++m) {
      values(raw[m], x);
#pragma unroll
      for (int i = 0; i < kPer16; ++i) {
        lo[i] = fminf(lo[i], x[i]);
        hi[i] = fmaxf(hi[i], x[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < kPer16; ++i) {
      extremes<kPieces, 64>(lo[i], hi[i]);                      // the lanes that hold the same piece of other rows
      sc[i] = (hi[i] - lo[i]) / levels;
      inv[i] = step_inverse(sc[i]);
    }
    if (rg == 0) {
      const int64_t n_groups = (cap + kGroup - 1) / kGroup;
      const int64_t o = (head * n_groups + tg) * D + q * kPer16;
      auto scale = in_memory(reinterpret_cast<f32x4*>(a.k_scale[ll] + o));
      auto zero = in_memory(reinterpret_cast<f32x4*>(a.k_zero[ll] + o));
#pragma unroll
      for (int i = 0; i < kPer16; i += 4) {
        scale[i / 4] = f32x4{sc[i], sc[i + 1], sc[i + 2], sc[i + 3]};
        zero[i / 4] = f32x4{lo[i], lo[i + 1], lo[i + 2], lo[i + 3]};
      }
    }
    uint8_t* out = a.k_codes[ll] + (head * cap + r0) * row_bytes + q * code_bytes;
    auto store = [&](int m, uint64_t packed) {
      const int r = m * kRowsPerLoad + rg;
      if (r < rows) store_codes(out + (int64_t)r * row_bytes, packed, code_bytes);
    };
#pragma unroll
    for (int m = 0; m < kLoads; ++m) {
      uint64_t packed;
      values(raw[m], x);
      if (__ballot(encode_piece<kBits>(x, [&](int i) { return lo[i]; }, [&](int i) { return sc[i]; }, [&](int i) { return inv[i]; }, packed))) redo |= 1u << m;
      store(m, packed);
    }
    for (; redo; redo &= redo - 1) {
      const int m = __builtin_ctz(redo);
      values(load_piece(m), x);
      store(m, encode_by_division<kBits>(x, [&](int i) { return lo[i]; }, [&](int i) { return sc[i]; }));
    }
  } else {
    // ---- values: per token over groups of 32 channels -----------------------------------
    uint8_t* out = a.v_codes[ll] + (head * cap + r0) * row_bytes + q * code_bytes;
    auto scale = in_memory(a.v_scale[ll]), zero = in_memory(a.v_zero[ll]);
    const int64_t o = (head * cap + r0) * kVGroups + q / kVLanes;
    auto group = [&](const float (&x)[kPer16], float& lo, float& sc) {
      float hi = lo = x[0];
#pragma unroll
      for (int i = 1; i < kPer16; ++i) {
        lo = fminf(lo, x[i]);
        hi = fmaxf(hi, x[i]);
      }
      extremes<1, kVLanes>(lo, hi);                              // the lanes of this row's channel group
      sc = (hi - lo) / levels;
    };
    auto store = [&](int m, uint64_t packed) {
      const int r = m * kRowsPerLoad + rg;
      if (r < rows) store_codes(out + (int64_t)r * row_bytes, packed, code_bytes);
    };
    float x[kPer16], lo, sc;
#pragma unroll
    for (int m = 0; m < kLoads; ++m) {
      uint64_t packed;
      values(raw[m], x);
      group(x, lo, sc);
      const float inv = step_inverse(sc);
      if (__ballot(encode_piece<kBits>(x, [&](int) { return lo; }, [&](int) { return sc; }, [&](int) { return inv; }, packed))) redo |= 1u << m;
      const int r = m * kRowsPerLoad + rg;
      if (r < rows && q % kVLanes == 0) {
        scale[o + r * kVGroups] = sc;
        zero[o + r * kVGroups] = lo;
      }
      store(m, packed);
    }
    for (; redo; redo &= redo - 1) {
      const int m = __builtin_ctz(redo);
      values(load_piece(m), x);
      group(x, lo, sc);
      store(m, encode_by_division<kBits>(x, [&](int) { return lo; }, [&](int) { return sc; }));
    }
  }
}

}  // namespace
}  // namespace cake

using namespace cake;

extern "C" int cake_quantize_kv(const cake_shape* shape, int32_t bits,
                                const void* const* k_hat, const void* const* v_hat, const int64_t* kv_strides,
                                const int32_t* keep,
                                uint8_t* const* k_codes, float* const* k_scale, float* const* k_zero,
                                uint8_t* const* v_codes, float* const* v_scale, float* const* v_zero,
                                void* stream) {
  if (int rc = check_shape_basic(shape)) return rc;
  CAKE_REQUIRE(bits == 2 || bits == 4 || bits == 8, "bits = %d must be 2, 4 or 8", bits);
  CAKE_REQUIRE(k_hat && v_hat && kv_strides && keep && k_codes && k_scale && k_zero && v_codes && v_scale && v_zero,
               "a pointer argument is NULL");
  const int B = shape->batch, L = shape->n_layers;
  const int eb = (int)elem_bytes(shape->dtype);
  for (int i = 0; i < L * B; ++i) CAKE_REQUIRE(keep[i] >= 0, "keep[%d] = %d is negative", i, keep[i]);
  for (int i = 0; i < 3 * L; ++i) {
    CAKE_REQUIRE(kv_strides[i] >= 0, "negative stride");
    CAKE_REQUIRE((kv_strides[i] * eb) % 16 == 0, "strides must be multiples of 16 bytes");
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  for (int l0 = 0; l0 < L;) {
    const int nl = launch_layers(L - l0, B);
    QuantArgs a{};
    LayerStrides ls{};
    a.k_hat = k_hat + l0; a.v_hat = v_hat + l0;
    a.k_codes = k_codes + l0; a.k_scale = k_scale + l0; a.k_zero = k_zero + l0;
    a.v_codes = v_codes + l0; a.v_scale = v_scale + l0; a.v_zero = v_zero + l0;
    a.batch = B; a.h_kv = shape->n_kv_heads; a.n_entries = nl * B;
    int64_t n_blocks = 0;
    for (int ll = 0; ll < nl; ++ll) {
      int ck = 0;
      for (int b = 0; b < B; ++b) {
        const int kp = keep[(l0 + ll) * B + b];
        a.keep[ll * B + b] = kp;
        a.first_block[ll * B + b] = (int32_t)n_blocks;
        n_blocks += ((kp + kGroup - 1) / kGroup + kGroupsPerBlock - 1) / kGroupsPerBlock;
        ck = std::max(ck, kp);
      }
      a.cap[ll] = ck;
      for (int j = 0; j < 3; ++j) ls.s[ll][j] = kv_strides[(l0 + ll) * 3 + j];
    }
    a.first_block[nl * B] = (int32_t)n_blocks;
    CAKE_REQUIRE(n_blocks <= 0x7fffffff, "too many rows for one launch");
    if (n_blocks > 0) {
      const dim3 grid((unsigned)n_blocks, shape->n_kv_heads), block(kThreads);
      const bool bf = shape->dtype == CAKE_BF16;
      auto launch = [&](auto bits_c) {
        constexpr int kBits = decltype(bits_c)::value;
        if (bf && shape->head_dim == 128) hipLaunchKernelGGL((quantize_kernel<__bf16, 128, kBits>), grid, block, 0, st, a, ls);
        else if (bf && shape->head_dim == 64) hipLaunchKernelGGL((quantize_kernel<__bf16, 64, kBits>), grid, block, 0, st, a, ls);
        else if (!bf && shape->head_dim == 128) hipLaunchKernelGGL((quantize_kernel<float, 128, kBits>), grid, block, 0, st, a, ls);
        else hipLaunchKernelGGL((quantize_kernel<float, 64, kBits>), grid, block, 0, st, a, ls);
      };
      if (shape->head_dim != 64 && shape->head_dim != 128) return fail(CAKE_ERR_UNSUPPORTED, "no quantiser for head_dim %d", shape->head_dim);
      if (bits == 2) launch(std::integral_constant<int, 2>{});
      else if (bits == 4) launch(std::integral_constant<int, 4>{});
      else launch(std::integral_constant<int, 8>{});
    }
    l0 += nl;
  }
  CAKE_HIP_TRY(hipGetLastError());
  return CAKE_OK;
}
