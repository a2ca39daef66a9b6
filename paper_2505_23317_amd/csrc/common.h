// Shared device/host helpers for the cfdetr kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace cfdetr {

constexpr int kWave = 64;
constexpr int kMaxLevels = 3;
constexpr int kMaxBatch = 64;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef uint16_t bf16_t;  // storage type: raw bf16 bit pattern

// Geometry of the patch pyramid, passed by value to kernels.
struct Pyramid {
  int n_levels;
  int patch[kMaxLevels];
  int rows[kMaxLevels];
  int cols[kMaxLevels];
  int img_h, img_w;
};

__device__ __forceinline__ float bf16_to_f32(bf16_t v) {
  return __uint_as_float(static_cast<uint32_t>(v) << 16);
}

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// Two floats -> two bf16 in one dword (lo in bits 0..15), round-to-nearest-even:
// this is the hardware's packed convert (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2 v = {lo, hi};
  bf16x2 b = __builtin_convertvector(v, bf16x2);
  return *reinterpret_cast<uint32_t*>(&b);
}

__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  return static_cast<bf16_t>(pack_bf16x2(f, 0.f) & 0xFFFFu);
}

__device__ __forceinline__ int tok_level(int32_t t) { return (t >> 28) & 0x7; }
__device__ __forceinline__ int tok_row(int32_t t) { return (t >> 14) & 0x3FFF; }
__device__ __forceinline__ int tok_col(int32_t t) { return t & 0x3FFF; }

// Frame index of global token t: the i with cu[i] <= t < cu[i+1] (cu[0] = 0, offsets
// ascending; frames may be empty, and the last i with cu[i] <= t is the one that holds t).
// A bisection: its loads depend on each other, and a walk from the front costs up to B of
// those round trips in front of a tile's first instruction.
__device__ __forceinline__ int frame_of_token(const int32_t* __restrict__ cu, int B, int t) {
  int lo = 0, hi = B - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cu[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// x * Phi(x) for the bf16 path, with Phi(x) ~ 1 / (1 + exp(-x (a + b x^2 + c x^4))),
// coefficients fitted to the erf form (maximum absolute error of the product 2.6e-5 over
// all x, two orders below the bf16 resolution of the values that matter); x is clamped
// to [-8, 8] inside the exponent, where the quartic is still positive.  The epilogue of
// the first FFN contraction evaluates this once per output element, and with K = d the
// main loop is short: seven plain operations and two transcendental ones per element
// keep it well below the cost of the MFMA loop.
constexpr float kGelu1 = -2.3011212e+00f, kGelu3 = -1.0677580e-01f, kGelu5 = 1.0142780e-03f;   // -log2(e) (a, b, c)
__device__ __forceinline__ float gelu_fast(float x) {
  const float xc = __builtin_amdgcn_fmed3f(x, -8.0f, 8.0f);
  const float x2 = xc * xc;
  const float t = fmaf(fmaf(kGelu5, x2, kGelu3), x2, kGelu1) * xc;
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

// Sum over the lanes of a wavefront, delivered to all: lane l adds the lanes l ^ 32, l ^ 16, .. l ^ 1, in
// that order.  Moves between lanes inside the vector unit, and no trips through the LDS (__shfl_xor: 130
// clocks each, one behind the other): a LayerNorm of 1,400 rows of width 768 takes 4.3 us instead of 4.5.
__device__ __forceinline__ float wave_sum(float v) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  u32x2 p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  auto from = [&](int old, auto ctrl, auto banks) {
    return __builtin_amdgcn_update_dpp(old, __float_as_int(v), decltype(ctrl)::value, 0xF, decltype(banks)::value, false);
  };
  const auto all = std::integral_constant<int, 0xF>{};
  v += __int_as_float(from(0, std::integral_constant<int, 0x128>{}, all));   // row_ror:8
  // l ^ 4: four lanes on for the even quads of a row, four back for the odd ones
  v += __int_as_float(from(from(0, std::integral_constant<int, 0x104>{}, std::integral_constant<int, 0x5>{}),
                           std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xA>{}));
  v += __int_as_float(from(0, std::integral_constant<int, 0x4E>{}, all));    // quad_perm [2, 3, 0, 1]
  v += __int_as_float(from(0, std::integral_constant<int, 0xB1>{}, all));    // quad_perm [1, 0, 3, 2]
  return v;
}

// LayerNorm of a row that a wavefront holds in quads of columns (quad lane + 64 j in v[j],
// zeros beyond `quads`): mean first, then the variance of the centred values.  Fused
// multiply-adds are written out, so that every kernel that does this gets the same bits.
template <int NQ>
__device__ __forceinline__ void ln_quad_stats(const float4 (&v)[NQ], int quads, int lane, int d, float eps, float& mean,
                                              float& rstd) {
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < NQ; ++j) sum += (v[j].x + v[j].y) + (v[j].z + v[j].w);
  mean = wave_sum(sum) / (float)d;
  float sq = 0.f;
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    if (lane + 64 * j < quads) {
      const float cx = v[j].x - mean, cy = v[j].y - mean, cz = v[j].z - mean, cw = v[j].w - mean;
      sq += fmaf(cx, cx, cy * cy) + fmaf(cz, cz, cw * cw);
    }
  }
  rstd = rsqrtf(wave_sum(sq) / (float)d + eps);
}
__device__ __forceinline__ float4 ln_quad(const float4& v, float mean, float rstd, const float4& g, const float4& b) {
  return make_float4(fmaf((v.x - mean) * rstd, g.x, b.x), fmaf((v.y - mean) * rstd, g.y, b.y),
                     fmaf((v.z - mean) * rstd, g.z, b.z), fmaf((v.w - mean) * rstd, g.w, b.w));
}

}  // namespace cfdetr
