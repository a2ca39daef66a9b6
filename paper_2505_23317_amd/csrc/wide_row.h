// What the kernels of the wider widths share (layer.hip, slim.hip).
#pragma once
#include "kernels.h"

namespace cfdetr {

// Tiles in contiguous runs per XCD (workgroups go round the eight XCDs).
__device__ __forceinline__ int tile_order(int pid, int total) {
  const int per = total >> 3;
  return (pid < (per << 3)) ? (pid & 7) * per + (pid >> 3) : pid;
}

// gemm.hip's gelu_fast
__device__ __forceinline__ float gelu_sig(float x) {
  const float xc = __builtin_amdgcn_fmed3f(x, -8.0f, 8.0f);
  const float x2 = xc * xc;
  const float t = fmaf(fmaf(1.0142780e-03f, x2, -1.0677580e-01f), x2, -2.3011212e+00f) * xc;
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

// Residual rows between the kernels of width 384 lie as these hold them, as MFMA results:
// tiles of 32 rows; in a tile, 32 columns by 32, four blocks of 1 KB, lane l of a wavefront's
// 64 with columns 8 q + 4 (l / 32) .. + 3 of row l % 32 at 16 l of block q.  Rows of floats
// instead would have every load touch 32 rows with 32 bytes each: 3 us for the rows of a
// workgroup when it is alone, 10 us with all CUs at it.

// Mean and 1/sigma of 32 MT rows that a workgroup of four wavefronts holds as MFMA results:
// wavefront w has columns [w D/4, (w + 1) D/4), D = 128 NT.  Each quarter's squares are taken
// about the quarter's own mean and put together exactly.  (Fused multiply-adds are written
// out: left to the compiler they would differ between kernels, and so would the bits.)
template <int NT, int MT>
__device__ __forceinline__ void wide_stats(const f32x16 (&acc)[NT][MT], float* s_red, int l32, int g, int wave, float eps,
                                           float (&mean)[MT], float (&rstd)[MT]) {
  constexpr int D = 128 * NT;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        s += (acc[j][i][4 * q] + acc[j][i][4 * q + 1]) + (acc[j][i][4 * q + 2] + acc[j][i][4 * q + 3]);
    s += __shfl_xor(s, 32, kWave);
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float e = fmaf(s, -4.0f / D, acc[j][i][r]);
        v = fmaf(e, e, v);
      }
    v += __shfl_xor(v, 32, kWave);
    if (g == 0) {
      s_red[(i * 32 + l32) * 8 + wave] = s;
      s_red[(i * 32 + l32) * 8 + 4 + wave] = v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const float4 s = *reinterpret_cast<const float4*>(s_red + (i * 32 + l32) * 8);
    const float4 v = *reinterpret_cast<const float4*>(s_red + (i * 32 + l32) * 8 + 4);
    mean[i] = ((s.x + s.y) + (s.z + s.w)) * (1.0f / D);
    const float d0 = fmaf(mean[i], -(D / 4), s.x), d1 = fmaf(mean[i], -(D / 4), s.y);
    const float d2 = fmaf(mean[i], -(D / 4), s.z), d3 = fmaf(mean[i], -(D / 4), s.w);
    const float between = fmaf(d0, d0, d1 * d1) + fmaf(d2, d2, d3 * d3);
    const float within = (v.x + v.y) + (v.z + v.w);
    rstd[i] = rsqrtf(fmaf(fmaf(between, 4.0f / D, within), 1.0f / D, eps));
  }
}

// The normalised rows in bf16 to LDS: rows of D, 16-byte chunks XORed by the row.  Ends with
// a barrier.
template <int NT, int MT>
__device__ __forceinline__ void wide_norm_to_lds(const f32x16 (&acc)[NT][MT], const float (&mean)[MT], const float (&rstd)[MT],
                                                 const float* gain, const float* offs, unsigned char* sA, int l32, int g,
                                                 int wave) {
  constexpr int D = 128 * NT;
  float shift[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) shift[i] = -mean[i] * rstd[i];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = wave * (D / 4) + j * 32 + 8 * q + 4 * g;
      const float4 ga = *reinterpret_cast<const float4*>(gain + col);
      const float4 of = *reinterpret_cast<const float4*>(offs + col);
      const int chunk = (wave * (D / 4) >> 3) + j * 4 + q;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const float r0 = fmaf(fmaf(acc[j][i][4 * q], rstd[i], shift[i]), ga.x, of.x);
        const float r1 = fmaf(fmaf(acc[j][i][4 * q + 1], rstd[i], shift[i]), ga.y, of.y);
        const float r2 = fmaf(fmaf(acc[j][i][4 * q + 2], rstd[i], shift[i]), ga.z, of.z);
        const float r3 = fmaf(fmaf(acc[j][i][4 * q + 3], rstd[i], shift[i]), ga.w, of.w);
        *reinterpret_cast<uint2*>(sA + (i * 32 + l32) * (2 * D) + ((chunk ^ (l32 & 15)) << 4) + g * 8) =
            make_uint2(pack_bf16x2(r0, r1), pack_bf16x2(r2, r3));
      }
    }
  __syncthreads();
}

}  // namespace cfdetr
