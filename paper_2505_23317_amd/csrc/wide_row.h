// What the kernels of the wider widths share (layer.hip, few_rows.hip).
#pragma once
#include "kernels.h"

namespace cfdetr {

// Tiles in contiguous runs per XCD (workgroups go round the eight XCDs).
__device__ __forceinline__ int tile_order(int pid, int total) {
  const int per = total >> 3;
  return (pid < (per << 3)) ? (pid & 7) * per + (pid >> 3) : pid;
}

// Addresses that follow from a lane's numbers are the same at every use, and the compiler keeps
// them from the first to the last, in scratch memory where registers run out.  Behind this call it
// does not know that they are.
__device__ __forceinline__ void work_out_here(int& v) { asm volatile("" : "+v"(v)); }

// Residual rows between the kernels of these widths lie as these hold them, as MFMA results:
// tiles of 32 rows; in a tile, 32 columns by 32, four blocks of 1 KB, lane l of a wavefront's
// 64 with columns 8 q + 4 (l / 32) .. + 3 of row l % 32 at 16 l of block q.  Rows of floats
// instead would have every load touch 32 rows with 32 bytes each: 3 us for the rows of a
// workgroup when it is alone, 10 us with all CUs at it.

// A residual and what is added to it.  An MFMA rounds its sum, so a product that is accumulated
// on top of the residual rounds at the residual's magnitude in every step.  Here it starts at the
// low part: residual_split leaves x - hi in acc, hi the bf16 next to x (the difference is exact),
// and residual_join gives hi + (acc + b), one rounding at x's magnitude.  The low part, 2^-9 of x
// at most, is what a sum from 0 would start at as far as rounding goes, and hi is half the bytes
// that x would be.
typedef __attribute__((ext_vector_type(8))) uint32_t u32x8;
__device__ __forceinline__ void residual_split(f32x16& acc, u32x8& hi) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    uint32_t h = pack_bf16x2(acc[2 * e], acc[2 * e + 1]);
    acc[2 * e] -= __uint_as_float(h << 16);
    acc[2 * e + 1] -= __uint_as_float(h & 0xffff0000u);
    asm volatile("" : "+v"(h));   // (or the compiler keeps both halves as floats)
    hi[e] = h;
  }
}
__device__ __forceinline__ void residual_join(f32x16& acc, const u32x8& hi, int q, const float4& b) {
  acc[4 * q] = __uint_as_float(hi[2 * q] << 16) + (acc[4 * q] + b.x);
  acc[4 * q + 1] = __uint_as_float(hi[2 * q] & 0xffff0000u) + (acc[4 * q + 1] + b.y);
  acc[4 * q + 2] = __uint_as_float(hi[2 * q + 1] << 16) + (acc[4 * q + 2] + b.z);
  acc[4 * q + 3] = __uint_as_float(hi[2 * q + 1] & 0xffff0000u) + (acc[4 * q + 3] + b.w);
}

// Mean and 1/sigma of 32 MT rows that a workgroup of NW (four or eight) wavefronts holds as
// MFMA results: wavefront w has columns [w D/NW, (w + 1) D/NW), D = 32 NT NW.  Each part's
// squares are taken about the part's own mean and put together exactly.  (Fused multiply-adds are written
// out: left to the compiler they would differ between kernels, and so would the bits.)
template <int NW, int NT, int MT>
__device__ __forceinline__ void wide_stats(const f32x16 (&acc)[NT][MT], float* s_red, int l32, int g, int wave, float eps,
                                           float (&mean)[MT], float (&rstd)[MT]) {
  constexpr int D = 32 * NT * NW;
  constexpr float kInvN = (float)NW / D;   // of a part's columns
  work_out_here(l32);
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
        const float e = fmaf(s, -kInvN, acc[j][i][r]);
        v = fmaf(e, e, v);
      }
    v += __shfl_xor(v, 32, kWave);
    if (g == 0) {
      s_red[(i * 32 + l32) * (2 * NW) + wave] = s;
      s_red[(i * 32 + l32) * (2 * NW) + NW + wave] = v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const float4* const part = reinterpret_cast<const float4*>(s_red + (i * 32 + l32) * (2 * NW));
    float sum = 0.f, within = 0.f, between = 0.f;
#pragma unroll
    for (int k = 0; k < NW / 4; ++k) {
      const float4 s = part[k], v = part[NW / 4 + k];
      sum += (s.x + s.y) + (s.z + s.w);
      within += (v.x + v.y) + (v.z + v.w);
    }
    mean[i] = sum / D;   // (1 / 384 is no float: times that, the mean of equal values would not be that value)
#pragma unroll
    for (int k = 0; k < NW / 4; ++k) {
      const float4 s = part[k];
      const float d0 = fmaf(mean[i], -(D / NW), s.x), d1 = fmaf(mean[i], -(D / NW), s.y);
      const float d2 = fmaf(mean[i], -(D / NW), s.z), d3 = fmaf(mean[i], -(D / NW), s.w);
      between += fmaf(d0, d0, d1 * d1) + fmaf(d2, d2, d3 * d3);
    }
    rstd[i] = rsqrtf(fmaf(fmaf(between, kInvN, within), 1.0f / D, eps));
  }
}

// The mean is taken off first: next to it x - mean is exact, while x rstd and mean rstd would
// each be rounded at the mean's magnitude.
__device__ __forceinline__ float wide_normed(float x, float mean, float rstd, float gain, float offs) {
  return fmaf((x - mean) * rstd, gain, offs);
}

// The normalised rows in bf16 to LDS: rows of D, 16-byte chunks XORed by the row.  Ends with
// a barrier.
template <int NW, int NT, int MT>
__device__ __forceinline__ void wide_norm_to_lds(const f32x16 (&acc)[NT][MT], const float (&mean)[MT], const float (&rstd)[MT],
                                                 const float* gain, const float* offs, unsigned char* sA, int l32, int g,
                                                 int wave) {
  constexpr int D = 32 * NT * NW;
  work_out_here(l32);
  work_out_here(g);
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = wave * (D / NW) + j * 32 + 8 * q + 4 * g;
      const float4 ga = *reinterpret_cast<const float4*>(gain + col);
      const float4 of = *reinterpret_cast<const float4*>(offs + col);
      const int chunk = (wave * (D / NW) >> 3) + j * 4 + q;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const float r0 = wide_normed(acc[j][i][4 * q], mean[i], rstd[i], ga.x, of.x);
        const float r1 = wide_normed(acc[j][i][4 * q + 1], mean[i], rstd[i], ga.y, of.y);
        const float r2 = wide_normed(acc[j][i][4 * q + 2], mean[i], rstd[i], ga.z, of.z);
        const float r3 = wide_normed(acc[j][i][4 * q + 3], mean[i], rstd[i], ga.w, of.w);
        *reinterpret_cast<uint2*>(sA + (i * 32 + l32) * (2 * D) + ((chunk ^ (l32 & 15)) << 4) + g * 8) =
            make_uint2(pack_bf16x2(r0, r1), pack_bf16x2(r2, r3));
      }
    }
  __syncthreads();
}

}  // namespace cfdetr
