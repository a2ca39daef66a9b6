// Layers of width 384 when there are few rows: wide_layer_kernel (layer.hip) gives every row to
// one CU, which streams all the weights of the layer past it; below some two thousand rows most
// CUs would have none.  Here a layer is four launches, each spread over the chip, with the same
// arithmetic in the same order (sums that start at the bias or at the residual's low part, its
// LayerNorm), so that a row's result does not depend on how many others there are.
#include "few_rows.h"
#include "wide_row.h"

namespace cfdetr {

namespace {

constexpr int kSlimPad = 32;   // blocks of 1 KB the weight rings read ahead of the end

struct SlimArgs {
  const bf16_t* rows;        // slim_residual_kernel's operand
  const float* x0;           // first layer: the rows as the embedding left them
  float* x;                  // residual blocks (wide_row.h)
  const float *ln_g, *ln_b;
  float eps;
  const unsigned char* w;    // launch_slim_pack's
  const float* bias;
  int parts;                 // 128-column parts of the result
  int K;
  int row_groups;            // XcdTiles
  float q_scale;
  bf16_t* out;               // q/k/v [M, 3D], or hidden blocks
  bf16_t* vt;
  int vt_ld;
  int32_t* vt_pos;
  const int32_t* cu;
  const int32_t* pcu;
  int nseq;
  const int32_t* m_ptr;
  int m_host;
};

template <int D>
__device__ __forceinline__ float* x_block(float* x, int m0, int c, int q, int lane) {
  return x + (((size_t)(m0 >> 5) * (D / 32) + (c >> 5)) * 4 + q) * 256 + lane * 4;
}

// kFirst: q/k/v of the first layer (reads x0, writes x and vt_pos); kQkv: of another one;
// kHidden: first feed-forward matrix and activation, as operands of the second.
constexpr int kFirst = 0, kQkv = 1, kHidden = 2;

// LayerNorm and the contraction behind it, 32 rows x 128 columns a workgroup.  Every workgroup
// of the same rows does their LayerNorm again, which costs 1.4 us in each and no launch (4.5 us).
// All loads of the rows are issued first, then all those of the weights (K = 384 is one ring of
// 24 blocks), which arrive while the rows are normalised.
// 920 rows: 8.5 us for q/k/v, 9.8 us for the hidden units, of which 3 us are the launch, 2 us
// the way of rows and weights into the XCDs; LayerNorm and 64 x 64 tiles took 4.5 and 8 us each.
template <int D, int kOut>
__global__ __launch_bounds__(256, 2) void slim_norm_kernel(SlimArgs p) {
  constexpr int KS = D / 16, NT = D / 128, ROWB = D * 2;
  static_assert(KS == kFewRing, "one ring of weights");
  __shared__ __attribute__((aligned(1024))) unsigned char sA[32 * ROWB];
  __shared__ float s_red[256], s_vec[2 * D];

  const int M = p.m_ptr ? *p.m_ptr : p.m_host;
  const XcdTiles tiles((M + 31) >> 5, p.parts, p.row_groups);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  const float4 vg = *reinterpret_cast<const float4*>(p.ln_g + min(tid * 4, D - 4));
  const float4 vb = *reinterpret_cast<const float4*>(p.ln_b + min(tid * 4, D - 4));

  for (int t = blockIdx.x >> 3; t < tiles.count; t += gridDim.x >> 3) {
    const int part = tiles.p0 + t / tiles.rows, m0 = (tiles.r0 + t % tiles.rows) * 32;
    const int m = min(m0 + l32, M - 1), n0 = part * 128 + wave * 32;
    const bool v_cols = kOut != kHidden && n0 >= 2 * D;
    int vpos = 0;
    if (kOut == kFirst && (v_cols || part == 0)) {
      const int f = frame_of_token(p.cu, p.nseq, m);
      vpos = p.pcu[f] + (m - p.cu[f]);
      if (part == 0 && wave == 0 && g == 0) p.vt_pos[m] = vpos;
    } else if (v_cols) {
      vpos = p.vt_pos[m];
    }
    f32x16 xa[NT][1];   // the wavefront's quarter of the rows' columns
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = wave * (D / 4) + j * 32;
        const float4 v = *reinterpret_cast<const float4*>(kOut == kFirst ? p.x0 + (size_t)m * D + c + 8 * q + 4 * g
                                                                         : x_block<D>(p.x, m0, c, q, lane));
        xa[j][0][4 * q] = v.x;
        xa[j][0][4 * q + 1] = v.y;
        xa[j][0][4 * q + 2] = v.z;
        xa[j][0][4 * q + 3] = v.w;
      }
    float4 b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) b[q] = *reinterpret_cast<const float4*>(p.bias + n0 + 8 * q + 4 * g);
    __builtin_amdgcn_sched_barrier(0);
    const unsigned char* wp = p.w + (size_t)(part * 4 + wave) * (KS * 1024) + lane * 16;
    bf16x8 wr[KS];
#pragma unroll
    for (int i = 0; i < KS; ++i) wr[i] = *reinterpret_cast<const bf16x8*>(wp + i * 1024);
    __builtin_amdgcn_sched_barrier(0);

    if (tid < D / 4) {
      *reinterpret_cast<float4*>(s_vec + tid * 4) = vg;
      *reinterpret_cast<float4*>(s_vec + D + tid * 4) = vb;
    }
    if (kOut == kFirst && part == 0) {
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(x_block<D>(p.x, m0, wave * (D / 4) + j * 32, q, lane)) =
              make_float4(xa[j][0][4 * q], xa[j][0][4 * q + 1], xa[j][0][4 * q + 2], xa[j][0][4 * q + 3]);
    }
    float mean[1], rstd[1];
    wide_stats<4>(xa, s_red, l32, g, wave, p.eps, mean, rstd);
    wide_norm_to_lds<4>(xa, mean, rstd, s_vec, s_vec + D, sA, l32, g, wave);

    f32x16 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc[4 * q] = b[q].x;
      acc[4 * q + 1] = b[q].y;
      acc[4 * q + 2] = b[q].z;
      acc[4 * q + 3] = b[q].w;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          wr[ks], *reinterpret_cast<const bf16x8*>(sA + l32 * ROWB + (((2 * ks + g) ^ (l32 & 15)) << 4)), acc, 0, 0, 0);

    const bool in = m0 + l32 < M;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int n = n0 + 8 * q + 4 * g;
      const float r0 = acc[4 * q], r1 = acc[4 * q + 1], r2 = acc[4 * q + 2], r3 = acc[4 * q + 3];
      if (kOut == kHidden) {
        // k-step n / 16 of the next contraction, the row's lane in it
        const size_t blk = (size_t)(m0 >> 5) * (p.parts * 8) + (n0 >> 4) + (q >> 1);
        *reinterpret_cast<uint2*>(reinterpret_cast<unsigned char*>(p.out) + blk * 1024 + (l32 + 32 * (q & 1)) * 16 + g * 8) =
            make_uint2(pack_bf16x2(gelu_fast(r0), gelu_fast(r1)), pack_bf16x2(gelu_fast(r2), gelu_fast(r3)));
      } else if (v_cols) {
        if (in) {
          bf16_t* vp = p.vt + (size_t)(n - 2 * D) * p.vt_ld + vpos;
          vp[0] = f32_to_bf16(r0);
          vp[(size_t)p.vt_ld] = f32_to_bf16(r1);
          vp[(size_t)2 * p.vt_ld] = f32_to_bf16(r2);
          vp[(size_t)3 * p.vt_ld] = f32_to_bf16(r3);
        }
      } else if (in) {
        const float sc = n0 < D ? p.q_scale : 1.0f;
        *reinterpret_cast<uint2*>(p.out + (size_t)m * (3 * D) + n) =
            make_uint2(pack_bf16x2(r0 * sc, r1 * sc), pack_bf16x2(r2 * sc, r3 * sc));
      }
    }
    __syncthreads();   // the rows' place is free
  }
}

// x += operand . W^T + bias: attention rows times the output projection, or (kBlocks) the
// hidden blocks times the second feed-forward matrix.  920 rows: 5.2 and 9.5 us (64 x 64 tiles
// took 9.5 and 17 us), the latter the K = 1536 of a wavefront at what a CU's vector-memory path
// gives.
template <int D, bool kBlocks>
__global__ __launch_bounds__(256, 2) void slim_residual_kernel(SlimArgs p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int M = p.m_ptr ? *p.m_ptr : p.m_host;
  const XcdTiles tiles((M + 31) >> 5, D / 128, p.row_groups);
  const int lane = threadIdx.x & 63, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int t = blockIdx.x >> 3; t < tiles.count; t += gridDim.x >> 3) {
    const int part = tiles.p0 + t / tiles.rows, m0 = (tiles.r0 + t % tiles.rows) * 32, n0 = part * 128 + wave * 32;
    float4 b[4];
    f32x16 x, acc[1];
    u32x8 hi;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      b[q] = *reinterpret_cast<const float4*>(p.bias + n0 + 8 * q + 4 * g);
      const float4 v = *reinterpret_cast<const float4*>(x_block<D>(p.x, m0, n0, q, lane));
      x[4 * q] = v.x;
      x[4 * q + 1] = v.y;
      x[4 * q + 2] = v.z;
      x[4 * q + 3] = v.w;
    }
    few_rows_product<1, kBlocks>(p.rows, p.K, M, m0, p.w + (size_t)(part * 4 + wave) * (p.K >> 4) * 1024, smem, acc, [&]() {
      acc[0] = x;
      residual_split(acc[0], hi);
    });
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      residual_join(acc[0], hi, q, b[q]);
      *reinterpret_cast<float4*>(x_block<D>(p.x, m0, n0, q, lane)) =
          make_float4(acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]);
    }
    __syncthreads();
  }
}

// wide_layer_kernel's final LayerNorm, 32 rows a workgroup.
template <int D>
__global__ __launch_bounds__(256) void wide_norm_kernel(float* x, const float* ln_g, const float* ln_b, float eps, float* out,
                                                        int split_row, float* out2, const int32_t* m_ptr, int m_host) {
  constexpr int NT = D / 128;
  __shared__ float s_red[256];
  const int M = m_ptr ? *m_ptr : m_host;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, g = lane >> 5, m0 = blockIdx.x * 32, m = m0 + l32;
  if (m0 >= M) return;
  f32x16 xa[NT][1];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = *reinterpret_cast<const float4*>(x_block<D>(x, m0, wave * (D / 4) + j * 32, q, lane));
      xa[j][0][4 * q] = v.x;
      xa[j][0][4 * q + 1] = v.y;
      xa[j][0][4 * q + 2] = v.z;
      xa[j][0][4 * q + 3] = v.w;
    }
  float mean[1], rstd[1];
  wide_stats<4>(xa, s_red, l32, g, wave, eps, mean, rstd);
  if (m >= M) return;
  const bool second = out2 != nullptr && m >= split_row;
  float* const o = (second ? out2 : out) + (size_t)(second ? m - split_row : m) * D;
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = wave * (D / 4) + j * 32 + 8 * q + 4 * g;
      const float4 ga = *reinterpret_cast<const float4*>(ln_g + col), of = *reinterpret_cast<const float4*>(ln_b + col);
      *reinterpret_cast<float4*>(o + col) = make_float4(wide_normed(xa[j][0][4 * q], mean[0], rstd[0], ga.x, of.x),
                                                        wide_normed(xa[j][0][4 * q + 1], mean[0], rstd[0], ga.y, of.y),
                                                        wide_normed(xa[j][0][4 * q + 2], mean[0], rstd[0], ga.z, of.z),
                                                        wide_normed(xa[j][0][4 * q + 3], mean[0], rstd[0], ga.w, of.w));
    }
}

// W [N, K] as MFMA operands: [N / 32][K / 16][64 lanes][8].  One thread per 16 bytes.
__global__ __launch_bounds__(256) void slim_pack_kernel(const bf16_t* __restrict__ W, int K, long units,
                                                        bf16_t* __restrict__ out) {
  const long u = (long)blockIdx.x * 256 + threadIdx.x;
  if (u >= units) return;
  const int lane = (int)(u & 63), ks = K >> 4;
  const long blk = u >> 6, n = (blk / ks) * 32 + (lane & 31);
  const int k = (int)(blk % ks) * 16 + (lane >> 5) * 8;
  reinterpret_cast<uint4*>(out)[u] = *reinterpret_cast<const uint4*>(W + n * K + k);
}

}  // namespace

bool few_rows_supported(int N, int K) { return N % 128 == 0 && K % (16 * kFewRing) == 0; }

uint64_t slim_packed_bytes(uint64_t N, uint64_t K) { return N * K * 2 + kSlimPad * 1024; }

hipError_t launch_slim_pack(const void* W, uint64_t N, int K, void* packed, hipStream_t s) {
  const long units = (long)(N * K / 8);
  hipLaunchKernelGGL(slim_pack_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, s,
                     static_cast<const bf16_t*>(W), K, units, static_cast<bf16_t*>(packed));
  return hipGetLastError();
}

hipError_t launch_slim(const SlimLayerArgs& a, SlimStep step, int d, int F, int rows, const int32_t* m_ptr, int m_host,
                       int m_capacity, hipStream_t s) {
  if (d != 384 || !few_rows_supported(F, F)) return hipErrorInvalidValue;
  SlimArgs p{};
  p.rows = static_cast<const bf16_t*>(a.rows);
  p.x0 = a.x0;
  p.x = a.x;
  p.ln_g = a.ln_g;
  p.ln_b = a.ln_b;
  p.eps = a.eps;
  p.w = static_cast<const unsigned char*>(a.w);
  p.bias = a.bias;
  p.parts = step == SlimStep::kHidden ? F / 128 : step == SlimStep::kOut || step == SlimStep::kDown ? d / 128 : 3 * d / 128;
  p.K = step == SlimStep::kDown ? F : d;
  p.q_scale = a.q_scale;
  p.out = static_cast<bf16_t*>(a.out);
  p.vt = static_cast<bf16_t*>(a.vt);
  p.vt_ld = a.vt_ld;
  p.vt_pos = a.vt_pos;
  p.cu = a.cu;
  p.pcu = a.pcu;
  p.nseq = a.nseq;
  p.m_ptr = m_ptr;
  p.m_host = m_host;
  const dim3 grid = few_rows_grid(rows, m_capacity, p.parts, p.K, 1, &p.row_groups);
  switch (step) {
    case SlimStep::kFirstQkv: {
      constexpr auto kern = slim_norm_kernel<384, kFirst>;
      hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, p);
      break;
    }
    case SlimStep::kQkv: {
      constexpr auto kern = slim_norm_kernel<384, kQkv>;
      hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, p);
      break;
    }
    case SlimStep::kHidden: {
      constexpr auto kern = slim_norm_kernel<384, kHidden>;
      hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, p);
      break;
    }
    case SlimStep::kOut: {
      constexpr auto kern = slim_residual_kernel<384, false>;
      hipLaunchKernelGGL(kern, grid, dim3(256), few_rows_lds(1), s, p);
      break;
    }
    case SlimStep::kDown: {
      constexpr auto kern = slim_residual_kernel<384, true>;
      hipLaunchKernelGGL(kern, grid, dim3(256), few_rows_lds(1), s, p);
      break;
    }
  }
  return hipGetLastError();
}

hipError_t launch_wide_norm(float* x, const float* ln_g, const float* ln_b, int d, float eps, float* out, int split_row,
                            float* out2, const int32_t* m_ptr, int m_host, int m_capacity, hipStream_t s) {
  if (d != 384) return hipErrorInvalidValue;
  hipLaunchKernelGGL(wide_norm_kernel<384>, dim3((m_capacity + 31) / 32), dim3(256), 0, s, x, ln_g, ln_b, eps, out, split_row,
                     out2, m_ptr, m_host);
  return hipGetLastError();
}

}  // namespace cfdetr
