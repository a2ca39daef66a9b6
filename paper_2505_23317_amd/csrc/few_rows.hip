// Layers of width 384 when there are few rows: wide_layer_kernel (layer.hip) gives every row to
// one CU, which streams all the weights of the layer past it; up to 15 rows a CU (3,840 rows on 256 CUs) half of the
// CUs and more would have none.  Here a layer is three launches, each spread over the chip, with the same
// arithmetic in the same order (sums that start at the bias or at the residual's low part, its
// LayerNorm), so that a row's result does not depend on how many others there are.
#include "few_rows.h"
#include "wide_row.h"

namespace cfdetr {

namespace {

constexpr int kAhead = 5;         // k-steps that operands are asked for ahead of their MFMAs (few_rows.h)
constexpr int kSlimMaxN = 2048;   // widest second matrix of slim_norm_kernel (its bias is in LDS)

// slim_norm_kernel's arguments behind those that it takes one by one: these are in scalar registers when a workgroup
// starts (build.py), a structure is a trip to memory away.
struct SlimArgs {
  const float* x0;           // first layer: the rows as the embedding left them, or x0_rows rows over and over
  int x0_rows;
  const float *ln_g, *ln_b;
  float eps;
  const float* bias;         // of the projection
  float* x_new;              // the new residual rows
  const float* bias2;
  int parts;                 // 128-column parts of the result
  float q_scale;
  bf16_t* out;               // q/k/v [M, 3D], other rows [M, D], or hidden blocks
  bf16_t* z;
  bf16_t* vt;
  int vt_ld;
  int32_t* vt_pos;
  const int32_t* cu;
  const int32_t* pcu;
  int nseq;
};

template <int D>
__device__ __forceinline__ float* x_block(float* x, int m0, int c, int q, int lane) {
  return x + (((size_t)(m0 >> 5) * (D / 32) + (c >> 5)) * 4 + q) * 256 + lane * 4;
}

// The activation of a wavefront's 32 rows x 32 columns, as operands of the next contraction: k-step
// n / 16 of it, the row's lane in that.
__device__ __forceinline__ void hidden_store(const SlimArgs& p, int m0, int n0, int l32, int g, const f32x16& r) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const size_t blk = (size_t)(m0 >> 5) * (p.parts * 8) + (n0 >> 4) + (q >> 1);
    *reinterpret_cast<uint2*>(reinterpret_cast<unsigned char*>(p.out) + blk * 1024 + (l32 + 32 * (q & 1)) * 16 + g * 8) =
        make_uint2(pack_bf16x2(gelu_fast(r[4 * q]), gelu_fast(r[4 * q + 1])),
                   pack_bf16x2(gelu_fast(r[4 * q + 2]), gelu_fast(r[4 * q + 3])));
  }
}

// What a kernel's contraction is.  kFirst: q/k/v of the first layer (reads x0, writes x and vt_pos); kQkv: of
// another one; kRelu: a square matrix with its activation (the normalised rows themselves go to z);
// kHidden: first feed-forward matrix and activation, as operands of the second; kQuery: the decoder's
// query projection.
constexpr int kFirst = 0, kQkv = 1, kRelu = 2, kHidden = 3, kQuery = 4;

// x: residual blocks (wide_row.h); w_rows, w_parts: the matrices of the projection and of the contraction, as
// launch_slim_pack leaves them; shares, per_share: shares of a row tile and parts of a share; row_bits: XcdTiles.
// LayerNorm of the residual rows and a contraction behind it.  kHidden and kQuery project the attention's
// rows first: x_new = x + rows . W^T + bias, and the LayerNorm is of x_new.  32 rows and a run of p.per_share
// 128-column parts of the contraction a workgroup: every workgroup of the same rows does their projection
// (D x D weights, 0.3 MB at D = 384) and their LayerNorm (1.4 us) again, which costs less than a launch
// of its own and rows that go through memory.  The first share writes x_new, which is not x because
// the others may not have read that yet.
// Wavefront w has columns [w D/4, (w + 1) D/4) of the rows, then 32 columns of every part; one ring of D/16
// weight blocks serves projection and parts, refilled behind each MFMA.
// Bounds: the chain launch (2.5 us) - first loads (1.5) - ring rounds at a CU's 64 B/clk (0.8 each; the projection
// is three) - LayerNorm (1.4) - stores, over 920 rows 7.3 us for q/k/v and 11.5 us for projection and
// hidden units.  Before, a launch each and an LDS wait in front of every MFMA: 8, 5.5 and 9.6 us.
template <int D, int kOut>
__global__ __launch_bounds__(256, 2) void slim_norm_kernel(const int32_t* m_ptr, const unsigned char* w_rows, const unsigned char* w_parts,
                                                            const bf16_t* rows, float* x, int m_host, int shares, int per_share,
                                                            int row_bits, SlimArgs p) {
  constexpr bool kProject = kOut == kHidden || kOut == kQuery;
  constexpr int KS = D / 16, NT = D / 128, ROWB = D * 2, UN = KS / NT;
  static_assert(UN == 8, "eight k-steps of the projection a ring round");
  __shared__ __attribute__((aligned(1024))) unsigned char sA[32 * ROWB];
  __shared__ float s_red[256], s_vec[3 * D], s_bias[kSlimMaxN];

  const int M = m_ptr ? *m_ptr : m_host;
  const XcdTiles tiles((M + 31) >> 5, shares, row_bits);
  if (tiles.none) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t voff;
  // 16 bytes a lane of block i at `base`, whose address is worked out in scalar registers and where it
  // is used: no vector arithmetic, and nothing kept
  typedef __attribute__((address_space(1))) unsigned char* gptr;
  auto at = [&](const void* base, int i) {
    gptr q = (gptr)base;
    asm volatile("" : "+s"(q));
    return q + i * 1024 + voff;
  };
  auto block = [&](const void* base, int i) { return *reinterpret_cast<const __attribute__((address_space(1))) bf16x8*>(at(base, i)); };

  const int share = tiles.part, part0 = share * per_share, part1 = min(part0 + per_share, p.parts);
  for (int t = tiles.r; t < tiles.r_end; t += tiles.step) {
    const int m0 = t * 32;
    int tid = threadIdx.x;
    work_out_here(tid);   // (or the addresses of a row tile are kept from tile to tile, in scratch memory)
    const int lane = tid & 63, l32 = lane & 31, g = lane >> 5, m = min(m0 + l32, M - 1);
    voff = lane * 16;
    int vpos = 0;   // place of the row in vt
    if ((kOut == kFirst || kOut == kQkv) && (part1 * 128 > 2 * D || share == 0)) {
      if (kOut == kQkv) {
        vpos = p.vt_pos[m];
      } else {
        const int f = frame_of_token(p.cu, p.nseq, m);
        vpos = p.pcu[f] + (m - p.cu[f]);
        if (share == 0 && wave == 0 && g == 0) p.vt_pos[m] = vpos;
      }
    }
    const int vat = min(tid * 4, D - 4);
    float4 vo;
    if (kProject) vo = *reinterpret_cast<const float4*>(p.bias + vat);
    const float4 vg = *reinterpret_cast<const float4*>(p.ln_g + vat);
    const float4 vb = *reinterpret_cast<const float4*>(p.ln_b + vat);
    static_assert(kSlimMaxN == 2048, "two pieces");   // the share's biases
    const float4 vc0 = *reinterpret_cast<const float4*>(p.bias2 + min(part0 * 128 + tid * 4, p.parts * 128 - 4));
    const float4 vc1 = *reinterpret_cast<const float4*>(p.bias2 + min(part0 * 128 + 1024 + tid * 4, p.parts * 128 - 4));
    // the attention's rows into LDS: 128 columns by 128, 32 rows of 256 bytes each, chunks XORed by the row
    if (kProject) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = (wave * 2 + i) * 4 + (lane >> 4);
        const unsigned char* src = reinterpret_cast<const unsigned char*>(rows + (size_t)min(m0 + row, M - 1) * D) +
                                   (((lane & 15) ^ (row & 15)) << 4);
#pragma unroll
        for (int j = 0; j < NT; ++j)
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                       : : "s"((uint32_t)(uintptr_t)sA + j * 8192 + (wave * 2 + i) * 1024), "v"(src + j * 256) : "memory");
      }
    }
    f32x16 acc[NT][1];
    u32x8 hi[NT];
    const size_t x0 = ((size_t)(m0 >> 5) * (D / 32) + wave * NT) * 1024;   // residual blocks of the wavefront
    const int row0 = kOut == kFirst && p.x0_rows > 0 ? m % p.x0_rows : m;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = kOut == kFirst
                            ? *reinterpret_cast<const f32x4*>(p.x0 + (size_t)row0 * D + wave * (D / 4) + j * 32 + 8 * q + 4 * g)
                            : *reinterpret_cast<const __attribute__((address_space(1))) f32x4*>(at(x + x0, j * 4 + q));
        acc[j][0][4 * q] = v[0];
        acc[j][0][4 * q + 1] = v[1];
        acc[j][0][4 * q + 2] = v[2];
        acc[j][0][4 * q + 3] = v[3];
      }
    __builtin_amdgcn_sched_barrier(0);
    // block ks NT + j of the ring: column tile j of k-step ks of the projection, then k-step ks of a part
    const unsigned char* const wo = w_rows + (size_t)(wave * NT) * (KS * 1024);
    const unsigned char* w2 = w_parts + (size_t)(part0 * 4 + wave) * (KS * 1024);
    bf16x8 wr[KS];
#pragma unroll
    for (int i = 0; i < KS; ++i) wr[i] = kProject ? block(wo, (i % NT) * KS + i / NT) : block(w2, i);
    __builtin_amdgcn_sched_barrier(0);
    if (tid < D / 4) {
      if (kProject) *reinterpret_cast<float4*>(s_vec + tid * 4) = vo;
      *reinterpret_cast<float4*>(s_vec + D + tid * 4) = vg;
      *reinterpret_cast<float4*>(s_vec + 2 * D + tid * 4) = vb;
    }
    *reinterpret_cast<float4*>(s_bias + tid * 4) = vc0;
    *reinterpret_cast<float4*>(s_bias + 1024 + tid * 4) = vc1;

    bf16x8 a[kAhead + 1];
    uint32_t ao[8];
    auto operand = [&](int ks, int next_8) {
      a[ks % (kAhead + 1)] = *reinterpret_cast<const bf16x8*>(sA + ao[ks & 7] + (ks >> 3) * next_8);
    };
    auto operand_addresses = [&](int row_bytes) {
      int lx = l32;
      work_out_here(lx);
#pragma unroll
      for (int k = 0; k < 8; ++k) ao[k] = lx * row_bytes + (((2 * k + g) ^ (lx & 15)) << 4);
    };
    if (kProject) {
#pragma unroll
      for (int j = 0; j < NT; ++j) residual_split(acc[j][0], hi[j]);
      // the rows' loads are older than the ring's
      asm volatile("s_waitcnt vmcnt(%0)" : : "n"(KS) : "memory");
      __syncthreads();
      operand_addresses(256);
#pragma unroll
      for (int ks = 0; ks < kAhead; ++ks) operand(ks, 8192);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + kAhead < KS) operand(ks + kAhead, 8192);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const int i = (ks % UN) * NT + j;
          acc[j][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[i], a[ks % (kAhead + 1)], acc[j][0], 0, 0, 0);
          wr[i] = ks + UN < KS ? block(wo, j * KS + ks + UN) : block(w2, i);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          residual_join(acc[j][0], hi[j], q, *reinterpret_cast<const float4*>(s_vec + wave * (D / 4) + j * 32 + 8 * q + 4 * g));
    }
    if ((kProject || kOut == kFirst) && share == 0) {
      float* const xo = (kProject ? p.x_new : x) + x0;
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<__attribute__((address_space(1))) f32x4*>(at(xo, j * 4 + q)) =
              f32x4{acc[j][0][4 * q], acc[j][0][4 * q + 1], acc[j][0][4 * q + 2], acc[j][0][4 * q + 3]};
    }
    float mean[1], rstd[1];
    wide_stats<4>(acc, s_red, l32, g, wave, p.eps, mean, rstd);
    wide_norm_to_lds<4>(acc, mean, rstd, s_vec + D, s_vec + 2 * D, sA, l32, g, wave);
    if (kOut == kRelu && share == 0) {
#pragma unroll
      for (int u0 = 0; u0 < 32 * (ROWB / 16); u0 += 256) {
        const int u = u0 + tid, row = u / (ROWB / 16), pos = u % (ROWB / 16);
        const int c = (pos & ~15) | ((pos ^ row) & 15);
        if (m0 + row < M)
          *reinterpret_cast<uint4*>(p.z + (size_t)(m0 + row) * D + c * 8) = *reinterpret_cast<const uint4*>(sA + u * 16);
      }
    }

    operand_addresses(ROWB);
    auto one_part = [&](int part, auto more_tag) {
      constexpr bool kMore = decltype(more_tag)::value;   // another part's weights are asked for
      const int n0 = part * 128 + wave * 32;
      const float* const bias = s_bias + n0 - part0 * 128 + 4 * g;
      f32x16 r;   // (kRelu: the bias is added to the sum, as the tiled contraction does)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 b = *reinterpret_cast<const float4*>(bias + 8 * q);
        r[4 * q] = kOut == kRelu ? 0.f : b.x;
        r[4 * q + 1] = kOut == kRelu ? 0.f : b.y;
        r[4 * q + 2] = kOut == kRelu ? 0.f : b.z;
        r[4 * q + 3] = kOut == kRelu ? 0.f : b.w;
      }
      w2 += 4 * KS * 1024;
#pragma unroll
      for (int ks = 0; ks < kAhead; ++ks) operand(ks, 256);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + kAhead < KS) operand(ks + kAhead, 256);
        __builtin_amdgcn_sched_barrier(0);
        r = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[ks], a[ks % (kAhead + 1)], r, 0, 0, 0);
        if (kMore) wr[ks] = block(w2, ks);
      }
      if (kOut == kHidden) {
        hidden_store(p, m0, n0, l32, g, r);
      } else if (m0 + l32 < M) {
        if ((kOut == kFirst || kOut == kQkv) && n0 >= 2 * D) {
          bf16_t* vp = p.vt + (size_t)(n0 + 4 * g - 2 * D) * p.vt_ld + vpos;
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            *vp = f32_to_bf16(r[e]);
            vp += (size_t)((e & 3) == 3 ? 5 : 1) * p.vt_ld;
          }
        } else {
          const float sc = kOut == kQuery || (kOut != kRelu && n0 < D) ? p.q_scale : 1.0f;
          bf16_t* const op = p.out + (size_t)m * (kOut == kFirst || kOut == kQkv ? 3 * D : D) + n0 + 4 * g;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (kOut == kRelu) {
              const float4 b = *reinterpret_cast<const float4*>(bias + 8 * q);
              r[4 * q] = fmaxf(r[4 * q] + b.x, 0.f);
              r[4 * q + 1] = fmaxf(r[4 * q + 1] + b.y, 0.f);
              r[4 * q + 2] = fmaxf(r[4 * q + 2] + b.z, 0.f);
              r[4 * q + 3] = fmaxf(r[4 * q + 3] + b.w, 0.f);
            }
            *reinterpret_cast<uint2*>(op + 8 * q) = make_uint2(pack_bf16x2(r[4 * q] * sc, r[4 * q + 1] * sc),
                                                               pack_bf16x2(r[4 * q + 2] * sc, r[4 * q + 3] * sc));
          }
        }
      }
    };
#pragma nounroll
    for (int part = part0; part + 1 < part1; ++part) one_part(part, std::true_type{});
    one_part(part1 - 1, std::false_type{});
    __syncthreads();   // the rows' place is free
  }
}

// x += hidden blocks . W^T + bias, the second feed-forward matrix: 32 MT rows x 32 NW columns a workgroup.
// 920 rows: 6.1 us (four wavefronts 7.3), the operands of a workgroup at what a CU's vector-memory path gives.  Two
// wavefronts are one a SIMD: their ring of 48 blocks does not fit beside another's.
template <int D, int MT, int NW>
__global__ __launch_bounds__(64 * NW, NW == 2 ? 1 : 2) void slim_residual_kernel(const int32_t* m_ptr, const unsigned char* w, const bf16_t* rows, float* x,
                                                                const float* bias, int m_host, int K, int row_bits) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int M = m_ptr ? *m_ptr : m_host;
  const XcdTiles tiles((M + 32 * MT - 1) / (32 * MT), D / (32 * NW), row_bits);
  if (tiles.none) return;
  const int lane = threadIdx.x & 63, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int part = tiles.part, n0 = part * (32 * NW) + wave * 32;
  for (int t = tiles.r; t < tiles.r_end; t += tiles.step) {
    const int m0 = t * (32 * MT);
    float4 b[4];
    f32x16 acc[MT];
    u32x8 hi[MT];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      b[q] = *reinterpret_cast<const float4*>(bias + n0 + 8 * q + 4 * g);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const float4 v = *reinterpret_cast<const float4*>(x_block<D>(x, m0 + i * 32, n0, q, lane));
        acc[i][4 * q] = v.x;
        acc[i][4 * q + 1] = v.y;
        acc[i][4 * q + 2] = v.z;
        acc[i][4 * q + 3] = v.w;
      }
    }
    few_rows_product<MT, true, NW>(rows, K, M, m0, w + (size_t)(part * NW + wave) * (K >> 4) * 1024, smem, acc, [&]() {
#pragma unroll
      for (int i = 0; i < MT; ++i) residual_split(acc[i], hi[i]);
    });
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      if (m0 + i * 32 >= M) break;   // (what is behind the last tile of 32 rows is not a residual row)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        residual_join(acc[i], hi[i], q, b[q]);
        *reinterpret_cast<float4*>(x_block<D>(x, m0 + i * 32, n0, q, lane)) =
            make_float4(acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]);
      }
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

uint64_t slim_packed_bytes(uint64_t N, uint64_t K) { return N * K * 2; }

hipError_t launch_slim_pack(const void* W, uint64_t N, int K, void* packed, hipStream_t s) {
  const long units = (long)(N * K / 8);
  hipLaunchKernelGGL(slim_pack_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, s,
                     static_cast<const bf16_t*>(W), K, units, static_cast<bf16_t*>(packed));
  return hipGetLastError();
}

hipError_t launch_slim(const SlimLayerArgs& a, SlimStep step, int d, int F, int rows, const int32_t* m_ptr, int m_host,
                       int m_capacity, hipStream_t s) {
  if (step == SlimStep::kOutQuery ? d != 256 && d != 384 : d != 384 || !few_rows_supported(F, F)) return hipErrorInvalidValue;
  SlimArgs p{};
  p.x0 = a.x0;
  p.x0_rows = a.x0_rows;
  p.x_new = a.x_new;
  p.ln_g = a.ln_g;
  p.ln_b = a.ln_b;
  p.eps = a.eps;
  p.bias = a.bias;
  p.bias2 = a.bias2;
  p.q_scale = a.q_scale;
  p.out = static_cast<bf16_t*>(a.out);
  p.z = static_cast<bf16_t*>(a.z);
  p.vt = static_cast<bf16_t*>(a.vt);
  p.vt_ld = a.vt_ld;
  p.vt_pos = a.vt_pos;
  p.cu = a.cu;
  p.pcu = a.pcu;
  p.nseq = a.nseq;
  const bf16_t* const in = static_cast<const bf16_t*>(a.rows);
  const unsigned char *const w = static_cast<const unsigned char*>(a.w), *const w2 = static_cast<const unsigned char*>(a.w2);
  int row_bits = 0;
  const int m = rows > 0 && rows < m_capacity ? rows : m_capacity, cus = cu_count();
  if (step == SlimStep::kDown) {
    const FewDown down = few_rows_down(m, d, F, cus);
    const dim3 grid = few_rows_grid(rows, m_capacity, d, F, down.mt, down.waves, cus, &row_bits);
    auto launch = [&](auto kern) {
      hipLaunchKernelGGL(kern, grid, dim3(64 * down.waves), few_rows_lds(down.mt, down.waves), s, m_ptr, w, in, a.x, a.bias, m_host, F,
                         row_bits);
    };
    if (down.waves == 2) launch(slim_residual_kernel<384, 1, 2>);
    else if (down.mt == 2) launch(slim_residual_kernel<384, 2, 4>);
    else launch(slim_residual_kernel<384, 1, 4>);
    return hipGetLastError();
  }
  const bool qkv = step == SlimStep::kFirstQkv || step == SlimStep::kQkv;
  const bool project = step == SlimStep::kOutHidden || step == SlimStep::kOutQuery;
  p.parts = (step == SlimStep::kOutHidden ? F : qkv ? 3 * d : d) / 128;
  if (p.parts * 128 > kSlimMaxN) return hipErrorInvalidValue;
  const int per_share = parts_of_a_share((m + 31) / 32, p.parts, d, project, cus);
  const int shares = (p.parts + per_share - 1) / per_share;
  const SlimBytes b = slim_bytes(d, per_share, project);
  const dim3 grid = few_rows_grid(rows, m_capacity, shares, [](int r) { return (r + 31) / 32; }, b.row, b.part, b.tile, cus, &row_bits);
  auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, m_ptr, w, w2, in, a.x, m_host, shares, per_share, row_bits, p);
  };
  switch (step) {
    case SlimStep::kFirstQkv: launch(slim_norm_kernel<384, kFirst>); break;
    case SlimStep::kQkv: launch(slim_norm_kernel<384, kQkv>); break;
    case SlimStep::kRelu: launch(slim_norm_kernel<384, kRelu>); break;
    case SlimStep::kOutHidden: launch(slim_norm_kernel<384, kHidden>); break;
    case SlimStep::kOutQuery:
      if (d == 256) launch(slim_norm_kernel<256, kQuery>);
      else launch(slim_norm_kernel<384, kQuery>);
      break;
    default: break;
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
