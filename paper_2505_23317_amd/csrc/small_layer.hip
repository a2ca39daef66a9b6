// Widths 64 and 128: everything of a layer after attention in one kernel (out-projection, residual,
// LayerNorm, feed-forward block, residual, the next LayerNorm and the next layer's q/k/v
// projection), as layer.hip does for the wider ones.
#include "kernels.h"
#include "wide_row.h"

namespace cfdetr {

namespace {

constexpr int kSmallMaxF = 1024;

// The arguments behind those that the kernel takes one by one: these are in scalar registers when a workgroup
// starts (build.py), a structure is a trip to memory away.
struct SmallArgs {
  const bf16_t* w_qkv;
  const float *b_o, *ln2_g, *ln2_b, *b1, *b2, *ln_g, *ln_b, *b_qkv;
  float eps;
  float *out, *out2;
  int split_row;
  float q_scale;
  bf16_t *qk, *vt;
  int vt_ld;
  int32_t* vt_pos;
  const int32_t *cu, *pcu;
  int nseq;
};

// What a launch does: the first layer's LayerNorm and projection only, a whole layer, or the
// last layer (which ends in the final LayerNorm).
constexpr int kHead = 0, kMid = 1, kLast = 2;

// Rows, hidden rows, statistics, and the vectors: b_o, ln2_g, ln2_b, b2, b1, and ln_g, ln_b, b_qkv, which at width 128
// take b1's place when the hidden units are done.  With a place of their own F = 1024 left room for one
// workgroup a CU there (83,456 bytes against 80,896).  At width 64 there is room, and writing them that late costs 0.2 us.
constexpr bool small_shares(int D) { return D == 128; }
template <int D>
constexpr int small_lds(int F) {
  return 32 * D * 2 + 32 * F * 2 + 32 * 8 * 4 + (4 * D + (!small_shares(D) ? F + 5 * D : F > 5 * D ? F : 5 * D)) * 4;
}
static_assert(small_lds<64>(kSmallMaxF) <= 80 * 1024 && small_lds<128>(kSmallMaxF) <= 80 * 1024, "two workgroups a CU");

// 16-byte chunks of an LDS row of `bytes` bytes are XORed by this, so that operand reads of 16
// rows hit disjoint banks.
__device__ __forceinline__ int small_key(int bytes, int row) { return bytes == 128 ? (row >> 1) & 7 : row & 15; }

// Mean and 1/sigma of rows whose columns [32 w, 32 w + 32) wavefront w < NP holds as an MFMA result, as
// wide_stats has them: parts about their own means, put together exactly.
template <int NP>
__device__ __forceinline__ void small_stats(const f32x16& x, float* s_red, int l32, int g, int wave, float eps, float& mean,
                                            float& rstd) {
  constexpr int D = 32 * NP;
  if (wave < NP) {
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) s += (x[4 * q] + x[4 * q + 1]) + (x[4 * q + 2] + x[4 * q + 3]);
    s += __shfl_xor(s, 32, kWave);
    // in pairs, as layernorm4_kernel has them: one after the other the sixteen squares leave a row 3 % more of rounding
    float v4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float e0 = fmaf(s, -1.0f / 32, x[4 * q]), e1 = fmaf(s, -1.0f / 32, x[4 * q + 1]);
      const float e2 = fmaf(s, -1.0f / 32, x[4 * q + 2]), e3 = fmaf(s, -1.0f / 32, x[4 * q + 3]);
      v4[q] = fmaf(e0, e0, e1 * e1) + fmaf(e2, e2, e3 * e3);
    }
    float v = (v4[0] + v4[1]) + (v4[2] + v4[3]);
    v += __shfl_xor(v, 32, kWave);
    if (g == 0) {
      s_red[l32 * 8 + wave] = s;
      s_red[l32 * 8 + 4 + wave] = v;
    }
  }
  __syncthreads();
  // The parts' squares in pairs, and what their last sum is rounded by with the distances of the means: as few
  // roundings at the sum's magnitude as layernorm4_kernel has.
  float s[NP], v[NP], between = 0.f;
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    s[k] = s_red[l32 * 8 + k];
    v[k] = s_red[l32 * 8 + 4 + k];
  }
  mean = (NP == 2 ? s[0] + s[1] : (s[0] + s[1]) + (s[NP - 2] + s[NP - 1])) / D;
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const float d = fmaf(mean, -32.0f, s[k]);
    between = fmaf(d, d, between);
  }
  const float a = NP == 2 ? v[0] : v[0] + v[1], b = NP == 2 ? v[1] : v[NP - 2] + v[NP - 1];
  const float sq = a + b, b_in = sq - a, rest = (a - (sq - b_in)) + (b - b_in);
  rstd = rsqrtf(fmaf(sq, 1.0f / D, fmaf(fmaf(between, 1.0f / 32, rest), 1.0f / D, eps)));
}

// 32 complete rows a workgroup of four wavefronts.  At these widths nothing is a rate: as kernels of
// their own the seven steps were 3.3 to 4 us each, of which 2.5 us are the launch and the rest is one
// trip to memory and its answer.  So every load whose address is known at the start is asked for at the
// start: rows, residual, vectors, and the first eight weight operands a wavefront needs of each of
// the four matrices (all there are at width 64 and F = 128); what is left of larger ones follows
// behind the MFMAs.  80 rows of width 64, F = 128: 11 launches -> 3 an encoder of one layer, 29 -> 16 us.
// No row limit: encoders of six layers in us, seven kernels a layer / this, 960 rows: width 64, F = 128 177 / 101, F = 1024
// 216 / 142, width 128, F = 128 193 / 121, F = 1024 238 / 199; 65,536 rows: 657 / 462, 944 / 751, 961 / 769, 1,332 /
// 1,339 (with one workgroup a CU 1,503); width 128, F = 512 1,123 / 1,017, F = 768 1,229 / 1,178.
// A row's result does not depend on the others, so no other form has to match this one's bits.
// m_ptr or m_host: rows; O: rows of the attention; x_rows: residual rows [M, D]; matrices [N, K].
template <int D, int kKind>
__global__ __launch_bounds__(256, 2) void small_layer_kernel(const int32_t* m_ptr, const bf16_t* O, float* x_rows,
                                                              const bf16_t* w_o, const bf16_t* w1, const bf16_t* w2, int m_host,
                                                              int F, SmallArgs p) {
  constexpr int NP = D / 32, KS = D / 16, TPR = 8 / KS, ROWB = D * 2;   // TPR: column tiles a ring round
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int HROWB = F * 2;
  unsigned char* const sA = smem;
  unsigned char* const sH = smem + 32 * ROWB;
  float* const s_red = reinterpret_cast<float*>(sH + 32 * HROWB);
  constexpr bool kLate = small_shares(D) && kKind != kHead;
  float* const s_vec = s_red + 32 * 8 + (small_shares(D) ? 4 * D : 0);   // [ln_g][ln_b][b_qkv: 3 D]
  float* const v_mid = small_shares(D) ? s_vec - 4 * D : s_vec + 5 * D;  // [b_o][ln2_g][ln2_b][b2][b1: F]

  const int M = m_ptr ? *m_ptr : m_host;
  const int m0 = blockIdx.x * 32;
  if (m0 >= M) return;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = min(m0 + l32, M - 1);
  const bool in = m0 + l32 < M, holds = wave < NP;
  const int xw = min(wave, NP - 1);   // column tile of the rows (wavefronts from NP on have none)

  // the attention's rows straight into LDS
  if (kKind != kHead) {
    constexpr int RPI = 1024 / ROWB, INST = 32 / RPI;   // rows of a load of 1 KB
#pragma unroll
    for (int i = 0; i < (INST + 3) / 4; ++i) {
      const int u = wave + 4 * i, row = u * RPI + lane / (ROWB / 16), c = (lane % (ROWB / 16)) ^ small_key(ROWB, row);
      const bf16_t* src = O + (size_t)min(m0 + row, M - 1) * D + c * 8;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                   : : "s"((uint32_t)(uintptr_t)sA + u * 1024), "v"(src) : "memory");
    }
  }
  f32x16 x;
  u32x8 hi;
  float* const xrow = x_rows + (size_t)m * D + xw * 32 + 4 * g;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 v = *reinterpret_cast<const float4*>(xrow + 8 * q);
    x[4 * q] = v.x;
    x[4 * q + 1] = v.y;
    x[4 * q + 2] = v.z;
    x[4 * q + 3] = v.w;
  }
  // vectors: a thread's four (or eight) of each, into LDS below
  const int v4 = min(tid * 4, D - 4), q4 = min(tid * 4, 3 * D - 4), f4 = min(tid * 4, F - 4);
  const float4 vg = *reinterpret_cast<const float4*>(p.ln_g + v4), vb = *reinterpret_cast<const float4*>(p.ln_b + v4);
  float4 vq, vo, vg2, vb2, vd, v1;
  if (kKind != kLast) vq = *reinterpret_cast<const float4*>(p.b_qkv + q4);
  if (kKind != kHead) {
    vo = *reinterpret_cast<const float4*>(p.b_o + v4);
    vg2 = *reinterpret_cast<const float4*>(p.ln2_g + v4);
    vb2 = *reinterpret_cast<const float4*>(p.ln2_b + v4);
    vd = *reinterpret_cast<const float4*>(p.b2 + v4);
    v1 = *reinterpret_cast<const float4*>(p.b1 + f4);
  }
  // weights: operand of k-step ks of 32 columns from n0, rows of K
  const int n_ff1 = F / 32, n_qkv = 3 * NP;   // column tiles; wavefront w takes w, w + 4, ...
  auto weights = [&](const bf16_t* W, int K, int n0, int ks) {
    return *reinterpret_cast<const bf16x8*>(W + (size_t)(n0 + l32) * K + ks * 16 + g * 8);
  };
  bf16x8 ro[KS], r1[8], r2[8], rq[8];
  if (kKind != kHead) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ro[ks] = weights(w_o, D, xw * 32, ks);
#pragma unroll
    for (int i = 0; i < 8; ++i) r1[i] = weights(w1, D, min(wave + 4 * (i / KS), n_ff1 - 1) * 32, i % KS);
#pragma unroll
    for (int i = 0; i < 8; ++i) r2[i] = weights(w2, F, xw * 32, i);
  }
  if (kKind != kLast) {
#pragma unroll
    for (int i = 0; i < 8; ++i) rq[i] = weights(p.w_qkv, D, min(wave + 4 * (i / KS), n_qkv - 1) * 32, i % KS);
  }
  int vpos = 0;   // place of the row in vt
  if (kKind == kHead) {
    const int f = frame_of_token(p.cu, p.nseq, m);
    vpos = p.pcu[f] + (m - p.cu[f]);
    if (wave == 0 && g == 0) p.vt_pos[m] = vpos;
  } else if (kKind == kMid) {
    vpos = p.vt_pos[m];
  }
  if (tid < D / 4) {
    if (!kLate) {
      *reinterpret_cast<float4*>(s_vec + tid * 4) = vg;
      *reinterpret_cast<float4*>(s_vec + D + tid * 4) = vb;
    }
    if (kKind != kHead) {
      *reinterpret_cast<float4*>(v_mid + tid * 4) = vo;
      *reinterpret_cast<float4*>(v_mid + D + tid * 4) = vg2;
      *reinterpret_cast<float4*>(v_mid + 2 * D + tid * 4) = vb2;
      *reinterpret_cast<float4*>(v_mid + 3 * D + tid * 4) = vd;
    }
  }
  if (!kLate && kKind != kLast && tid < 3 * D / 4) *reinterpret_cast<float4*>(s_vec + 2 * D + tid * 4) = vq;
  if (kKind != kHead && tid < F / 4) *reinterpret_cast<float4*>(v_mid + 4 * D + tid * 4) = v1;

  auto operand = [&](const unsigned char* rows, int bytes, int ks) {
    return *reinterpret_cast<const bf16x8*>(rows + l32 * bytes + (((2 * ks + g) ^ small_key(bytes, l32)) << 4));
  };
  auto join = [&](const float* b) {
#pragma unroll
    for (int q = 0; q < 4; ++q) residual_join(x, hi, q, *reinterpret_cast<const float4*>(b + xw * 32 + 8 * q + 4 * g));
  };
  float mean, rstd;
  auto normed = [&](int q, const float* gain, const float* offs) {
    const float4 ga = *reinterpret_cast<const float4*>(gain + xw * 32 + 8 * q + 4 * g);
    const float4 of = *reinterpret_cast<const float4*>(offs + xw * 32 + 8 * q + 4 * g);
    return make_float4(wide_normed(x[4 * q], mean, rstd, ga.x, of.x), wide_normed(x[4 * q + 1], mean, rstd, ga.y, of.y),
                       wide_normed(x[4 * q + 2], mean, rstd, ga.z, of.z), wide_normed(x[4 * q + 3], mean, rstd, ga.w, of.w));
  };
  // LayerNorm to sA, ends with a barrier (the first barrier of small_stats stands behind every read of sA)
  auto norm_to_lds = [&](const float* gain, const float* offs) {
    small_stats<NP>(x, s_red, l32, g, wave, p.eps, mean, rstd);
    if (holds) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 r = normed(q, gain, offs);
        *reinterpret_cast<uint2*>(sA + l32 * ROWB + (((wave * 4 + q) ^ small_key(ROWB, l32)) << 4) + g * 8) =
            make_uint2(pack_bf16x2(r.x, r.y), pack_bf16x2(r.z, r.w));
      }
    }
    __syncthreads();
  };
  // sA times the wavefront's column tiles of a matrix [32 tiles, D]: sums that start at the bias, done(tile, sum)
  auto contract = [&](const bf16_t* W, int tiles, bf16x8(&ring)[8], const float* bias, auto done) {
    bf16x8 a[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a[ks] = operand(sA, ROWB, ks);
#pragma nounroll
    for (int t0 = wave; t0 < tiles; t0 += 4 * TPR) {
      f32x16 r[TPR];
#pragma unroll
      for (int t = 0; t < TPR; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 b = *reinterpret_cast<const float4*>(bias + min(t0 + 4 * t, tiles - 1) * 32 + 8 * q + 4 * g);
          r[t][4 * q] = b.x;
          r[t][4 * q + 1] = b.y;
          r[t][4 * q + 2] = b.z;
          r[t][4 * q + 3] = b.w;
        }
      const bool more = t0 + 4 * TPR < tiles;
#pragma unroll
      for (int t = 0; t < TPR; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          r[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[t * KS + ks], a[ks], r[t], 0, 0, 0);
        }
      if (more) {
#pragma unroll
        for (int i = 0; i < 8; ++i) ring[i] = weights(W, D, min(t0 + 4 * (TPR + i / KS), tiles - 1) * 32, i % KS);
      }
#pragma unroll
      for (int t = 0; t < TPR; ++t)
        if (t0 + 4 * t < tiles) done(t0 + 4 * t, r[t]);
    }
  };

  if (kKind != kHead) {
    residual_split(x, hi);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ro[ks], operand(sA, ROWB, ks), x, 0, 0, 0);
    join(v_mid);
    norm_to_lds(v_mid + D, v_mid + 2 * D);
    contract(w1, n_ff1, r1, v_mid + 4 * D, [&](int tile, const f32x16& r) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<uint2*>(sH + l32 * HROWB + (((tile * 4 + q) ^ small_key(HROWB, l32)) << 4) + g * 8) =
            make_uint2(pack_bf16x2(gelu_fast(r[4 * q]), gelu_fast(r[4 * q + 1])),
                       pack_bf16x2(gelu_fast(r[4 * q + 2]), gelu_fast(r[4 * q + 3])));
    });
    residual_split(x, hi);
    __syncthreads();   // hidden units are complete, and their biases have been read
    if (holds) {
#pragma nounroll
      for (int k0 = 0; k0 < F / 16; k0 += 8) {
        bf16x8 a[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = operand(sH, HROWB, k0 + i);
#pragma unroll
        for (int i = 0; i < 8; ++i) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r2[i], a[i], x, 0, 0, 0);
        if (k0 + 8 < F / 16) {
#pragma unroll
          for (int i = 0; i < 8; ++i) r2[i] = weights(w2, F, xw * 32, k0 + 8 + i);
        }
      }
    }
    if (kLate) {   // (a barrier of small_stats is in front of their readers)
      if (tid < D / 4) {
        *reinterpret_cast<float4*>(s_vec + tid * 4) = vg;
        *reinterpret_cast<float4*>(s_vec + D + tid * 4) = vb;
      }
      if (kKind != kLast && tid < 3 * D / 4) *reinterpret_cast<float4*>(s_vec + 2 * D + tid * 4) = vq;
    }
    join(v_mid + 3 * D);
    if (kKind == kMid && holds && in) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(xrow + 8 * q) = make_float4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
    }
  } else {
    __syncthreads();   // the vectors
  }
  if (kKind == kLast) {
    small_stats<NP>(x, s_red, l32, g, wave, p.eps, mean, rstd);
    if (!holds || !in) return;
    const bool second = p.out2 != nullptr && m >= p.split_row;
    float* const o = (second ? p.out2 : p.out) + (size_t)(second ? m - p.split_row : m) * D + xw * 32 + 4 * g;
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<float4*>(o + 8 * q) = normed(q, s_vec, s_vec + D);
    return;
  }
  norm_to_lds(s_vec, s_vec + D);
  contract(p.w_qkv, n_qkv, rq, s_vec + 2 * D, [&](int tile, const f32x16& r) {
    if (!in) return;
    const int n0 = tile * 32;
    if (n0 >= 2 * D) {
      bf16_t* vp = p.vt + (size_t)(n0 - 2 * D + 4 * g) * p.vt_ld + vpos;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        *vp = f32_to_bf16(r[e]);
        vp += (size_t)((e & 3) == 3 ? 5 : 1) * p.vt_ld;
      }
    } else {
      const float sc = n0 < D ? p.q_scale : 1.0f;
      bf16_t* const o = p.qk + (size_t)m * (3 * D) + n0 + 4 * g;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<uint2*>(o + 8 * q) = make_uint2(pack_bf16x2(r[4 * q] * sc, r[4 * q + 1] * sc),
                                                          pack_bf16x2(r[4 * q + 2] * sc, r[4 * q + 3] * sc));
    }
  });
}

template <int D, int kKind>
hipError_t launch_small(const SmallLayerArgs& a, const SmallArgs& p, int F, const int32_t* m_ptr, int m_host, int m_capacity,
                        hipStream_t s) {
  const size_t lds = small_lds<D>(F);
  auto w = [](const void* q) { return static_cast<const bf16_t*>(q); };
  if (lds > 64 * 1024) {
    static DeviceOnce configured;
    if (hipError_t e = allow_lds(small_layer_kernel<D, kKind>, small_lds<D>(kSmallMaxF), &configured); e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((small_layer_kernel<D, kKind>), dim3((m_capacity + 31) / 32), dim3(256), lds, s, m_ptr, w(a.O),
                     a.x, w(a.w_o), w(a.w_ff1), w(a.w_ff2), m_host, F, p);
  return hipGetLastError();
}

}  // namespace

// F: whole ring rounds of the second feed-forward matrix, and a thread's four biases cover it.
bool small_layer_supported(int d, int F, bool use_bf16) {
  return use_bf16 && (d == 64 || d == 128) && F % 128 == 0 && F <= kSmallMaxF;
}

hipError_t launch_small_layer(const SmallLayerArgs& a, int d, int F, const int32_t* m_ptr, int m_host, int m_capacity,
                              hipStream_t s) {
  if (!small_layer_supported(d, F, true)) return hipErrorInvalidValue;
  SmallArgs p{};
  p.w_qkv = static_cast<const bf16_t*>(a.w_qkv);
  p.b_o = a.b_o;
  p.ln2_g = a.ln2_g;
  p.ln2_b = a.ln2_b;
  p.b1 = a.b_ff1;
  p.b2 = a.b_ff2;
  p.ln_g = a.ln_g;
  p.ln_b = a.ln_b;
  p.b_qkv = a.b_qkv;
  p.eps = a.eps;
  p.out = a.out;
  p.out2 = a.out2;
  p.split_row = a.split_row;
  p.q_scale = a.q_scale;
  p.qk = static_cast<bf16_t*>(a.qk);
  p.vt = static_cast<bf16_t*>(a.vt);
  p.vt_ld = a.vt_ld;
  p.vt_pos = a.vt_pos;
  p.cu = a.cu;
  p.pcu = a.pcu;
  p.nseq = a.nseq;
  const int kind = a.O == nullptr ? kHead : a.w_qkv == nullptr ? kLast : kMid;
  if (d == 64)
    return kind == kHead ? launch_small<64, kHead>(a, p, F, m_ptr, m_host, m_capacity, s)
                         : kind == kMid ? launch_small<64, kMid>(a, p, F, m_ptr, m_host, m_capacity, s) : launch_small<64, kLast>(a, p, F, m_ptr, m_host, m_capacity, s);
  return kind == kHead ? launch_small<128, kHead>(a, p, F, m_ptr, m_host, m_capacity, s)
                       : kind == kMid ? launch_small<128, kMid>(a, p, F, m_ptr, m_host, m_capacity, s) : launch_small<128, kLast>(a, p, F, m_ptr, m_host, m_capacity, s);
}

}  // namespace cfdetr
