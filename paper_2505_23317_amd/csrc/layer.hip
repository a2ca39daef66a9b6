// Widths 256 and 384: everything of a layer after attention in one kernel (out-projection,
// residual, LayerNorm, feed-forward block, residual, the next LayerNorm and the next layer's
// q/k/v projection).
#include "kernels.h"
#include "wide_row.h"

#include <type_traits>
#include <utility>

namespace cfdetr {

namespace {

constexpr int kRingMax = 16;    // most weight blocks of 1 KB a wavefront holds in registers

// The arguments behind those that the kernel takes one by one: these are in scalar registers when a workgroup
// starts (build.py), a structure is a trip to memory away.
struct WideArgs {
  const float *b_o, *ln2_g, *ln2_b, *b1, *b2;
  const float *ln_g, *ln_b;
  float eps;
  float* out;
  int split_row;
  float* out2;
  const float* b_qkv;
  float q_scale;
  bf16_t* qk;
  bf16_t* vt;
  int vt_ld;
  int32_t* vt_pos;
  const int32_t* cu;
  const int32_t* pcu;
  int nseq;
};

// LDS of a workgroup: operand rows, a hidden chunk (its place also serves the row sums and the
// staging of outputs), and the vectors of the layer.
template <int D, int NW, int MT>
struct WideLds {
  static constexpr int kFC = 32 * NW;                    // hidden units of a chunk: one 32-wide tile per wavefront
  static constexpr int kRow = D / NW * 2 + 16;           // staging row: the columns of a wavefront
  static constexpr int kA = MT * 32 * D * 2, kH = MT * 32 * kFC * 2, kStg = NW * 16 * kRow;
  static constexpr int kHS = kH > kStg ? kH : kStg;
  static constexpr int kVec = kA + kHS;                  // [b1 or b_qkv][ln2_g][ln2_b][b2][ln_g][ln_b][NW = 8: b_qkv]
  static int bytes(int F) { return kVec + ((F > 3 * D ? F : 3 * D) + 5 * D + (NW == 8 ? 3 * D : 0)) * 4; }
};

// What a launch does: the first layer's LayerNorm and projection only, a whole layer, or the
// last layer (which ends in the final LayerNorm).
constexpr int kHead = 0, kMid = 1, kLast = 2;

// A workgroup of NW wavefronts owns 32 MT complete rows; wavefront w owns columns
// [w D/NW, (w + 1) D/NW) of them.  The two products that end in the residual are not summed on
// top of it, where every MFMA would round at its magnitude (ten times the error where it is 30
// times what is added): the accumulators start at the residual's low part and its high part, a
// bf16, is added once (wide_row.h).  Through the feed-forward block the high parts wait in
// registers, where there is room for them (kKeep), or in memory in the rows' own place.  Per row
// only O and x are read and x, q, k, v written (half of x once more where it waits in memory); as
// separate kernels the same rows made 30 KB of traffic more per layer (bf16 rows of both
// LayerNorms, hidden activations, x twice).
// Weights: no wavefront shares one with another, so they skip the LDS.  They are packed in the
// order of use, 1 KB per MFMA operand, and stream through a ring of registers that is refilled
// right behind the MFMA that used a block.  Operand rows and hidden chunk lie in LDS with
// 16-byte chunks XORed by the row (row lengths are multiples of 256 bytes, all 64 banks).
// The feed-forward block goes in chunks of 32 NW hidden units; the activation of chunk c runs
// between the MFMAs of the second matrix on chunk c - 1, laid out instruction by instruction
// (the compiler puts it in front of them otherwise).  Vectors are in LDS because a global load
// that is waited for waits for the whole ring behind which it was issued.
//
// Bounds: the matrix cores at the clock the power limit leaves (1.9 GHz with all CUs busy),
// the activation's vector instructions (they exceed what its MFMAs hide: 60 clocks a value
// pair against 32), and the CU's vector-memory path: 64 B/clk for 3.5 MB of weights per
// workgroup, which is what taller tiles save.  Measured per layer at D = 384, F = 1536
// against q/k/v, out-projection, two LayerNorms and the two feed-forward matrices as kernels
// of their own: 22,400 rows 168 -> 99 us, 64,000 rows 430 -> 260 us, 3,520 rows 54 -> 43 us,
// 920 rows 45 -> 42 us (few_rows.hip takes those).  Of that the residual's two parts are 1 % of a pass
// (summed on top of it: eight frames of up to 8,000 tokens 8,262 us, so 8,349); the whole residual
// in memory would be 4 %.
//
// Width 384 has four wavefronts of 96 columns, width 256 eight of 32: two on each SIMD, so that
// one's waits (barriers, row sums, the activation's chain of dependent operations) are the
// other's work.  With four of 64 columns a layer of 1,200 rows took 24 us, with eight 18 us:
// 1.5 MB of weights per workgroup then come at two thirds of the CU's 64 B/clk.  Encoder passes
// of 6 layers against layer_tail_kernel (gemm.hip: 32 rows, a split of roles in the feed-forward
// block): 1,200 rows 224 -> 191 us, 6,400 rows 283 -> 260 us, 11,200 rows 470 -> 344 us,
// 24,000 rows 857 -> 676 us.
// m_ptr or m_host: rows; packed: weight streams of `stream` bytes, one per wavefront; x: residual blocks (wide_row.h);
// O: the attention's rows; x0 (kHead): the rows as the embedding left them, or x0_rows rows over and over.
template <int D, int NW, int MT, int kKind>
__global__ __launch_bounds__(64 * NW, NW == 4 && MT > 2 ? 1 : 2) void wide_layer_kernel(const int32_t* m_ptr, const unsigned char* packed,
                                                                                float* x, const bf16_t* O, const float* x0,
                                                                                int m_host, uint32_t stream, int F, int x0_rows,
                                                                                WideArgs p) {
  using L = WideLds<D, NW, MT>;
  // (96 rows of width 384, alone on a CU: a ring of 12 leaves registers for the residual's high parts.
  // 22,400 rows 105 us a layer with a ring of 24 and those in memory, 100 with 12 and 99 like this.)
  constexpr int kRing = NW == 8 ? 16 : 12;
  constexpr int kFC = L::kFC, kThreads = 64 * NW;
  constexpr bool kKeep = NW == 8 || MT == 1 || (MT == 3 && kKind != kLast);
  constexpr int NT = D / (32 * NW), KS = D / 16, BM = 32 * MT, ROWB = D * 2, HROWB = kFC * 2;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char* const sA = smem;
  unsigned char* const sH = smem + L::kA;
  float* const s_red = reinterpret_cast<float*>(smem + L::kA);

  const int M = m_ptr ? *m_ptr : m_host;
  const int total = (M + BM - 1) / BM;
  if ((int)blockIdx.x >= total) return;
  const int m0 = tile_order(blockIdx.x, total) * BM;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  unsigned char* const stg = smem + L::kA + wave * (16 * L::kRow);
  float* const v_b1 = reinterpret_cast<float*>(smem + L::kVec);
  float* const v_d = v_b1 + max(F, 3 * D);   // five vectors of D
  float* const v_qkv = NW == 8 ? v_d + 5 * D : v_b1;
  // (behind the row sums' place; the hidden chunk comes there later)
  float* const v_bo = reinterpret_cast<float*>(smem + L::kVec) - D;
  static_assert(L::kHS >= MT * 32 * 2 * NW * 4 + D * 4, "bias behind the row sums");
  const int c0 = wave * (D / NW);

  int vpos[MT];
  if (kKind == kHead) {
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int m = min(m0 + i * 32 + l32, M - 1);
      const int f = frame_of_token(p.cu, p.nseq, m);
      vpos[i] = p.pcu[f] + (m - p.cu[f]);
      if (wave == 0 && g == 0 && m0 + i * 32 + l32 < M) p.vt_pos[m] = vpos[i];
    }
  }

  // the vectors of the layer
  if (kKind != kHead) {
    for (int i = tid * 4; i < F; i += 4 * kThreads) *reinterpret_cast<float4*>(v_b1 + i) = *reinterpret_cast<const float4*>(p.b1 + i);
  }
  if (kKind == kHead || (NW == 8 && kKind == kMid)) {
    for (int i = tid * 4; i < 3 * D; i += 4 * kThreads) *reinterpret_cast<float4*>(v_qkv + i) = *reinterpret_cast<const float4*>(p.b_qkv + i);
  }
  if (tid < D / 4) {
    if (kKind != kHead) {
      *reinterpret_cast<float4*>(v_bo + tid * 4) = *reinterpret_cast<const float4*>(p.b_o + tid * 4);
      *reinterpret_cast<float4*>(v_d + tid * 4) = *reinterpret_cast<const float4*>(p.ln2_g + tid * 4);
      *reinterpret_cast<float4*>(v_d + D + tid * 4) = *reinterpret_cast<const float4*>(p.ln2_b + tid * 4);
      *reinterpret_cast<float4*>(v_d + 2 * D + tid * 4) = *reinterpret_cast<const float4*>(p.b2 + tid * 4);
    }
    *reinterpret_cast<float4*>(v_d + 3 * D + tid * 4) = *reinterpret_cast<const float4*>(p.ln_g + tid * 4);
    *reinterpret_cast<float4*>(v_d + 4 * D + tid * 4) = *reinterpret_cast<const float4*>(p.ln_b + tid * 4);
  }
  // weight stream
  const unsigned char* wp = packed + (size_t)wave * stream;
  const uint32_t voff = lane * 16;
  bf16x8 wr[kRing];
  // block i of the ring's next round: the base of every fourth one in scalar registers, so
  // that a load costs no vector arithmetic
  typedef const __attribute__((address_space(1))) unsigned char* gptr;
  gptr wq = (gptr)wp;
  auto next_block = [&](int i) {
    if (i % 4 == 0) {
      wq = (gptr)wp + i * 1024;
      asm volatile("" : "+s"(wq));
    }
    return *reinterpret_cast<const __attribute__((address_space(1))) bf16x8*>(wq + (i % 4) * 1024 + voff);
  };
#pragma unroll
  for (int i = 0; i < kRing; ++i) wr[i] = *reinterpret_cast<const bf16x8*>(wp + i * 1024 + voff);

  if (kKind != kHead) {
    // rows of O into sA
    constexpr int UNITS = BM * (ROWB / 16);
#pragma unroll
    for (int u0 = 0; u0 < UNITS; u0 += kThreads) {
      const int u = u0 + tid;
      const int row = u / (ROWB / 16), pos = u % (ROWB / 16);
      const int c = (pos & ~15) | ((pos ^ row) & 15);
      const bf16_t* src = O + (size_t)min(m0 + row, M - 1) * D + c * 8;
      const uint32_t dst = (uint32_t)(uintptr_t)sA + (u0 + wave * 64) * 16;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                   : : "s"(dst), "v"(src) : "memory");
    }
  }
  // residual rows: into the accumulators, in two parts where something is added to them
  unsigned char* const xw = reinterpret_cast<unsigned char*>(x) + (size_t)(m0 >> 5) * (D * 128) + wave * (NT * 4096);
  f32x16 acc[NT][MT];
  u32x8 hi[NT][MT];
  int row0[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    row0[i] = min(m0 + i * 32 + l32, M - 1);
    if (kKind == kHead && x0_rows > 0) row0[i] %= x0_rows;
  }
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const float4 v =
            kKind == kHead
                ? *reinterpret_cast<const float4*>(x0 + (size_t)row0[i] * D + c0 + j * 32 + 8 * q + 4 * g)
                : *reinterpret_cast<const float4*>(xw + i * (D * 128) + j * 4096 + q * 1024 + voff);
        acc[j][i][4 * q] = v.x;
        acc[j][i][4 * q + 1] = v.y;
        acc[j][i][4 * q + 2] = v.z;
        acc[j][i][4 * q + 3] = v.w;
      }
  auto split = [&]() {
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int i = 0; i < MT; ++i) residual_split(acc[j][i], hi[j][i]);
  };
  auto join = [&](const float* b) {   // `b` in LDS, the columns of D
    int g4 = 4 * g;
    work_out_here(g4);
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 bq = *reinterpret_cast<const float4*>(b + c0 + j * 32 + 8 * q + g4);
#pragma unroll
        for (int i = 0; i < MT; ++i) residual_join(acc[j][i], hi[j][i], q, bq);
      }
  };
  typedef __attribute__((address_space(1))) unsigned char* gwptr;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

  // LDS operand addresses (chunk swizzled with the row), k-step modulo 4
  uint32_t ao[8], ho[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    ao[k] = l32 * ROWB + (((2 * k + g) ^ (l32 & 15)) << 4);
    ho[k] = l32 * HROWB + (((2 * k + g) ^ (l32 & 15)) << 4);
  }

  // One product over NK k-steps of the operand rows at `rows` (row length RB bytes), NTX column
  // tiles per wavefront; `side(ks, mfma)` is work to put behind the MFMAs.
#define WIDE_PRODUCT(ACC_, NTX_, NK_, ROWS_, RB_, OFF_)                                          \
  do {                                                                                           \
    constexpr int UN_ = kRing / (NTX_);   /* k-steps of a ring round */                          \
    constexpr int BS_ = UN_ % 8 == 0 ? UN_ : UN_ == 4 ? 8 : 2 * UN_;                             \
    static_assert(BS_ % 8 == 0 && (NK_) % BS_ == 0, "k-steps");                                  \
    bf16x8 a_[2][MT];                                                                            \
    _Pragma("unroll") for (int i = 0; i < MT; ++i)                                               \
        a_[0][i] = *reinterpret_cast<const bf16x8*>((ROWS_) + OFF_[0] + i * (32 * (RB_)));       \
    const unsigned char* rp_ = (ROWS_);                                                          \
    _Pragma("nounroll") for (int k0_ = 0; k0_ < (NK_); k0_ += BS_) {                             \
      _Pragma("unroll") for (int u = 0; u < BS_; ++u) {                                          \
        if (u % UN_ == 0) wp += kRing * 1024;                                                    \
        _Pragma("unroll") for (int i = 0; i < MT; ++i)                                           \
            a_[(u + 1) & 1][i] = *reinterpret_cast<const bf16x8*>(                               \
                rp_ + OFF_[(u + 1) & 7] + ((u + 1) / 8) * 256 + i * (32 * (RB_)));               \
        _Pragma("unroll") for (int j = 0; j < (NTX_); ++j)                                       \
            _Pragma("unroll") for (int i = 0; i < MT; ++i) ACC_[j][i] =                          \
                __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[(u % UN_) * (NTX_) + j], a_[u & 1][i],        \
                                                        ACC_[j][i], 0, 0, 0);                    \
        _Pragma("unroll") for (int j = 0; j < (NTX_); ++j)                                       \
            wr[(u % UN_) * (NTX_) + j] = next_block((u % UN_) * (NTX_) + j);                     \
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                       \
        __builtin_amdgcn_sched_group_barrier(0x100, MT, 0);                                      \
        __builtin_amdgcn_sched_group_barrier(0x008, MT - 1, 0);                                  \
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                                       \
        _Pragma("unroll") for (int j = 1; j < (NTX_); ++j) {                                     \
          __builtin_amdgcn_sched_group_barrier(0x008, MT, 0);                                    \
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                                     \
        }                                                                                        \
        __builtin_amdgcn_sched_barrier(0);                                                       \
      }                                                                                          \
      rp_ += (BS_ / 8) * 256;                                                                    \
    }                                                                                            \
  } while (0)

  float mean[MT], rstd[MT];
  if (kKind != kHead) {
    split();
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    WIDE_PRODUCT(acc, NT, KS, sA, ROWB, ao);   // attention output times Wo
    join(v_bo);
    wide_stats<NW>(acc, s_red, l32, g, wave, p.eps, mean, rstd);
    wide_norm_to_lds<NW>(acc, mean, rstd, v_d, v_d + D, sA, l32, g, wave);
    if (kKeep) {
      split();
    } else {
      gwptr xo = (gwptr)xw;
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          asm volatile("" : "+s"(xo));   // addresses worked out here, not kept from the top of the kernel
          residual_split(acc[j][i], hi[j][i]);
#pragma unroll
          for (int h = 0; h < 2; ++h)
            *reinterpret_cast<__attribute__((address_space(1))) u32x4*>(xo + (i * (D * 128) + j * 4096 + h * 1024) + voff) =
                u32x4{hi[j][i][4 * h], hi[j][i][4 * h + 1], hi[j][i][4 * h + 2], hi[j][i][4 * h + 3]};
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    f32x16 hid[1][MT];
    uint2 pk[MT][4];
    auto hid_bias = [&](int c) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 b = *reinterpret_cast<const float4*>(v_b1 + c * kFC + wave * 32 + 8 * q + 4 * g);
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          hid[0][i][4 * q] = b.x;
          hid[0][i][4 * q + 1] = b.y;
          hid[0][i][4 * q + 2] = b.z;
          hid[0][i][4 * q + 3] = b.w;
        }
      }
    };
    auto put_hidden = [&]() {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<uint2*>(sH + (i * 32 + l32) * HROWB + (((wave * 4 + q) ^ (l32 & 15)) << 4) + g * 8) = pk[i][q];
    };
    const int nc = F / kFC;
    hid_bias(0);
    WIDE_PRODUCT(hid, 1, KS, sA, ROWB, ao);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        pk[i][q] = make_uint2(pack_bf16x2(gelu_fast(hid[0][i][4 * q]), gelu_fast(hid[0][i][4 * q + 1])),
                              pack_bf16x2(gelu_fast(hid[0][i][4 * q + 2]), gelu_fast(hid[0][i][4 * q + 3])));
#pragma nounroll
    for (int c = 1; c < nc; ++c) {
      // chunk c - 1 is in pk (every wavefront has passed its reads of sH): into LDS
      put_hidden();
      hid_bias(c);
      WIDE_PRODUCT(hid, 1, KS, sA, ROWB, ao);
      __syncthreads();
      // second matrix on chunk c - 1, the activation of chunk c between its MFMAs
      {
        constexpr int NM = NT * MT;
        bf16x8 a_[2][MT];
        // two registers of every hidden tile at a time: V values, gelu_fast in nine steps, step by step,
        // over TS k-steps
        constexpr int TS = kFC / 128, V = 2 * MT, OPS = 9 * V, PER = (OPS + NM * TS - 1) / (NM * TS);
        float ge[MT][4], gx[V], gc[V], gt[V], g2[V];
#pragma unroll
        for (int i = 0; i < MT; ++i)
          a_[0][i] = *reinterpret_cast<const bf16x8*>(sH + ho[0] + i * (32 * HROWB));
        // (t a constant of its own type: the registers below are indexed by it)
        auto step = [&](auto t_) {
          constexpr int t = decltype(t_)::value;
          constexpr int UN = kRing / NT;
          if (t % UN == 0) wp += kRing * 1024;
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            const int j = m / MT, i = m % MT;
            acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[(t % UN) * NT + j], a_[t & 1][i], acc[j][i], 0, 0, 0);
            if (m < MT)
              a_[(t + 1) & 1][m] = *reinterpret_cast<const bf16x8*>(sH + ho[(t + 1) & 7] + ((t + 1) / 8) * 256 + m * (32 * HROWB));
            if (i == MT - 1) wr[(t % UN) * NT + j] = next_block((t % UN) * NT + j);
#pragma unroll
            for (int o = (t % TS * NM + m) * PER; o < (t % TS * NM + m + 1) * PER && o < OPS; ++o) {
              const int s = o / V, v = o % V;
              const int vi = v / 2, r = 2 * (t / TS) + v % 2;
              if (s == 0) {
                gx[v] = hid[0][vi][r];
                asm volatile("" : "+v"(gx[v]));
                gc[v] = __builtin_amdgcn_fmed3f(gx[v], -8.0f, 8.0f);
                asm volatile("" : "+v"(gc[v]));
              } else if (s == 1) {
                g2[v] = gc[v] * gc[v];
                asm volatile("" : "+v"(g2[v]));
              } else if (s == 2) {
                gt[v] = fmaf(kGelu5, g2[v], kGelu3);
                asm volatile("" : "+v"(gt[v]));
              } else if (s == 3) {
                gt[v] = fmaf(gt[v], g2[v], kGelu1);
                asm volatile("" : "+v"(gt[v]));
              } else if (s == 4) {
                gt[v] = gt[v] * gc[v];
                asm volatile("" : "+v"(gt[v]));
              } else if (s == 5) {
                gt[v] = __builtin_amdgcn_exp2f(gt[v]);
                asm volatile("" : "+v"(gt[v]));
              } else if (s == 6) {
                gt[v] = 1.0f + gt[v];
                asm volatile("" : "+v"(gt[v]));
              } else if (s == 7) {
                gt[v] = __builtin_amdgcn_rcpf(gt[v]);
                asm volatile("" : "+v"(gt[v]));
              } else {
                ge[vi][r & 3] = gx[v] * gt[v];
                asm volatile("" : "+v"(ge[vi][r & 3]));
                if (r & 1) {
                  uint32_t w = pack_bf16x2(ge[vi][(r & 3) - 1], ge[vi][r & 3]);
                  asm volatile("" : "+v"(w));
                  if ((r & 3) == 1) pk[vi][r >> 2].x = w;
                  else pk[vi][r >> 2].y = w;
                }
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        [&]<int... kT>(std::integer_sequence<int, kT...>) { (step(std::integral_constant<int, kT>{}), ...); }
        (std::make_integer_sequence<int, kFC / 16>{});
      }
      __syncthreads();
    }
    put_hidden();
    __syncthreads();
    float4 bq0, bq1;
    if (kKind == kMid) {
#pragma unroll
      for (int i = 0; i < MT; ++i) vpos[i] = p.vt_pos[min(m0 + i * 32 + l32, M - 1)];
    }
    if (NW == 4 && kKind == kMid) {
      // the next projection's bias takes the place of b1 (everybody is done with that)
      static_assert(NW == 8 || (3 * D > 1024 && 3 * D <= 2048), "two pieces");
      bq0 = *reinterpret_cast<const float4*>(p.b_qkv + tid * 4);
      bq1 = *reinterpret_cast<const float4*>(p.b_qkv + min(tid * 4 + 1024, 3 * D - 4));
    }
    WIDE_PRODUCT(acc, NT, kFC / 16, sH, HROWB, ho);
    if (NW == 4 && kKind == kMid) {
      *reinterpret_cast<float4*>(v_b1 + tid * 4) = bq0;
      if (tid * 4 + 1024 < 3 * D) *reinterpret_cast<float4*>(v_b1 + tid * 4 + 1024) = bq1;
    }
    if (!kKeep) {
      gwptr xi = (gwptr)xw;
      asm volatile("" : "+s"(xi) : : "memory");   // (not what was stored there, still in registers)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const u32x4 v =
                *reinterpret_cast<const __attribute__((address_space(1))) u32x4*>(xi + (i * (D * 128) + j * 4096 + h * 1024) + voff);
#pragma unroll
            for (int e = 0; e < 4; ++e) hi[j][i][4 * h + e] = v[e];
          }
    }
    join(v_d + 2 * D);
    __syncthreads();   // (the row sums go where the hidden chunk was)
  }
  // the new residual rows
  if (kKind != kLast) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    gwptr xo = (gwptr)xw;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        asm volatile("" : "+s"(xo));
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<__attribute__((address_space(1))) f32x4*>(xo + (i * (D * 128) + j * 4096 + q * 1024) + voff) =
              f32x4{acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]};
      }
  }
  wide_stats<NW>(acc, s_red, l32, g, wave, p.eps, mean, rstd);
  if (kKind == kLast) {
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int col = c0 + j * 32 + 8 * q + 4 * g;
        const float4 ga = *reinterpret_cast<const float4*>(v_d + 3 * D + col);
        const float4 of = *reinterpret_cast<const float4*>(v_d + 4 * D + col);
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          const int m = m0 + i * 32 + l32;
          if (m >= M) continue;
          const bool second = p.out2 != nullptr && m >= p.split_row;
          float* o = (second ? p.out2 : p.out) + (size_t)(second ? m - p.split_row : m) * D + col;
          *reinterpret_cast<float4*>(o) =
              make_float4(wide_normed(acc[j][i][4 * q], mean[i], rstd[i], ga.x, of.x),
                          wide_normed(acc[j][i][4 * q + 1], mean[i], rstd[i], ga.y, of.y),
                          wide_normed(acc[j][i][4 * q + 2], mean[i], rstd[i], ga.z, of.z),
                          wide_normed(acc[j][i][4 * q + 3], mean[i], rstd[i], ga.w, of.w));
        }
      }
    return;
  }
  wide_norm_to_lds<NW>(acc, mean, rstd, v_d + 3 * D, v_d + 4 * D, sA, l32, g, wave);
  // q, k, v of these rows
#pragma nounroll
  for (int part = 0; part < 3; ++part) {
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 b = *reinterpret_cast<const float4*>(v_qkv + part * D + c0 + j * 32 + 8 * q + 4 * g);
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          acc[j][i][4 * q] = b.x;
          acc[j][i][4 * q + 1] = b.y;
          acc[j][i][4 * q + 2] = b.z;
          acc[j][i][4 * q + 3] = b.w;
        }
      }
    WIDE_PRODUCT(acc, NT, KS, sA, ROWB, ao);
    if (part < 2) {
      const float sc = part == 0 ? p.q_scale : 1.0f;
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          // 16 rows x the columns of a wavefront at a time through the wavefront's staging rows
          if ((l32 >> 4) == half) {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
              for (int q = 0; q < 4; ++q)
                *reinterpret_cast<uint2*>(stg + (l32 & 15) * L::kRow + j * 64 + q * 16 + g * 8) =
                    make_uint2(pack_bf16x2(acc[j][i][4 * q] * sc, acc[j][i][4 * q + 1] * sc),
                               pack_bf16x2(acc[j][i][4 * q + 2] * sc, acc[j][i][4 * q + 3] * sc));
          }
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const int u = t * 64 + lane, row = u / (4 * NT), c = u % (4 * NT);
            const uint4 v = *reinterpret_cast<const uint4*>(stg + row * L::kRow + c * 16);
            const int m = m0 + i * 32 + half * 16 + row;
            if (m < M)
              *reinterpret_cast<uint4*>(reinterpret_cast<unsigned char*>(p.qk + part * D + c0) +
                                        ((uint32_t)m * (6u * D) + (uint32_t)c * 16u)) = v;
          }
        }
    } else {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        // (in the global address space still after the pointer is made opaque: a flat store
        // would make every later wait one for all that is in flight)
        __attribute__((address_space(1))) bf16_t* vp =
            (__attribute__((address_space(1))) bf16_t*)(p.vt + (size_t)(c0 + 4 * g) * p.vt_ld + vpos[i]);
        asm volatile("" : "+v"(vp));
        if (m0 + i * 32 + l32 < M) {
#pragma unroll
          for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              *vp = f32_to_bf16(acc[j][i][r]);
              vp += (size_t)((r & 3) == 3 ? 5 : 1) * p.vt_ld;
            }
        }
      }
    }
  }
}

// The weights of a layer in the order the wavefronts stream them (see wide_layer_kernel).
// One thread per 16 bytes; with Wo null only the q/k/v part (the first layer's kernel).
template <int D, int NW>
__global__ __launch_bounds__(256) void wide_pack_kernel(const bf16_t* __restrict__ Wo, const bf16_t* __restrict__ W1,
                                                        const bf16_t* __restrict__ W2, const bf16_t* __restrict__ Wqkv,
                                                        int F, int blocks, bf16_t* __restrict__ out) {
  constexpr int NT = D / (32 * NW), KS = D / 16, kFC = 32 * NW;
  const long u = (long)blockIdx.x * 256 + threadIdx.x;
  if (u >= (long)blocks * NW * 64) return;
  const int lane = (int)(u & 63), l32 = lane & 31, g = lane >> 5;
  const long blk = u >> 6;
  const int w = (int)(blk / blocks);
  int b = (int)(blk % blocks);
  const int nc = F / kFC;
  const bf16_t* src = nullptr;
  const int c0 = w * (D / NW);
  bool done = false;
  if (Wo != nullptr) {
    if (b < KS * NT) {
      src = Wo + (size_t)(c0 + (b % NT) * 32 + l32) * D + (b / NT) * 16 + g * 8;
      done = true;
    }
    b -= KS * NT;
    // F1(0), then F1(c) F2(c - 1) ..., then F2(nc - 1)
    const int f1 = KS, f2 = (kFC / 16) * NT;
    if (!done && b < nc * (f1 + f2)) {
      int c, r;
      bool first;
      if (b < f1) { c = 0; r = b; first = true; }
      else if (b >= nc * (f1 + f2) - f2) { c = nc - 1; r = b - (nc * (f1 + f2) - f2); first = false; }
      else {
        const int t = b - f1, it = t / (f1 + f2), rr = t % (f1 + f2);
        first = rr < f1;
        c = first ? it + 1 : it;
        r = first ? rr : rr - f1;
      }
      if (first) src = W1 + (size_t)(c * kFC + w * 32 + l32) * D + r * 16 + g * 8;
      else src = W2 + (size_t)(c0 + (r % NT) * 32 + l32) * F + c * kFC + (r / NT) * 16 + g * 8;
      done = true;
    }
    b -= nc * (f1 + f2);
  }
  if (!done && Wqkv != nullptr && b < 3 * KS * NT) {
    const int part = b / (KS * NT), r = b % (KS * NT);
    src = Wqkv + (size_t)(part * D + c0 + (r % NT) * 32 + l32) * D + (r / NT) * 16 + g * 8;
  }
  if (src) reinterpret_cast<uint4*>(out)[u] = *reinterpret_cast<const uint4*>(src);
}

int wide_waves(int d) { return d == 256 ? 8 : 4; }

int wide_blocks(int d, int F, bool head) {
  const int nw = wide_waves(d), nt = d / (32 * nw), ks = d / 16, nc = F / (32 * nw);
  return (head ? 0 : ks * nt + nc * (ks + 2 * nw * nt)) + 3 * ks * nt;
}

template <int D, int NW, int MT, int kKind>
hipError_t launch_wide(const WideLayerArgs& a, const WideArgs& p, int F, const int32_t* m_ptr, int m_host, int m_capacity, hipStream_t s) {
  auto kern = wide_layer_kernel<D, NW, MT, kKind>;
  const size_t lds = WideLds<D, NW, MT>::bytes(F);
  static DeviceOnce configured;
  hipError_t e = allow_lds(kern, 160 * 1024, &configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((m_capacity + 32 * MT - 1) / (32 * MT)), dim3(64 * NW), lds, s, m_ptr,
                     static_cast<const unsigned char*>(a.packed), a.resid, static_cast<const bf16_t*>(a.O), a.x0, m_host,
                     (uint32_t)wide_blocks(D, F, kKind == kHead) * 1024, F, a.x0_rows, p);
  return hipGetLastError();
}

}  // namespace

// F: whole hidden chunks, and the vectors of a layer have to fit beside the tiles of the
// workgroups of a CU.  Rows: the
// kernel addresses rows of x and of q/k/v with 32-bit byte offsets.
bool wide_layer_supported(int d, int F, bool use_bf16, uint64_t rows) {
  return use_bf16 && ((d == 256 && F % 256 == 0) || (d == 384 && F % 128 == 0)) && F <= 2048 && rows * 6 * d < (1ull << 32);
}

uint64_t wide_layer_packed_bytes(int d, int F, bool head) {
  return ((uint64_t)wide_blocks(d, F, head) * wide_waves(d) + kRingMax) * 1024;   // (the ring reads ahead of the end)
}

hipError_t launch_wide_pack(const void* Wo, const void* W1, const void* W2, const void* Wqkv, int d, int F,
                            void* packed, hipStream_t s) {
  if (d != 256 && d != 384) return hipErrorInvalidValue;
  const int blocks = wide_blocks(d, F, Wo == nullptr);
  const long units = (long)blocks * wide_waves(d) * 64;
  auto a = [](const void* q) { return static_cast<const bf16_t*>(q); };
  hipLaunchKernelGGL((d == 256 ? wide_pack_kernel<256, 8> : wide_pack_kernel<384, 4>), dim3((unsigned)((units + 255) / 256)), dim3(256), 0, s, a(Wo), a(W1), a(W2),
                     a(Wqkv), F, blocks, static_cast<bf16_t*>(packed));
  return hipGetLastError();
}

// Rows per workgroup, by the rows expected (a guess is enough: every height gives the same
// bits).  Width 384: one workgroup per CU is the fastest there is, so the lowest tile that gets by with
// that; a workgroup of 96 rows has a CU to itself, one of 64 shares it with a second one,
// whose vector work then runs under its MFMAs, and is the best where CUs get several.
// Encoder passes of 4 layers over frames of 1,024 tokens in us, at 32 / 64 / 96 rows, F = 1536:
// 8,192 rows 309 / 348 / 444; 16,384 rows 519 / 470 / 561; 24,576 rows 762 / 690 / 654; 32,768 rows
// 1003 / 857 / 1077.  The same with F from 256 to 2048: 24,576 rows at F = 256 520 / 498 / 488, at 512 552 / 526 / 518, at
// 768 599 / 567 / 550; 18,432 rows at 512 478 / 460 / 444.
//
// Width 256: a workgroup of eight wavefronts fills a CU at every height, so the rounds of the
// busiest CU times what one costs decide.  A layer costs 19, 26 and 37 us at F = 1024, 12, 17 and 24
// at 256, 29, 39 and 55 at 2048: 1 : 1.4 : 1.95 at all of them, and only the ratio counts.  Passes as
// above, F = 1024: 8,192 rows 200 / 220 / 257; 16,384 rows 347 / 306 / 340; 24,576 rows 501 / 490 /
// 438; 32,768 rows 660 / 592 / 657; 102,400 rows 2,238 / 2,001 / 2,014; 112,896 rows 2,524 / 2,217 / 2,228.  At F =
// 256, 512, 1536 and 2048 the same heights win.
int wide_layer_tiles(int d, int rows, int cus) {
  if (d == 256) {
    const int cost[3] = {19, 26, 37};
    int best = 1;
    long least = 0;
    for (int mt = 1; mt <= 3; ++mt) {
      const long rounds = ((long)rows + 32L * mt * cus - 1) / (32L * mt * cus), t = rounds * cost[mt - 1];
      if (mt == 1 || t < least) {
        best = mt;
        least = t;
      }
    }
    return best;
  }
  for (int mt = 1; mt <= 3; ++mt)
    if (rows <= 32 * mt * cus) return mt;
  return 2;
}

hipError_t launch_wide_layer(const WideLayerArgs& a, int d, int F, int mt, const int32_t* m_ptr, int m_host,
                             int m_capacity, hipStream_t s) {
  if (!wide_layer_supported(d, F, true, m_capacity)) return hipErrorInvalidValue;
  WideArgs p{};
  const bool head = a.O == nullptr;
  p.b_o = a.b_o;
  p.ln2_g = a.ln2_g;
  p.ln2_b = a.ln2_b;
  p.b1 = a.b_ff1;
  p.b2 = a.b_ff2;
  p.ln_g = a.ln_g;
  p.ln_b = a.ln_b;
  p.eps = a.eps;
  p.out = a.out;
  p.split_row = a.split_row;
  p.out2 = a.out2;
  p.b_qkv = a.b_qkv;
  p.q_scale = a.q_scale;
  p.qk = static_cast<bf16_t*>(a.qk);
  p.vt = static_cast<bf16_t*>(a.vt);
  p.vt_ld = a.vt_ld;
  p.vt_pos = a.vt_pos;
  p.cu = a.cu;
  p.pcu = a.pcu;
  p.nseq = a.B;
  auto kind = [&](auto tiles) {
    constexpr int MT = decltype(tiles)::value;
    if (d == 256)
      return head ? launch_wide<256, 8, MT, kHead>(a, p, F, m_ptr, m_host, m_capacity, s)
                  : a.last ? launch_wide<256, 8, MT, kLast>(a, p, F, m_ptr, m_host, m_capacity, s) : launch_wide<256, 8, MT, kMid>(a, p, F, m_ptr, m_host, m_capacity, s);
    return head ? launch_wide<384, 4, MT, kHead>(a, p, F, m_ptr, m_host, m_capacity, s)
                : a.last ? launch_wide<384, 4, MT, kLast>(a, p, F, m_ptr, m_host, m_capacity, s) : launch_wide<384, 4, MT, kMid>(a, p, F, m_ptr, m_host, m_capacity, s);
  };
  return mt >= 3 ? kind(std::integral_constant<int, 3>{})
                 : mt == 2 ? kind(std::integral_constant<int, 2>{}) : kind(std::integral_constant<int, 1>{});
}

}  // namespace cfdetr
