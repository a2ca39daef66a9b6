// Variable-length multi-head self-attention (Sec. II-A: every token attends to
// every token of its own frame; A3, Sec. III-B: several frames in one batch).
// Frames are addressed by offsets, so no padding token is ever computed.
//
// bf16 kernel, flash style.  A work item is 128 (or 256) queries of one (frame, head); each
// of the four wavefronts of a workgroup owns 32 (or 64) of them.  Keys/values are walked in
// tiles of 64 that go from global memory straight into LDS (global_load_lds, a ring of three
// tiles, one wait and one barrier per tile).  Everything is computed transposed so that
// a query is a LANE:
//   S^T[key, q] = K . Q^T          (MFMA A = K rows from LDS, B = Q rows in registers)
//   O^T[dh, q] += V^T . P^T        (MFMA A = V^T rows from LDS, B = P from registers)
// In the MFMA result layout a lane then holds 16 keys of ONE query, so the sum of its
// probabilities is a per-lane scalar, the only cross-lane step is one exchange between
// lane l and l^32 at the end, and the probabilities feed the second MFMA straight from
// registers.  For that to work the 8 keys a
// lane contributes to one k-step must sit in 8 consecutive result registers: LDS row
// rho of a 32-key sub-tile therefore holds the key whose index is rho with bits 2
// and 3 swapped (result register r of lane group g holds row 8*(r/4)+4*g+r%4, which
// then is key 16*(r/8)+8*g+r%8); with direct loads that permutation is free, the
// lane that fills row rho simply fetches that key.  V^T comes from a feature-major
// copy of V ([d][positions], each frame padded to a multiple of 64 positions) that
// the QKV projection writes, so its tiles are plain row copies too.  LDS rows are
// unpadded; 16-byte chunks are XOR-swizzled by row so that operand reads of 16
// consecutive rows hit disjoint banks.
//
// What bounds the loop is that its parts depend on each other: the logits of a tile, their
// exponentials, the product with the values.  One after the other they leave the matrix unit
// idle through the exponentials and the vector unit idle through the MFMAs, and neither
// LDS nor occupancy makes up for it (the kernel that did so, with four wavefronts per SIMD,
// had the matrix unit busy 43 % of a launch, and at one wavefront per SIMD a 64-key tile took
// 0.93 us).  So the loop is a software pipeline over units of 32 keys: while the exponentials
// of unit u are worked out, the MFMAs of two other units run, the values of unit u - 1 and the
// logits of unit u + 1, in one fixed instruction order: an MFMA, then its share of two
// exponentials, two additions and a convert (32 clocks of the one beside about 34 of the
// others).  Measured, before -> after: one 4000-token frame of 6 heads of 64, 65.5 -> 43 us; 920
// tokens 17.9 -> 13 us; 24 470 tokens in 8 frames 149 -> 135 us; 8 x (1600 + 6400) tokens 488 ->
// 420 us (1.27 PFLOP/s, matrix unit busy 64 % at the 1.85 GHz that the load leaves).
//
// 64 queries per wavefront (head width 64 only) feed two MFMAs from every operand read, so LDS
// traffic per FLOP halves, but take 256 registers (two wavefronts per SIMD) and make items of
// 256 queries: the better form once there is far more work than the chip holds at once
// (attention_block_q).  Every query's arithmetic is the same in both, to the bit.
//
// Softmax arithmetic per element is one exp2, one add and half a convert: q arrives
// multiplied by log2(e)/sqrt(dh), so S is a base-2 logit, and the probabilities are taken as
// 2^S, relative to the reference 0 and not to a running maximum: O / l is the same quotient
// for any reference, floating point keeps the same relative precision at any magnitude, and
// no maximum has to be tracked, compared or applied.  What a fixed reference cannot do is
// stay inside the exponent range: when a query's sum of probabilities ends outside
// [2^-64, 2^100] (or is no number), some probability that matters may have been flushed to
// zero or have overflowed; such queries are computed again (exact_queries), with a walk for
// their largest logit and one with the probabilities relative to it, which is
// exact for any logits.  Trained or randomly initialised weights do not get there (|S| of
// a few tens); the parity tests force it.
//
// Work distribution: sequences differ in length by 2-3x, so a fixed item -> workgroup
// map leaves CUs idle while the longest items finish.  The grid is sized to what the
// chip holds at once (a multiple of 8) and workgroup w serves queue w mod 8: it starts
// with entry w/8 and fetches further entries (longest first) through an atomic counter
// until the queue is empty.  Every queue has grid/8 workgroups whatever the hardware's
// placement; with the usual round-robin placement those all sit on one XCD and share
// its L2.
//
// The fp32 kernel (check mode) is an online softmax (running maximum) with one query per
// thread.
#include <type_traits>

#include "kernels.h"

namespace cfdetr {

namespace {

constexpr int kBlockKV = 64;
constexpr int kWavesPerGroup = 4;
// sums of probabilities (relative to the reference 0) outside this range send an item
// through the exact walk: below, probabilities that matter may have been flushed to zero
// (normal numbers end at 2^-126; 2^24 flushed ones add up to less than 2^-100); above, one
// may have overflowed
constexpr float kSumLow = 0x1p-64f, kSumHigh = 0x1p+100f;

__device__ __forceinline__ int swap_bits_2_3(int i) {
  return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1);
}

// Swizzle key of LDS row r: 128-byte rows have 8 chunks and two rows cover the 64
// banks, 64-byte rows have 4 chunks and four rows cover them.
template <int ROWB>
__device__ __forceinline__ int swz(int r) {
  return ROWB == 128 ? ((r >> 1) & 7) : ((r >> 2) & 3);
}

// One 16-byte piece per lane from global memory straight into LDS (1 KB per wavefront at
// lds_addr, lane order): the address is a base in scalar registers plus the lane's 32-bit
// byte offset, so a tile that lies inside its sequence costs no vector arithmetic.  The
// compiler does not count these loads; the tile loop waits with vmcnt(0) itself.
__device__ __forceinline__ void attn_dma16(const void* sbase, uint32_t voff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_addr), "v"(voff), "s"(sbase)
               : "memory");
}

// Clears, in a V^T tile in LDS (row = feature, 8 chunks of 8 keys), the keys from `nvalid`
// on.  Not inlined on purpose: it runs once per work item, and inlined into the tile loop it
// costs the kernel an occupancy step (the loop's register budget is what sets it).
template <int DH>
__device__ __attribute__((noinline)) void clear_v_padding(unsigned char* wV, int nvalid, int tid) {
  for (int u = tid; u < DH * 8; u += 64 * kWavesPerGroup) {
    const int rho = u >> 3, c = u & 7;   // row (feature), logical chunk of 8 keys
    const int n = nvalid - 8 * c;        // keys of this chunk inside the sequence
    if (n < 8) {
      uint4* q = reinterpret_cast<uint4*>(wV + rho * 128 + ((c ^ swz<128>(rho)) << 4));
      uint4 w = *q;
      uint32_t* e = reinterpret_cast<uint32_t*>(&w);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        e[j] &= (2 * j < n ? 0x0000FFFFu : 0u) | (2 * j + 1 < n ? 0xFFFF0000u : 0u);
      *q = w;
    }
  }
}

// The exact walk of 32 queries per wavefront (see above), for an item whose sums left the safe
// range: the largest logit of every query, then the probabilities relative to it; only the
// queries with `redo` set are written.  Everything is fetched again; this is the rare path and
// it is a function of its own, so that the registers of the fast path are not its business (one for
// each kernel: a second caller at head width 32 took 32 bytes of scratch and 36 instructions more).
template <int DH, typename... Extra>
__device__ __attribute__((noinline)) void exact_queries(
    const bf16_t* q_row, const bf16_t* kbase, int k_ld, const bf16_t* vbase, int vt_ld, int TK,
    bf16_t* orow, bool redo, unsigned char* smem) {
  constexpr int KS = DH / 16, MO = DH / 32, KROWB = DH * 2, KCPR = KROWB / 16;
  unsigned char* const sK = smem;
  unsigned char* const sV = smem + kBlockKV * KROWB;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int n_kv = (TK + kBlockKV - 1) / kBlockKV;
  bf16x8 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(q_row + ks * 16 + g * 8);
  f32x16 acc_o[MO];
#pragma unroll
  for (int i = 0; i < MO; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_o[i][r] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;
#pragma nounroll
  for (int pass = 0; pass < 2; ++pass) {
#pragma nounroll
    for (int it = 0; it < n_kv; ++it) {
      const int kv0 = it * kBlockKV;
      __syncthreads();
      for (int u = tid; u < kBlockKV * KCPR; u += 64 * kWavesPerGroup) {
        const int rho = u / KCPR, c = u % KCPR;
        const int key = min(kv0 + ((rho & 32) | swap_bits_2_3(rho & 31)), TK - 1);
        *reinterpret_cast<uint4*>(sK + rho * KROWB + ((c ^ swz<KROWB>(rho)) << 4)) =
            *reinterpret_cast<const uint4*>(kbase + (size_t)key * k_ld + c * 8);
      }
      if (pass == 1)
        for (int u = tid; u < DH * 8; u += 64 * kWavesPerGroup) {
          const int rho = u >> 3, c = u & 7;
          *reinterpret_cast<uint4*>(sV + rho * 128 + ((c ^ swz<128>(rho)) << 4)) =
              *reinterpret_cast<const uint4*>(vbase + (size_t)rho * vt_ld + kv0 + c * 8);
        }
      __syncthreads();
      if (pass == 1 && kv0 + kBlockKV > TK) {
        clear_v_padding<DH>(sV, TK - kv0, tid);
        __syncthreads();
      }
      float l_tile = 0.f;
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        const int rho = sub * 32 + l32;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              *reinterpret_cast<const bf16x8*>(sK + rho * KROWB + (((2 * ks + g) ^ swz<KROWB>(rho)) << 4)),
              qf[ks], s, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kv0 + sub * 32 + 16 * (r >> 3) + 8 * g + (r & 7) >= TK) s[r] = -INFINITY;
        if (pass == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) m_ref = fmaxf(m_ref, s[r]);
          continue;
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          uint32_t w[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float p0 = __builtin_amdgcn_exp2f(s[8 * t + 2 * e] - m_ref);
            const float p1 = __builtin_amdgcn_exp2f(s[8 * t + 2 * e + 1] - m_ref);
            l_tile += p0 + p1;
            w[e] = pack_bf16x2(p0, p1);
          }
          uint4 packed = make_uint4(w[0], w[1], w[2], w[3]);
          const bf16x8 pf = *reinterpret_cast<bf16x8*>(&packed);
#pragma unroll
          for (int i = 0; i < MO; ++i) {
            const int rv = i * 32 + l32;
            acc_o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                *reinterpret_cast<const bf16x8*>(sV + rv * 128 + (((4 * sub + 2 * t + g) ^ swz<128>(rv)) << 4)),
                pf, acc_o[i], 0, 0, 0);
          }
        }
      }
      l_run += l_tile;
    }
    if (pass == 0) m_ref = fmaxf(m_ref, __shfl_xor(m_ref, 32, kWave));
  }
  __syncthreads();
  const float inv = 1.0f / (l_run + __shfl_xor(l_run, 32, kWave));
  if (redo) {
#pragma unroll
    for (int i = 0; i < MO; ++i)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq)
        *reinterpret_cast<uint2*>(orow + i * 32 + rq * 8 + g * 4) =
            make_uint2(pack_bf16x2(acc_o[i][4 * rq] * inv, acc_o[i][4 * rq + 1] * inv),
                       pack_bf16x2(acc_o[i][4 * rq + 2] * inv, acc_o[i][4 * rq + 3] * inv));
  }
}

// Few rows leave CUs without work in an attention launch, and the kernels behind it wait for weights that other
// work has driven out of the chip's memory-side cache.  kAheadGroups workgroups behind the others read them.  A
// kernel of its own (with Ahead), because the arguments and the branch cost the others 0.3 us a launch.
constexpr int kAheadGroups = 64;
struct Ahead {
  ReadAhead what;
  int from;  // the first of those workgroups
};
__device__ __forceinline__ void read_ahead(const ReadAhead& ahead, int group) {
  uint32_t sink = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint4* const p = static_cast<const uint4*>(ahead.at[r]);
    const uint32_t units = ahead.bytes[r] / 16;
#pragma unroll 8
    for (uint32_t u = group * (64 * kWavesPerGroup) + threadIdx.x; u < units; u += kAheadGroups * 64 * kWavesPerGroup) sink ^= p[u].x;
  }
  asm volatile("" : : "v"(sink));
}

// The first 14 words of arguments, as far as vt_ld and q_ld, arrive in scalar registers (build.py): what the first
// entry, keys and queries are asked for with.  The others are loaded meanwhile.  A launch is 0.2 to 0.3 us shorter for it: a
// coarse pass of 920 rows, 12 launches, 471 -> 469 us, one camera, 7 of them, 206.6 -> 205.0.
// QB: blocks of 32 queries per wavefront.  The second launch bound holds the compiler to the
// registers of two (64 queries), three or (head width 32) four wavefronts per SIMD.
template <int DH, int QB, typename... Extra>
__global__ __launch_bounds__(64 * kWavesPerGroup, QB == 2 ? 2 : DH == 64 ? 3 : 4) void attention_bf16_kernel(
    const int4* __restrict__ items, int32_t* __restrict__ queue_heads, const bf16_t* __restrict__ kbuf,
    const bf16_t* __restrict__ vt, const bf16_t* __restrict__ qbuf, int cap8, int k_ld, int vt_ld, int q_ld,
    const int32_t* __restrict__ cu_k, const int32_t* __restrict__ pcu_k, const int32_t* __restrict__ kv_len,
    bf16_t* __restrict__ out, int d, Extra... extra) {
  if constexpr (sizeof...(Extra) != 0) {
    const Ahead& ahead = (extra, ...);
    if ((int)blockIdx.x >= ahead.from) {
      read_ahead(ahead.what, blockIdx.x - ahead.from);
      return;
    }
  }
  constexpr int NW = kWavesPerGroup;
  constexpr int BQ = 32 * QB * NW;
  constexpr int KS = DH / 16;          // k-steps of Q.K^T
  constexpr int MO = DH / 32;          // 32-row blocks of O^T
  constexpr int KROWB = DH * 2;        // bytes per K row in LDS
  constexpr int KCPR = KROWB / 16;     // chunks per K row
  constexpr int KRPI = 1024 / KROWB;   // K rows per wave load instruction
  constexpr int KI = kBlockKV / KRPI / NW;   // K load instructions per wavefront
  constexpr int VI = DH / 8 / NW;            // V^T load instructions per wavefront (8 rows each)
  constexpr int KBYTES = kBlockKV * KROWB, VBYTES = DH * 128, TILE = KBYTES + VBYTES;
  constexpr int NB = 3;                // ring of key tiles
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NB * TILE];
  __shared__ int32_t s_item;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  const int home = blockIdx.x & 7;   // queue of this workgroup; w mod 8 is also its XCD
  // first item: entry blockIdx/8 of the home queue; later ones through the counter, which
  // starts behind the entries handed out this way
  int entry = blockIdx.x >> 3;
  // -1: the queue holds no more entries than were handed out by index (launch_plan)
  const bool drained = queue_heads[home] < 0;

  // Loader roles, as byte offsets of the lane's piece from the tile's first key (K) or
  // first position (V^T).  K: LDS row rho <- key (rho & 32) | swap23(rho & 31), chunk
  // swizzled.  V^T: LDS row rho = dh index; 64 keys = 8 chunks of 8.
  uint32_t k_off[KI], v_off[VI];
#pragma unroll
  for (int j = 0; j < KI; ++j) {
    const int rho = (wave * KI + j) * KRPI + lane / KCPR;
    const int key = (rho & 32) | swap_bits_2_3(rho & 31);
    k_off[j] = (uint32_t)key * (uint32_t)(k_ld * 2) + (uint32_t)(((lane % KCPR) ^ swz<KROWB>(rho)) * 16);
  }
#pragma unroll
  for (int j = 0; j < VI; ++j) {
    const int rho = (wave * VI + j) * 8 + (lane >> 3);
    v_off[j] = ((uint32_t)rho * (uint32_t)vt_ld + (uint32_t)(((lane & 7) ^ swz<128>(rho)) * 8)) * 2u;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  // operand addresses inside a tile: row l32 of a 32-row block, chunk swizzled
  uint32_t ka[KS], va[4];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) ka[ks] = l32 * KROWB + (((2 * ks + g) ^ swz<KROWB>(l32)) << 4);
#pragma unroll
  for (int c = 0; c < 4; ++c) va[c] = KBYTES + l32 * 128 + (((2 * c + g) ^ swz<128>(l32)) << 4);

  for (;;) {
    // An entry is four words: the item, then offset, length and padded offset of its
    // sequence; the index is uniform, so this is one scalar load and a workgroup needs
    // nothing else before it can ask for its queries and first keys.
    if (entry >= cap8) break;
    const int4 rec = items[home + 8 * entry];
    const int32_t item = rec.x;
    if (item < 0) break;   // entries are in use from the front: the queue is empty

    const int frame = item >> 24, head = (item >> 19) & 31, qt = item & 0x7FFFF;
    const int seq0 = rec.y, T = rec.z;
    // the keys come from sequence `frame` of cu_k (cross-attention) or are the queries' own
    // sequence, all of them unless the caller padded it
    const int kseq0 = cu_k ? cu_k[frame] : seq0;
    const int TKall = cu_k ? cu_k[frame + 1] - kseq0 : T;
    const int kpad0 = cu_k ? pcu_k[frame] : rec.w;
    const int TK = kv_len ? min(kv_len[frame], TKall) : TKall;
    const bf16_t* qbase = qbuf + (size_t)seq0 * q_ld + head * DH;
    const bf16_t* kbase = kbuf + (size_t)kseq0 * k_ld + head * DH;
    const bf16_t* vbase = vt + (size_t)(head * DH) * vt_ld + kpad0;
    const int n_kv = (TK + kBlockKV - 1) / kBlockKV;

    // Fill of tile j_: inside the sequence the lane offsets are the constants above; the
    // last, ragged tile clamps its keys to the sequence (the lanes that would read past it
    // fetch the last key again; their logits are masked).
    auto issue = [&](int j_, int slot_) {
      const int kv0_ = j_ * kBlockKV;
      const bf16_t* kb_ = kbase + (size_t)kv0_ * k_ld;
      const uint32_t lb_ = lds0 + slot_ * TILE;
      const uint32_t lk_ = lb_ + wave * (KI * 1024), lv_ = lb_ + KBYTES + wave * (VI * 1024);
      if (kv0_ + kBlockKV <= TK) {
#pragma unroll
        for (int j = 0; j < KI; ++j) attn_dma16(kb_, k_off[j], lk_ + j * 1024);
      } else {
#pragma unroll
        for (int j = 0; j < KI; ++j) {
          const int rho = (wave * KI + j) * KRPI + lane / KCPR;
          const int key = min((rho & 32) | swap_bits_2_3(rho & 31), TK - 1 - kv0_);
          attn_dma16(kb_, (uint32_t)key * (uint32_t)(k_ld * 2) +
                              (uint32_t)(((lane % KCPR) ^ swz<KROWB>(rho)) * 16), lk_ + j * 1024);
        }
      }
      const bf16_t* vb_ = vbase + kv0_;
#pragma unroll
      for (int j = 0; j < VI; ++j) attn_dma16(vb_, v_off[j], lv_ + j * 1024);
    };

    issue(0, 0);
    // Q operands: lane = query, 8 consecutive dh per k-step.
    bf16x8 qf[QB][KS];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const int q_load = min(qt * BQ + (wave * QB + qb) * 32 + l32, T - 1);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        qf[qb][ks] = *reinterpret_cast<const bf16x8*>(qbase + (size_t)q_load * q_ld + ks * 16 + g * 8);
    }
    f32x16 acc_o[QB][MO];
    // sums of probabilities: over all tiles so far, and over the tile in hand, which is added when
    // it is whole (thousands of keys added one pair at a time lose digits, equal ones 2e-5 at 6,400)
    float l_run[QB], l_tile[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      l_run[qb] = 0.f;
#pragma unroll
      for (int i = 0; i < MO; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[qb][i][r] = 0.f;
    }
    bf16x8 kf[KS], vf[MO][2];
    bf16x8 pA[QB][2], pB[QB][2];
    f32x16 sA[QB], sB[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) pB[qb][t][e] = (__bf16)0.f;

    auto read_k = [&](const unsigned char* tile, int sub) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        kf[ks] = *reinterpret_cast<const bf16x8*>(tile + ka[ks] + sub * (32 * KROWB));
    };
    auto read_v = [&](const unsigned char* tile, int sub) {
#pragma unroll
      for (int i = 0; i < MO; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          vf[i][t] = *reinterpret_cast<const bf16x8*>(tile + va[2 * sub + t] + i * (32 * 128));
    };
    auto qk1 = [&](f32x16(&s)[QB], int m) {   // MFMA m of the first product
      const int ks = m / QB, qb = m % QB;
      if (ks == 0) {
        f32x16 z;
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r] = 0.f;
        s[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[qb][ks], z, 0, 0, 0);
      } else {
        s[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[qb][ks], s[qb], 0, 0, 0);
      }
    };
    auto pv1 = [&](bf16x8(&p)[QB][2], int m) {   // MFMA m of the second product
      const int qb = m % QB, i = (m / QB) % MO, t = m / QB / MO;
      acc_o[qb][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i][t], p[qb][t], acc_o[qb][i], 0, 0, 0);
    };
    auto mask = [&](f32x16(&s)[QB], int key0) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (key0 + 16 * (r >> 3) + 8 * g + (r & 7) >= TK) s[qb][r] = -INFINITY;
    };
    // One stage: on the matrix unit the values of unit u - 1 (operands in vf) and then the
    // logits of unit u + 1 (keys read here, from ktile), between them the exponentials of
    // unit u: behind every MFMA its share of that arithmetic and of the LDS reads, in an order
    // the compiler is not to change.  The values of unit u are read behind the first product.
    auto stage = [&](f32x16(&s)[QB], f32x16(&sn)[QB], bf16x8(&pc)[QB][2], bf16x8(&pp)[QB][2],
                     const unsigned char* ktile, int ksub, const unsigned char* vtile, auto unit_tag,
                     auto more_tag) {
      constexpr bool kMore = decltype(more_tag)::value;   // there is a unit u + 1
      constexpr int vsub = decltype(unit_tag)::value;     // which half of its tile unit u is
      constexpr int NQK = QB * KS, NPV = QB * 2 * MO, NM = NQK + NPV;
      constexpr int PAIRS = QB * 8, PPM = PAIRS / NM;
      static_assert(PAIRS % NM == 0, "exponentials per MFMA");
      uint32_t w[QB][8];
      float e0 = 0.f, e1 = 0.f;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        if (m < NPV) {
          pv1(pp, m);
          if (kMore && m < KS) kf[m] = *reinterpret_cast<const bf16x8*>(ktile + ka[m] + ksub * (32 * KROWB));
        } else {
          if (kMore) qk1(sn, m - NPV);
          if (m - NPV < 2 * MO) {
            const int t_ = (m - NPV) / MO, i_ = (m - NPV) % MO;
            vf[i_][t_] = *reinterpret_cast<const bf16x8*>(vtile + va[2 * vsub + t_] + i_ * (32 * 128));
          }
        }
#pragma unroll
        for (int x = m * PPM; x < (m + 1) * PPM; ++x) {
          const int qb = x / 8, e = x % 8;
          // sum and conversion of the pair before: its exponentials have left the
          // transcendental pipe by now
          if (x > 0) {
            const int qy = (x - 1) / 8;
            l_tile[qy] = vsub == 0 && (x - 1) % 8 == 0 ? e0 + e1 : l_tile[qy] + (e0 + e1);
            w[qy][(x - 1) % 8] = pack_bf16x2(e0, e1);
            asm volatile("" : "+v"(w[qy][(x - 1) % 8]), "+v"(l_tile[qy]));
          }
          e0 = __builtin_amdgcn_exp2f(s[qb][2 * e]);
          e1 = __builtin_amdgcn_exp2f(s[qb][2 * e + 1]);
          asm volatile("" : "+v"(e0), "+v"(e1));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      l_tile[QB - 1] += e0 + e1;
      w[QB - 1][7] = pack_bf16x2(e0, e1);
      if (vsub == 1) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) l_run[qb] += l_tile[qb];
      }
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int t_ = 0; t_ < 2; ++t_) {
          uint4 packed = make_uint4(w[qb][4 * t_], w[qb][4 * t_ + 1], w[qb][4 * t_ + 2], w[qb][4 * t_ + 3]);
          pc[qb][t_] = *reinterpret_cast<bf16x8*>(&packed);
        }
    };

    // Tile j sits in slot j % 3.  The fills are waited for once per tile, between its two
    // units: tile j + 1 is then in LDS and every wavefront is past its last read of tile
    // j - 1, whose slot tile j + 2 takes.
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    if (n_kv > 1) issue(1, 1);
    else if (TK < kBlockKV) {
      clear_v_padding<DH>(smem + KBYTES, TK, tid);
      __syncthreads();
    }
    read_k(smem, 0);
#pragma unroll
    for (int m = 0; m < QB * KS; ++m) qk1(sA, m);
    read_v(smem, 0);   // (in front of the first unit: met with probabilities 0)
    const unsigned char* tcur = smem;
    int slot = 0;
    const auto half0 = std::integral_constant<int, 0>{};
    const auto half1 = std::integral_constant<int, 1>{};
    const auto yes = std::integral_constant<bool, true>{};
    const auto no = std::integral_constant<bool, false>{};
    // Three tiles at a time have constant slots, which makes every LDS address a lane constant
    // plus an immediate (with the slot in a register the additions are 8 % of a tile's vector
    // instructions); what is left over, and a ragged tile's padding, take the general form.
    auto tile_step = [&](int j, auto slot_tag) {
      constexpr int kSlot = decltype(slot_tag)::value, kNext = (kSlot + 1) % NB;
      const unsigned char* cur = smem + kSlot * TILE;
      const unsigned char* next = smem + kNext * TILE;
      stage(sA, sB, pA, pB, cur, 1, cur, half0, yes);    // unit 2j
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
      issue(j + 2, (kSlot + 2) % NB);
      stage(sB, sA, pB, pA, next, 0, cur, half1, yes);   // unit 2j + 1
    };
    int j = 0;
    for (; j + 5 <= n_kv; j += 3) {
      tile_step(j, std::integral_constant<int, 0>{});
      tile_step(j + 1, std::integral_constant<int, 1>{});
      tile_step(j + 2, std::integral_constant<int, 2>{});
    }
    for (; j < n_kv - 1; ++j) {
      stage(sA, sB, pA, pB, tcur, 1, tcur, half0, yes);    // unit 2j
      __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
      const int snext = slot == NB - 1 ? 0 : slot + 1;
      const unsigned char* tnext = smem + snext * TILE;
      if (j + 2 < n_kv) {
        issue(j + 2, snext == NB - 1 ? 0 : snext + 1);
      } else if (TK & (kBlockKV - 1)) {
        clear_v_padding<DH>(smem + snext * TILE + KBYTES, TK - (j + 1) * kBlockKV, tid);
        __syncthreads();
      }
      stage(sB, sA, pB, pA, tnext, 0, tcur, half1, yes);   // unit 2j + 1
      tcur = tnext;
      slot = snext;
    }
    {
      // the last tile, ragged or not
      const int kv0 = (n_kv - 1) * kBlockKV;
      if (TK & (kBlockKV - 1)) mask(sA, kv0);
      stage(sA, sB, pA, pB, tcur, 1, tcur, half0, yes);
      if (TK & (kBlockKV - 1)) mask(sB, kv0 + 32);
      stage(sB, sA, pB, pA, tcur, 0, tcur, half1, no);
#pragma unroll
      for (int m = 0; m < QB * 2 * MO; ++m) pv1(pB, m);
    }

    bool redo[QB], any = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const float l_tot = l_run[qb] + __shfl_xor(l_run[qb], 32, kWave);
      redo[qb] = !(l_tot >= kSumLow && l_tot <= kSumHigh);
      any |= redo[qb];
      const float inv = 1.0f / l_tot;
      const int q_local = qt * BQ + (wave * QB + qb) * 32 + l32;
      if (q_local < T) {
        bf16_t* orow = out + (size_t)(seq0 + q_local) * d + head * DH;
#pragma unroll
        for (int i = 0; i < MO; ++i)
#pragma unroll
          for (int rq = 0; rq < 4; ++rq) {
            // registers 4*rq..4*rq+3 of lane group g are dh = 32*i + 8*rq + 4*g + 0..3
            uint2 w;
            w.x = pack_bf16x2(acc_o[qb][i][4 * rq] * inv, acc_o[qb][i][4 * rq + 1] * inv);
            w.y = pack_bf16x2(acc_o[qb][i][4 * rq + 2] * inv, acc_o[qb][i][4 * rq + 3] * inv);
            *reinterpret_cast<uint2*>(orow + i * 32 + rq * 8 + g * 4) = w;
          }
      }
    }
    // A sum that left the range in which every probability that matters is a normal number
    // (some logit beyond +-100 or so in base 2; also inf and NaN): those queries are computed
    // again relative to their largest logit.  The barrier keeps the next item's first fill
    // behind every wavefront's last reads of this one's tiles.
    if (__syncthreads_or(any)) {
#pragma nounroll
      for (int qb = 0; qb < QB; ++qb) {
        const int q_local = qt * BQ + (wave * QB + qb) * 32 + l32;
        const bool again = QB == 1 ? redo[0] : (qb == 0 ? redo[0] : redo[QB - 1]);
        exact_queries<DH, Extra...>(qbase + (size_t)min(q_local, T - 1) * q_ld, kbase, k_ld, vbase, vt_ld, TK,
                              out + (size_t)(seq0 + min(q_local, T - 1)) * d + head * DH,
                              again && q_local < T, smem);
      }
    }
    if (drained) break;
    if (tid == 0) s_item = atomicAdd(&queue_heads[home], 1);
    __syncthreads();
    entry = __builtin_amdgcn_readfirstlane(s_item);
  }
}

// fp32 check mode: one query per thread, keys in tiles of 32 through LDS.
template <int DH>
__global__ __launch_bounds__(256) void attention_f32_kernel(
    const float* __restrict__ qkv, float* __restrict__ out, int d,
    const int4* __restrict__ items, float scale, const int32_t* __restrict__ kv_len) {
  constexpr int TILE = 32;
  __shared__ float sK[TILE][DH];
  __shared__ float sV[TILE][DH];
  const int4 rec = items[blockIdx.x];
  const int32_t item = rec.x;
  if (item < 0) return;
  const int frame = item >> 24, head = (item >> 19) & 31, qt = item & 0x7FFFF;
  const int seq0 = rec.y, T = rec.z;
  const int TK = kv_len ? min(kv_len[frame], T) : T;
  const int ld = 3 * d;
  const float* qbase = qkv + (size_t)seq0 * ld + head * DH;
  const int q_local = qt * (int)blockDim.x + threadIdx.x;   // block size = queries per tile
  const int q_load = min(q_local, T - 1);
  float q[DH], o[DH];
#pragma unroll
  for (int i = 0; i < DH; ++i) {
    q[i] = qbase[(size_t)q_load * ld + i] * scale;
    o[i] = 0.f;
  }
  float m_run = -INFINITY, l_run = 0.f;
  for (int kv0 = 0; kv0 < TK; kv0 += TILE) {
    __syncthreads();
    for (int e = threadIdx.x; e < TILE * DH; e += blockDim.x) {
      int r = e / DH, c = e - r * DH;
      int key = min(kv0 + r, TK - 1);
      sK[r][c] = qbase[(size_t)key * ld + d + c];
      sV[r][c] = qbase[(size_t)key * ld + 2 * d + c];
    }
    __syncthreads();
    float s[TILE];
    float m_tile = -INFINITY;
#pragma unroll
    for (int r = 0; r < TILE; ++r) {
      float acc = 0.f;
#pragma unroll
      for (int i = 0; i < DH; ++i) acc = fmaf(q[i], sK[r][i], acc);
      s[r] = (kv0 + r < TK) ? acc : -INFINITY;
      m_tile = fmaxf(m_tile, s[r]);
    }
    const float m_new = fmaxf(m_run, m_tile);
    const float alpha = expf(m_run - m_new);
    m_run = m_new;
    l_run *= alpha;
#pragma unroll
    for (int i = 0; i < DH; ++i) o[i] *= alpha;
#pragma unroll
    for (int r = 0; r < TILE; ++r) {
      float p = expf(s[r] - m_new);
      l_run += p;
#pragma unroll
      for (int i = 0; i < DH; ++i) o[i] = fmaf(p, sV[r][i], o[i]);
    }
  }
  if (q_local < T) {
    float* orow = out + (size_t)(seq0 + q_local) * d + head * DH;
    const float inv = 1.0f / l_run;
#pragma unroll
    for (int i = 0; i < DH; ++i) orow[i] = o[i] * inv;
  }
}

}  // namespace


// Queries per work item.  64 queries per wavefront win where the wavefronts of 32 would be
// more than the chip works on at once, with room for the coarser items' uneven end: at 2500 to
// 2800 of them 32 queries are 7 to 9 % faster (74 against 79 us, 32 against 35), at 4600 64
// queries are 5 % and at 16000 8 % faster (141 -> 135, 454 -> 420).  At head width 32 the
// exponentials bind whatever the LDS traffic is, and the small form is never slower.
// How well the sequences fill their items does not move the line.  Passes with items of 128 / 256
// in us: 300 decoder queries (384 / 512 places) of 64 frames x 6 heads 2546 / 2568, x 12 heads 3447 /
// 3434; coarse grids of 1,600 tokens (1,664 / 1,792), 12 frames 1968 / 1910, 24 3562 / 3592, 32 4648 /
// 4592; of 540 tokens (640 / 768) 1856 / 1804; of 121 tokens (128 / 256: two of an item's wavefronts
// have nothing), 64 frames x 16 heads, 398 / 400.
int attention_block_q(int d_head, bool use_bf16, int64_t rows, int heads) {
  return use_bf16 && d_head == 64 && rows * heads > (int64_t)3500 * 32 ? 256 : 128;
}

float attention_q_scale(int d_head) {
  return 1.44269504088896340736f / sqrtf((float)d_head);
}

namespace {

// Workgroups the chip holds at once for a kernel: the size of a fetch-from-queue grid.
template <typename K>
int resident_grid(K kern) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 64 * kWavesPerGroup, 0) != hipSuccess) return 0;
  if (cus <= 0 || per_cu <= 0) return 0;
  return (cus * per_cu + 7) & ~7;
}

}  // namespace

int attention_grid(int d_head, bool use_bf16, int block_q, int cap8) {
  const long all = 8L * cap8;
  if (!use_bf16) return (int)all;
  int resident = 0;
  if (d_head == 64 && block_q == 256) resident = resident_grid(attention_bf16_kernel<64, 2>);
  else if (d_head == 64) resident = resident_grid(attention_bf16_kernel<64, 1>);
  else if (d_head == 32) resident = resident_grid(attention_bf16_kernel<32, 1>);
  if (resident <= 0) return 0;
  return (int)(all < resident ? all : resident);
}

namespace {

// The bf16 kernel for a head width and item size; false: there is none.
bool launch_bf16(int dh, int block_q, int grid_size, hipStream_t s, const bf16_t* q, int q_ld,
                 const bf16_t* k, int k_ld, const bf16_t* v, int vt_ld, bf16_t* out,
                 const int32_t* cu_k, const int32_t* pcu_k, int d, const int4* recs, int cap8,
                 int32_t* queue_heads, const int32_t* kv_len, const ReadAhead& ahead) {
  const dim3 block(64 * kWavesPerGroup);
  auto go = [&](auto kernel, int groups, auto... extra) {
    hipLaunchKernelGGL(kernel, dim3(groups), block, 0, s, recs, queue_heads, k, v, q, cap8, k_ld, vt_ld, q_ld, cu_k, pcu_k,
                       kv_len, out, d, extra...);
  };
  const bool any = ahead.bytes[0] != 0;
  if (dh == 64 && block_q == 256)  // rows enough to fill the chip
    go(attention_bf16_kernel<64, 2>, grid_size);
  else if (dh == 64 && block_q == 128 && any)
    go(attention_bf16_kernel<64, 1, Ahead>, grid_size + kAheadGroups, Ahead{ahead, grid_size});
  else if (dh == 64 && block_q == 128)
    go(attention_bf16_kernel<64, 1>, grid_size);
  else if (dh == 32 && block_q == 128 && any)
    go(attention_bf16_kernel<32, 1, Ahead>, grid_size + kAheadGroups, Ahead{ahead, grid_size});
  else if (dh == 32 && block_q == 128)
    go(attention_bf16_kernel<32, 1>, grid_size);
  else
    return false;
  return true;
}

}  // namespace

hipError_t launch_attention(const void* qkv, const void* vt, int vt_ld, void* out, int d, int heads,
                            const int32_t* items, int cap8, int32_t* queue_heads, int grid_size,
                            int block_q, bool use_bf16, const int32_t* kv_len, hipStream_t s, const ReadAhead& ahead) {
  if (grid_size < 8 || grid_size % 8 != 0 || grid_size > 8 * cap8) return hipErrorInvalidValue;
  const int dh = d / heads;
  const int4* recs = reinterpret_cast<const int4*>(items);
  if (use_bf16) {
    // queries and keys are thirds of the same rows
    const bf16_t* in = static_cast<const bf16_t*>(qkv);
    if (!launch_bf16(dh, block_q, grid_size, s, in, 3 * d, in + d, 3 * d, static_cast<const bf16_t*>(vt),
                     vt_ld, static_cast<bf16_t*>(out), nullptr, nullptr, d, recs, cap8, queue_heads,
                     kv_len, ahead))
      return hipErrorInvalidValue;
  } else {
    if (block_q != 128) return hipErrorInvalidValue;
    const float scale = 1.0f / sqrtf((float)dh);
    dim3 grid(8 * cap8);
    const float* in = static_cast<const float*>(qkv);
    float* o = static_cast<float*>(out);
    if (dh == 64)
      hipLaunchKernelGGL(attention_f32_kernel<64>, grid, dim3(block_q), 0, s, in, o, d, recs, scale,
                         kv_len);
    else if (dh == 32)
      hipLaunchKernelGGL(attention_f32_kernel<32>, grid, dim3(block_q), 0, s, in, o, d, recs, scale,
                         kv_len);
    else
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_cross_attention(const void* q, const void* k, const void* vt, int vt_ld,
                                  void* out, const int32_t* cu_k,
                                  const int32_t* pcu_k, int d, int heads, const int32_t* items,
                                  int cap8, int32_t* queue_heads, int grid_size, int block_q,
                                  hipStream_t s, const ReadAhead& ahead) {
  if (grid_size < 8 || grid_size % 8 != 0 || grid_size > 8 * cap8) return hipErrorInvalidValue;
  if (!launch_bf16(d / heads, block_q, grid_size, s, static_cast<const bf16_t*>(q), d,
                   static_cast<const bf16_t*>(k), d, static_cast<const bf16_t*>(vt), vt_ld,
                   static_cast<bf16_t*>(out), cu_k, pcu_k, d, reinterpret_cast<const int4*>(items), cap8,
                   queue_heads, nullptr, ahead))
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace cfdetr
