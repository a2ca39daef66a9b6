// Contractions of few rows: what slim_residual_kernel (few_rows.hip) and
// gemm_bf16_few_kernel (gemm.hip) share.
//
// With few rows a contraction is latency and not throughput: the launch, one trip to memory
// for the rows and one for the weights.  A wavefront therefore takes 32 rows (or 64) by 32
// columns and the whole of K, a workgroup 128 columns, so that there are as many workgroups
// as the shape yields without cutting a sum; the weights, which no two wavefronts of a
// workgroup share, skip the LDS: packed 1 KB per MFMA operand they stream through a ring of
// 24 registers a lane, all of them asked for before the first row is looked at.
#pragma once
#include <type_traits>

#include "kernels.h"

namespace cfdetr {

// Which tiles a workgroup does.  Every XCD has an L2 of its own, and with few rows a good part
// of what a launch takes is its operands' way into the eight of them, so an XCD gets a
// rectangle of tiles: the row tiles are cut in 2^row_bits groups (1, 2, 4 or 8), the 128-column parts
// in 8 / that.  The grid (few_rows_grid) is a workgroup per part of a group, times eight, by the row tiles of
// a group; a workgroup has part `part` (or none) of row tiles r, r + step, .. below r_end.  Row tiles change
// slowest, so that the workgroups for rows that turn out not to be there come last: in between the others
// they cost CUs their turn (768 x 3072: 1,200 rows 19.8 against 13.8 us, 4,800 rows 42.2 against 32.5).
// (Shifts, no division: 150 dependent scalar instructions in front of a kernel's first load are 0.7 us.)
struct XcdTiles {
  int r, r_end, step, part;
  bool none;
  __device__ __forceinline__ XcdTiles(int mtiles, int parts, int row_bits) {
    const int x = blockIdx.x & 7, rg = x & ((1 << row_bits) - 1), pg = x >> row_bits, part_bits = 3 - row_bits;
    r = ((mtiles * rg) >> row_bits) + (int)blockIdx.y;
    r_end = (mtiles * (rg + 1)) >> row_bits;
    step = (int)gridDim.y;
    part = ((parts * pg) >> part_bits) + (int)(blockIdx.x >> 3);
    none = part >= (parts * (pg + 1)) >> part_bits;
  }
};

constexpr int kFewRing = 24;       // weight blocks in flight per wavefront; K is a multiple of 16 kFewRing
constexpr int few_rows_lds(int mt) { return 4 * mt * 8 * 1024; }

// acc[i] += rows m0 + 32 i .. of `rows` times the wavefront's 32 columns of weights (K / 16
// blocks from wp).  `rows`: bf16 rows [M, K], or operand blocks (kBlocks): tiles of 32 rows, one
// block of 1 KB per k-step.  They come through the LDS (few_rows_lds bytes) eight k-steps at a
// time, in four places, three stages ahead.  begin() runs when all first loads have been
// issued and sets acc.  Ends in front of a barrier that the caller has to pass before the next
// call.
template <int MT, bool kBlocks, typename Begin>
__device__ __forceinline__ void few_rows_product(const bf16_t* rows, int K, int M, int m0, const unsigned char* wp,
                                                 unsigned char* smem, f32x16 (&acc)[MT], Begin begin) {
  constexpr int kRing = kFewRing, kStage = MT * 8 * 1024, kLoads = 2 * MT;
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int NK = K >> 4, NS = NK >> 3;
  const uint32_t voff = lane * 16;
  uint32_t ao[8];   // operand of k-step k of a stage: a block, or rows of 256 bytes, chunks XORed by the row
#pragma unroll
  for (int k = 0; k < 8; ++k) ao[k] = kBlocks ? k * 1024 + voff : l32 * 256 + (((2 * k + g) ^ (l32 & 15)) << 4);
  // stage loads of this wavefront: 1 KB each, block u of the stage or rows 4 u .. 4 u + 3
  const unsigned char* src[kLoads];
#pragma unroll
  for (int i = 0; i < kLoads; ++i) {
    const int u = wave * kLoads + i;
    if (kBlocks) {
      const int tile = min((m0 >> 5) + (u >> 3), ((M + 31) >> 5) - 1);
      src[i] = reinterpret_cast<const unsigned char*>(rows) + ((size_t)tile * NK + (u & 7)) * 1024 + voff;
    } else {
      const int row = u * 4 + (lane >> 4);
      src[i] = reinterpret_cast<const unsigned char*>(rows) + (size_t)min(m0 + row, M - 1) * (K * 2) +
               (((lane & 15) ^ (row & 15)) << 4);
    }
  }
  auto stage = [&](int s) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const uint32_t dst = (uint32_t)(uintptr_t)smem + (s & 3) * kStage + (wave * kLoads + i) * 1024;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                   : : "s"(dst), "v"(src[i] + (size_t)s * (kBlocks ? 8192 : 256)) : "memory");
    }
  };
  for (int s = 0; s < 3; ++s) stage(s);
  __builtin_amdgcn_sched_barrier(0);
  // weight block i of a round, the base of every fourth one in scalar registers: no vector arithmetic
  typedef const __attribute__((address_space(1))) unsigned char* gptr;
  gptr wq = (gptr)wp;
  auto weights = [&](int i) {
    if (i % 4 == 0) {
      wq = (gptr)wp + i * 1024;
      asm volatile("" : "+s"(wq));
    }
    return *reinterpret_cast<const __attribute__((address_space(1))) bf16x8*>(wq + (i % 4) * 1024 + voff);
  };
  bf16x8 wr[kRing];
#pragma unroll
  for (int i = 0; i < kRing; ++i) wr[i] = weights(i);
  __builtin_amdgcn_sched_barrier(0);
  begin();
  auto round = [&](int s0, auto last_tag) {
    constexpr bool kLastRound = decltype(last_tag)::value;   // nothing is asked for any more
    wp += kRing * 1024;
#pragma unroll
    for (int h = 0; h < 3; ++h) {
      const int s = s0 + h;
      // stage s has arrived: its loads are older than the ring's, and loads return in order;
      // so has everybody's behind the barrier, where the place of stage s - 1 is free
      asm volatile("s_waitcnt vmcnt(%0)" : : "n"(kLastRound ? kRing - 8 * h : kRing) : "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" : : : "memory");
      if (!kLastRound) {
        if (s + 3 < NS) stage(s + 3);
      }
      // operands are asked for kAhead k-steps ahead: one by one in front of their MFMAs, as the
      // compiler has them otherwise, each is a wait for the LDS (900 clocks a stage against 400)
      constexpr int kAhead = MT == 1 ? 6 : 2;
      const unsigned char* ap = smem + (s & 3) * kStage;
      bf16x8 a[kAhead + 1][MT];
      auto operands = [&](int k) {
#pragma unroll
        for (int i = 0; i < MT; ++i) a[k % (kAhead + 1)][i] = *reinterpret_cast<const bf16x8*>(ap + ao[k] + i * 8192);
      };
#pragma unroll
      for (int k = 0; k < kAhead; ++k) operands(k);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (k + kAhead < 8) operands(k + kAhead);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < MT; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[h * 8 + k], a[k % (kAhead + 1)][i], acc[i], 0, 0, 0);
        if (!kLastRound) wr[h * 8 + k] = weights(h * 8 + k);
      }
      asm volatile("" : : : "memory");
    }
  };
  int s0 = 0;
#pragma nounroll
  for (; s0 + 3 < NS; s0 += 3) round(s0, std::false_type{});
  round(s0, std::true_type{});
}

// Grid for the rows expected (a quarter more workgroups, and they go on to further tiles if
// there are more rows after all), and the row_bits that go with it: a launch costs about the
// bytes into the XCDs at 5 TB/s and, per CU, its tiles' operands at 110 GB/s.  tiles(rows): row tiles;
// row_bytes, part_bytes: operands of a row tile and of a part, tile_bytes: of a workgroup; cus: of the device.
template <typename Tiles>
inline dim3 few_rows_grid(int rows, int m_capacity, int parts, Tiles tiles, double row_bytes, double part_bytes,
                          double tile_bytes, int cus, int* row_bits) {
  const int m = rows > 0 && rows < m_capacity ? rows : m_capacity, t = tiles(m);
  double best = 0;
  for (int bits = 0; bits <= 3; ++bits) {
    const int rg = 1 << bits, pg = 8 >> bits;
    const long most = (long)((t + rg - 1) / rg) * ((parts + pg - 1) / pg);
    const double us = (pg * t * row_bytes + rg * parts * part_bytes) / 5e6 + (most + cus / 8 - 1) / (cus / 8) * tile_bytes / 110e3;
    if (bits == 0 || us < best) {
      best = us;
      *row_bits = bits;
    }
  }
  const int rg = 1 << *row_bits, pg = 8 >> *row_bits, more = m + m / 4 < m_capacity ? m + m / 4 : m_capacity;
  const int rows_x = (tiles(more) + rg - 1) / rg, parts_x = (parts + pg - 1) / pg;
  return dim3(8 * parts_x, rows_x);
}
inline dim3 few_rows_grid(int rows, int m_capacity, int parts, int K, int mt, int cus, int* row_bits) {
  const int bm = 32 * mt;
  return few_rows_grid(rows, m_capacity, parts, [=](int m) { return (m + bm - 1) / bm; }, 2.0 * bm * K, 256.0 * K,
                       2.0 * K * (128 + bm), cus, row_bits);
}

}  // namespace cfdetr
