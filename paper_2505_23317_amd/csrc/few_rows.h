// Contractions of few rows: what slim_residual_kernel (few_rows.hip) and
// gemm_bf16_few_kernel (gemm.hip) share.
//
// With few rows a contraction is latency and not throughput: the launch, one trip to memory
// for the rows and one for the weights.  A wavefront therefore takes 32 rows (or 64) by 32
// columns and the whole of K, a workgroup 128 columns, or 64 where every one then has a CU of its own, so that there are
// as many workgroups as the shape yields without cutting a sum; the weights, which no two wavefronts of a
// workgroup share, skip the LDS: packed 1 KB per MFMA operand they stream through a ring of
// 24 registers a lane, 48 in workgroups of two wavefronts, all of them asked for before the first row is looked at.
#pragma once
#include <type_traits>

#include "kernels.h"

namespace cfdetr {

// Which tiles a workgroup does.  Every XCD has an L2 of its own, and with few rows a good part
// of what a launch takes is its operands' way into the eight of them, so an XCD gets a
// rectangle of tiles: the row tiles are cut in 2^row_bits groups (1, 2, 4 or 8), the column parts (128 or 64
// columns, or a share of them) in 8 / that.  The grid (few_rows_grid) is a workgroup per part of a group, times eight, by the row tiles of
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
constexpr int kDeepRing = 48;      // the same of a workgroup of two wavefronts
constexpr int few_rows_lds(int mt, int waves) { return (waves == 2 ? 8 : 4) * mt * 8 * 1024; }

// acc[i] += rows m0 + 32 i .. of `rows` times the wavefront's 32 columns of weights (K / 16
// blocks from wp).  `rows`: bf16 rows [M, K], or operand blocks (kBlocks): tiles of 32 rows, one
// block of 1 KB per k-step.  They come through the LDS (few_rows_lds bytes) eight k-steps at a
// time, in four places, three stages ahead (two wavefronts, which have 48 blocks in flight: in eight, six ahead).  begin() runs when all first loads have been
// issued and sets acc.  Ends in front of a barrier that the caller has to pass before the next
// call.
template <int MT, bool kBlocks, int NW = 4, typename Begin>
__device__ __forceinline__ void few_rows_product(const bf16_t* rows, int K, int M, int m0, const unsigned char* wp,
                                                 unsigned char* smem, f32x16 (&acc)[MT], Begin begin) {
  constexpr int kRing = NW == 2 ? kDeepRing : kFewRing, kStage = MT * 8 * 1024, kLoads = 8 * MT / NW;
  constexpr int kStages = kRing / 8, kPlaces = NW == 2 ? 8 : 4;   // of a ring round, and in the LDS
  static_assert(kStages < kPlaces, "a stage's place is free before it is asked for");
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
      const uint32_t dst = (uint32_t)(uintptr_t)smem + (s & (kPlaces - 1)) * kStage + (wave * kLoads + i) * 1024;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                   : : "s"(dst), "v"(src[i] + (size_t)s * (kBlocks ? 8192 : 256)) : "memory");
    }
  };
  for (int s = 0; s < kStages; ++s) stage(s);
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
    for (int h = 0; h < kStages; ++h) {
      const int s = s0 + h;
      // stage s has arrived: its loads are older than the ring's, and loads return in order;
      // so has everybody's behind the barrier, where the place of stage s - 1 is free
      asm volatile("s_waitcnt vmcnt(%0)" : : "n"(kLastRound ? kRing - 8 * h : kRing) : "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" : : : "memory");
      if (!kLastRound) {
        if (s + kStages < NS) stage(s + kStages);
      }
      // operands are asked for kAhead k-steps ahead: one by one in front of their MFMAs, as the
      // compiler has them otherwise, each is a wait for the LDS (900 clocks a stage against 400)
      constexpr int kAhead = MT == 1 ? 6 : 2;
      const unsigned char* ap = smem + (s & (kPlaces - 1)) * kStage;
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
  for (; s0 + kStages < NS; s0 += kStages) round(s0, std::false_type{});
  round(s0, std::true_type{});
}

// How `t` row tiles of `parts` column parts are cut for the XCDs (XcdTiles): row_bits, and the tiles of the XCD
// with the most.  A launch costs about the bytes into the XCDs at 5 TB/s and, per CU, its tiles' operands at
// 110 GB/s.  row_bytes, part_bytes: operands of a row tile and of a part, tile_bytes: of a workgroup; cus: of
// the device.
struct FewCut {
  int row_bits;
  long most;
};
inline FewCut few_rows_cut(int t, int parts, double row_bytes, double part_bytes, double tile_bytes, int cus) {
  const int per_xcd = cus < 8 ? 1 : cus / 8;
  FewCut cut{};
  double best = 0;
  for (int bits = 0; bits <= 3; ++bits) {
    const int rg = 1 << bits, pg = 8 >> bits;
    const long most = (long)((t + rg - 1) / rg) * ((parts + pg - 1) / pg);
    const double us = (pg * t * row_bytes + rg * parts * part_bytes) / 5e6 + (most + per_xcd - 1) / per_xcd * tile_bytes / 110e3;
    if (bits == 0 || us < best) {
      best = us;
      cut = {bits, most};
    }
  }
  return cut;
}
// Of a contraction N x K, 32 mt rows a tile.
inline FewCut few_rows_cut(int m, int N, int K, int mt, int cus) {
  const int bm = 32 * mt;
  return few_rows_cut((m + bm - 1) / bm, N / 128, 2.0 * bm * K, 256.0 * K, 2.0 * K * (128 + bm), cus);
}

// Operands of slim_norm_kernel in bytes: of a row tile, of a workgroup's `per` parts, and of both, with the
// projection's weights where there is one (few_rows_cut).
struct SlimBytes {
  double row, part, tile;
};
inline SlimBytes slim_bytes(int d, int per, bool project) {
  return {(project ? 6.0 : 4.0) * 32 * d, 256.0 * d * per, 2.0 * d * ((project ? d : 0) + 128.0 * per)};
}

// Parts of a workgroup of slim_norm_kernel.  It streams the weights of the projection (a matrix of D rows) and
// those of its parts, and is some 200 columns' worth of stream late at the start; what counts is what the
// busiest CU of the fullest XCD has, and fewer workgroups where that is the same.  (With tiles shared out over all CUs
// instead, encoder passes of width 384, 8 layers, F = 1536: 660 rows 287 and 267 us, 1,300 rows 325 and 297, 2,600 rows
// 418 and 378, the last with slim_residual_kernel's 64 rows by the same count.)
inline int parts_of_a_share(int tiles, int parts, int d, bool project, int cus) {
  int per = parts;
  long least = 0;
  for (int n = parts; n >= 1; --n) {
    const SlimBytes b = slim_bytes(d, n, project);
    const long cut = few_rows_cut(tiles, (parts + n - 1) / n, b.row, b.part, b.tile, cus).most, per_xcd = cus < 8 ? 1 : cus / 8;
    const long most = (cut + per_xcd - 1) / per_xcd * ((project ? d : 0) + 200 + n * 128);
    if (n == parts || most < least) {
      least = most;
      per = n;
    }
  }
  return per;
}

// Grid for the rows expected: a quarter more workgroups, and they go on to further tiles if there are more
// rows after all.  tiles(rows): row tiles.
template <typename Tiles>
inline dim3 few_rows_grid(int rows, int m_capacity, int parts, Tiles tiles, double row_bytes, double part_bytes,
                          double tile_bytes, int cus, int* row_bits) {
  const int m = rows > 0 && rows < m_capacity ? rows : m_capacity, more = m + m / 4 < m_capacity ? m + m / 4 : m_capacity;
  *row_bits = few_rows_cut(tiles(m), parts, row_bytes, part_bytes, tile_bytes, cus).row_bits;
  const int rg = 1 << *row_bits, pg = 8 >> *row_bits;
  const int rows_x = (tiles(more) + rg - 1) / rg, parts_x = (parts + pg - 1) / pg;
  return dim3(8 * parts_x, rows_x);
}
inline dim3 few_rows_grid(int rows, int m_capacity, int N, int K, int mt, int waves, int cus, int* row_bits) {
  const int bm = 32 * mt, bn = 32 * waves;
  return few_rows_grid(rows, m_capacity, N / bn, [=](int m) { return (m + bm - 1) / bm; }, 2.0 * bm * K, 2.0 * bn * K,
                       2.0 * K * (bn + bm), cus, row_bits);
}

// Do workgroups of 32 rows x 64 columns leave every CU with one at most? (And is K whole rings of theirs.)
inline bool few_rows_narrow(int m, int N, int K, int cus) {
  const double row = 64.0 * K, part = 128.0 * K;   // bytes of a tile's rows and columns
  return K % (16 * kDeepRing) == 0 &&
         few_rows_cut((m + 31) / 32, N / 64, row, part, row + part, cus).most <= (cus < 8 ? 1 : cus / 8);
}
// Tiles of slim_residual_kernel for m rows of N columns: 32 mt rows by 32 `waves` columns. 64 columns as long as no CU
// gets two workgroups: a workgroup's operands are half as much to bring into its CU, and two wavefronts have the registers
// for 48 blocks on the way each (with 24 that would be lost again). In us, 128 / 64 columns: K = 1536, 920 rows 7.3 / 6.1 (a
// pass of 12 layers 457 / 442), 1,200 rows 7.7 / 6.4 (a decoder of 6 layers 438.7 / 431.0). Else 64 rows where 32 would give CUs a
// second workgroup (3,520 rows: 14 -> 9 us).
struct FewDown {
  int mt, waves;
};
inline FewDown few_rows_down(int m, int N, int K, int cus) {
  if (few_rows_narrow(m, N, K, cus)) return {1, 2};
  return {few_rows_cut(m, N, K, 1, cus).most > (cus < 8 ? 1 : cus / 8) ? 2 : 1, 4};
}

// (gemm_bf16_few_kernel takes 64 columns by the same rule. Width 768, F = 3072, passes with some 200, 350 and 700 rows: 684 / 642
// us, 727 / 699 and 762 / 745, decoders of 300 and 600 queries 475 / 450 and 494 / 469.)
// Row tiles of 32 that a workgroup of gemm_bf16_few_kernel takes for m rows of an N x K contraction (`gelu`: with that
// activation behind it), or 0: the kernels for more rows.  32 rows as long as no CU gets two workgroups, else 64 as long as none
// does, else 32 with two.  What counts is the fullest XCD: with fewer tiles than CUs it may still have more than
// its share (41 tiles of 6 parts are 33 at best).  In us, 32 rows / 64 rows / packed tiles (gemm_bf16_packed_kernel),
// N x K = 768 x 3072: 1,200 rows 13.5 / 15.7 / 24.1, 1,300 rows 20.0 / 15.9 / 24.2, 2,200 rows 22.5 / 19.0 / 24.7, 2,600
// rows 23.6 / 28.9 / 25.1, 2,700 rows 31.0 / 30.4 / 25.4; 768 x 768: 1,200 rows 5.6 / 7.1 / 9.0, 2,200 rows 8.5 / 7.7 /
// 9.4, 2,600 rows 9.1 / 12.6 / 9.8, 2,700 rows 11.1 / 12.2 / 10.0.  q/k/v of width 384 (1152 x 384), this and tiles with the
// weights through the LDS: 700 rows 4.0 (32) and 5.9, 1,420 rows 5.2 (64) and 6.4, 2,000 rows 7.1 and 6.9.
// At width 768 what follows a LayerNorm comes here only as long as no CU gets two workgroups of 32 rows; behind that it is one
// launch with the LayerNorm (norm_cut) or a packed tile.  2304 x 768, 300 rows: 5.1 / 6.2 / 8.2.
// Then 64 rows with two workgroups a CU
//  - where the activation is behind it, which a tile of 64 x 256 does with half as many wavefronts: 2304 x 384 (feed-forward
//    widths past the layer kernel's), 1,420 rows 9.9 / 8.2 / 11.6;
//  - where the packed tiles do not fit (N no multiple of 256; the third figure is then for tiles with the weights through the LDS)
//    over a long K and the CUs are three quarters full: 384 x 3072: 6,400 rows 31.9 / 31.4 / 28.7, 8,500 rows
//    42.1 / 31.6 / 36.1, 10,700 rows 46.0 / 34.6 / 39.6, 10,900 rows 51.3 / 44.5 / 39.5.
inline int few_rows_tiles(int m, int N, int K, bool gelu, int cus) {
  const long per_xcd = cus < 8 ? 1 : cus / 8;
  const long most1 = few_rows_cut(m, N, K, 1, cus).most, most2 = few_rows_cut(m, N, K, 2, cus).most;
  if (most1 <= per_xcd) return 1;
  if (most2 <= per_xcd) return 2;
  if (most1 <= 2 * per_xcd) return 1;
  if (most2 <= 2 * per_xcd && ((gelu && N >= 2304) || (N % 256 != 0 && K >= 2048 && 2 * most2 > 3 * per_xcd))) return 2;
  return 0;
}

// How a LayerNorm and the contraction behind it (gemm_bf16_norm_kernel, width 768) are cut for `rows` rows and N
// columns: 32 mt rows by per_share strips of 32 columns a workgroup, the shares in 2^group_bits groups, each done by as
// many XCDs as there are for a group, and there tile by tile in runs of equal length. A CU holds one workgroup, so one
// round of them is all there may be (with a second one two launches are faster); eight strips are a round of a workgroup's
// wavefronts and take 5 us with 32 rows, 6.5 with 64, behind 4 and 8.5 us of launch, rows and LayerNorm. In us, the cuts mt /
// shares for 1,300 rows: q/k/v 1/4 13.8, 1/6 11.9, 2/9 14.4, 2/12 13.9; N = 3072 1/4 16.3, 1/6 14.1, 2/9 17.5, 2/12 14.8;
// 2,600 rows: q/k/v 1/2 23.7, 1/3 19.9, 2/4 23.0, 2/6 19.6; N = 3072 1/3 24.4, 2/4 25.1, 2/6 22.4; N = 1152, 1,200 rows 1/4 9.8
// (nine strips: two rounds), 1/5 8.5. Beyond four rounds it no longer gains: 3,200 rows in two shares 24.9 and 32.0, and two
// launches 25.3 and 30.7.
// Most rows: N = 384 and 768 16,384, 1152 to 1920 8,192, 2304 to 3072 5,440, 4608 some 3,200. Two launches / one near them:
// N = 384, 16,300 rows 28.3 / 21.2; 768, 8,100 rows 21.1 / 18.4, 16,300 rows 33.6 / 28.9; 1152, 8,100 rows 31.9 / 25.0; 1536 31.2 /
// 29.1; 1920 38.1 / 34.6; 2304, 5,400 rows 31.7 / 28.0; 3072 38.2 / 34.5; 4608, 2,400 rows 29.7 / 26.2, 3,200 rows 32.9 / 32.8.
// Fewest: as long as workgroups of 32 rows x 128 columns leave every CU with one at most, two launches are faster, whose weights
// are all on their way before the first row is looked at. Passes with two / one for that contraction, us, one context over
// and over, and three in turn, which find their weights in memory: q/k/v, 12 layers, up to 384 rows: 64 rows 407 / 421 and 484 /
// 527, 288 rows 483 / 488 and 566 / 583, 400 rows 543 / 520 and 617 / 612, 480 rows 535 / 511 and 614 / 608; N = 3072, up to 320
// rows: 288 rows 483 / 488 and 566 / 582, 324 rows 507 / 497 and 583 / 581, 480 rows 535 / 508 and 614 / 599; N = 1536, up to 640
// rows: 400 rows 495 / 499 and 554 / 569, 720 rows 547 / 534 and 632 / 626; N = 1152, up to 768 rows: 480 rows 496 / 498 and 566 /
// 579, 918 rows 570 / 551 and 672 / 664; N = 768, six layers of a decoder, up to 1,280 rows: 600 rows 416 / 427 and 459 / 472, 1,200
// rows 525 / 521 and 600 / 602, 1,500 rows 603 / 589 and 667 / 663.
constexpr int kNormWidth = 768, kNormRounds = 4;
struct NormCut {
  int mt = 0;   // 0: no cut
  int shares, per_share, group_bits;
};
// Workgroups of an XCD.
inline int norm_units(int rows, int mt, int shares, int group_bits) {
  const int g = 1 << group_bits, units = (rows + 32 * mt - 1) / (32 * mt) * ((shares + g - 1) / g);
  return (units + (8 >> group_bits) - 1) / (8 >> group_bits);
}
inline NormCut norm_cut(int rows, int N, int cus) {
  const int strips = N / 32, per_xcd = cus < 8 ? 1 : cus / 8;
  NormCut best;
  if (few_rows_cut(rows, N, kNormWidth, 1, cus).most <= per_xcd) return best;
  double least = 0;
  for (int mt = 1; mt <= 2; ++mt)
    for (int want = 1; want <= (strips + 7) / 8; ++want) {
      const int per = (strips + want - 1) / want, shares = (strips + per - 1) / per, rounds = (per + 7) / 8;
      if (rounds > kNormRounds) continue;
      for (int bits = 0; bits <= 3; ++bits) {
        if (norm_units(rows, mt, shares, bits) > per_xcd) continue;
        // operands into the XCDs: the matrix once for each XCD of a group, the rows once for each group
        const double bytes = 2.0 * kNormWidth * N * (8 >> bits) + 4.0 * kNormWidth * rows * (1 << bits);
        const double us = (mt == 1 ? 4 + 5 * rounds : 8.5 + 6.5 * rounds) + 0.1 * per + bytes / 50e6;
        if (best.mt == 0 || us < least) {
          least = us;
          best.mt = mt;
          best.shares = shares;
          best.per_share = per;
          best.group_bits = bits;
        }
      }
    }
  return best;
}

// Are the weights behind an attention launch asked for during it (read_ahead, attention.hip), at width 768 with q/k/v behind their
// LayerNorm in one launch? From 2.5 rows a CU on: with fewer the attention is over before they have come. Passes in us,
// without / with, one context over and over, and three in turn: 12 layers, F = 3072, 400 rows 516 / 536 and 620 / 624, 576 rows
// 510 / 541 and 618 / 630, 720 rows 592 / 627 and 738 / 717, 1,200 rows 696 / 691 and 852 / 777, 2,000 rows 1,002 / 970 and 1,047 /
// 1,005, 5,200 rows 1,755 / 1,656 and 1,758 / 1,662; F = 1536, 576 rows 473 / 492 and 553 / 563, 720 rows 533 / 531 and 642 / 611;
// decoders of 6 layers, 600 rows 387 / 408 and 447 / 455, 900 rows 454 / 473 and 540 / 520, 1,200 rows 476 / 489 and 581 / 547,
// 4,800 rows 992 / 1,007 and 1,111 / 1,051: a decoder alone on the chip pays 1.5 to 4 % for the 4 to 6 % of several.
inline bool norm_reads_ahead(int rows, int cus) { return 2 * rows > 5 * cus; }

}  // namespace cfdetr
