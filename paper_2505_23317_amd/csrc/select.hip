// A2 of CF-DETR (Sec. III-B): which cells are re-partitioned into finer patches,
// and the ordered token table that results.  Integer work only.
//
// Split rule: a cell of a non-finest level l is replaced by its four children iff
// a box of the same frame with tier > l overlaps it.  Such a box then also overlaps
// every ancestor of the cell with a tier above the ancestor's level, so a "hit"
// cell always has split ancestors.  Two consequences used here:
//   * a cell (l, r, c) is a token iff (l == 0 or its parent is hit) and
//     (l == finest or it is not hit itself): no recursion needed;
//   * a frame has N0 + 3 * (number of hit cells) tokens, and 4*S(l-1) - S(l) of them
//     at level l, with S(l) the hit cells of level l, S(finest) = 0, 4*S(-1) := N0.
// One kernel (select_kernel) as long as a bit per non-finest cell of all frames fits the LDS.
// Larger pyramids take two: kernel 1 tests every non-finest cell against the boxes of its
// frame (kBoxLanes threads share a cell, each taking every kBoxLanes-th box) and raises the
// cell's flag; kernel 2 counts the flags of all frames (offsets), then compacts the tokens
// of its own frame with wavefront ballots and popcount prefix sums, and clears the
// flag array that the NEXT call will use (two arrays alternate), so no memset is
// ever needed.
#include "kernels.h"

namespace cfdetr {

namespace {

constexpr int kHitThreads = 256;
constexpr int kBoxLanes = 8;
constexpr int kCompactThreads = 1024;

__global__ __launch_bounds__(kHitThreads) void select_hit_kernel(
    Pyramid pyr, const int32_t* __restrict__ boxes, const uint8_t* __restrict__ tier,
    const int32_t* __restrict__ box_offsets, int nonfinest, uint8_t* __restrict__ hit) {
  const int frame = blockIdx.y;
  const int cell = blockIdx.x * (kHitThreads / kBoxLanes) + threadIdx.x / kBoxLanes;
  const int boxlane = threadIdx.x % kBoxLanes;
  if (cell >= nonfinest) return;
  int id = cell, level = 0;
  while (id >= pyr.rows[level] * pyr.cols[level]) {
    id -= pyr.rows[level] * pyr.cols[level];
    ++level;
  }
  const int P = pyr.patch[level];
  const int row = id / pyr.cols[level], col = id % pyr.cols[level];
  const int cx0 = col * P, cx1 = cx0 + P, cy0 = row * P, cy1 = cy0 + P;
  const int lo = box_offsets[frame], hi = box_offsets[frame + 1];
  bool flag = false;
  for (int b = lo + boxlane; b < hi; b += kBoxLanes) {
    const int4 raw = *reinterpret_cast<const int4*>(boxes + 4 * (size_t)b);
    const int x0 = max(raw.x, 0), y0 = max(raw.y, 0);
    const int x1 = min(raw.z, pyr.img_w), y1 = min(raw.w, pyr.img_h);
    const bool nonempty = (x1 > x0) && (y1 > y0);
    flag |= nonempty && ((int)tier[b] > level) && (x0 < cx1) && (x1 > cx0) && (y0 < cy1) &&
            (y1 > cy0);
  }
  if (flag) hit[(size_t)frame * nonfinest + cell] = 1;   // several lanes may write the same 1
}

// Sequence list of one encoder run, and the attention work list over it.
// The sequences are `n_prefix` sequences of `prefix_len` tokens each (the coarse grids
// of a merged coarse+mixed run; n_prefix may be 0) followed by the B sequences that
// cu[0..B] delimits.  Outputs:
//   cu_all[0..nseq]  offsets of all sequences, m_all = their total
//   pcu[0..nseq]     offsets when every sequence is padded to a multiple of 64
//   items[0..8*cap8) attention work items of four words: sequence<<24 | head<<19 | query
//                    tile (or -1: no item), then the sequence's offset, length and padded
//                    offset, so that a workgroup gets all it needs to start in one load.
// Workgroups are dealt to the 8 XCDs round-robin (workgroup w runs on XCD w % 8), and
// every XCD has its own L2.  Sequences come longest first, and the items of those of as many
// tiles, sequence by sequence and head by head, are cut into eight runs of equal length, one for every XCD (whose
// workgroups 8*j + x take its run in order): all XCDs get the same work of every length, and an XCD
// reads the keys and values of an eighth of the heads and one or two more.  What
// does not divide by eight goes to the XCDs in turn, so the queues differ by one entry in
// all.  Whole (sequence, head) groups dealt to the XCDs read the least, but leave the fullest
// of them with 1.2 times the average where lengths are mixed: attention over four coarse
// grids of 1,600 tokens and sets of 5,803, 3,433, 4,612 and 2,257 (6 heads of 64) 132.5 us so,
// 115.8 in runs; sets of 3,000 to 6,000 153 and 137, twelve of 1,200 to 4,000 88 and 82; eight
// of 6,400, four of 6,400, eight of 3,200 or of 2,560 and 24 of 256 to 1,435 the same.
// The first entries of a queue, one for each CU of its XCD (p.round), are in turned order where there are more: CUs take
// a workgroup each before any takes a second, so the shortest of them share their CU with the longest of the next,
// and of 53 entries for 32 CUs the 11 longest have one to themselves.  In us, longest first throughout / so: six cameras
// (8 heads of 32, 640 to 1,300 tokens, 50 items an XCD) 262 / 254 a pass, one camera 205 / 203, two stages of six 836 /
// 822; sets of equal or far more items the same.
// Sequences of as many tiles share a cut, so that an XCD has whole heads of one of them and not an eighth of each: two
// stages of six cameras (decoders among them) 825 us a pass by sequences, 807 by such classes, six cameras 258 / 256, eight
// high-resolution frames of equal length 0.15 to 0.3 %.
// gated: no item at all.  The items are then not written (and not only counted as none): there
// is no barrier between the two loops over the entries, so where both wrote one, either could
// be the last, and an item that is left sends a workgroup to a sequence without keys.
// Inclusive sum over the lanes of a wavefront: inside the rows of 16 lanes, then the last lane
// of row 0 and 2 to the row behind, then that of row 1 to the upper half.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
  return v;
}

__device__ __forceinline__ int last_lane(int v) { return __builtin_amdgcn_readlane(v, kWave - 1); }

// The plan proper: the lengths of the nseq sequences are in s_len (shared, published by a
// barrier); all threads of a workgroup of at least 2 * kMaxBatch threads call it.
__device__ __forceinline__ void plan_body(const PlanArgs& p, int nseq, const int* s_len, bool gated) {
  // items of the sequences of more query tiles, of those of as many, and of the latter in front of this sequence's
  __shared__ int s_before[2 * kMaxBatch], s_class[2 * kMaxBatch], s_within[2 * kMaxBatch];
  __shared__ int s_count[8];
  __shared__ int s_cu[2 * kMaxBatch + 1], s_pcu[2 * kMaxBatch + 1];
  const int tid = threadIdx.x;
  // (no integer divisions: the kernel's time is latency, the way of its code to the CU included)
  const int heads = p.heads, cap8 = p.cap8, log_q = 31 - __clz(p.block_q);   // block_q: a power of two
  auto tiles = [&](int f) { return (s_len[f] + p.block_q - 1) >> log_q; };
  // XCD x's part of n items: an eighth, and one more for each of the n % 8 XCDs from `turn` on; `first` is the number
  // of those that the XCDs in front of it get.  With `turn` the items in front of these, modulo 8, XCD x has
  // (items >> 3) + (x < items % 8) of `items` items dealt so far.
  auto run_of = [&](int n, int turn, int x, int& first) {
    const int rest = n & 7, end = turn + rest;
    first = x * (n >> 3) + max(min(end, x) - turn, 0) + max(min(end - 8, x), 0);
    return (n >> 3) + (((x - turn) & 7) < rest ? 1 : 0);
  };
  auto dealt = [&](int items, int x) { return (items >> 3) + (x < (items & 7) ? 1 : 0); };
  int4* const items4 = reinterpret_cast<int4*>(p.items);
  if (tid < max(nseq, 8)) {
    const int len = tid < nseq ? s_len[tid] : 0, nt = (len + p.block_q - 1) >> log_q;
    int before = 0, of_class = 0, within = 0, all = 0;
    for (int j = 0; j < nseq; ++j) {
      const int lj = s_len[j], tj = tiles(j), n = heads * tj;
      all += n;
      before += tj > nt ? n : 0;
      of_class += tj == nt ? n : 0;
      within += tj == nt && (lj > len || (lj == len && j < tid)) ? n : 0;
    }
    if (tid < nseq) {
      s_before[tid] = before;
      s_class[tid] = of_class;
      s_within[tid] = within;
    }
    if (tid < 8) s_count[tid] = gated ? 0 : min(dealt(all, tid), cap8);
  }
  const int lane = tid & (kWave - 1), wave = tid / kWave, waves = blockDim.x / kWave;
  if (wave == waves - 1) {
    int pos = 0, ppos = 0;
    for (int i0 = 0; i0 < nseq; i0 += kWave) {
      const int i = i0 + lane;
      const int len = i < nseq ? s_len[i] : 0, plen = (len + 63) & ~63;
      const int end = wave_scan(len), pend = wave_scan(plen);
      if (i < nseq) {
        s_cu[i] = pos + end - len;
        s_pcu[i] = ppos + pend - plen;
      }
      pos += last_lane(end);
      ppos += last_lane(pend);
    }
    if (lane == 0) {
      s_cu[nseq] = pos;
      s_pcu[nseq] = ppos;
    }
  }
  __syncthreads();
  // (stores behind the barrier, which would wait for them; m_seen is in host memory)
  for (int i = tid; i <= nseq; i += blockDim.x) {
    p.cu_all[i] = s_cu[i];
    p.pcu[i] = s_pcu[i];
  }
  if (tid == 0) {
    *p.m_all = s_cu[nseq];
    if (p.m_seen != nullptr) *p.m_seen = s_cu[nseq];
  }
  for (int u = tid; !gated && u < nseq * 64; u += blockDim.x) {   // eight threads for a sequence's part of a run
    const int f = u >> 6, x = (u >> 3) & 7, nt = tiles(f), before = s_before[f], own = s_within[f];
    int first;
    const int n = run_of(s_class[f], before & 7, x, first), at = dealt(before, x) - first;   // of the class; its place
    const int i1 = min(min(first + n, own + heads * nt), cap8 - at);
    const int turned = s_count[x] > p.round ? p.round : 0;   // entries
    const float rcp = __builtin_amdgcn_rcpf((float)max(nt, 1));
    for (int i = max(first, own) + (u & 7); i < i1; i += 8) {
      const int item = i - own, j = at + i;
      int h = (int)((float)item * rcp);   // item / nt, or one off
      h += (h + 1) * nt <= item ? 1 : h * nt > item ? -1 : 0;
      items4[8 * (j < turned ? turned - 1 - j : j) + x] = make_int4((f << 24) | (h << 19) | (item - h * nt), s_cu[f], s_len[f], s_pcu[f]);
    }
  }
  for (int i = tid; i < 8 * cap8; i += blockDim.x)
    if ((i >> 3) >= s_count[i & 7]) items4[i] = make_int4(-1, 0, 0, 0);
  // fetch counters: behind the entries handed out by workgroup index, or -1 where those
  // are the whole queue (nothing to fetch: a workgroup need not ask)
  for (int i = tid; i < p.n_heads_q; i += blockDim.x)
    p.queue_heads[i] = s_count[i & 7] <= p.queue_start ? -1 : p.queue_start;
}

__global__ __launch_bounds__(256) void plan_kernel(const int32_t* __restrict__ cu, int B, PlanArgs p,
                                                   int max_total, int32_t* __restrict__ err_flag) {
  __shared__ int s_len[2 * kMaxBatch];
  const int tid = threadIdx.x;
  const int nseq = p.n_prefix + B;
  if (tid < nseq) s_len[tid] = tid < p.n_prefix ? p.prefix_len : cu[tid - p.n_prefix + 1] - cu[tid - p.n_prefix];
  __syncthreads();
  if (max_total > 0) {
    // offsets a caller wrote: no length may be negative and the total must fit;
    // otherwise the caller's sequences all get length 0 (nothing of them is computed or
    // written) and the error flag is raised
    if (tid == 0) {
      long long pos = 0;
      bool bad = false;
      for (int i = p.n_prefix; i < nseq; ++i) {
        const int len = s_len[i];
        if (len < 0) bad = true;
        pos += len > 0 ? len : 0;
      }
      if (pos > (long long)max_total) bad = true;
      if (bad) {
        for (int i = p.n_prefix; i < nseq; ++i) s_len[i] = 0;
        *err_flag = 1;
      }
    }
    __syncthreads();
  }
  plan_body(p, nseq, s_len, false);
}

// What a decoder run needs before its first layer, in one launch: the plan of the token sequences, whose offsets
// a caller wrote and every workgroup checks for itself (lengths of at least 1 that fit max_total; otherwise none is left
// and the error flag is raised), the plan of the queries, Q of every frame (no work after an error, this one or an
// earlier one), and the tokens in bf16.  As three launches, one behind the other, 13.5 us for 6,400 tokens of width 384;
// like this 6.4.
__global__ __launch_bounds__(256) void decode_plan_kernel(const int32_t* __restrict__ cu, int B, PlanArgs tokens, PlanArgs queries,
                                                          int Q, int max_total, int32_t* err_flag,
                                                          const float* __restrict__ memory, bf16_t* __restrict__ out, int d) {
  __shared__ int s_len[2 * kMaxBatch];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  static_assert(kMaxBatch <= kWave, "a sequence a lane");
  const int len = lane < B ? cu[lane + 1] - cu[lane] : 1;
  const int has = lane < B && len > 0 ? len : 0;
  const long long total = ((long long)last_lane(wave_scan(has >> 16)) << 16) + last_lane(wave_scan(has & 0xFFFF));
  const bool bad = __ballot(len < 1) != 0 || total > (long long)max_total;
  if (blockIdx.x == 0) {
    if (tid < B) s_len[tid] = bad ? 0 : len;
    if (tid == 0 && bad) *err_flag = 1;
    __syncthreads();
    plan_body(tokens, B, s_len, false);
  } else if (blockIdx.x == 1) {
    if (tid < B) s_len[tid] = Q;
    __syncthreads();
    plan_body(queries, B, s_len, bad || *err_flag != 0);
  } else {
    const size_t n = bad ? 0 : (size_t)total * d;   // d is a multiple of 64, so n is a multiple of 8
    const size_t i = ((size_t)(blockIdx.x - 2) * blockDim.x + tid) * 8;
    if (i >= n) return;
    const float4 a = *reinterpret_cast<const float4*>(memory + i), b = *reinterpret_cast<const float4*>(memory + i + 4);
    *reinterpret_cast<uint4*>(out + i) =
        make_uint4(pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w), pack_bf16x2(b.x, b.y), pack_bf16x2(b.z, b.w));
  }
}

__global__ __launch_bounds__(kCompactThreads) void select_compact_kernel(
    Pyramid pyr, int B, int nonfinest, const uint8_t* __restrict__ hit,
    uint8_t* __restrict__ hit_next, int hit_bytes, int max_tokens,
    int32_t* __restrict__ tok_desc,
    int32_t* __restrict__ cu_seqlens, int32_t* __restrict__ level_counts,
    int32_t* __restrict__ err_flag, const int32_t* __restrict__ hard, PlanArgs plan) {
  __shared__ int s_split[kMaxBatch][kMaxLevels];   // hit cells per (frame, level)
  __shared__ int s_wave[kCompactThreads / kWave];
  // Workgroup B, if there is one (plan.items set), compacts nothing: the lengths that every
  // workgroup works out for its offset are all the attention plan needs, so it makes that
  // plan while the others compact, and the encoder that follows has no launch for it.
  const int frame = blockIdx.x;
  const int tid = threadIdx.x;
  const int n = pyr.n_levels;
  const int lane = tid & (kWave - 1), wave = tid / kWave;

  // hit cells of every frame and level (each workgroup needs all of them for its offset)
  for (int i = tid; i < kMaxBatch * kMaxLevels; i += kCompactThreads) (&s_split[0][0])[i] = 0;
  __syncthreads();
  {
    int bound[kMaxLevels];   // end of level l inside one frame's flag array
    int acc = 0;
    for (int l = 0; l < kMaxLevels; ++l) {
      if (l + 1 < n) acc += pyr.rows[l] * pyr.cols[l];
      bound[l] = acc;
    }
    const int total = B * nonfinest;
    for (int start = 0; start < total; start += kCompactThreads) {
      const int i = start + tid;
      int f = 0, l = 0;
      bool h = false;
      if (i < total) {
        f = i / nonfinest;
        const int c = i - f * nonfinest;
        while (c >= bound[l]) ++l;
        h = hit[i] != 0;
      }
      // frames and levels change rarely inside a wavefront: vote per (frame, level) of lane 0
      // and let the few stragglers add on their own
      const int f0 = __shfl(f, 0, kWave), l0 = __shfl(l, 0, kWave);
      const bool same = (f == f0) && (l == l0);
      const unsigned long long m = __ballot(h && same);
      if (lane == 0 && m != 0) atomicAdd(&s_split[f0][l0], __popcll(m));
      if (h && !same) atomicAdd(&s_split[f][l], 1);
    }
  }
  __syncthreads();
  // A frame marked easy (hard given and 0 for it) has no fine stage: no token at all.
  long long total_tokens = 0;
  int base = 0;
  for (int j = 0; j < B; ++j) {
    int sj = 0;
    for (int l = 0; l + 1 < n; ++l) sj += s_split[j][l];
    const int tj = (hard != nullptr && hard[j] == 0) ? 0 : pyr.rows[0] * pyr.cols[0] + 3 * sj;
    if (j < frame) base += tj;
    total_tokens += tj;
  }
  if (frame >= B) {
    __shared__ int s_len[2 * kMaxBatch];
    const bool too_many = total_tokens > (long long)max_tokens;   // then every length is 0
    if (tid < plan.n_prefix + B) {
      int len = plan.prefix_len;
      if (tid >= plan.n_prefix) {
        int sj = 0;
        for (int l = 0; l + 1 < n; ++l) sj += s_split[tid - plan.n_prefix][l];
        len = too_many ? 0 : pyr.rows[0] * pyr.cols[0] + 3 * sj;
        if (hard != nullptr && hard[tid - plan.n_prefix] == 0) len = 0;
      }
      s_len[tid] = len;
    }
    __syncthreads();
    plan_body(plan, plan.n_prefix + B, s_len, false);
    return;
  }
  // The flag array of the call after this one starts from zero: all of it (that call
  // may have more frames than this one), shared out among the workgroups.
  {
    const int share = (hit_bytes + B - 1) / B;
    const int lo = frame * share, hi = min(lo + share, hit_bytes);
    for (int i = lo + tid; i < hi; i += kCompactThreads) hit_next[i] = 0;
  }
  const bool overflow = total_tokens > (long long)max_tokens;
  const bool skipped = hard != nullptr && hard[frame] == 0;
  if (tid == 0) {
    cu_seqlens[frame] = overflow ? 0 : base;
    if (frame == B - 1) cu_seqlens[B] = overflow ? 0 : (int)total_tokens;
    if (overflow && frame == 0) *err_flag = 1;
  }
  if (level_counts != nullptr && tid < n) {
    const int prev4 = tid == 0 ? pyr.rows[0] * pyr.cols[0] : 4 * s_split[frame][tid - 1];
    const int cur = (tid + 1 < n) ? s_split[frame][tid] : 0;
    level_counts[frame * n + tid] = (overflow || skipped) ? 0 : prev4 - cur;
  }
  if (overflow || skipped) return;

  const uint8_t* fhit = hit + (size_t)frame * nonfinest;
  int running = base;
  int off_prev = 0, off_cur = 0;  // start of level l-1 / level l inside the flag array
  for (int l = 0; l < n; ++l) {
    const int rows = pyr.rows[l], cols = pyr.cols[l], nl = rows * cols;
    const int pcols = (l > 0) ? pyr.cols[l - 1] : 0;
    for (int start = 0; start < nl; start += kCompactThreads) {
      const int id = start + tid;
      bool leaf = false;
      int row = 0, col = 0;
      if (id < nl) {
        row = id / cols;
        col = id - row * cols;
        bool parent_ok = (l == 0) || fhit[off_prev + (row >> 1) * pcols + (col >> 1)];
        bool self_split = (l + 1 < n) && fhit[off_cur + id];
        leaf = parent_ok && !self_split;
      }
      unsigned long long m = __ballot(leaf);
      int before = __popcll(m & ((1ull << lane) - 1ull));
      if (lane == 0) s_wave[wave] = __popcll(m);
      __syncthreads();
      int wave_off = 0, chunk = 0;
      for (int w = 0; w < kCompactThreads / kWave; ++w) {
        int c = s_wave[w];
        if (w < wave) wave_off += c;
        chunk += c;
      }
      if (leaf) tok_desc[running + wave_off + before] = (l << 28) | (row << 14) | col;
      running += chunk;
      __syncthreads();
    }
    off_prev = off_cur;
    off_cur += nl;
  }
}

// The bit maps of one frame: 32 columns a word, rows of whole words, level after level.
__host__ __device__ inline int row_words(const Pyramid& pyr, int level) { return (pyr.cols[level] + 31) >> 5; }

// 16 bits to 32, every bit twice (a parent's columns to its children's).
__device__ __forceinline__ uint32_t twice(uint32_t x) {
  x = (x | (x << 8)) & 0x00ff00ffu;
  x = (x | (x << 4)) & 0x0f0f0f0fu;
  x = (x | (x << 2)) & 0x33333333u;
  x = (x | (x << 1)) & 0x55555555u;
  return x | (x << 1);
}

// The whole selection: workgroup f does frame f, workgroup B (if there) makes the plan.
// A token's place depends on all frames, so every workgroup needs the hit cells of all of
// them, and two kernels with the flags in memory between them spent their time on launches
// and on memory's latency (a trip per 1024 cells).  Painting the boxes is cheap enough to do
// in every workgroup instead: up to eight lanes a box, one row each, an OR per 32 cells into a bit
// map in LDS.  Eight lanes halve the time of few boxes and do most of a box's work eight times, so
// there are fewer the more boxes the frame has, and the next box is on its way while one is painted.  Counts are popcounts of words; the tokens of a level's word are the children of
// the parents' bits without the word's own, so one scan over the words of the frame gives
// every token its place.
// Measured, two kernels / this one: six frames of 640 x 640 10.4 / 7.8 us, twelve of three
// levels at 1024 x 1024 with the plan 28 / 9 us; with 300 boxes a frame 64 frames of 640 x 640
// 43.0 / 21.6 us (eight lanes a box throughout 76.7), of 320 x 320 32.4 / 21.0 (76.1).  What counts is the frame's own
// number, for its own threads paint its boxes: 64 frames, 512 boxes in one of them, 22.0 us, and 90.1 by all frames' boxes.
constexpr int kPaintTrips = 4;          // boxes a lane paints before a box gets fewer lanes
constexpr int kSelectLds = 96 * 1024;   // most of its dynamic LDS (the plan's tables take 20 KB)

__global__ __launch_bounds__(kCompactThreads) void select_kernel(
    Pyramid pyr, const int32_t* __restrict__ boxes, const uint8_t* __restrict__ tier,
    const int32_t* __restrict__ box_offsets, int B, int frame_words, int leaf_words, int max_tokens,
    int32_t* __restrict__ tok_desc, int32_t* __restrict__ cu_seqlens, int32_t* __restrict__ level_counts,
    int32_t* __restrict__ err_flag, const int32_t* __restrict__ hard, PlanArgs plan) {
  extern __shared__ uint32_t s_select[];
  uint32_t* const s_bits = s_select;                        // [B][frame_words] hit cells
  uint32_t* const s_leaf = s_bits + B * frame_words;        // [leaf_words] tokens of this frame,
  int* const s_before = reinterpret_cast<int*>(s_leaf + leaf_words);   // those in front of the word,
  int* const s_desc = s_before + leaf_words;                // descriptor of its first column
  __shared__ int s_split[kMaxBatch][kMaxLevels];            // hit cells per (frame, level)
  __shared__ int s_wave[kCompactThreads / kWave];
  const int frame = blockIdx.x, tid = threadIdx.x, n = pyr.n_levels;
  const int lane = tid & (kWave - 1), wave = tid / kWave;

  // threads of a frame: 1024 over the next power of two of B
  const int per_frame = kCompactThreads >> (B > 1 ? 32 - __clz(B - 1) : 0);
  const int pf = tid / per_frame;
  int lo = 0, hi = 0;
  if (pf < B) {
    lo = box_offsets[pf];
    hi = box_offsets[pf + 1];
  }
  const bool easy = hard != nullptr && lane < B && hard[lane] == 0;
  for (int i = tid; i < B * frame_words; i += kCompactThreads) s_bits[i] = 0;
  for (int i = tid; i < kMaxBatch * kMaxLevels; i += kCompactThreads) (&s_split[0][0])[i] = 0;
  __syncthreads();
  // the most of eight, four, two and one with which the frame's boxes are kPaintTrips to a lane and fewer
  const int log_share = 31 - __clz(kPaintTrips * per_frame), log_boxes = 32 - __clz(max(hi - lo, 1) - 1);
  const int log_lanes = min(max(log_share - log_boxes, 0), 3);
  const int lanes = 1 << log_lanes, stride = per_frame >> log_lanes;
  int b = lo + ((tid & (per_frame - 1)) >> log_lanes);
  int4 next = make_int4(0, 0, 0, 0);
  int next_tier = 0;
  auto fetch = [&]() {
    if (b < hi) {
      next = *reinterpret_cast<const int4*>(boxes + 4 * (size_t)b);
      next_tier = tier[b];
    }
  };
  fetch();
  while (b < hi) {
    const int4 raw = next;
    const int levels = min(next_tier, n - 1);   // those that the box splits
    b += stride;
    fetch();
    const int x0 = max(raw.x, 0), y0 = max(raw.y, 0);
    const int x1 = min(raw.z, pyr.img_w), y1 = min(raw.w, pyr.img_h);
    if (x1 <= x0 || y1 <= y0) continue;
    uint32_t* map = s_bits + pf * frame_words;
    for (int l = 0; l < levels; ++l) {
      const int shift = __ffs(pyr.patch[l]) - 1, words = row_words(pyr, l);
      const int c0 = x0 >> shift, c1 = (x1 - 1) >> shift, r1 = (y1 - 1) >> shift;
      for (int r = (y0 >> shift) + (tid & (lanes - 1)); r <= r1; r += lanes)
        for (int w = c0 >> 5; w <= c1 >> 5; ++w) {
          const uint32_t from = w == c0 >> 5 ? ~0u << (c0 & 31) : ~0u;
          const uint32_t to = w == c1 >> 5 ? ~0u >> (31 - (c1 & 31)) : ~0u;
          atomicOr(&map[r * words + w], from & to);
        }
      map += pyr.rows[l] * words;
    }
  }
  __syncthreads();
  const int words0 = pyr.rows[0] * row_words(pyr, 0);   // of the coarsest level
  for (int i = tid; i < B * frame_words; i += kCompactThreads) {
    const int hits = __popc(s_bits[i]);
    if (hits) {
      const int f = i / frame_words;
      atomicAdd(&s_split[f][i - f * frame_words >= words0 ? 1 : 0], hits);
    }
  }
  if (frame < B) {
    const uint32_t* const map = s_bits + frame * frame_words;
    int running = 0;
    for (int start = 0; start < leaf_words; start += kCompactThreads) {
      const int i = start + tid;
      uint32_t leaf = 0;
      if (i < leaf_words) {
        int l = 0, first = 0, before = 0;   // level, its first word, the first of the level before
        while (i >= first + pyr.rows[l] * row_words(pyr, l)) {
          before = first;
          first += pyr.rows[l] * row_words(pyr, l);
          ++l;
        }
        const int words = row_words(pyr, l), row = (i - first) / words, w = (i - first) - row * words;
        const int rest = pyr.cols[l] - w * 32;
        leaf = rest < 32 ? (1u << rest) - 1 : ~0u;
        if (l > 0) leaf &= twice((map[before + (row >> 1) * row_words(pyr, l - 1) + (w >> 1)] >> (16 * (w & 1))) & 0xffffu);
        if (l + 1 < n) leaf &= ~map[i];
        s_leaf[i] = leaf;
        s_desc[i] = (l << 28) | (row << 14) | (w * 32);
      }
      const int mine = __popc(leaf), end = wave_scan(mine);
      if (lane == kWave - 1) s_wave[wave] = end;
      __syncthreads();
      int wave_off = 0, chunk = 0;
      for (int w = 0; w < kCompactThreads / kWave; ++w) {
        const int c = s_wave[w];
        if (w < wave) wave_off += c;
        chunk += c;
      }
      if (i < leaf_words) s_before[i] = running + wave_off + end - mine;
      running += chunk;
      __syncthreads();
    }
  } else {
    __syncthreads();
  }
  // tokens of frame `lane` (kMaxBatch is a wavefront), and those in front of it.  A frame
  // marked easy (hard given and 0 for it) has no fine stage: no token at all.
  int tokens = 0;
  if (lane < B && !easy) {
    tokens = pyr.rows[0] * pyr.cols[0];
    for (int l = 0; l + 1 < n; ++l) tokens += 3 * s_split[lane][l];
  }
  const int lower = wave_scan(tokens & 0xffff), upper = wave_scan(tokens >> 16);   // (the sum may pass 32 bits)
  const long long total = ((long long)last_lane(upper) << 16) + last_lane(lower);
  const bool overflow = total > (long long)max_tokens;   // then every length is 0
  if (frame >= B) {
    __shared__ int s_len[2 * kMaxBatch];
    if (wave == 0) {
      for (int i = lane; i < plan.n_prefix; i += kWave) s_len[i] = plan.prefix_len;
      if (lane < B) s_len[plan.n_prefix + lane] = overflow ? 0 : tokens;
    }
    __syncthreads();
    plan_body(plan, plan.n_prefix + B, s_len, false);
    return;
  }
  const int base = __builtin_amdgcn_readlane((upper << 16) + lower - tokens, frame);   // (right where nothing overflows)
  const bool skipped = __builtin_amdgcn_readlane((int)easy, frame) != 0;
  if (tid == 0) {
    cu_seqlens[frame] = overflow ? 0 : base;
    if (frame == B - 1) cu_seqlens[B] = overflow ? 0 : (int)total;
    if (overflow && frame == 0) *err_flag = 1;
  }
  if (level_counts != nullptr && tid < n) {
    const int prev4 = tid == 0 ? pyr.rows[0] * pyr.cols[0] : 4 * s_split[frame][tid - 1];
    const int cur = (tid + 1 < n) ? s_split[frame][tid] : 0;
    level_counts[frame * n + tid] = (overflow || skipped) ? 0 : prev4 - cur;
  }
  if (overflow || skipped) return;
  for (int i = tid; i < leaf_words * 32; i += kCompactThreads) {   // a half wavefront per word
    const uint32_t leaf = s_leaf[i >> 5], bit = 1u << (i & 31);
    if (leaf & bit) tok_desc[base + s_before[i >> 5] + __popc(leaf & (bit - 1))] = s_desc[i >> 5] + (i & 31);
  }
}

__global__ __launch_bounds__(256) void pad_tokens_kernel(const int32_t* __restrict__ tok_desc,
                                                         const int32_t* __restrict__ cu, int B,
                                                         int t_pad, int32_t* __restrict__ tok_pad,
                                                         int32_t* __restrict__ cu_pad,
                                                         int32_t* __restrict__ kv_len,
                                                         int32_t* __restrict__ err_flag) {
  const int f = blockIdx.y;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int t0 = cu[f], len = cu[f + 1] - t0;
  if (j == 0) {
    cu_pad[f] = f * t_pad;
    if (f == B - 1) cu_pad[B] = B * t_pad;
    // a frame without tokens cannot be padded (its keys would all be masked): it gets one
    // key, the rows hold the first coarse cell, and the error flag is raised
    kv_len[f] = max(min(len, t_pad), 1);
    if (len > t_pad || len < 1) *err_flag = 1;
  }
  if (j < t_pad) tok_pad[(size_t)f * t_pad + j] = len > 0 ? tok_desc[t0 + min(j, len - 1)] : 0;
}

}  // namespace

hipError_t launch_pad_tokens(const int32_t* tok_desc, const int32_t* cu_seqlens, int B, int t_pad,
                             int32_t* tok_pad, int32_t* cu_pad, int32_t* kv_len,
                             int32_t* err_flag, hipStream_t s) {
  hipLaunchKernelGGL(pad_tokens_kernel, dim3((t_pad + 255) / 256, B), dim3(256), 0, s, tok_desc,
                     cu_seqlens, B, t_pad, tok_pad, cu_pad, kv_len, err_flag);
  return hipGetLastError();
}

hipError_t launch_select(const Pyramid& pyr, const int32_t* boxes, const uint8_t* tier,
                         const int32_t* box_offsets, int B, int nonfinest, uint8_t* hit,
                         uint8_t* hit_next, int hit_bytes, int max_tokens, int32_t* tok_desc,
                         int32_t* cu_seqlens, int32_t* level_counts, int32_t* err_flag,
                         hipStream_t s, const PlanArgs* plan, const int32_t* hard) {
  const PlanArgs none{};
  // One kernel where its bit maps and word lists fit beside the plan's tables; frames are
  // counted at the capacity of the flag arrays, so that a context keeps to one of the two forms
  // (the two-kernel form relies on what its last call left in them).
  size_t frame_words = 0, leaf_words = 0;
  for (int l = 0; l < pyr.n_levels; ++l) {
    const size_t words = (size_t)pyr.rows[l] * row_words(pyr, l);
    leaf_words += words;
    if (l + 1 < pyr.n_levels) frame_words += words;
  }
  const size_t frames = hit_bytes > 0 && nonfinest > 0 ? (size_t)(hit_bytes / nonfinest) : (size_t)B;
  if ((frames * frame_words + 3 * leaf_words) * 4 <= (size_t)kSelectLds) {
    const size_t lds = (B * frame_words + 3 * leaf_words) * 4;
    static DeviceOnce configured;
    if (lds > 32 * 1024) {   // (64 KB with the plan's tables need no leave)
      hipError_t e = allow_lds(select_kernel, kSelectLds, &configured);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(select_kernel, dim3(B + (plan ? 1 : 0)), dim3(kCompactThreads),
                       lds, s, pyr, boxes, tier, box_offsets, B, (int)frame_words,
                       (int)leaf_words, max_tokens, tok_desc, cu_seqlens, level_counts, err_flag, hard,
                       plan ? *plan : none);
    return hipGetLastError();
  }
  if (nonfinest > 0) {
    const int cells_per_block = kHitThreads / kBoxLanes;
    dim3 grid((nonfinest + cells_per_block - 1) / cells_per_block, B);
    hipLaunchKernelGGL(select_hit_kernel, grid, dim3(kHitThreads), 0, s, pyr, boxes, tier,
                       box_offsets, nonfinest, hit);
  }
  hipLaunchKernelGGL(select_compact_kernel, dim3(B + (plan ? 1 : 0)), dim3(kCompactThreads), 0, s,
                     pyr, B, nonfinest, hit, hit_next, hit_bytes, max_tokens, tok_desc, cu_seqlens,
                     level_counts, err_flag, hard, plan ? *plan : none);
  return hipGetLastError();
}

hipError_t launch_plan(const int32_t* cu_seqlens, int B, const PlanArgs& plan, hipStream_t s,
                       int max_total, int32_t* err_flag) {
  hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(256), 0, s, cu_seqlens, B, plan, max_total, err_flag);
  return hipGetLastError();
}

hipError_t launch_decode_plan(const int32_t* cu_seqlens, int B, const PlanArgs& tokens, const PlanArgs& queries, int Q,
                              int max_total, int32_t* err_flag, const float* memory, void* out, int d, hipStream_t s) {
  const size_t n8 = ((size_t)max_total * d + 7) / 8;
  hipLaunchKernelGGL(decode_plan_kernel, dim3((unsigned)((n8 + 255) / 256) + 2), dim3(256), 0, s, cu_seqlens, B, tokens, queries, Q,
                     max_total, err_flag, memory, static_cast<bf16_t*>(out), d);
  return hipGetLastError();
}

}  // namespace cfdetr
