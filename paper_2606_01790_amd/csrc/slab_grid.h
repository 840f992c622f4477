// How a scoring pass's 64-token slabs are divided into blocks, and how a
// block walks its share.  Host code, kernels and tests share this file.
#pragma once
#include <algorithm>
#include <cstdint>

#ifdef __HIPCC__
#define STARKV_HD __host__ __device__
#else
#define STARKV_HD
#endif

namespace starkv {

constexpr int kSlab = 64;           // tokens per slab
constexpr int kSlabWaves = 8;       // waves of a persistent block
constexpr int kSmallRows = 256;     // tokens of a small-call block in pass 1
constexpr int kSmallWaves = 8;      // row blocks (a wave each) of a small-call block
constexpr int kSmallMost = 16;      // the same in the larger small-call block
constexpr int kUnrolledBlocks = 8;  // row blocks of the unrolled pass 2 at most

// Whether pass 2 runs the unrolled kernel, whose waves take whole slabs
// (whole_blocks: an output's rows are whole row blocks).
constexpr bool pass2_unrolled(int d, int esz, int nrb, bool whole_blocks) {
  return esz == 2 && d == 128 && nrb <= kUnrolledBlocks && whole_blocks;
}

STARKV_HD inline int slab_min(int a, int b) { return a < b ? a : b; }

// A pass's division of the slabs into blocks (slab_grid below):
// per_lg > 0: per_lg blocks per (layer, group), of q slabs and one more in
// the first r of them; per_lg = 0: the same over all slabs, so that a block
// may cross into the next (layer, group).
struct SlabGrid {
  int S;        // 64-token slabs per (layer, group)
  int per_lg, q, r;
  int rs;       // waves that share a slab, each with its part of the row blocks
};

// A pass's launch: its division and block count.
struct SlabLaunch {
  SlabGrid g;
  int blocks;
  bool small = false;   // the small-call kernels
};

// The block of slab x under per_lg = 0.  32 bits: the scores of 2^31 slabs
// would not fit the GPU's memory.
STARKV_HD inline int slab_owner(const SlabGrid& g, int x) {
  const int y = x - g.r * (g.q + 1);
  return y < 0 ? x / (g.q + 1) : g.r + y / g.q;
}

// A block's walk over its slabs: segments of one (layer, group) each.
struct SlabWalk {
  int lg, s0, s1;   // this segment
  int chunk;        // the block's index among the blocks of lg
  int left;         // slabs after this segment
};

STARKV_HD inline SlabWalk slab_walk(const SlabGrid& g, int b) {
  const bool aligned = g.per_lg > 0;
  const int x = b * g.q + slab_min(b, g.r);              // crossing: the first slab
  const int lg = aligned ? b / g.per_lg : x / g.S;
  const int i = b - lg * g.per_lg;                       // aligned: the block of lg
  const int s0 = aligned ? i * g.q + slab_min(i, g.r) : x - lg * g.S;
  const int n = g.q + ((aligned ? i : b) < g.r);
  const int s1 = slab_min(g.S, s0 + n);
  const int chunk = aligned ? i : b - slab_owner(g, lg * g.S);
  return SlabWalk{lg, s0, s1, chunk, n - (s1 - s0)};
}

// The walk's next segment, where left > 0.
STARKV_HD inline SlabWalk slab_next(const SlabGrid& g, const SlabWalk& w) {
  const int n = slab_min(g.S, w.left);
  return SlabWalk{w.lg + 1, 0, n, 0, w.left - n};
}

// Blocks whose slabs include some of (layer, group) lg's.
STARKV_HD inline int slab_chunks(const SlabGrid& g, int lg) {
  if (g.per_lg > 0) return g.per_lg;
  return slab_owner(g, lg * g.S + g.S - 1) - slab_owner(g, lg * g.S) + 1;
}

// A pass's blocks (one per CU at a time: the window rows fill the LDS).
// Either `per_lg` blocks per (layer, group), or one block per CU on equal
// ranges that cross groups.  The unit of the estimate is an eighth of a
// slab round, the time the block's eight waves take for a slab each.
//   aligned  whole rounds of the largest block, and a start
//   equal    pass 1: whole rounds, a start, and for every further segment a
//            start (its window rows and reference slab, two barriers) and
//            the rounding of its slabs to whole rounds;
//            pass 2: the slabs, half a round per segment for that rounding
//            (a wave goes to the next segment's rows while others finish),
//            a start, and a quarter round for every further segment.
// Pass 1's first slab is the reference, which the waves take together as
// part of the start.  Measured on 28 layers of 4 groups, 7 row blocks, us
// aligned / equal, at one to eight 1920x1080 frames:
//   pass 1  31/37 52/56 69/76 88/93 107/112 126/128 143/147 161/162
//   pass 2  27/30 45/48 65/64 91/84 111/105 134/128 157/148 178/166
// and pass 1 on 14 layers, one round of 224 blocks / two of 504, at three
// and five frames: 38/45 62/68.
// long_rounds: float32 keys and four row blocks, several times the matrix
// time per round, so that a start is a smaller part of one (14 layers of 4
// groups, d = 64, 13,679 tokens: 253 us of the call with the other start,
// 224 blocks per pass, 240 with this one, 504; 8,297 tokens 160 and 162).
// In a block of at most `share` slabs several waves share a slab, each with
// its part of the row blocks.
inline SlabLaunch slab_grid(int Lp, int nlg, int nrb, int n_cu, int max_per_lg, int share,
                            bool long_rounds, bool first) {
  SlabLaunch l;
  SlabGrid& g = l.g;
  g.S = (Lp + kSlab - 1) / kSlab;
  const int start = long_rounds ? 4 : first ? 10 : 8;
  auto waves_per_slab = [&](int64_t slabs) {
    int rs = 1;
    while (slabs <= share && rs * 2 * slabs <= kSlabWaves && rs * 2 <= nrb) rs *= 2;
    return rs;
  };
  auto rounds8 = [&](int64_t slabs) {
    const int rs = waves_per_slab(slabs);
    if (rs > 1) return (int64_t)(8 / rs);
    return (slabs - first + kSlabWaves - 1) / kSlabWaves * 8;
  };
  const int64_t total = (int64_t)g.S * nlg;
  int64_t best = -1;
  const int64_t p_max = std::min<int64_t>({(int64_t)max_per_lg, (int64_t)g.S,
                                           std::max<int64_t>(1, 4L * n_cu / nlg)});
  // of the block counts that run in k rounds on the CUs the largest costs
  // least; among equal costs the fewest rounds, though not fewer slabs
  for (int k = 1; k <= 4; ++k) {
    const int64_t p = std::min<int64_t>(p_max, std::max<int64_t>(1, (int64_t)k * n_cu / nlg));
    const int64_t q = (g.S + p - 1) / p;
    const int64_t cost = (p * nlg + n_cu - 1) / n_cu * (rounds8(q) + start);
    if (best < 0 || cost < best) {
      best = cost;
      g.per_lg = (int)p;
      g.q = (int)(g.S / p);
      g.r = (int)(g.S % p);
      g.rs = waves_per_slab(q);
      l.blocks = (int)(p * nlg);
    }
  }
  if (total > n_cu) {
    const int64_t q = (total + n_cu - 1) / n_cu, q_min = total / n_cu;
    const int64_t segs = (q + g.S - 2) / g.S + 1;           // of a block at most
    const int64_t chunks = (g.S + q_min - 2) / q_min + 1;   // blocks per group at most
    const int64_t cost = first ? (q + kSlabWaves - 1) / kSlabWaves * 8 + start +
                                     (segs - 1) * (8 + start)
                               : q + segs * 4 + start + (segs - 1) * 2;
    if (chunks <= max_per_lg && cost < best) {
      g.per_lg = 0;
      g.q = (int)q_min;
      g.r = (int)(total - q_min * n_cu);
      g.rs = 1;
      l.blocks = n_cu;
    }
  }
  return l;
}

// The two passes' launches for n_layers * G groups of nrb row blocks, at most
// max_chunks records per group in the workspace.  one_sum: one output per
// group; whole_blocks: an output's rows are whole row blocks.
//
// Waves share a slab only in pass 2 with one sum per group, outside the
// unrolled kernel, at most two slabs, and where a slab is long work for a
// wave: float32 keys, or more than ten row blocks.  us of the call, shared /
// not: float32, d = 64, 4 row blocks, 376 slabs on 256 CUs 32.9 / 33.6; bf16,
// 14 row blocks, d = 128, 376 slabs 30.3 / 30.3, 752 slabs 31.8 / 31.0, d =
// 64, 376 slabs 24.0 / 24.5; 9 row blocks, 376 slabs 26.6 / 25.3; pass 1, 9
// row blocks, 564 slabs 27.2 / 26.3.
//
// The small-call kernels run one short step per block and win while the
// blocks run side by side.  Pass 1 up to one block per CU: 28 heads on 4
// groups, d = 128, us of the call with it / with the persistent pass 1: 96
// blocks 19.7 / 22.2, 240 blocks 20.1 / 22.6, 260 blocks 26.3 / 23.8, 308
// blocks 27.3 / 24.7; with 14 row blocks 48 blocks 28.0 / 28.8, d = 64 22.0 /
// 23.3, but with 9 row blocks 24.9 / 24.1 and with 11 25.9 / 26.1.  Pass 2
// likewise (220 blocks 17.1 / 18.2, 264 blocks 19.0 / 18.3; 14 row blocks,
// 188 blocks 26.8 / 28.8, 376 blocks 33.8 / 29.9).  Up to eight row blocks it
// wins to one and a half blocks per CU for bf16 keys with d = 64 and several
// row blocks (460 blocks 16.4 / 17.0), an output per head (440 blocks 27.5 /
// 28.0) or four row blocks of float32 keys (376 blocks 27.6 / 29.0); it does
// not with one or two row blocks of bf16 keys and d = 128 (220 blocks 13.5 /
// 12.8), whose persistent kernel starts as soon.
inline void slab_launches(int Lp, int nlg, int nrb, int n_cu, int max_chunks, bool one_sum,
                          bool whole_blocks, int d, int esz, SlabLaunch* p1,
                          SlabLaunch* p2) {
  const bool unrolled = pass2_unrolled(d, esz, nrb, whole_blocks);
  const int share = !one_sum || unrolled ? 0 : esz == 4 || nrb > 10 ? 2 : 0;
  const bool long_rounds = esz == 4 && nrb >= 4;
  *p1 = slab_grid(Lp, nlg, nrb, n_cu, max_chunks, 0, long_rounds, true);
  *p2 = slab_grid(Lp, nlg, nrb, n_cu, 1 << 30, share, long_rounds, false);
  const int64_t chunks = (Lp + kSmallRows - 1) / kSmallRows;
  if (chunks <= max_chunks && chunks * nlg <= n_cu &&
      (nrb <= kSmallWaves || nrb > 11 || d == 64)) {
    p1->small = true;
    p1->g.per_lg = (int)chunks;
    p1->blocks = (int)(chunks * nlg);
  }
  int p2_small = n_cu;
  if (nrb <= kSmallWaves && (esz == 4 ? nrb >= 4 : d == 64 ? nrb >= 2 : nrb > 4 && !one_sum))
    p2_small += n_cu / 2;
  if (esz == 2 && d == 128 && nrb <= 2) p2_small = 0;
  if (whole_blocks && (int64_t)p2->g.S * nlg <= p2_small) {
    p2->small = true;
    p2->blocks = p2->g.S * nlg;
  }
}

}  // namespace starkv
