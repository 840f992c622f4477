// Window attention scoring (sec. 3.3): A_raw summed over the window rows of
// each scoring subspace.
//
// The window softmax of every query row needs that row's sum over all L_p
// past keys before any key's normalised mass is known, so scoring runs in
// two passes over K, with y = q.k * log2(e)/sqrt(d):
//   pass 1  per (layer, group, block): for each window row r a reference
//           M_r and the sum of 2^(y - M_r) over the block's tokens;
//   pass 2  merges the blocks' statistics into c_r = M_r + log2(sum_r) and
//           sums 2^(y_rt - c_r) over the rows of each subspace for every
//           token t.
//
// Both passes are one persistent design.  A 512-thread block (one per CU)
// takes a range of one or more (layer, group)'s 64-token slabs and stages
// the group's R window rows in LDS (rows padded by 16 bytes: no bank
// conflicts).  Each wave takes whole slabs: the slab's K rows go straight
// from global memory into MFMA fragment registers, and the wave walks the
// group's 32-row blocks, reading each Q fragment from LDS once for the
// slab's two 32-token tiles.  No barrier inside the slab loop.
//   - bf16: a slab's tiles form one sequence; the MFMAs of a tile are
//     interleaved with the exponentials of the tile before it, two
//     accumulator tiles in all.  The next slab's K is loaded behind the last
//     tile's exponentials; the other wave of the SIMD covers its latency (a
//     second register set for it, loaded a slab ahead, gained nothing).
//   - The row-block loop is rolled (nothing per row block stays in
//     registers), so one kernel serves every R.
//   - What bounds it: power.  With normal random operands an MFMA loop alone
//     runs at 1.74 PFLOP/s (1.70 GHz; 2.4 PFLOP/s and 2.4 GHz with zeros),
//     with this epilogue at 1.30 and with the LDS reads at 1.23; the slab
//     loop reaches 1.13 at 13,679 tokens of 28 layers.  A K load, a row per
//     lane, takes 64 address cycles against 16 for contiguous lanes, about
//     3.5 us for the first slabs of a block's eight waves.
// Pass 1 puts tokens on the MFMA M axis: a lane owns one window row of the
// tile and its reference is one register.  Pass 2 puts rows on M: a lane
// owns one token and its sum over the rows completes in the wave; it takes a
// segment's slabs from the last to the first, since the last ones pass 1 read
// are those the last-level cache still holds (first to last, 16 layers of 16
// groups, 32 rows: 73 us against 63 at 5,606 tokens, 172 against 162 at
// 13,679; 32 layers of 8 groups, 128 rows: 82 against 73 at 5,606).  Against
// a pass 1 with K tiles in LDS and a wave per row block, one fragment read
// per MFMA: 2209 -> 1772 us at 140,190 tokens and 14 row blocks, 80 -> 74 at
// 8,297 and 7, and 114 -> 113 at 13,679; fp32 at d = 64 with one row block
// (there a block of one wave) 39 -> 23 us, and its pass 2 44 -> 22.
//
// fp32 keys run v_mfma_f32_32x32x2f32 (64 cycles per 2 k): the matrix core
// bounds them, so their tiles are not interleaved.
#pragma once
#include "device_common.h"
#include "internal.h"
#include "slab_grid.h"

namespace starkv {

struct ScoreArgs {
  const void* q;
  const void* k;
  int64_t ls, gs, ts;   // element strides of the K cache
  int H, G, W, R, nrb, Lp;
  int n_chunks_max;
  bool far;             // the records' references may lie far below their maxima
  float scale;          // log2(e) / sqrt(d)
  float2* part;         // [n_layers][G][n_chunks_max][nrb * 32]  (M, sum)
  float* sraw;          // [n_layers][Ns][Lp]
  // subspaces per KV group (1, or H/G per head), and the row blocks
  // (kHeadBlocks) or 8-row groups (kHeadGroups) per head
  int n_out, upo;
};

namespace {

constexpr int kSlabThreads = kSlabWaves * 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1e30f;
// A row's sum over a block against its reference stays below this unless a
// logit rises about 32 log2 units above the reference slab.  An exponent's
// rounding grows with its size (up to 2^-20 below 32), so such a block's
// sums are taken again, against a higher reference (sum_again).
constexpr float kSumLimit = 4294967296.0f;   // 2^32

// Pass-2 output: one sum per group; one per head, a head being whole row
// blocks; one per head, a head being whole 8-row groups.
enum HeadLayout { kGroup = 0, kHeadBlocks = 1, kHeadGroups = 2 };

// 16 bytes of a row: one bf16 MFMA step, or four fp32 ones.  Lane half h
// supplies bytes 32 j + 16 h of its row in step j for both operands, so the
// contraction pairs equal elements whatever order the hardware takes them.
template <typename T>
__device__ __forceinline__ f32x16 mma16(i32x4 a, i32x4 b, f32x16 c);
template <>
__device__ __forceinline__ f32x16 mma16<__bf16>(i32x4 a, i32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
template <>
__device__ __forceinline__ f32x16 mma16<float>(i32x4 a, i32x4 b, f32x16 c) {
  const f32x4 fa = __builtin_bit_cast(f32x4, a), fb = __builtin_bit_cast(f32x4, b);
#pragma unroll
  for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i], fb[i], c, 0, 0, 0);
  return c;
}

template <typename T, int D>
struct Shape {
  static constexpr int kRowBytes = D * (int)sizeof(T);
  static constexpr int kNP = kRowBytes / 32;        // 16-byte pieces per lane and row
  static constexpr int kQStride = kRowBytes + 16;   // LDS bytes per window row
  // 32-token tiles of a slab held at a time: 64 registers of K per set
  static constexpr int kTB = kNP > 8 ? 1 : 2;
};

template <typename T, int D>
using KFrags = i32x4[Shape<T, D>::kTB][Shape<T, D>::kNP];

// The value lane l ^ 32 holds.  v_permlane32_swap exchanges the upper lane
// half of its first operand with the lower half of its second, so with both
// operands = v the first result holds the lower half's values in the upper
// lanes and the second the upper half's values in the lower lanes.
__device__ inline float other_half(float v, int half) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(half ? sw[0] : sw[1]);
}

// The two waves of a SIMD take turns at the higher issue priority, slab by
// slab: the older one would otherwise finish its slabs early and leave the
// other to run alone at the end of the block.
__device__ __forceinline__ void take_turn(int& turn) {
  if ((turn ^= 1)) __builtin_amdgcn_s_setprio(0);
  else __builtin_amdgcn_s_setprio(1);
}

// 2^((m - mn) * scale) for a running max m <= mn, ms = mn * scale.  Exactly 1
// when the max did not move: with the -1e30 start value the fma would
// otherwise return the rounding residual of the product, not 0.
__device__ inline float rescale(float m, float mn, float ms, float scale) {
  return m == mn ? 1.0f : __builtin_amdgcn_exp2f(fmaf(m, scale, -ms));
}

// Lanes 0-31: both halves of v0 added; lanes 32-63: both halves of v1.
__device__ inline float add_halves(float v0, float v1) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v0), __float_as_uint(v1), false, false);
  return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

// Blocks are dealt to the 8 XCDs round-robin by id; the id is permuted so
// that each XCD walks one contiguous part of the slab space (a bijection of
// [0, gridDim.x), correct whatever the placement).
__device__ inline int slab_block() {
  const int n = gridDim.x, b = blockIdx.x;
  const int xcd = b & 7, local = b >> 3, per = n >> 3, rem = n & 7;
  return xcd < rem ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
}

// threadIdx.x, opaque to the compiler: what is computed from it stays where
// it is written.  The slab loops need nearly every register, and thread
// constants hoisted above them (staging indices, row offsets) end in
// scratch memory, whose reloads wait for the K loads in flight.
__device__ __forceinline__ int tid_here() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

template <typename T, int D>
__device__ inline const T* group_q(const ScoreArgs& a, int lg) {
  const int layer = lg / a.G, g = lg - layer * a.G;
  return reinterpret_cast<const T*>(a.q) +
         ((size_t)layer * a.H + (size_t)g * (a.H / a.G)) * (size_t)a.W * D;
}

template <typename T>
__device__ inline const T* group_k(const ScoreArgs& a, int lg) {
  const int layer = lg / a.G, g = lg - layer * a.G;
  return reinterpret_cast<const T*>(a.k) + (int64_t)layer * a.ls + (int64_t)g * a.gs;
}

// The group's window rows to LDS, rows R .. nrb * 32 zero.  The first batch
// of 16-byte vectors is issued by q_issue; q_commit stores it and moves the
// rest, so that a segment's other first loads can be issued between.
constexpr int kQBatch = 7;
template <typename T, int D>
__device__ __forceinline__ void q_issue(const ScoreArgs& a, const T* qg, int i0,
                                        i32x4 (&v)[kQBatch]) {
  constexpr int VPR = Shape<T, D>::kRowBytes / 16;
  const char* src = reinterpret_cast<const char*>(qg);
#pragma unroll
  for (int j = 0; j < kQBatch; ++j) {
    const int i = min(i0 + j * kSlabThreads, a.R * VPR - 1);
    v[j] = *reinterpret_cast<const i32x4*>(src + (size_t)i * 16);
  }
}
template <typename T, int D>
__device__ __forceinline__ void q_commit(const ScoreArgs& a, const T* qg, char* qs,
                                         i32x4 (&v)[kQBatch]) {
  using SH = Shape<T, D>;
  constexpr int VPR = SH::kRowBytes / 16;
  const int nv = a.nrb * 32 * VPR;
  for (int i0 = tid_here();;) {
#pragma unroll
    for (int j = 0; j < kQBatch; ++j) {
      const int i = i0 + j * kSlabThreads, row = i / VPR, part = i % VPR;
      if (row >= a.R) v[j] = i32x4{0, 0, 0, 0};
      if (i < nv) *reinterpret_cast<i32x4*>(qs + row * SH::kQStride + part * 16) = v[j];
      __builtin_amdgcn_sched_barrier(0);   // one condition at a time
    }
    i0 += kQBatch * kSlabThreads;
    if (i0 - (int)threadIdx.x >= nv) break;
    q_issue<T, D>(a, qg, i0, v);
  }
}

// One slab of K to LDS, rows as the window rows; vectors of this thread.
template <typename T, int D>
constexpr int slab_vecs() { return kSlab * (Shape<T, D>::kRowBytes / 16) / kSlabThreads; }
template <typename T, int D>
__device__ __forceinline__ void slab_issue(const ScoreArgs& a, const T* kg, int slab,
                                           i32x4 (&v)[slab_vecs<T, D>()]) {
  constexpr int VPR = Shape<T, D>::kRowBytes / 16;
  const int tid = tid_here();
  const int last = a.Lp - 1 - slab * kSlab;
  const char* base = reinterpret_cast<const char*>(kg + (int64_t)slab * kSlab * a.ts);
#pragma unroll
  for (int j = 0; j < slab_vecs<T, D>(); ++j) {
    const int i = tid + j * kSlabThreads, row = min(i / VPR, last), part = i % VPR;
    v[j] = *reinterpret_cast<const i32x4*>(base + (int64_t)row * (a.ts * (int64_t)sizeof(T)) +
                                           part * 16);
  }
}
template <typename T, int D>
__device__ __forceinline__ void slab_commit(char* ks, const i32x4 (&v)[slab_vecs<T, D>()]) {
  using SH = Shape<T, D>;
  constexpr int VPR = SH::kRowBytes / 16;
  const int tid = tid_here();
#pragma unroll
  for (int j = 0; j < slab_vecs<T, D>(); ++j) {
    const int i = tid + j * kSlabThreads, row = i / VPR, part = i % VPR;
    *reinterpret_cast<i32x4*>(ks + row * SH::kQStride + part * 16) = v[j];
  }
}

// K fragments of tiles cb0 .. cb0 + kTB - 1 of one slab: the token of row
// l32 of each tile, this lane half's pieces.  Tokens past L_p re-read the
// last one.
template <typename T, int D>
__device__ __forceinline__ void load_k(const ScoreArgs& a, const T* kg, int slab, int cb0,
                                       KFrags<T, D>& kf) {
  using SH = Shape<T, D>;
  const int lane = tid_here() & 63, half = lane >> 5, l32 = lane & 31;
  const char* base = reinterpret_cast<const char*>(kg + (int64_t)slab * kSlab * a.ts);
  const int last = a.Lp - 1 - slab * kSlab;
#pragma unroll
  for (int cb = 0; cb < SH::kTB; ++cb) {
    const int rel = min((cb0 + cb) * 32 + l32, last);
    const char* row = base + (int64_t)rel * (a.ts * (int64_t)sizeof(T)) + half * 16;
#pragma unroll
    for (int j = 0; j < SH::kNP; ++j) kf[cb][j] = *reinterpret_cast<const i32x4*>(row + j * 32);
  }
}

template <typename T, int D>
__device__ __forceinline__ void load_q(const char* qrow, i32x4 (&qf)[Shape<T, D>::kNP]) {
#pragma unroll
  for (int j = 0; j < Shape<T, D>::kNP; ++j)
    qf[j] = *reinterpret_cast<const i32x4*>(qrow + j * 32);
}

// One tile's MFMA chain.  TOK_M: tokens on the M axis (pass 1), else rows.
template <typename T, int D, bool TOK_M>
__device__ __forceinline__ f32x16 chain(const i32x4 (&qf)[Shape<T, D>::kNP],
                                        const i32x4 (&kf)[Shape<T, D>::kNP]) {
  f32x16 acc = {};
#pragma unroll
  for (int j = 0; j < Shape<T, D>::kNP; ++j)
    acc = TOK_M ? mma16<T>(kf[j], qf[j], acc) : mma16<T>(qf[j], kf[j], acc);
  return acc;
}

// Tokens on M: element e of this lane is token tb + 8 (e / 4) + 4 half + e % 4.
__device__ __forceinline__ void mask_tokens(f32x16& acc, int tb, int Lp) {
  const int left = Lp - tb - 4 * ((tid_here() & 63) >> 5);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    if (8 * (e >> 2) + (e & 3) >= left) acc[e] = -INFINITY;
    __builtin_amdgcn_sched_barrier(0);   // one condition at a time
  }
}

// ---------------------------------------------------------------- stages
// One tile's step of the bf16 sequence: the MFMAs of the next tile (nxt, K
// fragments kf) interleaved with cur's 16 exponentials per lane.  RELOAD:
// each Q fragment is replaced by the next row block's once it is used.
// The order is pinned one MFMA at a time.  The exponentials start behind
// the second MFMA: cur's own last MFMA, just before this step, has then
// left the matrix core.
// A tile's 16 values are added up in two chains of their own before they
// join a longer sum.
__device__ __forceinline__ void add_to(float& s, float v, bool first) { s = first ? v : s + v; }

template <int NP>
constexpr int stage_elem(int j) {   // cur's elements before step j
  return j <= 1 ? 0 : (j - 1) * 16 / (NP - 1);
}

template <int D, bool RELOAD>
__device__ __forceinline__ float stage1(i32x4 (&qf)[D / 16], const i32x4 (&kf)[D / 16],
                                        const char* qnext, f32x16& nxt, const f32x16& cur,
                                        float scale, float ms) {
  constexpr int NP = D / 16;
  float s[2];
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    nxt = mma16<__bf16>(kf[j], qf[j], j ? nxt : f32x16{});
    if (RELOAD) qf[j] = *reinterpret_cast<const i32x4*>(qnext + j * 32);
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (e >= stage_elem<NP>(j) && e < stage_elem<NP>(j + 1))
        add_to(s[e & 1], __builtin_amdgcn_exp2f(fmaf(cur[e], scale, -ms)), e < 2);
    __builtin_amdgcn_sched_barrier(0);
  }
  return s[0] + s[1];
}

template <int D, bool RELOAD>
__device__ __forceinline__ float stage2(i32x4 (&qf)[D / 16], const i32x4 (&kf)[D / 16],
                                        const char* qnext, f32x16& nxt, const f32x16& cur,
                                        float scale, const float (&c)[16]) {
  constexpr int NP = D / 16;
  float s[2];
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    nxt = mma16<__bf16>(qf[j], kf[j], j ? nxt : f32x16{});
    if (RELOAD) qf[j] = *reinterpret_cast<const i32x4*>(qnext + j * 32);
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (e >= stage_elem<NP>(j) && e < stage_elem<NP>(j + 1))
        add_to(s[e & 1], __builtin_amdgcn_exp2f(fmaf(cur[e], scale, -c[e])), e < 2);
    __builtin_amdgcn_sched_barrier(0);
  }
  return s[0] + s[1];
}

// The same sums with no MFMAs to interleave.
__device__ __forceinline__ float tile_sum1(const f32x16& acc, float scale, float ms) {
  float s[2];
#pragma unroll
  for (int e = 0; e < 16; ++e)
    add_to(s[e & 1], __builtin_amdgcn_exp2f(fmaf(acc[e], scale, -ms)), e < 2);
  return s[0] + s[1];
}
__device__ __forceinline__ float tile_sum2(const f32x16& acc, float scale, const float (&c)[16]) {
  float s[2];
#pragma unroll
  for (int e = 0; e < 16; ++e)
    add_to(s[e & 1], __builtin_amdgcn_exp2f(fmaf(acc[e], scale, -c[e])), e < 2);
  return s[0] + s[1];
}

// Waits for every load of the wave, at the end of a step whose other register
// set was loaded meanwhile: a loop that uses registers whose loads may (as
// far as the compiler can tell) be outstanding would wait for the newer
// loads behind them too.
__device__ __forceinline__ void loads_landed() {
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
}

// c of the 16 rows this lane receives of a row block: 8 i + 4 half + j
__device__ __forceinline__ void load_c(const float* cs, int half, float (&c)[16]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x4 c4 = *reinterpret_cast<const f32x4*>(cs + 4 * half + 8 * i);
#pragma unroll
    for (int j = 0; j < 4; ++j) c[4 * i + j] = c4[j];
  }
}

// ---------------------------------------------------------------- pass 1
// LDS: window rows, ms[nrb * 32] (references times scale), a flag,
// l[wave][nrb * 64] (each wave's sums, one per lane).
template <typename T, int D>
__host__ __device__ constexpr size_t pass1_lds(int nrb) {
  const size_t sums = (size_t)kSlabWaves * nrb * 64 * 4;
  const size_t slab = (size_t)kSlab * Shape<T, D>::kQStride;   // the reference slab, before
  return (size_t)nrb * 32 * Shape<T, D>::kQStride + (size_t)nrb * 32 * 4 + 16 +
         (sums > slab ? sums : slab);
}

// Row r's sum over the block: every wave's part, both lane halves.
__device__ __forceinline__ float row_sum(const ScoreArgs& a, const float* l_s, int r) {
  float l = 0.f;
  const float* lr = l_s + (r >> 5) * 64 + (r & 31);
#pragma unroll
  for (int v = 0; v < kSlabWaves; ++v) l += lr[v * a.nrb * 64] + lr[v * a.nrb * 64 + 32];
  return l;
}

// The sums of slabs [s0, s1) again where a row's (out) left its range: that
// row's reference rises to M_r + log2(sum), within log2 of the token count of
// its maximum.  True if a sum is not finite.  Apart from the first sums' loop, whose schedule suffers
// from a second use; it takes whole slabs per wave without loading ahead.
// Every group with a key 98 log2 units above the others, 28 layers of 4
// groups, whole score call: 77 us at 2,915 tokens and 303 at 13,679; with
// exact_rows instead 128 and 528; without such keys 60 and 212.
template <typename T, int D>
__device__ bool sum_again(const ScoreArgs& a, const T* kg, const char* qs, float* ms_s, float* l_s,
                          int s0, int s1, float2* out) {
  using SH = Shape<T, D>;
  const int tid = tid_here(), lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
  bool bad = false;
  for (int r = tid; r < a.nrb * 32; r += kSlabThreads) {
    const float l = out[r].y;   // this thread's own store
    bad |= !(l < INFINITY);
    if (l >= kSumLimit) ms_s[r] += log2f(l);
  }
  float* lw = l_s + wave * a.nrb * 64 + lane;
  for (int rb = 0; rb < a.nrb; ++rb) lw[rb * 64] = 0.f;
  __syncthreads();
  for (int slab = s0 + wave; slab < s1; slab += kSlabWaves) {
    for (int cb = 0; cb < 2; cb += SH::kTB) {
      KFrags<T, D> kf;
      load_k<T, D>(a, kg, slab, cb, kf);
      for (int rb = 0; rb < a.nrb; ++rb) {
        i32x4 qf[SH::kNP];
        load_q<T, D>(qs + (rb * 32 + l32) * SH::kQStride + half * 16, qf);
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < SH::kTB; ++u) {
          f32x16 acc = chain<T, D, true>(qf, kf[u]);
          if (slab == s1 - 1) mask_tokens(acc, slab * kSlab + (cb + u) * 32, a.Lp);
          s += tile_sum1(acc, a.scale, ms_s[rb * 32 + l32]);
        }
        lw[rb * 64] += s;
      }
    }
  }
  __syncthreads();
  for (int r = tid; r < a.nrb * 32; r += kSlabThreads)
    out[r] = make_float2(ms_s[r], row_sum(a, l_s, r));
  return bad;
}

// Exact row statistics of slabs [s0, s1) against running maxima, for blocks
// with sums that are not finite: a wave per row block, K re-read for each.
template <typename T, int D>
__device__ void exact_rows(const ScoreArgs& a, const T* kg, const char* qs, int s0, int s1,
                           float2* out) {
  using SH = Shape<T, D>;
  const int tid = tid_here(), lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
  for (int rb = wave; rb < a.nrb; rb += kSlabWaves) {
    i32x4 qf[SH::kNP];
    load_q<T, D>(qs + (rb * 32 + l32) * SH::kQStride + half * 16, qf);
    float m = kNegBig, l = 0.f;
    for (int slab = s0; slab < s1; ++slab) {
      for (int cb = 0; cb < 2; cb += SH::kTB) {
        KFrags<T, D> kf;
        load_k<T, D>(a, kg, slab, cb, kf);
#pragma unroll
        for (int u = 0; u < SH::kTB; ++u) {
          f32x16 acc = chain<T, D, true>(qf, kf[u]);
          mask_tokens(acc, slab * kSlab + (cb + u) * 32, a.Lp);
          float mt = acc[0];
#pragma unroll
          for (int e = 1; e < 16; ++e) mt = fmaxf(mt, acc[e]);
          const float mn = fmaxf(m, mt), msn = mn * a.scale;
          const float sum = tile_sum1(acc, a.scale, msn);
          l = l * rescale(m, mn, msn, a.scale) + sum;
          m = mn;
        }
      }
    }
    // the two lane halves hold the same row over other tokens
    const float mo = other_half(m, half), lo = other_half(l, half);
    const float mn = fmaxf(m, mo), msn = mn * a.scale;
    l = l * rescale(m, mn, msn, a.scale) + lo * rescale(mo, mn, msn, a.scale);
    if (half == 0) out[rb * 32 + l32] = make_float2(msn, l);
  }
}

template <typename T, int D, bool PIPE>
__global__ __launch_bounds__(kSlabThreads) void score_pass1(ScoreArgs a, SlabGrid sg) {
  using SH = Shape<T, D>;
  extern __shared__ __align__(16) unsigned char smem[];
  char* qs = reinterpret_cast<char*>(smem);
  float* ms_s = reinterpret_cast<float*>(smem + (size_t)a.nrb * 32 * SH::kQStride);
  int* redo = reinterpret_cast<int*>(ms_s + a.nrb * 32);   // a sum left its range
  float* l_s = ms_s + a.nrb * 32 + 4;
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const char* qlane = qs + l32 * SH::kQStride + half * 16;
  const float* mslane = ms_s + l32;
  float* lw = l_s + wave * a.nrb * 64 + lane;
  constexpr int kRB = 32 * SH::kQStride;      // LDS bytes of a row block

  for (SlabWalk w = slab_walk(sg, slab_block());; w = slab_next(sg, w)) {
    const T* kg = group_k<T>(a, w.lg);
    // the segment's last slab gives the references (below); the waves then
    // take the others, all of them whole
    const int end = w.s1 - 1;
    int slab = w.s0 + wave;
    const bool any = slab < end;
    KFrags<T, D> kf;
    char* ks = reinterpret_cast<char*>(l_s);
    {
      const T* qg = group_q<T, D>(a, w.lg);
      i32x4 kv[slab_vecs<T, D>()], qv[kQBatch];
      slab_issue<T, D>(a, kg, end, kv);
      q_issue<T, D>(a, qg, tid_here(), qv);
      if (any) load_k<T, D>(a, kg, slab, 0, kf);
      __builtin_amdgcn_sched_barrier(0);
      slab_commit<T, D>(ks, kv);
      q_commit<T, D>(a, qg, qs, qv);
    }
    if (threadIdx.x == 0) *redo = 0;
    __syncthreads();
    // References: each row's max over that slab, and the slab's own sums; a
    // wave per row block (up to two each).
    float ref[2], rsum[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int rb = wave + i * kSlabWaves;
      if (rb < a.nrb) {
        i32x4 qf[SH::kNP];
        load_q<T, D>(qlane + rb * kRB, qf);
        f32x16 acc[2];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          i32x4 kf[SH::kNP];
          load_q<T, D>(ks + (cb * 32 + l32) * SH::kQStride + half * 16, kf);
          acc[cb] = chain<T, D, true>(qf, kf);
        }
        const int tb = end * kSlab;
        if (tb + kSlab > a.Lp) {
          mask_tokens(acc[0], tb, a.Lp);
          mask_tokens(acc[1], tb + 32, a.Lp);
        }
        float mt = fmaxf(acc[0][0], acc[1][0]);
#pragma unroll
        for (int e = 1; e < 16; ++e) mt = fmaxf(mt, fmaxf(acc[0][e], acc[1][e]));
        mt = fmaxf(mt, other_half(mt, half));
        const float ms = mt * a.scale;
        rsum[i] = tile_sum1(acc[0], a.scale, ms) + tile_sum1(acc[1], a.scale, ms);
        ref[i] = ms;
      }
    }
    __syncthreads();   // the slab's LDS becomes the sums
    for (int rb = 0; rb < a.nrb; ++rb) lw[rb * 64] = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int rb = wave + i * kSlabWaves;
      if (rb < a.nrb) {
        lw[rb * 64] = rsum[i];
        if (half == 0) ms_s[rb * 32 + l32] = ref[i];
      }
    }
    __syncthreads();

    if (any) {
      if constexpr (PIPE) {
        i32x4 qf[SH::kNP];
        load_q<T, D>(qlane, qf);
        f32x16 acc0 = chain<T, D, true>(qf, kf[0]), acc1;
        int turn = wave >> 2;
        for (;;) {
          take_turn(turn);
          const int next = slab + kSlabWaves;
          for (int rb = 0; rb + 1 < a.nrb; ++rb) {
            const float ms = mslane[rb * 32];
            const float l = lw[rb * 64];
            const float s = stage1<D, true>(qf, kf[1], qlane + (rb + 1) * kRB, acc1, acc0,
                                            a.scale, ms);
            lw[rb * 64] = l + (s + stage1<D, false>(qf, kf[0], nullptr, acc0, acc1, a.scale, ms));
          }
          const int rb = a.nrb - 1;
          const float ms = mslane[rb * 32], l = lw[rb * 64];
          const float s0 = stage1<D, true>(qf, kf[1], qlane, acc1, acc0, a.scale, ms);
          // the slab's K is used up: the next slab's, behind the last tile's sums
          if (next < end) load_k<T, D>(a, kg, next, 0, kf);
          __builtin_amdgcn_sched_barrier(0);
          lw[rb * 64] = l + (s0 + tile_sum1(acc1, a.scale, ms));
          if ((slab = next) >= end) break;
          acc0 = chain<T, D, true>(qf, kf[0]);
        }
      } else {
        // kTB tiles at a time
        auto process = [&](KFrags<T, D>& k) {
          for (int rb = 0; rb < a.nrb; ++rb) {
            const float ms = mslane[rb * 32];
            i32x4 qf[SH::kNP];
            load_q<T, D>(qlane + rb * kRB, qf);
            const float l = lw[rb * 64];
            float s = 0.f;
#pragma unroll
            for (int cb = 0; cb < SH::kTB; ++cb)
              s += tile_sum1(chain<T, D, true>(qf, k[cb]), a.scale, ms);
            lw[rb * 64] = l + s;
          }
        };
        KFrags<T, D> kB;
        for (;;) {
          const int nx = min(slab + kSlabWaves, end);
          if constexpr (SH::kTB == 2) {
            load_k<T, D>(a, kg, nx, 0, kB);
            process(kf);
            loads_landed();
            if ((slab += kSlabWaves) >= end) break;
            load_k<T, D>(a, kg, min(slab + kSlabWaves, end), 0, kf);
            process(kB);
            loads_landed();
            if ((slab += kSlabWaves) >= end) break;
          } else {
            load_k<T, D>(a, kg, slab, 1, kB);
            process(kf);
            loads_landed();
            load_k<T, D>(a, kg, nx, 0, kf);
            process(kB);
            loads_landed();
            if ((slab += kSlabWaves) >= end) break;
          }
        }
      }
    }
    __syncthreads();
    // the block's sums: every wave's, both lane halves, one reference per row
    float2* out = a.part + ((size_t)w.lg * a.n_chunks_max + w.chunk) * (a.nrb * 32);
    bool bad = false;
    for (int r = tid_here(); r < a.nrb * 32; r += kSlabThreads) {
      const float l = row_sum(a, l_s, r);
      out[r] = make_float2(ms_s[r], l);
      bad |= !(l < kSumLimit);
    }
    if (bad) *redo = 1;
    __syncthreads();
    if (*redo) {
      __syncthreads();   // the flag is read
      if (threadIdx.x == 0) *redo = 0;
      if (sum_again<T, D>(a, kg, qs, ms_s, l_s, w.s0, w.s1, out)) *redo = 1;
      __syncthreads();
      if (*redo) exact_rows<T, D>(a, kg, qs, w.s0, w.s1, out);
    }
    if (w.left <= 0) break;
    __syncthreads();   // the next segment overwrites the LDS
  }
}

// ---------------------------------------------------------------- merge
// c_r = M_r + log2(l_r) of row r of one (layer, group) from its blocks'
// statistics, in a fixed merge order; rows past R get +inf so that their
// 2^(y - c) vanishes in pass 2.  The first records are loaded ahead by
// merge_issue.
constexpr int kMergeBatch = 8;
// M + log2(l).  The logarithm is off by up to an ulp of its result, to one
// side.  Taken of l against the persistent pass 1's references, about 2^10 in
// ordinary calls and up to 2^32 under high logits, that was most of S's
// error; of l's mantissa in [0.5, 1) it is off by 2^-24 at most, and the sum
// is rounded once.  28 layers of 4 groups, 2,915 tokens, S against 64 bits:
// 3.1e-7 and 6.3e-8; with a key 24 log2 units above the others in every group
// 3.6e-7 and 6.2e-8.  Not for the small pass 1 (exact maxima, at most 256
// tokens a record, 1.7e-7): the statistics rank S, and a last bit that moves
// may swap two ranks at a bin's edge, so those calls keep theirs.
__device__ __forceinline__ float add_log2(float M, float l) {
  int e;
  const float m = frexpf(l, &e);
  return (float)((double)M + ((double)e + (double)log2f(m)));
}
__device__ __forceinline__ void merge_issue(const ScoreArgs& a, const float2* part, int n_chunks,
                                            int c0, int r, float2 (&p)[kMergeBatch]) {
#pragma unroll
  for (int j = 0; j < kMergeBatch; ++j)
    p[j] = part[(size_t)min(c0 + j, n_chunks - 1) * (a.nrb * 32) + r];
}
__device__ __forceinline__ float merge_row(const ScoreArgs& a, const float2* part, int n_chunks,
                                           int r, float2 (&p)[kMergeBatch]) {
  float Mx = kNegBig, lx = 0.f;
  for (int c0 = 0;;) {
    // one reference per batch; the records past the last repeat it with
    // nothing to add
    float mn = Mx;
#pragma unroll
    for (int j = 0; j < kMergeBatch; ++j) mn = fmaxf(mn, p[j].x);
    lx *= __builtin_amdgcn_exp2f(Mx - mn);
#pragma unroll
    for (int j = 0; j < kMergeBatch; ++j)
      lx += (c0 + j < n_chunks ? p[j].y : 0.f) * __builtin_amdgcn_exp2f(p[j].x - mn);
    Mx = mn;
    if ((c0 += kMergeBatch) >= n_chunks) break;
    merge_issue(a, part, n_chunks, c0, r, p);
  }
  if (r >= a.R) return INFINITY;
  return a.far ? add_log2(Mx, lx) : Mx + log2f(lx);
}

// ---------------------------------------------------------------- pass 2
// LDS: window rows, c[nrb * 32]; with row blocks split over waves (rs > 1)
// the waves' token sums [wave][64].
template <typename T, int D>
__host__ __device__ constexpr size_t pass2_lds(int nrb) {
  return (size_t)nrb * 32 * Shape<T, D>::kQStride + (size_t)nrb * 32 * 4 +
         (size_t)kSlabWaves * 64 * 4;
}

template <typename T, int D, int HL, bool PIPE>
__global__ __launch_bounds__(kSlabThreads) void score_pass2(ScoreArgs a, SlabGrid sg,
                                                              SlabGrid sg1) {
  using SH = Shape<T, D>;
  extern __shared__ __align__(16) unsigned char smem[];
  char* qs = reinterpret_cast<char*>(smem);
  float* cs = reinterpret_cast<float*>(smem + (size_t)a.nrb * 32 * SH::kQStride);
  float* red = cs + a.nrb * 32;
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int units = kSlabWaves / sg.rs, unit = wave / sg.rs, sub = wave % sg.rs;
  const int rb0 = a.nrb * sub / sg.rs, rb1 = a.nrb * (sub + 1) / sg.rs;
  const char* qlane = qs + l32 * SH::kQStride + half * 16;
  constexpr int kRB = 32 * SH::kQStride;

  for (SlabWalk w = slab_walk(sg, slab_block());; w = slab_next(sg, w)) {
    const int lg = w.lg, first = w.s0, end = w.s1;
    const T* kg = group_k<T>(a, lg);
    // the group's first output row: its only one, or its first head's
    float* srow = a.sraw + (size_t)lg * (HL ? a.n_out : 1) * a.Lp;

    KFrags<T, D> kf;
    int slab = end - 1 - unit;
    const bool any = slab >= first && rb0 < rb1;
    {
      const T* qg = group_q<T, D>(a, lg);
      const float2* part = a.part + (size_t)lg * a.n_chunks_max * (a.nrb * 32);
      const int n_chunks = slab_chunks(sg1, lg), r = tid_here();
      // one row per thread (at most 512 rows)
      float2 pv[kMergeBatch];
      i32x4 qv[kQBatch];
      if (r < a.nrb * 32) merge_issue(a, part, n_chunks, 0, r, pv);
      q_issue<T, D>(a, qg, tid_here(), qv);
      if (any) load_k<T, D>(a, kg, slab, 0, kf);
      __builtin_amdgcn_sched_barrier(0);
      if (r < a.nrb * 32) cs[r] = merge_row(a, part, n_chunks, r, pv);
      q_commit<T, D>(a, qg, qs, qv);
    }
    __syncthreads();

    // lane's token sum(s) of a finished slab or head: tile 0's in the lower
    // lane half, tile 1's in the upper
    auto store = [&](float* row, float v0, float v1) {
      const float v = add_halves(v0, v1);
      const int tok = slab * kSlab + lane;
      if (tok < a.Lp) row[tok] = v;
    };
    if (any) {
      if constexpr (PIPE) {
        i32x4 qf[SH::kNP];
        load_q<T, D>(qlane + rb0 * kRB, qf);
        f32x16 acc0 = chain<T, D, false>(qf, kf[0]), acc1;
        int turn = wave >> 2;
        for (;;) {
          take_turn(turn);
          const int next = slab - units;
          float s0 = 0.f, s1 = 0.f;   // the lane's tokens of the two tiles
          int left = a.upo;
          float* hrow = srow;
          auto flush = [&]() {
            if (HL == kHeadBlocks && --left == 0) {
              store(hrow, s0, s1);
              s0 = s1 = 0.f;
              hrow += a.Lp;
              left = a.upo;
            }
          };
          float c[16];
          for (int rb = rb0; rb + 1 < rb1; ++rb) {
            load_c(cs + rb * 32, half, c);
            s0 += stage2<D, true>(qf, kf[1], qlane + (rb + 1) * kRB, acc1, acc0, a.scale, c);
            s1 += stage2<D, false>(qf, kf[0], nullptr, acc0, acc1, a.scale, c);
            flush();
          }
          load_c(cs + (rb1 - 1) * 32, half, c);
          s0 += stage2<D, true>(qf, kf[1], qlane + rb0 * kRB, acc1, acc0, a.scale, c);
          // the slab's K is used up: the next slab's, behind the last tile's sums
          if (next >= first) load_k<T, D>(a, kg, next, 0, kf);
          __builtin_amdgcn_sched_barrier(0);
          s1 += tile_sum2(acc1, a.scale, c);
          flush();
          if (HL == kGroup) {
            if (sg.rs == 1) store(srow, s0, s1);
            else red[wave * 64 + lane] = add_halves(s0, s1);
          }
          if ((slab = next) < first) break;
          acc0 = chain<T, D, false>(qf, kf[0]);
        }
      } else {
        auto process = [&](KFrags<T, D>& k, int cb0) {
          constexpr int TB = SH::kTB;
          float s[2] = {0.f, 0.f};
          int left = a.upo, heads = a.n_out;
          float* hrow = srow;
          // one 32-token tile (kTB = 1): only the lower lanes' tokens exist
          auto put = [&](float* row) {
            const float v = add_halves(s[0], s[1]);
            const int tok = slab * kSlab + cb0 * 32 + lane;
            if (tok < a.Lp && (TB == 2 || half == 0)) row[tok] = v;
            s[0] = s[1] = 0.f;
          };
          for (int rb = rb0; rb < rb1; ++rb) {
            i32x4 qf[SH::kNP];
            load_q<T, D>(qlane + rb * kRB, qf);
            float c[16];
            load_c(cs + rb * 32, half, c);
            f32x16 acc[TB];
#pragma unroll
            for (int cb = 0; cb < TB; ++cb) acc[cb] = chain<T, D, false>(qf, k[cb]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
              for (int cb = 0; cb < TB; ++cb) {
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                  v[j] = __builtin_amdgcn_exp2f(fmaf(acc[cb][4 * i + j], a.scale, -c[4 * i + j]));
                s[cb] += (v[0] + v[1]) + (v[2] + v[3]);
              }
              // a head ends with this 8-row group, or with this row block;
              // the 8-row groups past the last head's are padding
              if ((HL == kHeadGroups || (HL == kHeadBlocks && i == 3)) && --left == 0 &&
                  heads > 0) {
                put(hrow);
                hrow += a.Lp;
                left = a.upo;
                --heads;
              }
            }
          }
          if (HL == kGroup) {
            if (sg.rs == 1) put(srow);
            else {
              const float v = add_halves(s[0], s[1]);
              if (TB == 2 || half == 0) red[wave * 64 + cb0 * 32 + lane] = v;
            }
          }
        };
        KFrags<T, D> kB;
        for (;;) {
          const int nx = max(slab - units, first);
          if constexpr (SH::kTB == 2) {
            load_k<T, D>(a, kg, nx, 0, kB);
            process(kf, 0);
            loads_landed();
            if ((slab -= units) < first) break;
            load_k<T, D>(a, kg, max(slab - units, first), 0, kf);
            process(kB, 0);
            loads_landed();
            if ((slab -= units) < first) break;
          } else {
            load_k<T, D>(a, kg, slab, 1, kB);
            process(kf, 0);
            loads_landed();
            load_k<T, D>(a, kg, nx, 0, kf);
            process(kB, 1);
            loads_landed();
            if ((slab -= units) < first) break;
          }
        }
      }
    }
    if (HL == kGroup && sg.rs > 1) {
      // one slab per unit of rs waves: add their parts in wave order
      if (!any) red[wave * 64 + lane] = 0.f;
      __syncthreads();
      const int u = wave, tok = (end - 1 - u) * kSlab + lane;
      if (u < units && end - 1 - u >= first && tok < a.Lp) {
        float v = 0.f;
        for (int w = 0; w < sg.rs; ++w) v += red[(u * sg.rs + w) * 64 + lane];
        srow[tok] = v;
      }
    }
    if (w.left <= 0) break;
    __syncthreads();   // the next segment overwrites the LDS
  }
}

// ---------------------------------------------------------------- pass 2, unrolled
// bf16 with d = 128 and up to eight row blocks, one sum per group or heads
// of whole row blocks (PH).  The row blocks are unrolled and a row block's
// two tiles computed together, with four accumulator tiles: each Q fragment
// read feeds two MFMAs in a row, and the exponentials of a row block (two
// tiles) run behind the MFMAs of the next.  7 row blocks, 28 layers of 4
// groups, this against the rolled kernel above: 26.2 / 27.8 us at 2,915
// tokens, 42.8 / 46.5 at 5,600, 106 / 112 at 13,679.  At 14 row blocks its
// registers spill and the rolled one is the faster (1771 / 1792 us at
// 140,190 tokens).
template <int NRB, bool PH>
__global__ __launch_bounds__(kSlabThreads) void score_pass2_unrolled(ScoreArgs a, SlabGrid sg,
                                                                     SlabGrid sg1) {
  constexpr int NW = kSlabWaves, TB = 2;
  constexpr int QS = Shape<__bf16, 128>::kQStride / 2;     // padded Q row
  extern __shared__ __align__(16) unsigned char smem[];
  __bf16* qs = reinterpret_cast<__bf16*>(smem);
  float* cs = reinterpret_cast<float*>(smem + (size_t)NRB * 32 * QS * 2);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const __bf16* qlane = qs + l32 * QS + half * 8;
  const float* clane = cs + 4 * half;

  for (SlabWalk w = slab_walk(sg, slab_block());; w = slab_next(sg, w)) {
    const int s0 = w.s0, s1 = w.s1;
    const __bf16* kg = group_k<__bf16>(a, w.lg);
    // the group's first output row: its only one, or its first head's
    float* srow = a.sraw + (size_t)w.lg * (PH ? a.n_out : 1) * a.Lp;
    {
      const __bf16* qg = group_q<__bf16, 128>(a, w.lg);
      constexpr int NV = NRB * 32 * 16;
      constexpr int PER = (NV + kSlabThreads - 1) / kSlabThreads;
      constexpr int BATCH = PER < 7 ? PER : 7;
#pragma unroll
      for (int j0 = 0; j0 < PER; j0 += BATCH) {
        i32x4 v[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
          const int i = threadIdx.x + (j0 + j) * kSlabThreads, row = i >> 4, part = i & 15;
          v[j] = i32x4{0, 0, 0, 0};
          if (j0 + j < PER && i < NV && row < a.R)
            v[j] = *reinterpret_cast<const i32x4*>(qg + (size_t)row * 128 + part * 8);
        }
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
          const int i = threadIdx.x + (j0 + j) * kSlabThreads, row = i >> 4, part = i & 15;
          if (j0 + j < PER && i < NV) *reinterpret_cast<i32x4*>(qs + row * QS + part * 8) = v[j];
        }
      }
    }
    if (threadIdx.x < NRB * 32) {
      const float2* part = a.part + (size_t)w.lg * a.n_chunks_max * (NRB * 32);
      const int n_chunks = slab_chunks(sg1, w.lg);
      float2 pv[kMergeBatch];
      merge_issue(a, part, n_chunks, 0, threadIdx.x, pv);
      cs[threadIdx.x] = merge_row(a, part, n_chunks, threadIdx.x, pv);
    }
    KFrags<__bf16, 128> kf;
    if (s1 - 1 - wave >= s0) load_k<__bf16, 128>(a, kg, s1 - 1 - wave, 0, kf);
    __syncthreads();

    for (int slab = s1 - 1 - wave; slab >= s0; slab -= NW) {
      // two partial sums per token block keep the add chains short
      float s[TB][2];
#pragma unroll
      for (int cb = 0; cb < TB; ++cb) { s[cb][0] = 0.f; s[cb][1] = 0.f; }
      f32x16 accA[TB], accB[TB];
      i32x4 qf[8];
      // row block 0's chain; the fragments of row block 1 are read as
      // those of row block 0 are consumed
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) qf[kk] = *reinterpret_cast<const i32x4*>(qlane + kk * 16);
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
#pragma unroll
        for (int cb = 0; cb < TB; ++cb) accA[cb] = mma16<__bf16>(qf[kk], kf[cb][kk], kk ? accA[cb] : f32x16{});
        if (NRB > 1) qf[kk] = *reinterpret_cast<const i32x4*>(qlane + 32 * QS + kk * 16);
      }
      __builtin_amdgcn_sched_barrier(0);
      // stage rb: MFMAs of row block rb+1 (reading the Q fragments of rb+2
      // behind them), interleaved with the exponentials of row block rb
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        f32x16 (&cur)[TB] = (rb & 1) ? accB : accA;
        f32x16 (&nxt)[TB] = (rb & 1) ? accA : accB;
        // c of the rows this lane receives: rb*32 + 8i + 4*half + j
        float c[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 c4 = *reinterpret_cast<const f32x4*>(clane + rb * 32 + 8 * i);
#pragma unroll
          for (int j = 0; j < 4; ++j) c[4 * i + j] = c4[j];
        }
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
          if (rb + 1 < NRB) {
#pragma unroll
            for (int cb = 0; cb < TB; ++cb) nxt[cb] = mma16<__bf16>(qf[kk], kf[cb][kk], kk ? nxt[cb] : f32x16{});
            if (rb + 2 < NRB) qf[kk] = *reinterpret_cast<const i32x4*>(qlane + (rb + 2) * 32 * QS + kk * 16);
          }
#pragma unroll
          for (int cb = 0; cb < TB; ++cb)
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2)
              s[cb][h2] += __builtin_amdgcn_exp2f(fmaf(cur[cb][2 * kk + h2], a.scale, -c[2 * kk + h2]));
          if (rb + 1 < NRB) {
            // one MFMA, then the epilogue's share of six VALU operations
#pragma unroll
            for (int cb = 0; cb < TB; ++cb) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
            }
            if (rb + 2 < NRB) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
        }
        // pin the partial sums to this stage: the compiler would otherwise
        // sink every stage's exponentials to the end of the slab and keep
        // all accumulators alive
#pragma unroll
        for (int cb = 0; cb < TB; ++cb) {
          asm volatile("" : "+v"(s[cb][0]));
          asm volatile("" : "+v"(s[cb][1]));
        }
        if (PH && (rb + 1) % a.upo == 0) {
          // the last row block of head rb / upo: its output, then a fresh sum
          float* hrow = srow + (size_t)(rb / a.upo) * a.Lp;
#pragma unroll
          for (int cb = 0; cb < TB; ++cb) {
            const float sc = s[cb][0] + s[cb][1];
            const float v = sc + other_half(sc, half);
            const int tok = slab * kSlab + cb * 32 + l32;
            if ((cb & 1) == half && tok < a.Lp) hrow[tok] = v;
            s[cb][0] = 0.f;
            s[cb][1] = 0.f;
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      const int t0 = slab * kSlab;
      if (slab - NW >= s0) load_k<__bf16, 128>(a, kg, slab - NW, 0, kf);
      // lanes l and l ^ 32 hold the same token's two row halves; half h
      // stores token block h
      if (!PH) {
#pragma unroll
        for (int cb = 0; cb < TB; ++cb) {
          const float sc = s[cb][0] + s[cb][1];
          const float v = sc + other_half(sc, half);
          const int tok = t0 + cb * 32 + l32;
          if ((cb & 1) == half && tok < a.Lp) srow[tok] = v;
        }
      }
    }
    if (w.left <= 0) break;
    __syncthreads();   // the next segment overwrites the LDS
  }
}

template <int NRB>
void launch_unrolled(const ScoreArgs& a, const SlabLaunch& p2, const SlabGrid& g1,
                     hipStream_t st) {
  const size_t lds = (size_t)NRB * 32 * (Shape<__bf16, 128>::kQStride + 4);
  if (a.n_out > 1)
    score_pass2_unrolled<NRB, true><<<p2.blocks, kSlabThreads, lds, st>>>(a, p2.g, g1);
  else
    score_pass2_unrolled<NRB, false><<<p2.blocks, kSlabThreads, lds, st>>>(a, p2.g, g1);
}

// ---------------------------------------------------------------- small calls
// Few slabs for the GPU: a launch is then its start and one short chain of
// dependent steps, and the persistent kernels' steps (window rows to LDS,
// references, the slab loop) come one after another.  Here the waves of a
// block have a row block each (NW of them at most; with few row blocks,
// several waves share one and split its tokens), whose window rows go
// straight into registers, and K is read once through LDS.

// Rows [0, n) of K from token t0 on to LDS, coalesced; n_rows rows are
// written, those past n repeating the last.
template <typename T, int D, int NW>
__device__ __forceinline__ void stage_rows(const ScoreArgs& a, const T* kg, int t0, int n,
                                           int n_rows, char* ks) {
  using SH = Shape<T, D>;
  constexpr int VPR = SH::kRowBytes / 16, BATCH = 8;
  constexpr int NT = NW * 64;
  const int nv = n_rows * VPR;
  const char* base = reinterpret_cast<const char*>(kg + (int64_t)t0 * a.ts);
  for (int i0 = threadIdx.x; i0 < nv; i0 += BATCH * NT) {
    i32x4 v[BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int i = i0 + j * NT, row = min(i / VPR, n - 1), part = i % VPR;
      if (i < nv)
        v[j] = *reinterpret_cast<const i32x4*>(base + (int64_t)row * (a.ts * (int64_t)sizeof(T)) +
                                               part * 16);
    }
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int i = i0 + j * NT, row = i / VPR, part = i % VPR;
      if (i < nv) *reinterpret_cast<i32x4*>(ks + row * SH::kQStride + part * 16) = v[j];
    }
  }
}

// The wave's row block of window rows, zero past R.
template <typename T, int D>
__device__ __forceinline__ void load_rows(const ScoreArgs& a, const T* qg, int rb,
                                          i32x4 (&qf)[Shape<T, D>::kNP]) {
  const int lane = threadIdx.x & 63, half = lane >> 5, row = rb * 32 + (lane & 31);
  const char* q = reinterpret_cast<const char*>(qg + (size_t)min(row, a.R - 1) * D) + half * 16;
#pragma unroll
  for (int j = 0; j < Shape<T, D>::kNP; ++j) {
    qf[j] = *reinterpret_cast<const i32x4*>(q + j * 32);
    if (row >= a.R) qf[j] = i32x4{0, 0, 0, 0};
  }
}

// Pass 1: block (lg, chunk) of per_lg = ceil(L_p / 256) chunks; exact
// running maxima, slab by slab.  parts waves share a row block, slab by slab.
template <typename T, int D, int NW>
__global__ __launch_bounds__(NW * 64) void score_pass1_small(ScoreArgs a, int per_lg, int parts) {
  using SH = Shape<T, D>;
  __shared__ float2 ml[NW * 32];
  extern __shared__ __align__(16) unsigned char smem[];
  char* ks = reinterpret_cast<char*>(smem);
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int part = wave / a.nrb, rb = wave - part * a.nrb;
  const int b = slab_block(), lg = b / per_lg, chunk = b - lg * per_lg;
  const int t0 = chunk * kSmallRows, n = min(kSmallRows, a.Lp - t0);
  const int slabs = (n + kSlab - 1) / kSlab;
  i32x4 qf[SH::kNP];
  load_rows<T, D>(a, group_q<T, D>(a, lg), rb, qf);
  stage_rows<T, D, NW>(a, group_k<T>(a, lg), t0, n, slabs * kSlab, ks);
  __syncthreads();
  float m = kNegBig, l = 0.f;
  const char* krow = ks + l32 * SH::kQStride + half * 16;
  for (int s = part < parts ? part : slabs; s < slabs; s += parts) {
    f32x16 acc[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      i32x4 kf[SH::kNP];
      load_q<T, D>(krow + (s * kSlab + cb * 32) * SH::kQStride, kf);
      acc[cb] = chain<T, D, true>(qf, kf);
    }
    if ((s + 1) * kSlab > n) {
      mask_tokens(acc[0], t0 + s * kSlab, a.Lp);
      mask_tokens(acc[1], t0 + s * kSlab + 32, a.Lp);
    }
    float mt = fmaxf(acc[0][0], acc[1][0]);
#pragma unroll
    for (int e = 1; e < 16; ++e) mt = fmaxf(mt, fmaxf(acc[0][e], acc[1][e]));
    const float mn = fmaxf(m, mt), msn = mn * a.scale;
    const float sum = tile_sum1(acc[0], a.scale, msn) + tile_sum1(acc[1], a.scale, msn);
    l = l * rescale(m, mn, msn, a.scale) + sum;
    m = mn;
  }
  const float mo = other_half(m, half), lo = other_half(l, half);
  float mn = fmaxf(m, mo), msn = mn * a.scale;
  l = l * rescale(m, mn, msn, a.scale) + lo * rescale(mo, mn, msn, a.scale);
  if (parts > 1) {   // the row block's waves, in order (an idle one adds 0)
    if (half == 0) ml[wave * 32 + l32] = make_float2(mn, l);
    __syncthreads();
    if (part > 0) return;
    for (int p = 1; p < parts; ++p) {
      const float2 o = ml[(p * a.nrb + rb) * 32 + l32];
      const float mm = fmaxf(mn, o.x);
      msn = mm * a.scale;
      l = l * rescale(mn, mm, msn, a.scale) + o.y * rescale(o.x, mm, msn, a.scale);
      mn = mm;
    }
  } else if (part > 0) {
    return;
  }
  if (half == 0)
    a.part[((size_t)lg * a.n_chunks_max + chunk) * (a.nrb * 32) + rb * 32 + l32] =
        make_float2(msn, l);
}

// Pass 2: block (lg, slab); the records of pass 1's division sg1.  n_out
// outputs, of upo row blocks each.  With at most half as many row blocks as
// waves two waves share one, a tile each.
template <typename T, int D, int NW>
__global__ __launch_bounds__(NW * 64) void score_pass2_small(ScoreArgs a, int S, SlabGrid sg1) {
  using SH = Shape<T, D>;
  __shared__ __align__(16) float cs[NW * 32];
  __shared__ float red[NW * 64];
  extern __shared__ __align__(16) unsigned char smem[];
  char* ks = reinterpret_cast<char*>(smem);
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool split = 2 * a.nrb <= NW;
  const int part = wave / a.nrb, rb = wave - part * a.nrb;
  const int b = slab_block(), lg = b / S, slab = b - lg * S;
  const int t0 = slab * kSlab;
  const float2* rec = a.part + (size_t)lg * a.n_chunks_max * (a.nrb * 32);
  const int n_chunks = slab_chunks(sg1, lg), row = threadIdx.x;
  float2 pv[kMergeBatch];
  i32x4 qf[SH::kNP];
  if (row < a.nrb * 32) merge_issue(a, rec, n_chunks, 0, row, pv);
  load_rows<T, D>(a, group_q<T, D>(a, lg), rb, qf);
  stage_rows<T, D, NW>(a, group_k<T>(a, lg), t0, min(kSlab, a.Lp - t0), kSlab, ks);
  if (row < a.nrb * 32) cs[row] = merge_row(a, rec, n_chunks, row, pv);
  __syncthreads();
  if (part < (split ? 2 : 1)) {
    float c[16];
    load_c(cs + rb * 32, half, c);
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      if (split && part != cb) continue;
      i32x4 kf[SH::kNP];
      load_q<T, D>(ks + (cb * 32 + l32) * SH::kQStride + half * 16, kf);
      const float s = tile_sum2(chain<T, D, false>(qf, kf), a.scale, c);
      const float v = s + other_half(s, half);
      if (half == 0) red[rb * 64 + cb * 32 + l32] = v;
    }
  }
  __syncthreads();
  if (wave >= a.n_out || t0 + lane >= a.Lp) return;
  const int upo = a.n_out == 1 ? a.nrb : a.upo;
  float v = 0.f;
  for (int u = wave * upo; u < (wave + 1) * upo; ++u) v += red[u * 64 + lane];
  a.sraw[((size_t)lg * a.n_out + wave) * a.Lp + t0 + lane] = v;
}

// Pass 2 with one sum per group, or heads of whole row blocks.  The unrolled
// kernels are compiled only for the keys they serve.
template <typename T, int D>
void run_pass2_blocks(const ScoreArgs& a, const SlabLaunch& p2, const SlabGrid& g1,
                      hipStream_t st) {
  constexpr bool kPipe = sizeof(T) == 2;   // tiles interleaved
  if constexpr (pass2_unrolled(D, (int)sizeof(T), 1, true)) {
    switch (a.nrb) {
#define STARKV_NRB(n) \
  case n: return launch_unrolled<n>(a, p2, g1, st);
      STARKV_NRB(1) STARKV_NRB(2) STARKV_NRB(3) STARKV_NRB(4) STARKV_NRB(5) STARKV_NRB(6)
      STARKV_NRB(7) STARKV_NRB(8)
#undef STARKV_NRB
    }
    static_assert(kUnrolledBlocks == 8, "a case for every unrolled row-block count");
  }
  const size_t lds = pass2_lds<T, D>(a.nrb);
  if (a.n_out == 1)
    score_pass2<T, D, kGroup, kPipe><<<p2.blocks, kSlabThreads, lds, st>>>(a, p2.g, g1);
  else
    score_pass2<T, D, kHeadBlocks, kPipe><<<p2.blocks, kSlabThreads, lds, st>>>(a, p2.g, g1);
}

template <typename T, int D>
int run_passes(const ScoreArgs& a, const SlabLaunch& p1, const SlabLaunch& p2, hipStream_t st) {
  constexpr bool kPipe = sizeof(T) == 2;   // tiles interleaved
  const size_t lds2 = pass2_lds<T, D>(a.nrb);
  // float32 has four row blocks at most
  constexpr int kMost = sizeof(T) == 2 ? kSmallMost : kSmallWaves;
  const bool most = a.nrb > kSmallWaves;
  if (p1.small) {
    const size_t lds = (size_t)kSmallRows * Shape<T, D>::kQStride;
    const int slabs = kSmallRows / kSlab, parts = std::min(slabs, kSmallWaves / a.nrb);
    if (most)
      score_pass1_small<T, D, kMost><<<p1.blocks, kMost * 64, lds, st>>>(a, p1.g.per_lg, 1);
    else
      score_pass1_small<T, D, kSmallWaves><<<p1.blocks, kSmallWaves * 64, lds, st>>>(
          a, p1.g.per_lg, parts);
  } else {
    score_pass1<T, D, kPipe><<<p1.blocks, kSlabThreads, pass1_lds<T, D>(a.nrb), st>>>(a, p1.g);
  }
  const size_t slab_lds = (size_t)kSlab * Shape<T, D>::kQStride;
  if (p2.small && most)
    score_pass2_small<T, D, kMost><<<p2.blocks, kMost * 64, slab_lds, st>>>(a, p2.g.S, p1.g);
  else if (p2.small)
    score_pass2_small<T, D, kSmallWaves><<<p2.blocks, kSmallWaves * 64, slab_lds, st>>>(a, p2.g.S,
                                                                                    p1.g);
  else if (a.n_out > 1 && a.W % 32 != 0)
    score_pass2<T, D, kHeadGroups, false><<<p2.blocks, kSlabThreads, lds2, st>>>(a, p2.g, p1.g);
  else
    run_pass2_blocks<T, D>(a, p2, p1.g, st);
  return (int)hipGetLastError();
}

}  // namespace

// The two passes, one translation unit per element type.
int run_score_bf16(const ScoreArgs& a, int d, const SlabLaunch& p1, const SlabLaunch& p2,
                   hipStream_t st);
int run_score_f32(const ScoreArgs& a, int d, const SlabLaunch& p1, const SlabLaunch& p2,
                  hipStream_t st);

}  // namespace starkv
