// Block shape of the statistics kernel (threads per block) for a call, from
// its block count, the GPU's CU count and the binning parameters.  Host and
// tests share this code; the kernel's LDS partitions per shape live in
// state.hip (StatsShape).
//   1024  the wide shape, one block per CU: when every block fits on the GPU
//         at once, or the bins need its LDS;
//   512   the narrow shape, two blocks per CU (n_bins <= kNarrowMaxBins);
//   256   the small shape, four blocks per CU, when even two per CU leave
//         blocks for a second round (n_bins <= kSmallMaxBins and
//         grid^2 <= kSmallMaxCells).
// A layer's blocks: one per subspace (MI), one for the AEB statistic and
// stats_stab_blocks for the stability means, kStabSubspaces subspaces each;
// the shape is chosen by these.  A wide launch at a long context has
// kEntropyBlocks - 1 more per layer (stats_entropy_blocks).
#pragma once

namespace starkv {

constexpr int kNarrowMaxBins = 17;
constexpr int kSmallMaxBins = 9;
constexpr int kSmallMaxCells = 64;
constexpr int kStabSubspaces = 8;

inline int stats_stab_blocks(int n_sub) { return (n_sub + kStabSubspaces - 1) / kStabSubspaces; }
inline int stats_layer_blocks(int n_sub) { return n_sub + 1 + stats_stab_blocks(n_sub); }

// Entropy blocks of a layer.  A block adds up all of s-bar for the
// normaliser, then its part of p log p in float64.  One block takes 137 us at
// 140,190 tokens, longer than the MI blocks; from about 96K tokens four share
// it, while the launch stays within five blocks per four CUs (the last ones
// then start as the first entropy and stability blocks end).  us of the fused
// call, four blocks / one:
//   140,254 tokens: 1 layer of 4 groups 236 / 254, 28 layers 265 / 275, 37
//     layers (333 blocks) 266 / 282, 42 layers (378) 295 / 286
//    93,332 tokens: 1 layer 164 / 173, 28 layers 188 / 187, 25 layers of 8
//     groups (325 blocks) 206 / 190
//    35,495 tokens: 1 layer 83 / 82, 28 layers 92 / 88, 25 layers of 8 groups
//     112 / 91
constexpr int kEntropyBlocks = 4;
constexpr int kEntropySplitTokens = 96 * 1024;
inline int stats_entropy_blocks(int Lp, bool entropy, long n_layers, int n_sub, int n_cu) {
  const long blocks = n_layers * (stats_layer_blocks(n_sub) + kEntropyBlocks - 1);
  return entropy && Lp >= kEntropySplitTokens && blocks <= n_cu + n_cu / 4 ? kEntropyBlocks : 1;
}

inline int stats_shape_for(long blocks, int n_cu, int n_bins, int grid) {
  if (blocks <= n_cu || n_bins > kNarrowMaxBins) return 1024;
  if (blocks > 2L * n_cu && n_bins <= kSmallMaxBins && grid * grid <= kSmallMaxCells)
    return 256;
  return 512;
}

}  // namespace starkv
