// Checks the scoring passes' division of slabs into blocks (slab_grid.h, the
// same source the library compiles) for each "Lp nlg nrb n_cu max_chunks
// one_sum whole_blocks [d element-bytes]" line of stdin: prints "ok", or what
// is wrong, the two passes' kinds, their block counts and the waves that share
// a slab in pass 2.
#include <cstdio>
#include <string>
#include <vector>

#include "slab_grid.h"

using namespace starkv;

static const char* check(const SlabLaunch& l, int nlg, int max_chunks, bool records) {
  const SlabGrid& g = l.g;
  if (l.blocks < 1) return "no blocks";
  std::vector<int> next(nlg, 0), chunks(nlg, 0);
  for (int b = 0; b < l.blocks; ++b) {
    for (SlabWalk w = slab_walk(g, b);; w = slab_next(g, w)) {
      if (w.lg < 0 || w.lg >= nlg) return "group out of range";
      if (w.s1 <= w.s0) return "empty segment";
      if (w.s0 != next[w.lg]) return "slab missed or repeated";
      if (w.chunk != chunks[w.lg]) return "record index not in block order";
      next[w.lg] = w.s1;
      ++chunks[w.lg];
      if (g.rs > 1 && (w.s1 - w.s0) * g.rs > kSlabWaves) return "shared slabs do not fit";
      if (w.left <= 0) break;
    }
  }
  for (int i = 0; i < nlg; ++i) {
    if (next[i] != g.S) return "slabs left over";
    if (slab_chunks(g, i) != chunks[i]) return "record count";
    if (records && chunks[i] > max_chunks) return "too many records";
  }
  return nullptr;
}

int main() {
  char line[256];
  while (std::fgets(line, sizeof line, stdin)) {
    int Lp, nlg, nrb, n_cu, mc, one, whole, d = 64, esz = 2;
    if (std::sscanf(line, "%d %d %d %d %d %d %d %d %d", &Lp, &nlg, &nrb, &n_cu, &mc, &one,
                    &whole, &d, &esz) < 7)
      return 1;
    SlabLaunch p1, p2;
    slab_launches(Lp, nlg, nrb, n_cu, mc, one != 0, whole != 0, d, esz, &p1, &p2);
    const char* bad = nullptr;
    if (p1.small) {   // its blocks take kSmallRows tokens each
      const int n = (Lp + kSmallRows - 1) / kSmallRows;
      if (p1.g.per_lg != n || slab_chunks(p1.g, 0) != n || p1.blocks != n * nlg || n > mc)
        bad = "small pass 1";
    } else {
      bad = check(p1, nlg, mc, true);
    }
    if (!bad && p2.small) bad = p2.blocks == p2.g.S * nlg && whole ? nullptr : "small pass 2";
    else if (!bad) bad = check(p2, nlg, mc, false);
    if (!bad && !one && p2.g.rs != 1) bad = "shared slabs with several outputs";
    if (!bad && pass2_unrolled(d, esz, nrb, whole != 0) && p2.g.rs != 1)
      bad = "shared slabs in the unrolled kernel";
    if (!bad && p1.g.rs != 1) bad = "shared slabs in pass 1";
    std::printf("%s %s %s %d %d %d\n", bad ? bad : "ok",
                p1.small ? "small" : p1.g.per_lg ? "aligned" : "crossing",
                p2.small ? "small" : p2.g.per_lg ? "aligned" : "crossing", p1.blocks, p2.blocks,
                p2.g.rs);
  }
  return 0;
}
