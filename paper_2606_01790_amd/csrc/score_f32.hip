// float32 instantiations of the scoring passes (v_mfma_f32_32x32x2f32), for
// up to four 32-row blocks of window rows per group.
#include "score_slab.h"

namespace starkv {

int run_score_f32(const ScoreArgs& a, int d, const SlabLaunch& p1, const SlabLaunch& p2,
                  hipStream_t st) {
  return d == 128 ? run_passes<float, 128>(a, p1, p2, st)
                  : run_passes<float, 64>(a, p1, p2, st);
}

}  // namespace starkv
