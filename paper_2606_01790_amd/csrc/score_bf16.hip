// bf16 instantiations of the scoring passes (v_mfma_f32_32x32x16_bf16).
#include "score_slab.h"

namespace starkv {

int run_score_bf16(const ScoreArgs& a, int d, const SlabLaunch& p1, const SlabLaunch& p2,
                   hipStream_t st) {
  return d == 128 ? run_passes<__bf16, 128>(a, p1, p2, st)
                  : run_passes<__bf16, 64>(a, p1, p2, st);
}

}  // namespace starkv
