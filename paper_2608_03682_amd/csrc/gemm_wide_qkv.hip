#include "gemm_wide.hpp"

namespace phyai {

void gemm_wide(const GemmArgs& g, const EpiQkv<bf16_t>& e, WideTile t, hipStream_t s) {
  if (g.A_lo) {
    if (g.kind == W_FP8) wide_launch<EpiQkv<bf16_t>, true, W_FP8>(g, e, t, s);
    else wide_launch<EpiQkv<bf16_t>, true, W_BF16>(g, e, t, s);
    return;
  }
  if (g.kind == W_FP8) wide_launch<EpiQkv<bf16_t>, false, W_FP8>(g, e, t, s);
  else wide_launch<EpiQkv<bf16_t>, false, W_BF16>(g, e, t, s);
}

}  // namespace phyai
