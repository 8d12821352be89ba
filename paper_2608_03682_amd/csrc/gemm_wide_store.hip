#include "gemm_wide.hpp"

namespace phyai {

void gemm_wide(const GemmArgs& g, const EpiStore<bf16_t>& e, WideTile t, hipStream_t s) {
  if (g.kind == W_FP8) wide_launch<EpiStore<bf16_t>, false, W_FP8>(g, e, t, s);
  else wide_launch<EpiStore<bf16_t>, false, W_BF16>(g, e, t, s);
}

void gemm_wide(const GemmArgs& g, const EpiStore<float>& e, WideTile t, hipStream_t s) {
  if (g.kind == W_FP8) wide_launch<EpiStore<float>, false, W_FP8>(g, e, t, s);
  else wide_launch<EpiStore<float>, false, W_BF16>(g, e, t, s);
}

}  // namespace phyai
