#include "gemm_wide.hpp"

namespace phyai {

void gemm_wide(const GemmArgs& g, const EpiGeglu<bf16_t>& e, WideTile t, hipStream_t s) {
  if (g.kind == W_FP8) wide_launch<EpiGeglu<bf16_t>, false, W_FP8>(g, e, t, s);
  else wide_launch<EpiGeglu<bf16_t>, false, W_BF16>(g, e, t, s);
}

void gemm_wide(const GemmArgs& g, const EpiGegluLo& e, WideTile t, hipStream_t s) {
  if (g.kind == W_FP8) wide_launch<EpiGegluLo, true, W_FP8>(g, e, t, s);
  else wide_launch<EpiGegluLo, true, W_BF16>(g, e, t, s);
}

}  // namespace phyai
