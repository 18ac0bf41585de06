// Sixteen-column rollout kernel in one wavefront: bf16 operands.
#include "rollout_cols.hpp"

namespace es {

int launch_cols_bf16(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  if (a.nh <= 32) return launch_cols_bf16<2>(ctx, a, fitness, st);
  return a.nh <= 48 ? launch_cols_bf16<3>(ctx, a, fitness, st) : launch_cols_bf16<4>(ctx, a, fitness, st);
}

}  // namespace es
