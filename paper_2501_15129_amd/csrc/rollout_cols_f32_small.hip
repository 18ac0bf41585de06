// Sixteen-column rollout kernel in one wavefront: binary32, up to 32 hidden units.
#include "rollout_cols.hpp"

namespace es {

int launch_cols_f32_small(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  return a.nh <= 16 ? launch_cols_f32<1>(ctx, a, fitness, st) : launch_cols_f32<2>(ctx, a, fitness, st);
}

}  // namespace es
