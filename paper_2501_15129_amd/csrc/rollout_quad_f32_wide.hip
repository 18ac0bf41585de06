// Four-copy rollout kernel, binary32: 129..256 hidden units, one or two hidden layers, obs <= 64, act <= 16.
#include "rollout_quad.hpp"

namespace es {

int launch_quad_f32_wide(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  return ctx->shp.m == 1 ? launch_quad_obs64<false, 4, 1, false>(ctx, a, fitness, st) : launch_quad_obs64<false, 4, 2, false>(ctx, a, fitness, st);
}

}  // namespace es
