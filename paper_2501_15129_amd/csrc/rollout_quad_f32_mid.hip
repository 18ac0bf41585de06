// Four-copy rollout kernel, binary32, two wavefronts: 65..128 hidden units, one to three hidden layers, obs <= 64, act <= 16.
#include "rollout_quad.hpp"

namespace es {

int launch_quad_f32_mid(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  if (ctx->shp.m == 1) return launch_quad_obs64<false, 2, 1, false>(ctx, a, fitness, st);
  return ctx->shp.m == 2 ? launch_quad_obs64<false, 2, 2, false>(ctx, a, fitness, st) : launch_quad_obs64<false, 2, 3, false>(ctx, a, fitness, st);
}

}  // namespace es
