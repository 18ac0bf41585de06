// Four-copy rollout kernel in one wavefront, binary32 and bf16: up to 64 hidden units, two hidden layers, obs <= 64, act <= 16,
// for populations that fill the chip.
#include "rollout_quad.hpp"

namespace es {

int launch_quad_narrow(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  if (ctx->cfg.dtype == 1)
    return a.no <= 32 && !a.obs_mean ? launch_quad_options<true, 1, 8, 2, 4, false, false>(ctx, a, fitness, st) : launch_quad_options<true, 1, 16, 2, 4, true, false>(ctx, a, fitness, st);
  if (a.no <= 16) return launch_quad_options<false, 1, 4, 2, 4, true, false>(ctx, a, fitness, st);
  return a.no <= 32 ? launch_quad_options<false, 1, 8, 2, 4, true, false>(ctx, a, fitness, st) : launch_quad_options<false, 1, 16, 2, 4, true, false>(ctx, a, fitness, st);
}

}  // namespace es
