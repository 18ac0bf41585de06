// Narrow policies in numbers that fill the chip, binary32 and bf16: up to 64 hidden units, two hidden layers, obs <= 64, act <= 16, in passes of four
// or sixteen copies, one wavefront each.
#include "rollout_cols.hpp"

namespace es {

int launch_quad_narrow(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  if (ctx->rollout().kind == ROLLOUT_COLS) {
    if (ctx->cfg.dtype == 1) return launch_cols_bf16(ctx, a, fitness, st);
    if (a.nh <= 32) return launch_cols_f32_small(ctx, a, fitness, st);
    return a.nh <= 48 ? launch_cols_f32_48(ctx, a, fitness, st) : launch_cols_f32_64(ctx, a, fitness, st);
  }
  if (ctx->cfg.dtype == 1)
    return a.no <= 32 && !a.obs_mean ? launch_quad_options<true, 1, 8, 2, 4, false, false>(ctx, a, fitness, st) : launch_quad_options<true, 1, 16, 2, 4, true, false>(ctx, a, fitness, st);
  if (a.no <= 16) return launch_quad_options<false, 1, 4, 2, 4, true, false>(ctx, a, fitness, st);
  return a.no <= 32 ? launch_quad_options<false, 1, 8, 2, 4, true, false>(ctx, a, fitness, st) : launch_quad_options<false, 1, 16, 2, 4, true, false>(ctx, a, fitness, st);
}

}  // namespace es
