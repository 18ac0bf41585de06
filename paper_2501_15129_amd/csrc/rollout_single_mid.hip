// One copy per workgroup of four wavefronts: binary32, 65 to 128 hidden units.
#include "rollout_single.hpp"

namespace es {

template <int M>
static int launch_obs(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  if (a.no <= 20) return launch_single_mode<4, 5, M>(ctx, a, fitness, st);
  return a.no <= 32 ? launch_single_mode<4, 8, M>(ctx, a, fitness, st) : launch_single_mode<4, 16, M>(ctx, a, fitness, st);
}

int launch_single_mid(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  if (ctx->shp.m == 1) return launch_obs<1>(ctx, a, fitness, st);
  return ctx->shp.m == 2 ? launch_obs<2>(ctx, a, fitness, st) : launch_obs<3>(ctx, a, fitness, st);
}

}  // namespace es
