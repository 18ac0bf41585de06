// One copy per workgroup of eight wavefronts: binary32, 129 to 256 hidden units.
#include "rollout_single.hpp"

namespace es {

template <int M>
static int launch_obs(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  if (a.no <= 12) return launch_single_mode<8, 3, M>(ctx, a, fitness, st);
  return a.no <= 20 ? launch_single_mode<8, 5, M>(ctx, a, fitness, st) : launch_single_mode<8, 8, M>(ctx, a, fitness, st);
}

int launch_single_wide(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  return ctx->shp.m == 1 ? launch_obs<1>(ctx, a, fitness, st) : launch_obs<2>(ctx, a, fitness, st);
}

}  // namespace es
