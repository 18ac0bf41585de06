// Narrow policies in four wavefronts per episode: binary32.
#include "rollout_wave_team.hpp"

namespace es {

template <int M>
static int launch_mode(es_ctx* ctx, int mode, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a) {
  return mode == 2 ? launch_team_obs<2, false, M>(ctx, grid, lds, st, a) : launch_team_obs<-1, false, M>(ctx, grid, lds, st, a);
}

int launch_team_f32(es_ctx* ctx, int mode, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a) {
  if (ctx->shp.m == 2) return launch_mode<2>(ctx, mode, grid, lds, st, a);
  return ctx->shp.m == 3 ? launch_mode<3>(ctx, mode, grid, lds, st, a) : launch_mode<4>(ctx, mode, grid, lds, st, a);
}

}  // namespace es
