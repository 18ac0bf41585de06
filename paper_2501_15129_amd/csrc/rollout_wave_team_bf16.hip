// Narrow policies in four wavefronts per episode: bf16 operands.
#include "rollout_wave_team.hpp"

namespace es {

int launch_team_bf16(es_ctx* ctx, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a) {
  if (ctx->shp.m == 2) return launch_team_obs<-1, true, 2>(ctx, grid, lds, st, a);
  return ctx->shp.m == 3 ? launch_team_obs<-1, true, 3>(ctx, grid, lds, st, a) : launch_team_obs<-1, true, 4>(ctx, grid, lds, st, a);
}

}  // namespace es
