// Four-copy rollout kernel, bf16 operands: 128..256 hidden units, four hidden layers, obs <= 64, act <= 16.
#include "rollout_quad.hpp"

namespace es {

int launch_quad_bf16_deep4(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  return launch_quad_obs64<true, 4, 4, false>(ctx, a, fitness, st);
}

}  // namespace es
