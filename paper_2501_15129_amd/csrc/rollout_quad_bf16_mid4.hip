// Four-copy rollout kernel, bf16 operands: 65..127 hidden units, four hidden layers, obs <= 64, act <= 16.  tanh_near, as in
// rollout_quad_bf16_mid.hip (24 random shapes, three and four layers: rms error 2.5e-5 on the LDS kernel, 3.5e-5 with tanh_fast,
// 2.3e-5 here; 1 to 4 % of the time).
#include "rollout_quad.hpp"

namespace es {

int launch_quad_bf16_mid4(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  return launch_quad_obs64<true, 4, 4, true>(ctx, a, fitness, st);
}

}  // namespace es
