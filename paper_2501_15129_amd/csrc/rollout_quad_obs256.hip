// Four-copy rollout kernel, bf16 operands, four wavefronts: 129..256 hidden units, two hidden layers, obs <= 256, act <= 32.
#include "rollout_quad.hpp"

namespace es {

int launch_quad_obs256(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) { return launch_quad_copies<true, 4, 64, 2, true, false>(ctx, a, fitness, st); }

}  // namespace es
