// Four-copy rollout kernel, bf16 operands, two wavefronts: 65..128 hidden units, one or two hidden layers; obs <= 64 with act <= 16,
// or obs <= 128 with act <= 32 (state rows spread over the wavefronts).
// tanh_near, because the LDS kernel that served these shapes is that accurate (error of the returns against binary64, rms and
// geometric mean over 43 random shapes: 2.7e-5 and 5.0e-6 there, 6.0e-5 and 1.7e-5 with tanh_fast, 3.5e-5 and 6.1e-6 with
// tanh_near; 27-100-100-8, 128 x 5 copies x 400 steps: 0.335 -> 0.352 ms).
#include "rollout_quad.hpp"

namespace es {

int launch_quad_bf16_mid(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  const bool one = ctx->shp.m == 1;
  if (a.no <= 64 && a.na <= 16) return one ? launch_quad_obs64<true, 2, 1, true>(ctx, a, fitness, st) : launch_quad_obs64<true, 2, 2, true>(ctx, a, fitness, st);
  // (per 200 steps, four copies a pass / as many as the chip has room for: 70-100-100-17 64 x 4 copies 237 / 194 us, 512 x 1 247 / 198, 512 x 2 242 / 208,
  // 128-128-128-32 64 x 16 223 / 205, 1024 x 4 458 / 455, one layer 64 x 4 179 / 135)
  return one ? launch_quad_copies<true, 2, 32, 1, true, true>(ctx, a, fitness, st) : launch_quad_copies<true, 2, 32, 2, true, true>(ctx, a, fitness, st);
}

}  // namespace es
