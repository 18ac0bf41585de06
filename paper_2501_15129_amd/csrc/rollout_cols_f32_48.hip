// Sixteen-column rollout kernel in one wavefront: binary32, up to 48 hidden units.
#include "rollout_cols.hpp"

namespace es {

int launch_cols_f32_48(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) { return launch_cols_f32<3>(ctx, a, fitness, st); }

}  // namespace es
