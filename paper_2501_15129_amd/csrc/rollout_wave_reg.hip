// Narrow policies in one wavefront per episode: choice of the variant, the exact shapes.
#include <algorithm>

#include "rollout_wave_team.hpp"

namespace es {

// ---- variants: two exact shapes, and classes for everything else ----
constexpr int REG_EXACT = 2;
struct RegExact { uint32_t no, nh, na; };
static const RegExact kRegExact[REG_EXACT] = {{11, 32, 3}, {17, 64, 6}};
// class variant index = REG_EXACT + 9 * (obs class) + 3 * (hidden class) + (act class)
static int class_of(uint32_t v, uint32_t a, uint32_t b) { return v <= a ? 0 : (v <= b ? 1 : 2); }

int reg_variant_for(const es_config& c) {
  const uint32_t m = c.num_hidden ? c.num_hidden : 2;
  if (c.dtype > 1 || m > 4) return -1;
  if (c.obs_dim > 64 || c.hid_dim > 64 || c.act_dim > 16) return -1;
  for (int v = 0; v < REG_EXACT && c.dtype == 0 && m == 2; ++v)
    if (c.obs_dim == kRegExact[v].no && c.hid_dim == kRegExact[v].nh && c.act_dim == kRegExact[v].na) return v;
  return REG_EXACT + 9 * class_of(c.obs_dim, 16, 32) + 3 * class_of(c.hid_dim, 16, 32) + class_of(c.act_dim, 4, 8);
}

std::string reg_variant_name(int v, bool bf16, uint32_t m) {
  if (v < 0) return "none";
  if (v < REG_EXACT)
    return "rollout_wave_reg_f32<" + std::to_string(kRegExact[v].no) + "," + std::to_string(kRegExact[v].nh) + "," +
           std::to_string(kRegExact[v].na) + ">";
  v -= REG_EXACT;
  static const char* obs[] = {"16", "32", "64"}, *hid[] = {"16", "32", "64"}, *act[] = {"4", "8", "16"};
  std::string s = std::string(bf16 ? "rollout_wave_reg_bf16<obs<=" : "rollout_wave_reg_f32<obs<=") + obs[v / 9] + ",hid<=" + hid[(v / 3) % 3] + ",act<=" + act[v % 3] + ">";
  return m == 2 ? s : s + ",depth" + std::to_string(m);
}

template <int CJ, int NQ, int NAR>
static void launch_fixed(int mode, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a) {
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(64), lds, st, a); };
  switch (mode) {
    case 0: go(rollout_reg_kernel<CJ, NQ, NAR, 0, false, 2>); break;
    case 1: go(rollout_reg_kernel<CJ, NQ, NAR, 1, false, 2>); break;
    case 2: go(rollout_reg_kernel<CJ, NQ, NAR, 2, false, 2>); break;
    case 3: go(rollout_reg_kernel<CJ, NQ, NAR, 3, false, 2>); break;
    case 4: go(rollout_reg_kernel<CJ, NQ, NAR, 4, false, 2>); break;
    case 5: go(rollout_reg_kernel<CJ, NQ, NAR, 5, false, 2>); break;
    case 6: go(rollout_reg_kernel<CJ, NQ, NAR, 6, false, 2>); break;
    default: go(rollout_reg_kernel<CJ, NQ, NAR, 7, false, 2>); break;
  }
}
// Four wavefronts share an episode (rollout_wave_team.hpp) while every episode has a compute unit of its own; two episodes on a compute
// unit only with four layers.  Per 200 steps, four wavefronts against one: 256 episodes of 17-64-64-6 84 us against 90, 512 episodes 108 against
// 91; three layers of 64 97 against 145, 145 against 147; 30-40x4-6 124 against 212, 178 against 218, 640 episodes 241 against 219.
bool reg_team(const es_config& c, uint64_t copies, int cus) {
  const uint32_t m = c.num_hidden ? c.num_hidden : 2;
  return c.hid_dim > 32 && m >= 2 && m <= 4 && c.pop * copies <= (uint64_t)cus * (m == 4 ? 2u : 1u);
}

std::string team_variant_name(const es_config& c) {
  const uint32_t m = c.num_hidden ? c.num_hidden : 2;
  const char *obs = c.obs_dim <= 20 ? "20" : c.obs_dim <= 32 ? "32" : c.obs_dim <= 48 ? "48" : "64", *act = c.act_dim <= 4 ? "4" : c.act_dim <= 6 ? "6" : c.act_dim <= 8 ? "8" : "16";
  const std::string s = std::string(c.dtype == 1 ? "rollout_wave_reg_team_bf16<obs<=" : "rollout_wave_reg_team_f32<obs<=") + obs + ",hid<=64,act<=" + act + ">";
  return m == 2 ? s : s + ",depth" + std::to_string(m);
}

int launch_rollout_reg(es_ctx* ctx, uint32_t gen, const float* theta, const void* noise, const float* A,
                       const float* B, float* returns, int32_t* ep_len, float* fitness, void* /*ws*/,
                       hipStream_t st) {
  const Shape& s = ctx->shp;
  const es_config& c = ctx->cfg;
  RegArgs a;
  const NoiseView nv = noise_view(ctx, noise);
  a.theta = theta; a.noise = nv.base; a.noise_offs = nv.offs; a.A = A; a.B = B; a.obs_mean = ctx->obs_mean; a.obs_inv = ctx->obs_inv_std; a.returns = returns; a.ep_len = ep_len;
  a.fitness = s.E == 1u ? fitness : nullptr;
  a.N = s.N; a.E = s.E; a.T = s.T; a.ld = s.ld; a.D = s.D;
  a.no = s.no; a.nh = s.nh; a.na = s.na;
  a.oW1 = s.oW1; a.ob1 = s.ob1; a.oW2 = s.oW2; a.ob2 = s.ob2; a.oW3 = s.oW3; a.ob3 = s.ob3;
  a.gen = gen; a.k0 = (uint32_t)c.seed; a.k1 = (uint32_t)(c.seed >> 32);
  a.antithetic = c.antithetic; a.noise_mode = nv.mode; a.hidden_relu = c.hidden_act == 1; a.out_tanh = c.out_tanh != 0;
  a.env_f32 = (c.dtype == 1 && c.env_dtype == 1) ? 1u : 0u;
  a.sigma = c.sigma; a.done_thresh = c.done_thresh; a.act_cost = c.act_cost;
  const dim3 grid(s.N * s.E);
  // the parameters of an individual pass through the LDS at once (one round of memory latency instead of one per layer) where the
  // wavefronts of a CU have room for it, else one layer at a time: at most 65 * 64 values
  const size_t whole = sizeof(float) * (size_t)s.D, per_cu = ((size_t)s.N * s.E + ctx->num_cus - 1) / ctx->num_cus;
  a.whole = whole <= 48u * 1024u && whole * per_cu <= 128u * 1024u ? 1u : 0u;
  const size_t lds = a.whole ? whole : sizeof(float) * (size_t)std::max(s.nh * (s.no + 1u), std::max(s.m > 1u ? s.nh * (s.nh + 1u) : 0u, s.na * (s.nh + 1u)));
  const int mode = (c.hidden_act == 1 ? 4 : 0) | (c.out_tanh ? 2 : 0) | (ctx->obs_mean ? 1 : 0);
  const int v = ctx->reg_variant;
  if (v < 0 || s.no > 64 || s.nh > 64 || s.na > 16 || s.m > 4)
    return fail(ctx, ES_EUNSUPPORTED, "es_rollout: no register-resident binary32 variant for this shape");
  int rc = ES_OK;
  if (ctx->rollout().kind == ROLLOUT_WAVE_TEAM) {
    rc = c.dtype == 1 ? launch_team_bf16(ctx, grid, whole, st, a) : launch_team_f32(ctx, mode, grid, whole, st, a);
    if (rc != ES_OK) return rc;
  } else if (v == 0) launch_fixed<3, 2, 3>(mode, grid, lds, st, a);
  else if (v == 1) launch_fixed<5, 4, 6>(mode, grid, lds, st, a);
  else {
    const uint32_t cls = (uint32_t)(v - REG_EXACT);
    if (c.dtype == 1) launch_reg_bf16(s.m, cls, grid, lds, st, a);
    else if (s.m == 2) launch_reg_f32_two(cls, mode, grid, lds, st, a);
    else launch_reg_f32_deep(s.m, cls, mode, grid, lds, st, a);
  }
  rc = check_launch(ctx, "es_rollout (register-resident f32)");
  if (rc != ES_OK || s.E == 1u) return rc;
  return launch_fitness(ctx, returns, fitness, st);
}

}  // namespace es
