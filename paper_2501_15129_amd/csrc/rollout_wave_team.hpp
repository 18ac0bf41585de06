// es_rollout, register-resident kernel for narrow policies (obs, 33 to 64 hidden units, act <= 16, two to four hidden layers), binary32
// or bf16 operands: FOUR wavefronts per episode, for populations that leave compute units idle otherwise.
//
// Paper Sec. 3.2 / 5.2: population x environment-copy evaluation of a deterministic MLP policy, fitness = mean undiscounted
// return.  The layouts are those of rollout_wave_reg.hpp (state element k in row k % 4, column k / 4; hidden unit u in lane u; every product
// broadcasts its inputs within the 16-lane rows, fused into the multiply-add).  Bound there: a lone wavefront issues one DPP multiply-add every
// 4.5 cycles whatever else it does, and two thirds of a step are multiply-adds.  Here the hidden layers are taken in pairs and shared:
//   * the first of a pair is split over its outputs: wavefront w computes units 16 w .. 16 w + 15, whose totals the two row-swap stages
//     leave in every row;
//   * the second is split over its inputs: wavefront w multiplies the sixteen units it has just computed with all 64 outputs, one output
//     per lane, sixteen multiply-adds and no row stages;
//   * only these partial sums cross the LDS, [wavefront][unit], once per pair; every wavefront adds the four in the same order and
//     goes on with the whole layer.
// The state, the action layer and the environment are kept by every wavefront for itself from the same operands in the same order
// (bit-identical, so all of them take the same branches).  A s, which is off the chain, is computed where the hand-over would be waited for: part of
// it before the barrier (the LDS write), the rest behind it (the reads).  An odd first layer is computed by every wavefront.
// Its four wavefronts then have a SIMD each: used up to one episode per compute unit (reg_team in rollout_wave_reg.hip).  Two wavefronts on a
// SIMD do not overlap their DPP multiply-adds (10.7 cycles a pair), so beyond that one wavefront per episode is faster.
// Bound: 660 cycles of issue per step of 17-64-64-6 and the hand-over, 820 to 890 in all (the barrier takes 100 to 200 of them: four wavefronts that
// leave it together fetch their code together; the spread is that of the code's alignment in 32-byte windows).
// Whole rollout, against one wavefront per episode: 256 episodes x 1000 steps of 17-64-64-6 391 -> 374 us (439 before either was tuned),
// 128 episodes x 400 steps of three layers 266 -> 187 us.
#pragma once

#include "rollout_wave_reg.hpp"

namespace es {

// CJ: state elements per row (class of ceil(obs / 4)); NAR: length of the action run; MODE as in rollout_reg_kernel; M: hidden layers.
template <int CJ, int NAR, int MODE, bool BF16, int M>
__global__ __launch_bounds__(256) void rollout_team_kernel(const RegArgs a) {
  static_assert(M >= 2 && M <= 4, "pairs of hidden layers");
  constexpr bool FIXED = MODE >= 0;
  constexpr bool NORM = !FIXED || (MODE & 1);
  constexpr int P = action_period(NAR);
  constexpr bool ODD = (M & 1) != 0;             // the first layer stands alone
  constexpr int PAIRS = M / 2;
  extern __shared__ float sp[];                  // the individual's perturbed parameters, once
  __shared__ float xch[2][4][64];                // partial sums; hand-overs alternate between the two buffers
  const int u = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t i = blockIdx.x / a.E, e = blockIdx.x % a.E;
  const uint32_t row = a.antithetic ? (i >> 1) : i;
  const float scale = (a.antithetic && (i & 1u)) ? -a.sigma : a.sigma;
  const int no = (int)a.no, nh = (int)a.nh, na = (int)a.na;
  const int lr = u >> 4, lc = u & 15;
  const int ks = 4 * lc + lr;                    // the state element of this lane
  const bool sval = lc < CJ && ks < no;
  const int um = 16 * w + lc;                    // its unit of a layer that is split over the outputs
  auto opnd = [](float v) { return BF16 ? bf16_round(v) : v; };
  uint32_t envf_l = a.env_f32;                   // (a select, not a branch)
  if (BF16) asm volatile("" : "+v"(envf_l));
  auto opnd_env = [&](float v) { return BF16 ? (envf_l ? v : bf16_round(v)) : v; };

  // ---- environment matrices and statistics: requested first (masked elements read the matrix's first entry) ----
  float ar[4 * CJ], br[NAR];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
      const int el = 4 * lc + r, k = 4 * j + lr;
      const bool ok = lc < CJ && el < no && k < no;
      const float v = a.A[ok ? el * no + k : 0];
      ar[CJ * r + j] = ok ? opnd_env(v) : 0.f;
    }
#pragma unroll
  for (int c = 0; c < NAR; ++c) {
    const bool ok = sval && c < na;
    const float v = a.B[ok ? ks * na + c : 0];
    br[c] = ok ? opnd_env(v) : 0.f;
  }
  const bool stats = a.obs_mean != nullptr;
  const float mu = (NORM && stats && sval) ? a.obs_mean[ks] : 0.f;
  const float iv = (NORM && stats && sval) ? a.obs_inv[ks] : 1.f;
  float s = sval ? reset_value((uint32_t)ks, e, a.gen, a.k0, a.k1) : 0.f;

  // ---- this lane's weights: all layers pass through the LDS at once ----
  param_stage(a, row, scale).stage<256, BF16>(sp, 0u, a.D);
  auto pick = [&](bool ok, int idx) { const float v = sp[ok ? idx : 0]; return ok ? v : 0.f; };
  // the layer that reads the state: of unit um (split), or of all units as in rollout_reg_kernel
  constexpr int Q1 = ODD ? 4 : 1;
  float w1[Q1 * CJ], b1, wm[PAIRS][16], bm[PAIRS], wk[PAIRS][16], bk[PAIRS], w3[P], b3;
#pragma unroll
  for (int q = 0; q < Q1; ++q)
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
      const int unit = ODD ? lc + 16 * q : um, k = 4 * j + lr;
      w1[CJ * q + j] = pick(unit < nh && k < no, (int)a.oW1 + unit * no + k);
    }
  { const int unit = ODD ? u : um; b1 = pick(unit < nh, (int)a.ob1 + unit); }
  const int layer = nh * nh + nh;
#pragma unroll
  for (int p = 0; p < PAIRS; ++p) {
    // hidden layers of the pair, counted from the second: its first (none for the first pair of an even depth: that is w1), its second
    const int l0 = (int)a.oW2 + (ODD ? 0 : 2 * p - 1) * layer, l1 = (int)a.oW2 + (ODD ? 1 : 2 * p) * layer;
    bm[p] = 0.f;
    if (ODD || p > 0) {
#pragma unroll
      for (int j = 0; j < 16; ++j) wm[p][j] = pick(um < nh && 16 * lr + j < nh, l0 + um * nh + 16 * lr + j);
      bm[p] = pick(um < nh, l0 + nh * nh + um);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) wk[p][j] = pick(u < nh && 16 * w + j < nh, l1 + u * nh + 16 * w + j);
    bk[p] = pick(u < nh, l1 + nh * nh + u);
  }
  // action layer: column c adds up action c % P over inputs c, c - 1, .., c - P + 1 (mod 16) of its row
  const int ac = lc % P;
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const int k = 16 * lr + ((lc - j) & 15);
    w3[j] = pick(ac < na && k < nh, (int)a.oW3 + ac * nh + k);
  }
  b3 = pick(ac < na, (int)a.ob3 + ac);

  uint32_t relu_l = a.hidden_relu, otanh_l = a.out_tanh;
  if (!FIXED) asm volatile("" : "+v"(relu_l), "+v"(otanh_l));
  float R = 0.f;                      // per-lane share of the return
  // (every action is held 4 * 16 / P times)
  const float ninv_no = -1.0f / (float)no, nq_cost = -(float)P / 64.0f * a.act_cost;
  const RegAct<MODE, BF16 && M != 2> act{};
  const auto c1 = act.bias(b1), c3 = act.bias(b3);
  typename RegAct<MODE, BF16 && M != 2>::Bias cm[PAIRS], ck[PAIRS];
#pragma unroll
  for (int p = 0; p < PAIRS; ++p) { cm[p] = act.bias(bm[p]); ck[p] = act.bias(bk[p]); }

  // one step, the k-th of its turn; the lanes whose state is above the threshold
  auto step = [&](auto k) {
    constexpr int BUF = PAIRS == 1 ? decltype(k)::value & 1 : 0;      // the buffer of the first hand-over: a step makes one or two
    const float xp = opnd(NORM ? (s - mu) * iv : s), se = opnd_env(s);
    float ev[4], h = 0.f, pre = 0.f;
    // (A s: four accumulators in two runs, whose swaps have their distance without a wait state of the runs' own)
    auto env_front = [&] { row_bcast_dot<2, CJ, false>(reinterpret_cast<float(&)[2]>(ev[0]), se, reinterpret_cast<const float(&)[2 * CJ]>(ar[0])); };
    auto env_back = [&] {
      row_bcast_dot<2, CJ, false>(reinterpret_cast<float(&)[2]>(ev[2]), se, reinterpret_cast<const float(&)[2 * CJ]>(ar[2 * CJ]));
      pre = rows_transpose_add(ev[0], ev[1], ev[2], ev[3]);
    };
    auto bar = [] { __builtin_amdgcn_sched_barrier(0); };
    if constexpr (ODD) {
      float p[4];
      row_bcast_dot<4, CJ>(p, xp, reinterpret_cast<const float(&)[4 * CJ]>(w1[0]));
      h = opnd(act.hidden(rows_transpose_add(p[0], p[1], p[2], p[3]), c1, relu_l));
    }
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
      float hm;
      if (!ODD && p == 0) hm = act.hidden(rows_add(row_bcast_chain<CJ>(xp, reinterpret_cast<const float(&)[CJ]>(w1[0]))), c1, relu_l);
      else hm = act.hidden(rows_add(row_bcast_chain<16>(h, wm[p])), cm[p], relu_l);
      float* x = &xch[(BUF + p) & 1][0][u];
      x[64 * w] = row_bcast_chain<16>(opnd(hm), wk[p]);
      bar();
      if (PAIRS == 1) env_front();
      bar();
      __syncthreads();
      const float x0 = x[0], x1 = x[64], x2 = x[128], x3 = x[192];
      bar();
      if (PAIRS > 1 && p == 0) env_front();
      if (p == PAIRS - 1) env_back();
      bar();
      h = opnd(act.hidden((x0 + x1) + (x2 + x3), ck[p], relu_l));
    }
    // a = tanh(W3 h + b3): every row holds every action, P columns apart
    float pv = rows_add(row_rotate_chain<P>(h, w3));
    if (P == 4) pv += dpp_rotate<4>(pv);
    if (P <= 8) pv += dpp_rotate<8>(pv);
    const float tv = act.out(pv, c3, otanh_l);
    // reward from the pre-step state, 1 - |s|^2 / obs - cost |a|^2: this lane's share, the lanes are added after the last step
    R += __fmaf_rn(ninv_no * s, s, nq_cost * (tv * tv));
    // s' = tanh(A s + B a)
    pre = row_bcast_mac<NAR>(pre, opnd_env(tv), br);
    s = act.state(pre);                               // lanes without a state element: zero weights, tanh(0) = 0
    return __ballot(fabsf(s) > a.done_thresh);
  };
  const uint32_t len = run_episode(a.T, R, step);
  R = (float)len + row_total(rows_add(R));      // ends in lane 15
  if (threadIdx.x == 15) {
    a.returns[(size_t)i * a.E + e] = R;
    if (a.fitness) a.fitness[i] = R;
    a.ep_len[(size_t)i * a.E + e] = (int32_t)len;
  }
}

// launchers, one source file each (compile time)
int launch_team_f32(es_ctx* ctx, int mode, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a);
int launch_team_bf16(es_ctx* ctx, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a);

// classes of the action run (the six of 17-64-6 among them) and of the observation width
template <int CJ, int MODE, bool BF16, int M>
int launch_team_act(es_ctx* ctx, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a) {
  auto go = [&](auto kernel) {
    if (lds > 60u * 1024u) {      // (more dynamic LDS than a kernel has without asking)
      const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (err != hipSuccess) return fail(ctx, ES_EHIP, std::string("hipFuncSetAttribute: ") + hipGetErrorString(err));
    }
    hipLaunchKernelGGL(kernel, grid, dim3(256), lds, st, a);
    return (int)ES_OK;
  };
  if (a.na <= 4) return go(rollout_team_kernel<CJ, 4, MODE, BF16, M>);
  if (a.na <= 6) return go(rollout_team_kernel<CJ, 6, MODE, BF16, M>);
  if (a.na <= 8) return go(rollout_team_kernel<CJ, 8, MODE, BF16, M>);
  return go(rollout_team_kernel<CJ, 16, MODE, BF16, M>);
}
template <int MODE, bool BF16, int M>
int launch_team_obs(es_ctx* ctx, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a) {
  if (a.no <= 20) return launch_team_act<5, MODE, BF16, M>(ctx, grid, lds, st, a);
  if (a.no <= 32) return launch_team_act<8, MODE, BF16, M>(ctx, grid, lds, st, a);
  if (a.no <= 48) return launch_team_act<12, MODE, BF16, M>(ctx, grid, lds, st, a);
  return launch_team_act<16, MODE, BF16, M>(ctx, grid, lds, st, a);
}

}  // namespace es
