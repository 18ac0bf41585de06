// es_rollout, ONE environment copy per workgroup on the vector ALU: binary32 policies of 65 to 256 hidden units, obs <= 64 (more than 128 units:
// <= 32), act <= 16, one or two hidden layers (up to 128 units: three).
//
// Paper Sec. 5.1 / 5.2: population x environment-copy evaluation of a deterministic MLP policy, fitness = mean undiscounted return.  For a single copy
// the matrix cores are the slower place in binary32: a 4x4x1 product does 64 useful multiply-adds in 8.3 cycles (three of its four rows are idle), a
// multiply-add with its input broadcast within the 16-lane rows (DPP, as in rollout_wave_reg.hpp) does them in 4.5.  A workgroup of HW wavefronts takes
// one episode; wavefront w owns units 32 w .. 32 w + 31 of every hidden layer, whose weights live in its registers for all T steps:
//   * lane (row r, column c) adds up units 32 w + c and 32 w + 16 + c over the inputs that its row holds; two row-swap stages add the four rows' sums and
//     leave the first sixteen units in the even rows, the others in the odd ones;
//   * a layer crosses the LDS once ([unit], one barrier) and every wavefront reads all of it, HW / 2 registers a lane;
//   * the action layer is split over the wavefronts' own units (its sixteen columns share eight actions' inputs, row_ror; rows 2 and 3 take actions 8 to 15),
//     partial sums [action][wavefront] cross the LDS, every wavefront adds them in the same order;
//   * state, action and environment are kept by every wavefront for itself from the same operands in the same order (bit-identical, no
//     exchange); A s is computed where a hand-over would be waited for.
// Bound: the multiply-adds of the wavefronts on a SIMD, which do not overlap (256 units: 128 each, two wavefronts), then the two hand-overs of a step.
// Whole rollout, 1000 steps of 8-256-256-2, 128 individuals: 1.56 ms on the four-copy kernel -> 1.03 ms; 17-128-128-6, 128 x 100 steps 126 -> 70 us.  Which
// populations: single_pays (rollout_quad.hip).
#pragma once

#include "rollout_quad.hpp"
#include "rollout_wave_reg.hpp"

namespace es {

template <int HW, int CJ>
struct SingleMap {
  static constexpr int HID = 32 * HW, NI = HW / 2, PW = 64 + 4, PW3 = HID + 4;
  // More than 32 observations: the environment's matrices pass through the LDS.  Its lanes fetching their own elements is a line per lane and load, 64 loads a
  // wavefront of A alone: 60-100-100-8, 128 x 4 copies, 2 steps 36 -> 29 us; up to 32 observations the additional round costs as much as it saves
  static constexpr bool ENV_LDS = CJ > 8;
  static_assert(!ENV_LDS || CJ == 16, "a column each");
  static constexpr int ROWS = 4 * CJ, PA = ROWS + 4, PB = 16 + 4;
  // LDS (bytes): exchange buffers, the staging window, the environment's matrices
  static constexpr int OFF_H = 0, OFF_P = 2 * 4 * HID, OFF_WIN = OFF_P + 2 * 4 * 16 * HW;
  static constexpr int WIN = 4 * HID * PW > 4 * 16 * PW3 ? 4 * HID * PW : 4 * 16 * PW3;
  static constexpr int OFF_A = OFF_WIN + WIN, OFF_B = OFF_A + 4 * ROWS * PA;
  static constexpr int LDS_BYTES = ENV_LDS ? OFF_B + 4 * ROWS * PB : OFF_A;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

// HW: wavefronts; CJ: state elements per row; NAR: length of the action run; MODE as in rollout_reg_kernel; M: hidden layers.
template <int HW, int CJ, int NAR, int MODE, int M>
__global__ __launch_bounds__(64 * HW) __attribute__((amdgpu_waves_per_eu(HW / 4, HW / 4)))
void rollout_single_kernel(const QuadArgs a, const uint32_t hidden_relu) {
  using Map = SingleMap<HW, CJ>;
  constexpr int HID = Map::HID, NI = Map::NI;
  constexpr bool NORM = MODE < 0 || (MODE & 1);
  extern __shared__ __align__(16) unsigned char lds[];
  float* xh = reinterpret_cast<float*>(lds + Map::OFF_H);      // [2][HID]: layers alternate
  float* xa = reinterpret_cast<float*>(lds + Map::OFF_P);      // [2][16][HW]: steps alternate where this is the only hand-over
  float* win = reinterpret_cast<float*>(lds + Map::OFF_WIN);
  const int u = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t i = blockIdx.x / a.E, e = blockIdx.x % a.E;
  const uint32_t row = a.antithetic ? (i >> 1) : i;
  const float scale = (a.antithetic && (i & 1u)) ? -a.sigma : a.sigma;
  const int no = (int)a.no, nh = (int)a.nh, na = (int)a.na;
  const int lr = u >> 4, lc = u & 15;
  const int ks = 4 * lc + lr;                    // the state element of this lane
  const bool sval = lc < CJ && ks < no;
  const int own = 32 * w + 16 * (lr & 1) + lc;   // its unit after a layer

  // ---- environment matrices and statistics, requested first (masked elements read the matrix's first entry) ----
  float ar[4 * CJ], br[NAR];
  float* ea = reinterpret_cast<float*>(lds + Map::OFF_A);
  float* eb = reinterpret_cast<float*>(lds + Map::OFF_B);
  if constexpr (Map::ENV_LDS) {
    stage_cols<Map::ROWS, false>(ea, Map::PA, Map::ROWS, no, no, 0, a.A, NoiseRow{}, 0.0f, 0u);
    stage_cols<16, false>(eb, Map::PB, Map::ROWS, no, na, 0, a.B, NoiseRow{}, 0.0f, 0u);
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < CJ; ++j) {
        const int el = 4 * lc + r, k = 4 * j + lr;
        const bool ok = lc < CJ && el < no && k < no;
        const float v = a.A[ok ? el * no + k : 0];
        ar[CJ * r + j] = ok ? v : 0.f;
      }
#pragma unroll
    for (int c = 0; c < NAR; ++c) {
      const bool ok = sval && c < na;
      const float v = a.B[ok ? ks * na + c : 0];
      br[c] = ok ? v : 0.f;
    }
  }
  const bool stats = a.obs_mean != nullptr;
  const float mu = (NORM && stats && sval) ? a.obs_mean[ks] : 0.f;
  const float iv = (NORM && stats && sval) ? a.obs_inv[ks] : 1.f;
  float s = sval ? reset_value((uint32_t)ks, e, a.gen, a.k0, a.k1) : 0.f;

  // ---- perturbed parameters -> LDS window -> registers ----
  NoiseRow nz;
  nz.mode = a.noise_mode; nz.row = row; nz.gen = a.gen; nz.k0 = a.k0; nz.k1 = a.k1; nz.ptr = nullptr;
  if (a.noise_offs) nz.ptr = table_row_base(a.noise_mode, a.noise, a.noise_offs, row);
  else if (a.noise_mode == 1u) nz.ptr = static_cast<const uint16_t*>(a.noise) + (size_t)row * a.ld;
  else if (a.noise_mode == 0u) nz.ptr = static_cast<const float*>(a.noise) + (size_t)row * a.ld;
  auto bias_of = [&](bool ok, uint32_t idx) { const uint32_t ix = ok ? idx : 0u; const float v = __fmaf_rn(scale, row_noise(nz, ix), a.theta[ix]); return ok ? v : 0.f; };
  float b[M];
#pragma unroll
  for (int l = 0; l < M; ++l) b[l] = bias_of(own < nh, (l == 0 ? a.ob1 : a.ob2 + (uint32_t)(l - 1) * (uint32_t)(nh * nh + nh)) + (uint32_t)own);
  const float b3 = bias_of(lc < na, a.ob3 + (uint32_t)lc);
  // first layer: w1[CJ t + j] = W1[32 w + 16 t + lc][4 j + lr]
  float w1[2 * CJ], wh[M > 1 ? M - 1 : 1][M > 1 ? NI : 1][32], w3[8];
  stage_cols<64, true>(win, Map::PW, HID, nh, no, 0, a.theta, nz, scale, a.oW1);
  __syncthreads();
  if constexpr (Map::ENV_LDS) {      // (staged before the barrier above, zero beyond the matrices; all sixteen columns hold elements)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < CJ; ++j) ar[CJ * r + j] = ea[(4 * lc + r) * Map::PA + 4 * j + lr];
#pragma unroll
    for (int c = 0; c < NAR; ++c) br[c] = eb[ks * Map::PB + c];
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int j = 0; j < CJ; ++j) w1[CJ * t + j] = win[(32 * w + 16 * t + lc) * Map::PW + 4 * j + lr];
  __syncthreads();
  // further layers: wh[l][q][16 t + j] = W[32 w + 16 t + lc][64 q + 16 lr + j]
#pragma unroll
  for (int l = 0; l < M - 1; ++l)
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      stage_cols<64, true>(win, Map::PW, HID, nh, nh, 64 * q, a.theta, nz, scale, a.oW2 + (uint32_t)l * (uint32_t)(nh * nh + nh));
      __syncthreads();
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 16; j += 4) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(win + (32 * w + 16 * t + lc) * Map::PW + 16 * lr + j);
          wh[l][q][16 * t + j] = v.x; wh[l][q][16 * t + j + 1] = v.y; wh[l][q][16 * t + j + 2] = v.z; wh[l][q][16 * t + j + 3] = v.w;
        }
      __syncthreads();
    }
  // action layer: rows 0 and 1 actions 0 .. 7, rows 2 and 3 actions 8 .. 15; columns eight apart share an action's sixteen inputs of the row
  stage_cols<HID, true>(win, Map::PW3, 16, na, nh, 0, a.theta, nz, scale, a.oW3);
  __syncthreads();
  const int act_row = 8 * (lr >> 1) + (lc & 7);
#pragma unroll
  for (int j = 0; j < 8; ++j) w3[j] = win[act_row * Map::PW3 + 32 * w + 16 * (lr & 1) + ((lc - j) & 15)];

  uint32_t relu_l = hidden_relu, otanh_l = a.out_tanh;      // (selects, not branches)
  if (MODE < 0) asm volatile("" : "+v"(relu_l), "+v"(otanh_l));
  float R = 0.f;                      // per-lane share of the return
  const float ninv_no = -1.0f / (float)no, nq_cost = -0.25f * a.act_cost;      // (every action is held four times)
  const RegAct<MODE, false> act{};
  typename RegAct<MODE, false>::Bias cb[M];
#pragma unroll
  for (int l = 0; l < M; ++l) cb[l] = act.bias(b[l]);
  const auto c3 = act.bias(b3);

  // one step, the k-th of its turn; the lanes whose state is above the threshold
  auto step = [&](auto k) {
    auto bar = [] { __builtin_amdgcn_sched_barrier(0); };
    const float xp = NORM ? (s - mu) * iv : s;
    float ev[4], p[2];
    auto env_front = [&] { row_bcast_dot<2, CJ, false>(reinterpret_cast<float(&)[2]>(ev[0]), s, reinterpret_cast<const float(&)[2 * CJ]>(ar[0])); };
    auto env_back = [&] { row_bcast_dot<2, CJ>(reinterpret_cast<float(&)[2]>(ev[2]), s, reinterpret_cast<const float(&)[2 * CJ]>(ar[2 * CJ])); };
    row_bcast_dot<2, CJ>(p, xp, w1);
    float h = act.hidden(rows_transpose_add(p[0], p[1]), cb[0], relu_l);
#pragma unroll
    for (int l = 0; l < M - 1; ++l) {
      float* x = xh + (l & 1) * HID;
      if (u < 32) x[32 * w + u] = h;
      bar();
      if (l == 0) env_front();
      bar();
      __syncthreads();
      float hq[NI];
#pragma unroll
      for (int q = 0; q < NI; ++q) hq[q] = x[64 * q + u];
      bar();
      row_bcast_dot<2, 16>(p, hq[0], wh[l][0]);
#pragma unroll
      for (int q = 1; q < NI; ++q) row_bcast_dot_add(p, hq[q], wh[l][q]);
      h = act.hidden(rows_transpose_add(p[0], p[1]), cb[l + 1], relu_l);
    }
    float pv = row_rotate_chain<8>(h, w3);
    pv = swap16_add(pv, pv);
    pv += dpp_rotate<8>(pv);
    float* x = xa + (M == 1 ? (decltype(k)::value & 1) * 16 * HW : 0);
    if ((u & 24) == 0) x[act_row * HW + w] = pv;
    bar();
    if (M == 1) env_front();
    bar();
    __syncthreads();
    f32x4 part[HW / 4];
#pragma unroll
    for (int q = 0; q < HW / 4; ++q) part[q] = *reinterpret_cast<const f32x4*>(x + lc * HW + 4 * q);
    bar();
    env_back();
    float pre = rows_transpose_add(ev[0], ev[1], ev[2], ev[3]);
    bar();
    f32x4 sum = part[0];
#pragma unroll
    for (int q = 1; q < HW / 4; ++q) sum += part[q];
    const float tv = act.out((sum.x + sum.y) + (sum.z + sum.w), c3, otanh_l);      // actions >= act: weights and bias are zero
    R += __fmaf_rn(ninv_no * s, s, nq_cost * (tv * tv));
    pre = row_bcast_mac<NAR>(pre, tv, br);
    s = act.state(pre);
    return __ballot(fabsf(s) > a.done_thresh);
  };
  __syncthreads();
  const uint32_t len = run_episode(a.T, R, step);
  R = (float)len + row_total(rows_add(R));      // ends in lane 15
  if (threadIdx.x == 15) {
    a.returns[(size_t)i * a.E + e] = R;
    if (a.fitness) a.fitness[i] = R;
    a.ep_len[(size_t)i * a.E + e] = (int32_t)len;
  }
}

template <int HW, int CJ, int MODE, int M>
int launch_single_act(es_ctx* ctx, QuadArgs a, float* fitness, hipStream_t st) {
  a.fitness = a.E == 1u ? fitness : nullptr;
  constexpr int lds = SingleMap<HW, CJ>::LDS_BYTES;
  auto go = [&](auto kernel) {
    const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (err != hipSuccess) return fail(ctx, ES_EHIP, std::string("hipFuncSetAttribute: ") + hipGetErrorString(err));
    hipLaunchKernelGGL(kernel, dim3(a.N * a.E), dim3(64 * HW), lds, st, a, ctx->cfg.hidden_act == 1 ? 1u : 0u);
    const int rc = check_launch(ctx, "es_rollout (one copy per workgroup)");
    return rc != ES_OK || a.E == 1u ? rc : launch_fitness(ctx, a.returns, fitness, st);
  };
  if constexpr (MODE >= 0) {
    if (a.na <= 4) return go(rollout_single_kernel<HW, CJ, 4, MODE, M>);
    if (a.na <= 8) return go(rollout_single_kernel<HW, CJ, 8, MODE, M>);
  }
  return go(rollout_single_kernel<HW, CJ, 16, MODE, M>);
}
template <int HW, int CJ, int M>
int launch_single_mode(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  const bool plain = ctx->cfg.hidden_act == 0 && a.out_tanh != 0u && a.obs_mean == nullptr;
  return plain ? launch_single_act<HW, CJ, 2, M>(ctx, a, fitness, st) : launch_single_act<HW, CJ, -1, M>(ctx, a, fitness, st);
}

// one source file each (compile time)
int launch_single_mid(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);      // four wavefronts: up to 128 units
int launch_single_wide(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);     // eight

}  // namespace es
