// es_rollout, register-resident kernel for narrow policies (obs, hidden <= 64, act <= 16, one to four hidden layers), binary32
// or bf16 operands.
//
// Paper Sec. 3.2 / 5.2: population x environment-copy evaluation of a deterministic
// MLP policy, fitness = mean undiscounted return.  One wavefront runs one
// (individual, environment copy) episode.  Lane u owns hidden unit u (with at most 16 hidden units every
// 16-lane row owns all of them), and the state vector is spread over the four 16-lane rows of the
// wavefront (element k in row k % 4, column k / 4).  The individual's perturbed weights
// (theta + sign*sigma*eps) pass through LDS once, layer by layer in coalesced order, and then live in registers for all
// T steps, as do the environment matrices.
// Every matrix-vector product broadcasts its inputs within the 16-lane rows by DPP, fused into the
// multiply-add (v_fmac_f32_dpp ... row_newbcast:j, one instruction per multiply-add, no scalar hop):
// the lane in row r, column c adds up the inputs that live in ITS row into partial sums for the outputs
// that belong to ITS column (hidden units c, c + 16, ...; state elements 4 c .. 4 c + 3), and two
// row-swap stages (v_permlane32_swap, v_permlane16_swap + add) add the four rows' partial sums and
// leave each output's total in the lane that owns it.  A step is one straight-line block: no LDS, no
// barriers, no masks (lanes without a unit have zero weights, and tanh and ReLU map 0 to 0), the return is
// accumulated per lane and reduced after the last step, termination is one compare whose mask is the
// branch condition.
// The run lengths (inputs per row, rows of hidden units, action width) are compile-time: exact for the
// benchmark shapes 11-32-3 and 17-64-6, whose activations and observation statistics are compile-time
// variants too, and rounded up to a few classes for every other shape (padding has zero weights), where
// the activations are chosen by branch-free selects.
// A layer of at most 32 units, which four rows would hold twice, is shared by the rows that hold the same inputs; the action layer of at most
// eight actions is summed by sixteen columns, each over a part of its row's inputs (row_ror instead of row_newbcast).
// Bound: one wavefront's instructions (32-256 episodes for 1024 SIMDs).  A lone wavefront issues a DPP multiply-add (8 bytes) every 4.5
// cycles, a plain one (4 bytes) every 4, dependent or not; a transcendental takes 8, the two wait states before a DPP read 8, a taken
// branch 70.  So the count of instructions and bytes of a step is what matters, and everything that ends a step comes once in four.
// 11-32-32-3 (8 x 4 episodes, 100 steps, whole generation): 43.8 -> 36.2 us, some of it the staging (all layers in one round of loads); 17-64-64-6, 256
// episodes x 1000 steps: 439 -> 391 us; 17-64-64-64-6, 128 episodes x 400 steps: 274 -> 266 us.
#pragma once

#include <type_traits>

#include "es_internal.hpp"
#include "rollout_stage.hpp"

namespace es {

struct RegArgs {
  const float* theta;
  const void* noise;
  const uint32_t* noise_offs;   // shared noise table: start of every row, else null
  const float* A;
  const float* B;
  const float* obs_mean;     // frozen observation statistics, or null
  const float* obs_inv;
  float* returns;
  int32_t* ep_len;
  float* fitness;            // one episode per individual: its return is the fitness; else null
  uint32_t N, E, T, ld, D;
  uint32_t no, nh, na;
  uint32_t oW1, ob1, oW2, ob2, oW3, ob3;
  uint32_t gen, k0, k1;
  uint32_t antithetic, noise_mode, hidden_relu, out_tanh;
  uint32_t env_f32;          // bf16 operands: keep the environment's products binary32
  uint32_t whole;            // all parameters of an individual pass through the LDS at once
  float sigma, done_thresh, act_cost;
};

#include "dpp_runs.inc"

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_zero(float v) {      // lanes without a source (or masked off) read 0
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xF, ROW_MASK == 0xF));
}
// x + y after a row swap: permlane16_swap exchanges the odd rows of x with the even rows of y, permlane32_swap the
// upper two rows of x with the lower two of y
__device__ __forceinline__ float swap16_add(float x, float y) {
  const auto p = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
  return __builtin_bit_cast(float, (unsigned)p[0]) + __builtin_bit_cast(float, (unsigned)p[1]);
}
__device__ __forceinline__ float swap32_add(float x, float y) {
  const auto p = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
  return __builtin_bit_cast(float, (unsigned)p[0]) + __builtin_bit_cast(float, (unsigned)p[1]);
}
// out[row q] = sum over the four rows of x_q: two row-swap stages
__device__ __forceinline__ float rows_transpose_add(float x0, float x1, float x2, float x3) {
  return swap16_add(swap32_add(x0, x2), swap32_add(x1, x3));
}
// the same for two registers whose sums go to rows 0 and 1 (and again to rows 2 and 3)
__device__ __forceinline__ float rows_transpose_add(float x0, float x1) {
  const float t = swap16_add(x0, x1);
  return swap32_add(t, t);
}
// the sum over the four rows, in every row
__device__ __forceinline__ float rows_add(float x) {
  const float t = swap16_add(x, x);
  return swap32_add(t, t);
}
// sum over the lanes of each 16-lane row, result in lane 15 of the row (lanes without a source read 0)
__device__ __forceinline__ float row_total(float v) {
  v += dpp_zero<0x111, 0xF>(v);
  v += dpp_zero<0x112, 0xF>(v);
  v += dpp_zero<0x114, 0xF>(v);
  return v + dpp_zero<0x118, 0xF>(v);
}
// the value n columns away, (c - n) mod 16 of the row
template <int N>
__device__ __forceinline__ float dpp_rotate(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xF, 0xF, true));
}
// Columns after which the action vector repeats within a row: a column that adds up action c % P needs P of its row's sixteen
// inputs, the columns P apart hold the other parts
constexpr int action_period(int run) { return run <= 4 ? 4 : run <= 8 ? 8 : 16; }

// Activations of the one- and four-wavefront kernels.  tanh(x + b) is 1 - 2 / (1 + 2^(c x + c b)), the bias in the multiply-add;
// MODE < 0 chooses between the activations by selects (no branches).  NEAR: the tanh that is accurate near zero, for bf16 policies of one, three and
// four layers, like the LDS kernel's, which served them (error of the returns against binary64, geometric mean of 50 random
// shapes: 3.9e-6 there, 8.4e-6 with the short form, 3.7e-6 with this one; 0 to 6 % of the time)
template <int MODE, bool NEAR>
struct RegAct {
  static constexpr bool FIXED = MODE >= 0, RELU = FIXED && (MODE & 4), OUT_TANH = FIXED && (MODE & 2);
  float c;
  // c in a scalar register: a multiplication is four bytes then, not eight
  __device__ __forceinline__ RegAct() : c(2.88539008f) { asm volatile("" : "+s"(c)); }      // 2 log2(e), as in tanh_fast
  __device__ __forceinline__ float squash(float t) const {
    if (NEAR) return tanh_near(t);
    return __fmaf_rn(-2.0f, __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(t) + 1.0f), 1.0f);
  }
  // a bias, as ReLU and the linear output take it and as tanh does (the fixed modes drop the other)
  struct Bias { float b, cb; };
  __device__ __forceinline__ Bias bias(float b) const { return Bias{b, c * b}; }
  __device__ __forceinline__ float tanh_of(float x, Bias b) const { return squash(__fmaf_rn(x, c, b.cb)); }
  __device__ __forceinline__ float hidden(float x, Bias b, uint32_t relu) const {
    if (FIXED) return RELU ? fmaxf(x + b.b, 0.f) : tanh_of(x, b);
    const float z = fmaxf(x + b.b, 0.f), t = tanh_of(x, b);
    return relu ? z : t;
  }
  __device__ __forceinline__ float out(float x, Bias b, uint32_t otanh) const {
    if (FIXED) return OUT_TANH ? tanh_of(x, b) : x + b.b;
    const float z = x + b.b, t = tanh_of(x, b);
    return otanh ? t : z;
  }
  __device__ __forceinline__ float state(float x) const { return squash(x * c); }
};

// Steps until the horizon or until step(k) names lanes above the threshold; returns their number, with R as it was after the last of them.
// A taken branch costs a lone wavefront 70 cycles and the test of a compare's mask 31 (it waits for the compare), so both come once
// in a turn of four steps.  Nothing outside the registers depends on the steps a turn makes beyond an episode's end; R is kept for each.
template <class Step>
__device__ __forceinline__ uint32_t run_episode(uint32_t T, float& R, Step&& step) {
  // (the share of a step is added within it, where its instructions fill waits, not all four behind the last)
  auto booked = [](float& r) { asm volatile("" : "+v"(r)); return r; };
  uint32_t left = T, stop;
  unsigned long long m0, m1, m2, m3;
  float r0, r1, r2;
  do {
    m0 = step(std::integral_constant<int, 0>{});
    r0 = booked(R);
    m1 = step(std::integral_constant<int, 1>{});
    r1 = booked(R);
    m2 = step(std::integral_constant<int, 2>{});
    r2 = booked(R);
    m3 = step(std::integral_constant<int, 3>{});
    booked(R);
    const unsigned long long m = (m0 | m1) | (m2 | m3);
    asm volatile("s_cmp_lt_u32 %1, 5\n\ts_cselect_b32 %0, 1, 0" : "=s"(stop) : "s"(left) : "scc");      // (scalar: the compiler would make it a vector compare)
    stop |= (uint32_t)m | (uint32_t)(m >> 32);
    left -= 4u;
  } while (stop == 0u);
  left += 4u;
  const uint32_t n = min(left, m0 != 0ull ? 1u : m1 != 0ull ? 2u : m2 != 0ull ? 3u : 4u);
  R = n == 1u ? r0 : n == 2u ? r1 : n == 3u ? r2 : R;
  return T - left + n;
}

// The perturbed parameters of one individual (one binary32 rounding each, then bf16 where they are operands in bf16), a range
// of consecutive ones at a time into LDS, in coalesced order; the loads of eight iterations are in flight together.
struct ParamStage {
  NoiseRow nz;
  const float* theta;
  float scale;
  // sp[k] = perturbed parameter off + k, k < count, by THREADS threads; barriers on both sides
  template <int THREADS, bool BF16 = false>
  __device__ __forceinline__ void stage(float* sp, uint32_t off, uint32_t count) const {
    constexpr uint32_t U = 8u, NT = (uint32_t)THREADS;
    const uint32_t tid = threadIdx.x;
    auto opnd = [](float v) { return BF16 ? bf16_round(v) : v; };
    __syncthreads();
    auto batch = [&](auto fetch) {
      for (uint32_t q0 = tid; q0 < count; q0 += NT * U) {
        float th[U];
        decltype(fetch(0u)) ez[U];
#pragma unroll
        for (uint32_t v = 0; v < U; ++v) {
          const uint32_t idx = off + min(q0 + NT * v, count - 1u);
          th[v] = theta[idx];
          ez[v] = fetch(idx);
        }
#pragma unroll
        for (uint32_t v = 0; v < U; ++v)
          if (q0 + NT * v < count) sp[q0 + NT * v] = opnd(__fmaf_rn(scale, widen1(ez[v]), th[v]));
      }
    };
    if (nz.mode >= 2u) {            // regenerated noise: one counter block gives four consecutive parameters
      for (uint32_t d0 = (off & ~3u) + 4u * tid; d0 < off + count; d0 += 4u * NT) {
        float z[4];
        noise_regen4(nz.row, d0, nz.gen, nz.k0, nz.k1, nz.mode == 3u, z);
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k)
          if (d0 + k >= off && d0 + k < off + count) sp[d0 + k - off] = opnd(__fmaf_rn(scale, z[k], theta[d0 + k]));
      }
    } else if (nz.mode == 1u) {
      batch([&](uint32_t idx) { return static_cast<const uint16_t*>(nz.ptr)[idx]; });
    } else {
      batch([&](uint32_t idx) { return static_cast<const float*>(nz.ptr)[idx]; });
    }
    __syncthreads();
  }
};
__device__ __forceinline__ ParamStage param_stage(const RegArgs& a, uint32_t row, float scale) {
  ParamStage p;
  p.nz.mode = a.noise_mode; p.nz.row = row; p.nz.gen = a.gen; p.nz.k0 = a.k0; p.nz.k1 = a.k1; p.nz.ptr = nullptr;
  if (a.noise_offs) p.nz.ptr = table_row_base(a.noise_mode, a.noise, a.noise_offs, row);
  else if (a.noise_mode == 1u) p.nz.ptr = static_cast<const uint16_t*>(a.noise) + (size_t)row * a.ld;
  else if (a.noise_mode == 0u) p.nz.ptr = static_cast<const float*>(a.noise) + (size_t)row * a.ld;
  p.theta = a.theta; p.scale = scale;
  return p;
}

// CJ: state elements per row (ceil(obs / 4), or its class); NQ: 16-lane rows of hidden units (1, 2, 4); NAR: action
// run length (act, or its class).  MODE 0..7 = ReLU (4) | tanh on the action layer (2) | observation statistics (1)
// fixed at compile time; MODE < 0: read from the arguments and applied by selects.  BF16: every operand of a product
// (weights, biases, environment matrices, state, activations, action) is rounded to bf16; sums, tanh, reward binary32.
// M: hidden layers.
template <int CJ, int NQ, int NAR, int MODE, bool BF16, int M>
__global__ __launch_bounds__(64) void rollout_reg_kernel(const RegArgs a) {
  static_assert(NQ == 1 || NQ == 2 || NQ == 4, "rows of hidden units");
  constexpr bool FIXED = MODE >= 0;
  constexpr bool NORM = !FIXED || (MODE & 1);
  extern __shared__ float sp[];      // the individual's perturbed parameters, once
  const int u = threadIdx.x;
  const uint32_t i = blockIdx.x / a.E, e = blockIdx.x % a.E;
  const uint32_t row = a.antithetic ? (i >> 1) : i;
  const float scale = (a.antithetic && (i & 1u)) ? -a.sigma : a.sigma;
  const int no = (int)a.no, nh = (int)a.nh, na = (int)a.na;
  const int lr = u >> 4, lc = u & 15;
  const int ks = 4 * lc + lr;                    // the state element of this lane
  const bool sval = lc < CJ && ks < no;
  // Units of a hidden layer, by lane.  NQ = 4: unit u in lane u; NQ = 1: unit c in column c of every row.  NQ = 2: two rows hold the same
  // sixteen, alternately rows r and r + 2 (after layers 1, 3) and the rows of a pair (after layers 2, 4): a layer of a pair of rows that
  // hold the same inputs is shared by them, each sums one half of the outputs, and one row stage adds the two halves of the inputs.
  auto tile_of = [&](int layer) { return NQ == 4 ? lr : NQ == 1 ? 0 : (layer & 1) ? lr & 1 : lr >> 1; };      // of hidden layer 1, 2, ..
  auto opnd = [](float v) { return BF16 ? bf16_round(v) : v; };      // a value as an operand of a product
  // ... of one of the ENVIRONMENT's products: rounded like the policy's unless the environment stays binary32 (a select,
  // not a branch: the flag is read into a vector register the compiler cannot prove uniform)
  uint32_t envf_l = a.env_f32;
  if (BF16) asm volatile("" : "+v"(envf_l));
  auto opnd_env = [&](float v) { return BF16 ? (envf_l ? v : bf16_round(v)) : v; };

  // ---- environment matrices and statistics, requested first (masked elements read the matrix's first entry) ----
  // partial sums of the four state elements of column lc: ar[CJ r + j] = A[4 lc + r][4 j + lr]; action term of this lane's own
  // element: br[c] = B[ks][c]
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
  // frozen observation statistics of this lane's state element (identity when none are set: (s - 0) * 1 = s exactly)
  const bool stats = a.obs_mean != nullptr;
  const float mu = (NORM && stats && sval) ? a.obs_mean[ks] : 0.f;
  const float iv = (NORM && stats && sval) ? a.obs_inv[ks] : 1.f;
  float s = sval ? reset_value((uint32_t)ks, e, a.gen, a.k0, a.k1) : 0.f;

  // ---- this lane's weights ----
  // first layer: partial sums of the units lc, lc + 16, ... over the inputs of row lr: w1[CJ q + j] = W1[lc + 16 q][4 j + lr]
  // further layers, NQ = 4 and 1: the same over the hidden units of row lr: w2[16 q + j] = W2[lc + 16 q][16 lr + j]; NQ = 2: of the one tile of
  //   outputs this row has after the layer
  // action layer: column lc adds up action lc % P over units lc, lc - 1, .., lc - P + 1 (mod 16) of its row (rows that hold the same: one of them)
  constexpr int P = action_period(NAR), Q2 = NQ == 4 ? 4 : 1;
  float w1[NQ * CJ], w2[M > 1 ? M - 1 : 1][Q2 * 16], w3[P], b1, b2[M > 1 ? M - 1 : 1], b3;
  // all layers through the LDS at once, or one layer's window after the other (at most 16.6 KB: room for nine wavefronts per CU)
  const ParamStage ps = param_stage(a, row, scale);
  if (a.whole) ps.stage<64, BF16>(sp, 0u, a.D);
  auto window = [&](uint32_t off, uint32_t count) -> const float* {
    if (a.whole) return sp + off;
    ps.stage<64, BF16>(sp, off, count);
    return sp;
  };
  const float* wp = window(a.oW1, (uint32_t)(nh * no + nh));
  auto pick = [&](bool ok, int idx) { const float v = wp[ok ? idx : 0]; return ok ? v : 0.f; };
#pragma unroll
  for (int qq = 0; qq < NQ; ++qq)
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
      const int unit = lc + 16 * qq, k = 4 * j + lr;
      w1[CJ * qq + j] = pick(unit < nh && k < no, unit * no + k);
    }
  { const int unit = 16 * tile_of(1) + lc; b1 = pick(unit < nh, nh * no + unit); }
#pragma unroll
  for (int l = 0; l < M - 1; ++l) {
    wp = window(a.oW2 + (uint32_t)l * (uint32_t)(nh * nh + nh), (uint32_t)(nh * nh + nh));
    const int own = 16 * tile_of(l + 2) + lc;
#pragma unroll
    for (int qq = 0; qq < Q2; ++qq)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int unit = NQ == 4 ? lc + 16 * qq : own, k = 16 * tile_of(l + 1) + j;
        w2[l][16 * qq + j] = pick(unit < nh && k < nh, unit * nh + k);
      }
    b2[l] = pick(own < nh, nh * nh + own);
  }
  wp = window(a.oW3, (uint32_t)(na * nh + na));
  const int ac = lc % P;
  const bool sole = NQ != 2 || ((M & 1) ? lr < 2 : (lr & 1) == 0);      // the first row that holds these units
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const int k = 16 * tile_of(M) + ((lc - j) & 15);
    w3[j] = pick(sole && ac < na && k < nh, ac * nh + k);
  }
  b3 = pick(ac < na, na * nh + ac);

  // run-time activation choices as per-lane values the compiler cannot prove uniform: selects, not branches
  uint32_t relu_l = a.hidden_relu, otanh_l = a.out_tanh;
  if (!FIXED) asm volatile("" : "+v"(relu_l), "+v"(otanh_l));
  float R = 0.f;                      // per-lane share of the return
  // (every action is held 4 * 16 / P times)
  const float ninv_no = -1.0f / (float)no, nq_cost = -(float)P / 64.0f * a.act_cost;
  const RegAct<MODE, BF16 && M != 2> act{};
  const auto c1 = act.bias(b1), c3 = act.bias(b3);
  typename RegAct<MODE, BF16 && M != 2>::Bias c2[M > 1 ? M - 1 : 1];
#pragma unroll
  for (int l = 0; l < M - 1; ++l) c2[l] = act.bias(b2[l]);

  // one step; the lanes whose state is above the threshold
  auto step = [&](auto) {
    // h1 = act(W1 s + b1)
    const float xp = opnd(NORM ? (s - mu) * iv : s);      // the policy's input (paper App. B: fixed normalisation statistics)
    float p[NQ];
    row_bcast_dot<NQ, CJ>(p, xp, w1);
    float l1;
    if constexpr (NQ == 4) l1 = rows_transpose_add(p[0], p[1], p[2], p[3]);
    else if constexpr (NQ == 2) l1 = rows_transpose_add(p[0], p[1]);
    else l1 = rows_add(p[0]);
    float h = opnd(act.hidden(l1, c1, relu_l));      // the last hidden layer so far
    // further hidden layers: h = act(W h + b)
#pragma unroll
    for (int l = 0; l < M - 1; ++l) {
      float l2;
      if constexpr (NQ == 4) {
        row_bcast_dot<4, 16>(p, h, w2[l]);
        l2 = rows_transpose_add(p[0], p[1], p[2], p[3]);
      } else {
        l2 = row_bcast_chain<16>(h, w2[l]);
        if (NQ == 2) l2 = (l & 1) ? swap32_add(l2, l2) : swap16_add(l2, l2);      // the other half of the inputs: in the row's partner of the layer before
      }
      h = opnd(act.hidden(l2, c2[l], relu_l));
    }
    // a = tanh(W3 h + b3): every row holds every action, P columns apart; one tanh serves all of them
    float pv = row_rotate_chain<P>(h, w3);
    if (NQ != 1) pv = rows_add(pv);
    else if (P <= 8) pv += 0.0f;      // (the wait states before a DPP read are counted from instructions the compiler sees)
    if (P == 4) pv += dpp_rotate<4>(pv);
    if (P <= 8) pv += dpp_rotate<8>(pv);
    const float tv = act.out(pv, c3, otanh_l);      // actions >= act: weights and bias are zero
    // reward from the pre-step state, 1 - |s|^2 / obs - cost |a|^2: a sum over all 64 lanes; this lane's share, the lanes are added after the
    // last step
    R += __fmaf_rn(ninv_no * s, s, nq_cost * (tv * tv));
    // s' = tanh(A s + B a): partial sums of the four elements of this column over the inputs of this row, rows added
    // and moved to their element's lane; the action term straight from the row's action vector
    float ev[4];
    row_bcast_dot<4, CJ>(ev, opnd_env(s), ar);
    float pre = rows_transpose_add(ev[0], ev[1], ev[2], ev[3]);
    pre = row_bcast_mac<NAR>(pre, opnd_env(tv), br);
    s = act.state(pre);                               // lanes without a state element: zero weights, tanh(0) = 0
    return __ballot(fabsf(s) > a.done_thresh);
  };
  const uint32_t len = run_episode(a.T, R, step);
  R = (float)len + row_total(rows_add(R));      // ends in lane 15
  if (u == 15) {
    a.returns[(size_t)i * a.E + e] = R;
    if (a.fitness) a.fitness[i] = R;
    a.ep_len[(size_t)i * a.E + e] = (int32_t)len;
  }
}


// launchers of the class variants, one source file each (compile time): hidden layers m, classes of the three widths
int launch_reg_f32_two(uint32_t cls, int mode, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a);
int launch_reg_f32_deep(uint32_t m, uint32_t cls, int mode, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a);
int launch_reg_bf16(uint32_t m, uint32_t cls, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a);

// two hidden layers: every class; other depths share the wider classes (hidden 32 or 64, action 8 or 16).  MODE 2: tanh
// everywhere and no statistics, fixed at compile time; -1: read from the arguments
template <int CJ, int NQ, int MODE, bool BF16, int M>
void launch_class_act(int act_class, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a) {
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(64), lds, st, a); };
  if constexpr (M == 2) {
    if (act_class == 0) return go(rollout_reg_kernel<CJ, NQ, 4, MODE, BF16, M>);
  }
  if (act_class <= 1) go(rollout_reg_kernel<CJ, NQ, 8, MODE, BF16, M>);
  else go(rollout_reg_kernel<CJ, NQ, 16, MODE, BF16, M>);
}
template <int CJ, int MODE, bool BF16, int M>
void launch_class_hid(int hid_class, int act_class, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a) {
  if constexpr (M == 2) {
    if (hid_class == 0) return launch_class_act<CJ, 1, MODE, BF16, M>(act_class, grid, lds, st, a);
  }
  if (hid_class <= 1) launch_class_act<CJ, 2, MODE, BF16, M>(act_class, grid, lds, st, a);
  else launch_class_act<CJ, 4, MODE, BF16, M>(act_class, grid, lds, st, a);
}
template <int MODE, bool BF16, int M>
void launch_class(uint32_t cls, dim3 grid, size_t lds, hipStream_t st, const RegArgs& a) {
  const int obs_class = (int)cls / 9, hid_class = (int)(cls / 3) % 3, act_class = (int)cls % 3;
  if (obs_class == 0) launch_class_hid<4, MODE, BF16, M>(hid_class, act_class, grid, lds, st, a);
  else if (obs_class == 1) launch_class_hid<8, MODE, BF16, M>(hid_class, act_class, grid, lds, st, a);
  else launch_class_hid<16, MODE, BF16, M>(hid_class, act_class, grid, lds, st, a);
}

}  // namespace es
