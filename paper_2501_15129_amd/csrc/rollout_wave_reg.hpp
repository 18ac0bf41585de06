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
// Bound: one wavefront's instructions (32-256 episodes for 1024 SIMDs).  A lone wavefront is fed 8 bytes of code every 5.2
// cycles, which is one DPP multiply-add, and no number of independent instructions hides that; so the count of instructions and
// bytes of a step is what matters (18 KB per 10 steps of 17-64-64-6), and a taken branch, which costs 70 cycles, comes once in
// four steps.  Splitting an episode over four wavefronts measured the same (two LDS hand-overs of 140 cycles per step).
// 17-64-64-6, 256 episodes x 1000 steps: 465 -> 447 us; 11-40-40-3: 455 -> 425 us; three layers, which used to stream their
// weights from the LDS: 17-64-64-64-6, 128 episodes x 400 steps: 4.2 -> 0.28 ms.
#pragma once

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
  constexpr int UNROLL = 4;
  constexpr bool RELU = FIXED && (MODE & 4), OUT_TANH = FIXED && (MODE & 2), NORM = !FIXED || (MODE & 1);
  extern __shared__ float sp[];      // the individual's perturbed parameters, once
  const int u = threadIdx.x;
  const uint32_t i = blockIdx.x / a.E, e = blockIdx.x % a.E;
  const uint32_t row = a.antithetic ? (i >> 1) : i;
  const float scale = (a.antithetic && (i & 1u)) ? -a.sigma : a.sigma;
  const int no = (int)a.no, nh = (int)a.nh, na = (int)a.na;
  const int lr = u >> 4, lc = u & 15;
  const int ks = 4 * lc + lr;                    // the state element of this lane
  const bool sval = lc < CJ && ks < no;
  const int hu = NQ == 1 ? lc : u;               // the hidden unit of this lane
  const bool hid = hu < nh;
  auto opnd = [](float v) { return BF16 ? bf16_round(v) : v; };      // a value as an operand of a product
  // ... of one of the ENVIRONMENT's products: rounded like the policy's unless the environment stays binary32 (a select,
  // not a branch: the flag is read into a vector register the compiler cannot prove uniform)
  uint32_t envf_l = a.env_f32;
  if (BF16) asm volatile("" : "+v"(envf_l));
  auto opnd_env = [&](float v) { return BF16 ? (envf_l ? v : bf16_round(v)) : v; };

  // ---- this lane's weights ----
  // first layer: partial sums of the units lc, lc + 16, ... over the inputs of row lr: w1[CJ q + j] = W1[lc + 16 q][4 j + lr]
  // second layer and action layer: the same over the 16 hidden units of row lr: w2[16 q + j] = W2[lc + 16 q][16 lr + j],
  //   w3[j] = W3[lc][16 lr + j] (with one row of hidden units every row holds all of them: input j)
  // environment: partial sums of the four state elements of column lc: ar[CJ r + j] = A[4 lc + r][4 j + lr];
  //   action term of this lane's own element: br[c] = B[ks][c]
  float w1[NQ * CJ], w2[M > 1 ? M - 1 : 1][NQ * 16], w3[16], ar[4 * CJ], br[NAR], b1, b2[M > 1 ? M - 1 : 1], b3;
  // (one layer's window, at most 16.6 KB, leaves room for nine wavefronts per CU)
  const ParamStage ps = param_stage(a, row, scale);
  ps.stage<64, BF16>(sp, a.oW1, (uint32_t)(nh * no + nh));
#pragma unroll
  for (int qq = 0; qq < NQ; ++qq)
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
      const int unit = lc + 16 * qq, k = 4 * j + lr;
      w1[CJ * qq + j] = (unit < nh && k < no) ? sp[unit * no + k] : 0.f;
    }
  b1 = hid ? sp[nh * no + hu] : 0.f;
#pragma unroll
  for (int l = 0; l < M - 1; ++l) {
    ps.stage<64, BF16>(sp, a.oW2 + (uint32_t)l * (uint32_t)(nh * nh + nh), (uint32_t)(nh * nh + nh));
#pragma unroll
    for (int qq = 0; qq < NQ; ++qq)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int unit = lc + 16 * qq, k = (NQ == 1 ? 0 : 16 * lr) + j;
        w2[l][16 * qq + j] = (unit < nh && k < nh) ? sp[unit * nh + k] : 0.f;
      }
    b2[l] = hid ? sp[nh * nh + hu] : 0.f;
  }
  ps.stage<64, BF16>(sp, a.oW3, (uint32_t)(na * nh + na));
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int k = (NQ == 1 ? 0 : 16 * lr) + j;
    w3[j] = (lc < na && k < nh) ? sp[lc * nh + k] : 0.f;
  }
  b3 = lc < na ? sp[na * nh + lc] : 0.f;            // in every row: the action vector is kept once per row
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
      const int el = 4 * lc + r, k = 4 * j + lr;
      ar[CJ * r + j] = (lc < CJ && el < no && k < no) ? opnd_env(a.A[el * no + k]) : 0.f;
    }
#pragma unroll
  for (int c = 0; c < NAR; ++c) br[c] = (sval && c < na) ? opnd_env(a.B[ks * na + c]) : 0.f;

  // frozen observation statistics of this lane's state element (identity when none are set: (s - 0) * 1 = s exactly)
  const bool stats = a.obs_mean != nullptr;
  const float mu = (NORM && stats && sval) ? a.obs_mean[ks] : 0.f;
  const float iv = (NORM && stats && sval) ? a.obs_inv[ks] : 1.f;
  // run-time activation choices as per-lane values the compiler cannot prove uniform: selects, not branches
  uint32_t relu_l = a.hidden_relu, otanh_l = a.out_tanh;
  if (!FIXED) asm volatile("" : "+v"(relu_l), "+v"(otanh_l));
  float s = sval ? reset_value((uint32_t)ks, e, a.gen, a.k0, a.k1) : 0.f;
  float R = 0.f;                      // per-lane share of the return
  const float ninv_no = -1.0f / (float)no, nq_cost = -0.25f * a.act_cost;

  // c of tanh(x) = 1 - 2 / (1 + 2^(c x)) in a scalar register: the multiplication is four bytes then, not eight
  float tanh_c = 2.88539008f;      // 2 log2(e), as in tanh_fast
  asm volatile("" : "+s"(tanh_c));
  // bf16 policies of one, three and four layers: the tanh that is accurate near zero, like the LDS kernel's, which served them
  // (error of the returns against binary64, geometric mean of 50 random shapes: 3.9e-6 there, 8.4e-6 with the short form, 3.7e-6
  // with this one; 0 to 6 % of the time)
  auto tanh_s = [&](float x) {
    if (BF16 && M != 2) return tanh_near(x * tanh_c);
    return __fmaf_rn(-2.0f, __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(x * tanh_c) + 1.0f), 1.0f);
  };
  auto hidden = [&](float l) {
    if (FIXED) return RELU ? fmaxf(l, 0.f) : tanh_s(l);
    const float t = tanh_s(l);
    return relu_l ? fmaxf(l, 0.f) : t;
  };
  // one step; true: the episode is over
  auto step = [&]() {
    // h1 = act(W1 s + b1)
    const float xp = opnd(NORM ? (s - mu) * iv : s);      // the policy's input (paper App. B: fixed normalisation statistics)
    float p[NQ];
    row_bcast_dot<NQ, CJ>(p, xp, w1);
    float l1;
    if constexpr (NQ == 4) l1 = rows_transpose_add(p[0], p[1], p[2], p[3]);
    else if constexpr (NQ == 2) l1 = rows_transpose_add(p[0], p[1]);
    else l1 = rows_add(p[0]);
    float h2 = opnd(hidden(l1 + b1));      // the last hidden layer so far
    // further hidden layers: h = act(W h + b)
#pragma unroll
    for (int l = 0; l < M - 1; ++l) {
      row_bcast_dot<NQ, 16>(p, h2, w2[l]);
      float l2;
      if constexpr (NQ == 4) l2 = rows_transpose_add(p[0], p[1], p[2], p[3]);
      else if constexpr (NQ == 2) l2 = swap16_add(p[0], p[1]);      // the units' own rows 0 and 1 hold all of their inputs
      else l2 = p[0];                                               // every row holds all inputs
      h2 = opnd(hidden(l2 + b2[l]));
    }
    // a = tanh(W3 h2 + b3): column c of every row ends up with unit c's total, one tanh serves all units
    float pa[1];
    row_bcast_dot<1, 16>(pa, h2, w3);
    float pv = NQ == 1 ? pa[0] : rows_add(pa[0]);
    pv = pv + b3;
    float tv;
    if (FIXED) tv = OUT_TANH ? tanh_s(pv) : pv;      // columns >= act: weights and bias are zero
    else { const float tt = tanh_s(pv); tv = otanh_l ? tt : pv; }
    // reward from the pre-step state, 1 - |s|^2 / obs - cost |a|^2: a sum over all 64 lanes (the action vector is held
    // once per row, hence the quarter); this lane's share, the lanes are added after the last step
    R += __fmaf_rn(ninv_no * s, s, nq_cost * (tv * tv));
    // s' = tanh(A s + B a): partial sums of the four elements of this column over the inputs of this row, rows added
    // and moved to their element's lane; the action term straight from the row's action vector
    float ev[4];
    row_bcast_dot<4, CJ>(ev, opnd_env(s), ar);
    float pre = rows_transpose_add(ev[0], ev[1], ev[2], ev[3]);
    pre = row_bcast_mac<NAR>(pre, opnd_env(tv), br);
    s = tanh_s(pre);                                  // lanes without a state element: zero weights, tanh(0) = 0
    // max |s| > threshold: some lane exceeds it
    return __ballot(fabsf(s) > a.done_thresh) != 0ull;
  };
  // A taken branch costs a lone wavefront 70 cycles, a branch not taken 5: UNROLL steps per turn
  uint32_t len = 0u;
  for (uint32_t turns = a.T / (uint32_t)UNROLL; turns != 0u; --turns) {
#pragma unroll
    for (int k = 0; k < UNROLL; ++k) {
      ++len;
      asm volatile("" : "+s"(len));      // (one register, counted here: the exits would each need their own count otherwise)
      if (__builtin_expect(step(), 0)) goto end;
    }
  }
  for (uint32_t rest = a.T % (uint32_t)UNROLL; rest != 0u; --rest) {
    ++len;
    if (__builtin_expect(step(), 0)) break;
  }
end:
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
