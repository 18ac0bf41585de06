// es_rollout in passes of SIXTEEN environment copies, one wavefront each: up to 64 hidden units, two hidden layers, obs <= 64, act <= 16,
// binary32 or bf16 operands, for populations whose episodes outnumber the wavefronts of the chip.
//
// Paper Sec. 3.2 / 5.1: population x environment-copy evaluation of a deterministic MLP policy, fitness = mean undiscounted
// return.  The copies are the columns of the 16-row matrix-core shapes (binary32 16x16x4: lane (g, n) of sixteen lanes a group supplies A[row n][k = g]
// and B[k = g][column n]; bf16 16x16x32: eight consecutive k each), the weights the A operand, parked in registers for all T steps.  Lane (g, n)
// gets rows 4 g .. 4 g + 3 of column n in the four result registers, and any order of the rows and of K is as good as another as long as
// both operands agree.  So unit (state element, action) 16 t + 4 r + g is row 4 g + r of tile t: what a lane holds of a layer is what it supplies to
// the next product - K step 4 t + r takes result register r of tile t - and a whole step is products and activations on registers the lane owns.
// No LDS, no exchange between lanes, no barrier; a layer of n units costs ceil(n / 4) K steps.  Each lane accumulates its share of its copy's
// return; a copy that ends is a bit of a compare mask behind a branch that is not taken.
// Bound, binary32: matrix issue (32 cycles per 16x16x4) plus vector issue, which do not overlap - binary32 products and vector instructions share
// the multipliers, in one wavefront and between two.  19-48-48-5 (ReLU, statistics), 1000 x 16 copies: 77 products a step, 2464 of 3300 cycles;
// 4.29 ms in passes of four copies -> 1.40 ms per 1000 steps.
// bf16: the activations (29 cycles per tanh of a register); 17-64-64-6, 1000 x 16 copies x 60 steps: 137 -> 64 us.
#pragma once

#include "rollout_quad.hpp"

namespace es {

namespace cols {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The perturbed parameters of one individual, all of them, into LDS in coalesced order by one wavefront: four consecutive ones per lane and
// load where the row has them, the loads of eight iterations in flight together.
template <class Elem>
__device__ __forceinline__ void stage_all(Elem* sp, const float* __restrict__ theta, const NoiseRow nz, float scale, uint32_t count) {
  constexpr uint32_t U = STAGE_BATCH;
  const uint32_t lane = threadIdx.x, quads = count / 4u;
  auto batch = [&](auto fetch) {
    for (uint32_t q0 = lane; q0 < quads; q0 += 64u * U) {
      f32x4 tv[U];
      decltype(fetch(0u)) ev[U];
#pragma unroll
      for (uint32_t v = 0; v < U; ++v) {
        const uint32_t idx = 4u * min(q0 + 64u * v, quads - 1u);
        tv[v] = *reinterpret_cast<const f32x4*>(theta + idx);
        ev[v] = fetch(idx);
      }
#pragma unroll
      for (uint32_t v = 0; v < U; ++v) {
        const f32x4 e = widen4(ev[v]);
        if (q0 + 64u * v < quads)
          put4(sp + 4u * (q0 + 64u * v), f32x4{__fmaf_rn(scale, e.x, tv[v].x), __fmaf_rn(scale, e.y, tv[v].y), __fmaf_rn(scale, e.z, tv[v].z), __fmaf_rn(scale, e.w, tv[v].w)});
      }
    }
    const uint32_t k = 4u * quads + lane;      // the last one to three
    if (k < count) put1(sp + k, __fmaf_rn(scale, row_noise(nz, k), theta[k]));
  };
  if (nz.mode >= 2u) {
#pragma unroll 1
    for (uint32_t d0 = 4u * lane; d0 < count; d0 += 256u) {
      float z[4];
      noise_regen4(nz.row, d0, nz.gen, nz.k0, nz.k1, nz.mode == 3u, z);
#pragma unroll
      for (uint32_t k = 0; k < 4u; ++k)
        if (d0 + k < count) put1(sp + d0 + k, __fmaf_rn(scale, z[k], theta[d0 + k]));
    }
  } else if (nz.mode == 1u) {
    batch([&](uint32_t idx) { return *reinterpret_cast<const u32x2*>(static_cast<const uint16_t*>(nz.ptr) + idx); });
  } else {
    batch([&](uint32_t idx) { return *reinterpret_cast<const f32x4*>(static_cast<const float*>(nz.ptr) + idx); });
  }
  __syncthreads();
}

// LDS of an individual's parameters
template <class Elem>
constexpr uint32_t param_bytes(uint32_t count) { return ((uint32_t)sizeof(Elem) * count + 15u) / 16u * 16u; }

}  // namespace cols

// KS: groups of four state elements (class of ceil(obs / 4)); HT: tiles of sixteen hidden units; NAK: groups of four actions.
template <bool BF16_, int KS_, int HT_, int NAK_, bool RELU_, bool NORM_>
struct ColsShape {
  static constexpr bool BF16 = BF16_, RELU = RELU_, NORM = NORM_;
  static constexpr int KS = KS_, HT = HT_, NAK = NAK_;
  static constexpr int OT = (KS + 3) / 4;                                  // tiles of the state
  static constexpr int NA = 4;                                             // result registers of the action tile
  // operands of a product along K: binary32 one register a K step, bf16 a pair of tiles (four registers)
  static constexpr int K1 = BF16 ? (OT + 1) / 2 : KS, KH = BF16 ? (HT + 1) / 2 : 4 * HT, KA = BF16 ? 1 : NAK;
  static constexpr int WREGS = (BF16 ? 4 : 1) * (HT * K1 + HT * KH + KH + OT * K1 + OT * KA) + 8 * HT + 4;      // weights and biases of a lane
  static constexpr int WORK = 12 * OT + 8 * HT + 40 + (NORM ? 8 * OT : 0);
  static constexpr int OCC = WREGS + WORK <= 168 ? 3 : WREGS + WORK <= 256 ? 2 : 1;       // wavefronts per SIMD the registers leave room for
};

template <class S>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(S::OCC, S::OCC)))
void rollout_cols_kernel(const QuadArgs a) {
  using namespace cols;
  constexpr bool BF16 = S::BF16, NORM = S::NORM;
  constexpr int HT = S::HT, OT = S::OT, K1 = S::K1, KH = S::KH, KA = S::KA;
  using Op = std::conditional_t<BF16, bf16x8, float>;
  extern __shared__ __align__(16) unsigned char lds[];
  using Elem = std::conditional_t<BF16, uint16_t, float>;
  Elem* sp = reinterpret_cast<Elem*>(lds);
  const int lane = threadIdx.x, g = lane >> 4, n = lane & 15;
  const int no = (int)a.no, nh = (int)a.nh, na = (int)a.na;
  const uint32_t i = blockIdx.x / a.split, pass0 = blockIdx.x - i * a.split;
  const uint32_t row = a.antithetic ? i >> 1 : i;
  const float scale = (a.antithetic && (i & 1u)) ? -a.sigma : a.sigma;
  // matrix row of this lane as an A operand, and element of result register r, of tile t
  auto row_of = [&](int t) { return 16 * t + 4 * (n & 3) + (n >> 2); };
  auto elem = [&](int t, int r) { return 16 * t + 4 * r + g; };
  // K operand kk of a matrix row: src(k) for the K indices this lane supplies
  auto operand = [&](int kk, auto src) -> Op {
    if constexpr (BF16) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = src(elem(2 * kk + (j >> 2), j & 3));
      const u32x2 lo = pack_bf16x4(v[0], v[1], v[2], v[3]), hi = pack_bf16x4(v[4], v[5], v[6], v[7]);
      return __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
    } else {
      return src(4 * kk + g);
    }
  };
  auto mma = [](Op w, Op x, f32x4 c) {
    if constexpr (BF16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x4f32(w, x, c, 0, 0, 0);
  };

  // one wavefront per SIMD: the wide layers sit in the accumulation half of the register file, where the products read them directly
  auto pin = [](Op& w) { asm volatile("" : "+a"(w)); };

  // ---- environment matrices and statistics, requested first (masked elements read the matrix's first entry) ----
  Op Ae[OT][K1], Be[OT][KA];
#pragma unroll
  for (int t = 0; t < OT; ++t) {
    const int el = row_of(t);
#pragma unroll
    for (int kk = 0; kk < K1; ++kk)
      Ae[t][kk] = operand(kk, [&](int k) { const bool ok = el < no && k < no; const float v = a.A[ok ? el * no + k : 0]; return ok ? v : 0.0f; });
#pragma unroll
    for (int kk = 0; kk < KA; ++kk)
      Be[t][kk] = operand(kk, [&](int k) { const bool ok = el < no && k < na; const float v = a.B[ok ? el * na + k : 0]; return ok ? v : 0.0f; });
  }
  f32x4 mu[NORM ? OT : 1], iv[NORM ? OT : 1];
  if constexpr (NORM) {
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool ok = elem(t, r) < no;
        mu[t][r] = ok ? a.obs_mean[elem(t, r)] : 0.0f;
        iv[t][r] = ok ? a.obs_inv[elem(t, r)] : 0.0f;
      }
  }

  // ---- perturbed parameters -> LDS -> registers ----
  NoiseRow nz;
  nz.mode = a.noise_mode; nz.row = row; nz.gen = a.gen; nz.k0 = a.k0; nz.k1 = a.k1; nz.ptr = nullptr;
  if (a.noise_offs) nz.ptr = table_row_base(a.noise_mode, a.noise, a.noise_offs, row);
  else if (a.noise_mode == 1u) nz.ptr = static_cast<const uint16_t*>(a.noise) + (size_t)row * a.ld;
  else if (a.noise_mode == 0u) nz.ptr = static_cast<const float*>(a.noise) + (size_t)row * a.ld;
  stage_all(sp, a.theta, nz, scale, a.ob3 + a.na);
  auto pick = [&](bool ok, int idx) { const float v = widen1(sp[ok ? idx : 0]); return ok ? v : 0.0f; };
  Op W1[HT][K1], W2[HT][KH], W3[KH];
  f32x4 b1[HT], b2[HT], b3;
#pragma unroll
  for (int u = 0; u < HT; ++u) {
    const int unit = row_of(u);
#pragma unroll
    for (int kk = 0; kk < K1; ++kk) W1[u][kk] = operand(kk, [&](int k) { return pick(unit < nh && k < no, (int)a.oW1 + unit * no + k); });
#pragma unroll
    for (int kk = 0; kk < KH; ++kk) W2[u][kk] = operand(kk, [&](int k) { return pick(unit < nh && k < nh, (int)a.oW2 + unit * nh + k); });
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      b1[u][r] = pick(elem(u, r) < nh, (int)a.ob1 + elem(u, r));
      b2[u][r] = pick(elem(u, r) < nh, (int)a.ob2 + elem(u, r));
    }
  }
#pragma unroll
  for (int kk = 0; kk < KH; ++kk) W3[kk] = operand(kk, [&](int k) { return pick(row_of(0) < na && k < nh, (int)a.oW3 + row_of(0) * nh + k); });
#pragma unroll
  for (int r = 0; r < 4; ++r) b3[r] = pick(elem(0, r) < na, (int)a.ob3 + elem(0, r));

  // a layer's tiles as K operands
  auto supply = [&](auto& x, const auto& v) {
    constexpr int T = (int)(sizeof(v) / sizeof(f32x4)), K = (int)(sizeof(x) / sizeof(Op));
#pragma unroll
    for (int kk = 0; kk < K; ++kk) {
      if constexpr (BF16) {
        const f32x4 p = v[2 * kk], q = 2 * kk + 1 < T ? v[2 * kk + 1 < T ? 2 * kk + 1 : 0] : f32x4{0.f, 0.f, 0.f, 0.f};
        const u32x2 lo = pack_bf16x4(p.x, p.y, p.z, p.w), hi = 2 * kk + 1 < T ? pack_bf16x4(q.x, q.y, q.z, q.w) : u32x2{0u, 0u};
        x[kk] = __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
      } else {
        x[kk] = v[kk >> 2][kk & 3];
      }
    }
  };
  auto squash = [](f32x4 v) { return f32x4{tanh_fast(v.x), tanh_fast(v.y), tanh_fast(v.z), tanh_fast(v.w)}; };
  // max(x, 0) as a median with an upper bound the compiler does not know: it would quieten the argument of a maximum with an instruction of its own
  float inf = __builtin_inff();
  asm volatile("" : "+s"(inf));
  auto relu = [&](float x) { return __builtin_amdgcn_fmed3f(x, 0.0f, inf); };
  auto hidden = [&](f32x4 v) { return S::RELU ? f32x4{relu(v.x), relu(v.y), relu(v.z), relu(v.w)} : squash(v); };
  const f32x4 zero4 = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint32_t npass = (a.E + 15u) / 16u;
  const float ninv = -1.0f / (float)no, ncost = -a.act_cost;
  // A copy that has ended goes on with the others and may run into infinities, so its share of the return is put aside when it ends (not multiplied
  // by zero from then on): one per lane, behind the parameters
  float* ends = reinterpret_cast<float*>(lds + param_bytes<Elem>(a.ob3 + a.na));
  uint32_t squash_l = a.out_tanh;      // (a select, not a branch)
  asm volatile("" : "+v"(squash_l));

  float fit_sum = 0.0f;
  for (uint32_t pass = pass0; pass < npass; pass += a.split) {
    const uint32_t e = 16u * pass + (uint32_t)n, cnt = min(16u, a.E - 16u * pass);
    const bool on = e < a.E;
    uint32_t alive = cnt == 16u ? 0xFFFFu : (1u << cnt) - 1u;      // copies still running (uniform)
    uint32_t len = a.T;
    float thr = on ? a.done_thresh : __builtin_inff(), R = 0.0f;      // of this lane's copy, while it runs
    f32x4 s[OT];
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) s[t][r] = on && elem(t, r) < no ? reset_value((uint32_t)elem(t, r), e, a.gen, a.k0, a.k1) : 0.0f;

    uint32_t t = 0u;
    while (true) {
      Op x[K1], xe[K1], h[KH], ax[KA];
      f32x4 acc[HT], accE[OT], v[HT];
      supply(xe, s);
      if constexpr (NORM) {
        f32x4 sn[OT];
#pragma unroll
        for (int q = 0; q < OT; ++q) sn[q] = (s[q] - mu[q]) * iv[q];
        supply(x, sn);
      }
      // ---- the hidden layers ----
#pragma unroll
      for (int u = 0; u < HT; ++u) {
        acc[u] = b1[u];
#pragma unroll
        for (int kk = 0; kk < K1; ++kk) {
          if (S::OCC == 1) pin(W1[u][kk]);
          acc[u] = mma(W1[u][kk], NORM ? x[kk] : xe[kk], acc[u]);
        }
      }
      // the reward's state term, from the pre-step state
      float ss = 0.0f;
#pragma unroll
      for (int q = 0; q < OT; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) ss = q + r == 0 ? s[0][0] * s[0][0] : __fmaf_rn(s[q][r], s[q][r], ss);
      R = __fmaf_rn(ss, ninv, R);
#pragma unroll
      for (int u = 0; u < HT; ++u) v[u] = hidden(acc[u]);
      supply(h, v);
#pragma unroll
      for (int u = 0; u < HT; ++u) {
        acc[u] = b2[u];
#pragma unroll
        for (int kk = 0; kk < KH; ++kk) {
          if (S::OCC == 1) pin(W2[u][kk]);
          acc[u] = mma(W2[u][kk], h[kk], acc[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < HT; ++u) v[u] = hidden(acc[u]);
      supply(h, v);
      // ---- the action and its cost, under it A s ----
      f32x4 av = b3;
#pragma unroll
      for (int kk = 0; kk < KH; ++kk) av = mma(W3[kk], h[kk], av);
#pragma unroll
      for (int q = 0; q < OT; ++q) {
        accE[q] = zero4;
#pragma unroll
        for (int kk = 0; kk < K1; ++kk) accE[q] = mma(Ae[q][kk], xe[kk], accE[q]);
      }
      const f32x4 ta = squash(av);
#pragma unroll
      for (int r = 0; r < S::NAK; ++r) av[r] = squash_l ? ta[r] : av[r];
#pragma unroll
      for (int r = S::NAK; r < 4; ++r) av[r] = 0.0f;
      float aa = av[0] * av[0];
#pragma unroll
      for (int r = 1; r < S::NAK; ++r) aa = __fmaf_rn(av[r], av[r], aa);
      R = __fmaf_rn(aa, ncost, R);
      { const f32x4 one[1] = {av}; supply(ax, one); }
      // ---- s' = tanh(A s + B a) ----
      float top = 0.0f;
#pragma unroll
      for (int q = 0; q < OT; ++q) {
#pragma unroll
        for (int kk = 0; kk < KA; ++kk) accE[q] = mma(Be[q][kk], ax[kk], accE[q]);
      }
#pragma unroll
      for (int q = 0; q < OT; ++q) {
        s[q] = squash(accE[q]);                // padded rows: tanh(0) = 0
        top = fmaxf(fmaxf(fmaxf(top, fabsf(s[q].x)), fmaxf(fabsf(s[q].y), fabsf(s[q].z))), fabsf(s[q].w));
      }
      // ---- termination: max |s| > threshold ends a copy after this step ----
      const unsigned long long over = __ballot(top > thr);
      ++t;
      if (__builtin_expect(over != 0ull || t == a.T, 0)) {
        uint32_t m = (uint32_t)(over | over >> 32);
        m = t == a.T ? alive : (m | m >> 16) & alive;
        if (m >> n & 1u) { len = t; thr = __builtin_inff(); ends[lane] = R; }
        alive &= ~m;
        if (alive == 0u) break;
      }
    }
    R = ends[lane];      // (written by this lane)
    // ---- outputs: return = length + the shares of the four lanes of a copy ----
    R += __shfl_xor(R, 16, 64);
    R += __shfl_xor(R, 32, 64);
    const float total = (float)len + R;
    if (g == 0 && on) {
      a.returns[(size_t)i * a.E + e] = total;
      a.ep_len[(size_t)i * a.E + e] = (int32_t)len;
    }
    for (uint32_t r = 0; r < cnt; ++r) fit_sum += __shfl(total, (int)r, 64);
  }
  if (a.fitness && lane == 0) a.fitness[i] = fit_sum / (float)a.E;
}

template <class S>
int launch_cols_shape(es_ctx* ctx, QuadArgs a, float* fitness, hipStream_t st) {
  const size_t lds = cols::param_bytes<std::conditional_t<S::BF16, uint16_t, float>>(a.ob3 + a.na) + 64u * sizeof(float);      // at most 38 KB
  const uint32_t npass = (a.E + 15u) / 16u, per_cu = (uint32_t)std::max<size_t>(1, std::min<size_t>(4 * S::OCC, (size_t)ctx->lds_limit / lds));
  a.split = quad_split(a.N, npass, (uint32_t)std::max(1, ctx->num_cus) * per_cu);
  a.fitness = a.split == 1u ? fitness : nullptr;
  hipLaunchKernelGGL(rollout_cols_kernel<S>, dim3(a.N * a.split), dim3(64), lds, st, a);
  int rc = check_launch(ctx, "es_rollout (passes of sixteen copies, one wavefront)");
  if (rc != ES_OK || a.split == 1u) return rc;
  return launch_fitness(ctx, a.returns, fitness, st);
}

template <bool BF16, int KS, int HT, int NAK>
int launch_cols_options(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  const bool relu = ctx->cfg.hidden_act == 1;
  if (a.obs_mean)
    return relu ? launch_cols_shape<ColsShape<BF16, KS, HT, NAK, true, true>>(ctx, a, fitness, st) : launch_cols_shape<ColsShape<BF16, KS, HT, NAK, false, true>>(ctx, a, fitness, st);
  return relu ? launch_cols_shape<ColsShape<BF16, KS, HT, NAK, true, false>>(ctx, a, fitness, st) : launch_cols_shape<ColsShape<BF16, KS, HT, NAK, false, false>>(ctx, a, fitness, st);
}
template <int KS, int HT>
int launch_cols_act(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  return a.na <= 8 ? launch_cols_options<false, KS, HT, 2>(ctx, a, fitness, st) : launch_cols_options<false, KS, HT, 4>(ctx, a, fitness, st);
}
// classes of the widths: hidden units in tiles of sixteen, the state in groups of four (bf16: in tiles)
template <int HT>
int launch_cols_f32(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  if (a.no <= 16) return launch_cols_act<4, HT>(ctx, a, fitness, st);
  if (a.no <= 20) return launch_cols_act<5, HT>(ctx, a, fitness, st);
  if (a.no <= 32) return launch_cols_act<8, HT>(ctx, a, fitness, st);
  if (a.no <= 48) return launch_cols_act<12, HT>(ctx, a, fitness, st);
  return launch_cols_act<16, HT>(ctx, a, fitness, st);
}
template <int HT>
int launch_cols_bf16(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  if (a.no <= 16) return launch_cols_options<true, 4, HT, 4>(ctx, a, fitness, st);
  if (a.no <= 32) return launch_cols_options<true, 8, HT, 4>(ctx, a, fitness, st);
  return launch_cols_options<true, 16, HT, 4>(ctx, a, fitness, st);
}

// one source file each (compile time)
int launch_cols_f32_small(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);     // up to 32 hidden units
int launch_cols_f32_48(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);
int launch_cols_f32_64(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);
int launch_cols_bf16(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);

}  // namespace es
