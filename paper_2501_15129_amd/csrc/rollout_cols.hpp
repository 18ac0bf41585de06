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
// Binary32 runs on the bf16 shape too, values cut into three pieces (Split), wherever the pieces fit the registers (all but the widest classes): binary32 products take 32 cycles
// for four inputs and share the multipliers with vector instructions, in one wavefront and between two, so that the two add up - 19-48-48-5 (ReLU, statistics),
// 1000 x 16 copies: 77 products, 2464 of 3300 cycles a step, and 809 of vector issue.  Now 70 products (1120 cycles) beside 331 vector instructions, 2500 cycles:
// 4.29 ms in passes of four copies -> 1.40 -> 1.04 ms per 1000 steps.  100 steps of 1000 x 16 copies: 10-16-4 70 -> 72 us (4000 x 16: 280 -> 171), 18-32-4 135 -> 112, 30-64-12 292 -> 189,
// 44-48-4 264 -> 172, 60-48-12 350 -> 217; widest, as before: 60-64-4 419.  Bound: vector issue of a lone wavefront, and products with nothing beside them (state, first and last products of a layer).
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

// Binary32 products on the bf16 shapes.  A value is the sum of three bf16 values h + m + l, each the rest of the ones before it rounded to nearest, exactly (3 x 8 bits), and a
// product is h h' + h m' + m h' + h l' + m m' + l h': what is left out, m l' + l m' + l l', is 2^-24 of the product at most.  Products of bf16 values are exact and the sums are
// binary32's.  Three 16x16x32 products take 50 cycles for sixteen inputs, four 16x16x4 ones 128; and vector instructions run beside them.
//
// A lane's values in pairs, V of them: operands of four pairs' h, m and l; of two pairs' (h, m) and (l, h); of one pair's (h, m, l, h).
constexpr int split_full(int v) { return (v + 1) / 2 == 3 ? 4 : (v + 1) / 2; }                                       // pairs
constexpr int split_inputs(int v) { return split_full(v) / 4 * 3 + split_full(v) % 4; }                                // operands of the inputs
constexpr int split_weights(int v) { return split_full(v) / 4 * 3 + (split_full(v) % 4 ? split_full(v) % 4 + 1 : 0); }  // ... of the weights of an output tile
constexpr int split_products(int v) { return split_full(v) / 4 * 6 + (split_full(v) % 4 ? split_full(v) % 4 + 1 : 0); }
// registers of a lane's weights and biases, beside them, and whether there are as many (the widest stay with the binary32 shape)
constexpr int split_held(int ks, int ht, int nak) {
  const int ot = (ks + 3) / 4;
  return 4 * ((ht + ot) * split_weights(ks) + (ht + 1) * split_weights(4 * ht) + ot * split_weights(nak)) + 8 * ht + 4;
}
constexpr int split_work(int ks, int ht, bool norm) {
  const int ot = (ks + 3) / 4;
  return 12 * ot + 4 * (norm ? 2 : 1) * split_inputs(ks) + 8 * ht + 4 * split_inputs(4 * ht) + 40 + (norm ? 8 * ot : 0);
}
constexpr bool split_fits(int ks, int ht, int nak, bool norm) { return split_held(ks, ht, nak) + split_work(ks, ht, norm) <= 512; }
constexpr int wavefronts(int regs) { return regs <= 168 ? 3 : regs <= 256 ? 2 : 1; }                                   // per SIMD
// bf16's largest value: the first piece of a larger one would be infinite and the rest not a number
constexpr float LARGEST = 3.38953139e38f;
__device__ __forceinline__ float finite(float v) { return fabsf(v) > LARGEST ? copysignf(LARGEST, v) : v; }

template <int V>
struct Split {
  static constexpr int P = (V + 1) / 2, FULL = split_full(V), G = FULL / 4, REST = FULL % 4;
  static constexpr int NX = split_inputs(V), NW = split_weights(V), MF = split_products(V);
  static_assert(REST != 3, "pairs of a lane");
  // Cutting N pairs of values into pieces in stages: convert, widen, subtract, convert, widen, subtract, convert.  (A rest as one two-element bf16 product on top of the value,
  // v_dot2c_f32_bf16, whose result must not be used within three instructions: 1 055 us instead of 1 018 at 19-48-48-5, 1000 x 16 copies.)
  static constexpr int STAGES = 7;
  template <int STAGE, int N>
  static __device__ __forceinline__ void cut_stage(float (&a)[2 * N], float (&piece)[2 * N], uint32_t (&r)[N][3]) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      if constexpr (STAGE % 3 == 0) {
        r[k][STAGE / 3] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a[2 * k], a[2 * k + 1]}, bf16x2));
      } else if constexpr (STAGE % 3 == 1) {
        piece[2 * k] = __uint_as_float(r[k][STAGE / 3] << 16);
        piece[2 * k + 1] = __uint_as_float(r[k][STAGE / 3] & 0xFFFF0000u);
      } else {
        a[2 * k] -= piece[2 * k];
        a[2 * k + 1] -= piece[2 * k + 1];
      }
    }
  }
  static __device__ __forceinline__ bf16x8 four(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return __builtin_bit_cast(bf16x8, u32x4{a, b, c, d}); }
  // val(v), v < V -> the pieces of all pairs (of pairs past the last one: zero)
  template <class F>
  static __device__ __forceinline__ void cut(uint32_t (&r)[FULL][3], F val) {
    float a[2 * FULL], piece[2 * FULL];
#pragma unroll
    for (int v = 0; v < 2 * FULL; ++v) a[v] = v < V ? val(v < V ? v : 0) : 0.0f;
    quad::static_for<0, STAGES>([&](auto sc) { cut_stage<decltype(sc)::value, FULL>(a, piece, r); });
  }
  // all pairs' pieces -> inputs (of the groups of four from FROM on, and the rest)
  template <int FROM = 0>
  static __device__ __forceinline__ void inputs(bf16x8 (&x)[NX], const uint32_t (&r)[FULL][3]) {
#pragma unroll
    for (int g = FROM; g < G; ++g)
#pragma unroll
      for (int j = 0; j < 3; ++j) x[3 * g + j] = four(r[4 * g][j], r[4 * g + 1][j], r[4 * g + 2][j], r[4 * g + 3][j]);
    constexpr int e = 4 * G;
    if constexpr (REST == 2) {
      x[3 * G] = four(r[e][0], r[e + 1][0], r[e][1], r[e + 1][1]);
      x[3 * G + 1] = four(r[e][2], r[e + 1][2], r[e][0], r[e + 1][0]);
    } else if constexpr (REST == 1) {
      x[3 * G] = four(r[e][0], r[e][1], r[e][2], r[e][0]);
    }
  }
  // ... -> weights, the counterpart
  template <class F>
  static __device__ __forceinline__ void weights(bf16x8 (&w)[NW], F val) {
    uint32_t r[FULL][3];
    cut(r, [&](int v) { return finite(val(v)); });
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int j = 0; j < 3; ++j) w[3 * g + j] = four(r[4 * g][j], r[4 * g + 1][j], r[4 * g + 2][j], r[4 * g + 3][j]);
    constexpr int e = 4 * G;
    if constexpr (REST == 2) {
      w[3 * G] = four(r[e][0], r[e + 1][0], r[e][0], r[e + 1][0]);
      w[3 * G + 1] = four(r[e][1], r[e + 1][1], r[e][1], r[e + 1][1]);
      w[3 * G + 2] = four(r[e][0], r[e + 1][0], r[e][2], r[e + 1][2]);
    } else if constexpr (REST == 1) {
      w[3 * G] = four(r[e][0], r[e][0], r[e][0], r[e][1]);
      w[3 * G + 1] = four(r[e][2], r[e][1], 0u, 0u);
    }
  }
  // product K of MF, a group's small terms first
  template <int K, class M>
  static __device__ __forceinline__ f32x4 step(const bf16x8 (&w)[NW], const bf16x8 (&x)[NX], f32x4 acc, M mma) {
    if constexpr (K < 6 * G) {
      constexpr int wi[6] = {2, 1, 0, 1, 0, 0}, xi[6] = {0, 1, 2, 0, 1, 0};
      return mma(w[3 * (K / 6) + wi[K % 6]], x[3 * (K / 6) + xi[K % 6]], acc);
    } else if constexpr (REST == 2) {
      return mma(w[3 * G + MF - 1 - K], x[3 * G + (K == 6 * G ? 1 : 0)], acc);
    } else {
      return mma(w[3 * G + MF - 1 - K], x[3 * G], acc);
    }
  }
};

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
  using SX = cols::Split<KS>; using SH = cols::Split<4 * HT>; using SA = cols::Split<NAK>;
  static constexpr bool SPLIT = !BF16 && cols::split_fits(KS, HT, NAK, NORM);      // binary32: products of three-piece values
  // operands of a product along K: bf16 a pair of tiles (four registers), split see there, else one register a K step; inputs and weights of an output tile
  static constexpr int K1 = BF16 ? (OT + 1) / 2 : SPLIT ? SX::NX : KS, KH = BF16 ? (HT + 1) / 2 : SPLIT ? SH::NX : 4 * HT, KA = BF16 ? 1 : SPLIT ? SA::NX : NAK;
  static constexpr int W1N = SPLIT ? SX::NW : K1, WHN = SPLIT ? SH::NW : KH, WAN = SPLIT ? SA::NW : KA;
  static constexpr int WREGS = (BF16 || SPLIT ? 4 : 1) * (HT * W1N + HT * WHN + WHN + OT * W1N + OT * WAN) + 8 * HT + 4;      // weights and biases of a lane
  static constexpr int WORK = SPLIT ? cols::split_work(KS, HT, NORM) : 12 * OT + 8 * HT + 40 + (NORM ? 8 * OT : 0);
  static constexpr int OCC = cols::wavefronts(WREGS + WORK);
};

template <class S>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(S::OCC, S::OCC)))
void rollout_cols_kernel(const QuadArgs a) {
  using namespace cols;
  constexpr bool BF16 = S::BF16, NORM = S::NORM, SPLIT = S::SPLIT;
  constexpr int HT = S::HT, OT = S::OT, K1 = S::K1, KH = S::KH, KA = S::KA;
  using Op = std::conditional_t<BF16 || SPLIT, bf16x8, float>;
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
    if constexpr (BF16 || SPLIT) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x4f32(w, x, c, 0, 0, 0);
  };

  // one wavefront per SIMD: the wide layers sit in the accumulation half of the register file, where the products read them directly
  auto pin = [](Op& w) { asm volatile("" : "+a"(w)); };

  // ---- environment matrices and statistics, requested first (masked elements read the matrix's first entry) ----
  using SX = typename S::SX; using SH = typename S::SH; using SA = typename S::SA;
  Op Ae[OT][S::W1N], Be[OT][S::WAN];
#pragma unroll
  for (int t = 0; t < OT; ++t) {
    const int el = row_of(t);
    auto of_A = [&](int k) { const bool ok = el < no && k < no; const float v = a.A[ok ? el * no + k : 0]; return ok ? v : 0.0f; };
    auto of_B = [&](int k) { const bool ok = el < no && k < na; const float v = a.B[ok ? el * na + k : 0]; return ok ? v : 0.0f; };
    if constexpr (SPLIT) {
      SX::weights(Ae[t], [&](int v) { return of_A(elem(v >> 2, v & 3)); });
      SA::weights(Be[t], [&](int v) { return of_B(elem(v >> 2, v & 3)); });
    } else {
#pragma unroll
      for (int kk = 0; kk < K1; ++kk) Ae[t][kk] = operand(kk, of_A);
#pragma unroll
      for (int kk = 0; kk < KA; ++kk) Be[t][kk] = operand(kk, of_B);
    }
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
        if constexpr (SPLIT) {      // (an infinite input has no pieces)
          if (fabsf(mu[t][r]) > 1e8f) mu[t][r] = copysignf(1e8f, mu[t][r]);
          if (fabsf(iv[t][r]) > 1e30f) iv[t][r] = copysignf(1e30f, iv[t][r]);
        }
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
  Op W1[HT][S::W1N], W2[HT][S::WHN], W3[S::WHN];
  f32x4 b1[HT], b2[HT], b3;
#pragma unroll
  for (int u = 0; u < HT; ++u) {
    const int unit = row_of(u);
    auto of_1 = [&](int k) { return pick(unit < nh && k < no, (int)a.oW1 + unit * no + k); };
    auto of_2 = [&](int k) { return pick(unit < nh && k < nh, (int)a.oW2 + unit * nh + k); };
    if constexpr (SPLIT) {
      SX::weights(W1[u], [&](int v) { return of_1(elem(v >> 2, v & 3)); });
      SH::weights(W2[u], [&](int v) { return of_2(elem(v >> 2, v & 3)); });
    } else {
#pragma unroll
      for (int kk = 0; kk < K1; ++kk) W1[u][kk] = operand(kk, of_1);
#pragma unroll
      for (int kk = 0; kk < KH; ++kk) W2[u][kk] = operand(kk, of_2);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      b1[u][r] = pick(elem(u, r) < nh, (int)a.ob1 + elem(u, r));
      b2[u][r] = pick(elem(u, r) < nh, (int)a.ob2 + elem(u, r));
    }
  }
  auto of_3 = [&](int k) { return pick(row_of(0) < na && k < nh, (int)a.oW3 + row_of(0) * nh + k); };
  if constexpr (SPLIT) {
    SH::weights(W3, [&](int v) { return of_3(elem(v >> 2, v & 3)); });
  } else {
#pragma unroll
    for (int kk = 0; kk < KH; ++kk) W3[kk] = operand(kk, of_3);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) b3[r] = pick(elem(0, r) < na, (int)a.ob3 + elem(0, r));

  // a layer's tiles as K operands
  auto supply = [&](auto& x, auto split, const auto& v) {
    if constexpr (SPLIT) {
      uint32_t r[decltype(split)::FULL][3];
      decltype(split)::cut(r, [&](int k) { return v[k >> 2][k & 3]; });
      decltype(split)::inputs(x, r);
      return;
    }
    constexpr int T = (int)(sizeof(v) / sizeof(f32x4)), K = (int)(sizeof(x) / sizeof(Op));
#pragma unroll
    for (int kk = 0; kk < K; ++kk) {
      if constexpr (BF16) {
        const f32x4 p = v[2 * kk], q = 2 * kk + 1 < T ? v[2 * kk + 1 < T ? 2 * kk + 1 : 0] : f32x4{0.f, 0.f, 0.f, 0.f};
        const u32x2 lo = pack_bf16x4(p.x, p.y, p.z, p.w), hi = 2 * kk + 1 < T ? pack_bf16x4(q.x, q.y, q.z, q.w) : u32x2{0u, 0u};
        x[kk] = __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
      } else if constexpr (!SPLIT) {
        x[kk] = v[kk >> 2][kk & 3];
      }
    }
  };
  auto squash = [](f32x4 v) { return f32x4{tanh_fast(v.x), tanh_fast(v.y), tanh_fast(v.z), tanh_fast(v.w)}; };
  // max(x, 0) as a median with an upper bound the compiler does not know: it would quieten the argument of a maximum with an instruction of its own
  float inf = SPLIT ? LARGEST : __builtin_inff();
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
      f32x4 acc[HT], accE[OT], v[HT], av;
      if constexpr (SPLIT) {
        // The vector work of one tile beside the products of the next, by hand: left to itself the compiler issues one after the other.  products(k), k < M, over the
        // stages of the vector work, stage(i), i < V, before each its share
        auto weave = [](auto mc, auto products, auto vc, auto stage) {
          constexpr int M = decltype(mc)::value, V = decltype(vc)::value;
          quad::static_for<0, V>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            quad::static_for<M * i / V, M * (i + 1) / V>(products);
            __builtin_amdgcn_sched_barrier(0);
            stage(ic);
            __builtin_amdgcn_sched_barrier(0);
          });
        };
        auto hold = [&](auto& W) {
          if constexpr (S::OCC == 1) {
#pragma unroll
            for (int kk = 0; kk < (int)(sizeof(W) / sizeof(Op)); ++kk) pin(W[kk]);
          }
        };
        constexpr int M1 = SX::MF, MH = SH::MF;
        // activation of a tile of four registers, then its pieces, in stages
        constexpr int ACT = S::RELU ? 1 : 5, TILE = ACT + SH::STAGES;
        uint32_t pieces[SH::FULL][3], cutting[2][3];
        float a4[4], rest4[4];
        auto tile_stage = [&](auto uc, auto ic) {
          constexpr int u = decltype(uc)::value, i = decltype(ic)::value;
          if constexpr (i < ACT) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              if constexpr (S::RELU) a4[r] = relu(acc[u][r]);
              else if constexpr (i == 0) a4[r] = acc[u][r] * quad::TANH_C;
              else if constexpr (i == 1) a4[r] = __builtin_amdgcn_exp2f(a4[r]);
              else if constexpr (i == 2) a4[r] = a4[r] + 1.0f;
              else if constexpr (i == 3) a4[r] = __builtin_amdgcn_rcpf(a4[r]);
              else a4[r] = __fmaf_rn(-2.0f, a4[r], 1.0f);
            }
          } else {
            SH::template cut_stage<i - ACT, 2>(a4, rest4, cutting);
            if constexpr (i == TILE - 1) {
#pragma unroll
              for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int j = 0; j < 3; ++j) pieces[2 * u + k][j] = cutting[k][j];
            }
          }
        };
        if constexpr (NORM) {
          f32x4 sn[OT];
#pragma unroll
          for (int q = 0; q < OT; ++q) sn[q] = (s[q] - mu[q]) * iv[q];
          supply(x, SX{}, sn);
        } else {
          supply(xe, SX{}, s);
        }
        __builtin_amdgcn_sched_barrier(0);
        quad::static_for<0, HT>([&](auto uc) {
          constexpr int u = decltype(uc)::value;
          hold(W1[u]);
          acc[u] = b1[u];
          auto products = [&](auto kc) {
            if constexpr (NORM) acc[u] = SX::template step<decltype(kc)::value>(W1[u], x, acc[u], mma);
            else acc[u] = SX::template step<decltype(kc)::value>(W1[u], xe, acc[u], mma);
          };
          if constexpr (u == 0) {
            quad::static_for<0, M1>(products);
            if constexpr (NORM) supply(xe, SX{}, s);
            // the reward's state term, from the pre-step state
            float ss = 0.0f;
#pragma unroll
            for (int q = 0; q < OT; ++q)
#pragma unroll
              for (int r = 0; r < 4; ++r) ss = q + r == 0 ? s[0][0] * s[0][0] : __fmaf_rn(s[q][r], s[q][r], ss);
            R = __fmaf_rn(ss, ninv, R);
            __builtin_amdgcn_sched_barrier(0);
          } else {
            weave(std::integral_constant<int, M1>{}, products, std::integral_constant<int, TILE>{}, [&](auto ic) { tile_stage(std::integral_constant<int, u - 1>{}, ic); });
          }
        });
        // Under a layer's last tile, which its own inputs do not wait for: the next product's groups that are complete, or, where there are none, products of A s; what is left of
        // these goes under the action's activation
        constexpr int G0 = (HT - 1) / 2, E1 = G0 ? 0 : M1, E2 = G0 || OT == 1 ? E1 : E1 + M1;
        quad::static_for<0, OT>([&](auto qc) { accE[decltype(qc)::value] = zero4; });
        auto env = [&](auto kc) {
          constexpr int q = decltype(kc)::value / M1, k = decltype(kc)::value % M1;
          accE[q] = SX::template step<k>(Ae[q], xe, accE[q], mma);
        };
        auto ready = [&](auto gc) {      // groups whose tiles are cut
          constexpr int g = decltype(gc)::value;
#pragma unroll
          for (int j = 0; j < 3; ++j) h[3 * g + j] = SH::four(pieces[4 * g][j], pieces[4 * g + 1][j], pieces[4 * g + 2][j], pieces[4 * g + 3][j]);
        };
        auto last_tile = [&](auto ic) { tile_stage(std::integral_constant<int, HT - 1>{}, ic); };
        using Stages = std::integral_constant<int, TILE>;
        quad::static_for<0, G0>(ready);
        hold(W2[0]);
        f32x4 next = b2[0];
        auto into_next = [&](auto kc) { next = SH::template step<decltype(kc)::value>(W2[0], h, next, mma); };
        if constexpr (G0 > 0) weave(std::integral_constant<int, 6 * G0>{}, into_next, Stages{}, last_tile);
        else weave(std::integral_constant<int, E1>{}, env, Stages{}, last_tile);
        SH::template inputs<G0>(h, pieces);
        quad::static_for<6 * G0, MH>(into_next);
        acc[0] = next;
        quad::static_for<1, HT>([&](auto uc) {
          constexpr int u = decltype(uc)::value;
          hold(W2[u]);
          acc[u] = b2[u];
          weave(std::integral_constant<int, MH>{}, [&](auto kc) { acc[u] = SH::template step<decltype(kc)::value>(W2[u], h, acc[u], mma); },
                Stages{}, [&](auto ic) { tile_stage(std::integral_constant<int, u - 1>{}, ic); });
        });
        quad::static_for<0, G0>(ready);
        av = b3;
        auto into_action = [&](auto kc) { av = SH::template step<decltype(kc)::value>(W3, h, av, mma); };
        if constexpr (G0 > 0) weave(std::integral_constant<int, 6 * G0>{}, into_action, Stages{}, last_tile);
        else weave(std::integral_constant<int, E2 - E1>{}, [&](auto kc) { env(std::integral_constant<int, E1 + decltype(kc)::value>{}); }, Stages{}, last_tile);
        SH::template inputs<G0>(h, pieces);
        quad::static_for<6 * G0, MH>(into_action);
        // ---- the action, its cost and pieces ----
        constexpr int NAK = S::NAK, NP = SA::FULL;
        uint32_t cuts[NP][3];
        float aa = 0.0f;
        weave(std::integral_constant<int, OT * M1 - E2>{}, [&](auto kc) { env(std::integral_constant<int, E2 + decltype(kc)::value>{}); },
              std::integral_constant<int, 5 + SA::STAGES>{}, [&](auto ic) {
          constexpr int i = decltype(ic)::value;
          if constexpr (i < 5) {
#pragma unroll
            for (int r = 0; r < NAK; ++r) {
              if constexpr (i == 0) a4[r] = av[r] * quad::TANH_C;
              else if constexpr (i == 1) a4[r] = __builtin_amdgcn_exp2f(a4[r]);
              else if constexpr (i == 2) a4[r] = a4[r] + 1.0f;
              else if constexpr (i == 3) a4[r] = __builtin_amdgcn_rcpf(a4[r]);
              else { a4[r] = __fmaf_rn(-2.0f, a4[r], 1.0f); a4[r] = squash_l ? a4[r] : av[r]; }
            }
          } else {
            if constexpr (i == 5) {
#pragma unroll
              for (int r = 0; r < NAK; ++r) aa = r == 0 ? a4[0] * a4[0] : __fmaf_rn(a4[r], a4[r], aa);
              R = __fmaf_rn(aa, ncost, R);
#pragma unroll
              for (int r = 0; r < NAK; ++r) a4[r] = finite(a4[r]);      // (of a linear output)
            }
            auto& pairs = reinterpret_cast<float (&)[2 * NP]>(a4);
            auto& rests = reinterpret_cast<float (&)[2 * NP]>(rest4);
            SA::template cut_stage<i - 5, NP>(pairs, rests, cuts);
          }
        });
        SA::inputs(ax, cuts);
      } else {
        supply(xe, SX{}, s);
        if constexpr (NORM) {
          f32x4 sn[OT];
#pragma unroll
          for (int q = 0; q < OT; ++q) sn[q] = (s[q] - mu[q]) * iv[q];
          supply(x, SX{}, sn);
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
        supply(h, SH{}, v);
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
        supply(h, SH{}, v);
        // ---- the action and its cost, under it A s ----
        av = b3;
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
        const f32x4 one[1] = {av};
        supply(ax, SA{}, one);
      }
      // ---- s' = tanh(A s + B a) ----
      float top = 0.0f;
#pragma unroll
      for (int q = 0; q < OT; ++q) {
        if constexpr (SPLIT) {
          quad::static_for<0, SA::MF>([&](auto kc) { accE[q] = SA::template step<decltype(kc)::value>(Be[q], ax, accE[q], mma); });
        } else {
#pragma unroll
          for (int kk = 0; kk < KA; ++kk) accE[q] = mma(Be[q][kk], ax[kk], accE[q]);
        }
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
