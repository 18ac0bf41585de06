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
// Binary32 runs on the bf16 shape too, values cut into three pieces (Split), wherever the pieces fit the registers (all but the widest classes) and carry the individual's values (P_BITS): binary32 products take 32 cycles
// for four inputs and share the multipliers with vector instructions, in one wavefront and between two, so that the two add up - 19-48-48-5 (ReLU, statistics),
// 1000 x 16 copies: 77 products, 2464 of 3300 cycles a step, and 809 of vector issue.  Now 70 products (1120 cycles) beside 325 vector instructions, 2440 cycles:
// 4.29 ms in passes of four copies -> 1.40 -> 1.02 ms per 1000 steps.  100 steps of 1000 x 16 copies: 10-16-4 60 -> 58 us (4000 x 16: 213 -> 186), 18-32-4 135 -> 112, 30-64-12 292 -> 189,
// 44-48-4 264 -> 172, 60-48-12 350 -> 217; widest, as before: 60-64-4 419.  Bound: vector issue of a lone wavefront, and products with nothing beside them (state, first and last products of a layer).
// bf16: the activations (29 cycles per tanh of a register); 17-64-64-6, 1000 x 16 copies x 60 steps: 137 -> 64 us.
#pragma once

#include "rollout_quad.hpp"

namespace es {

namespace cols {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The perturbed parameters of one individual, all of them, into LDS in coalesced order by one wavefront: four consecutive ones per lane and
// load where the row has them, the loads of eight iterations in flight together.  put(at, v): one or four parameters.
template <class Elem, class F>
__device__ __forceinline__ void stage_all(Elem* sp, const float* __restrict__ theta, const NoiseRow nz, float scale, uint32_t count, F put) {
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
          put(sp + 4u * (q0 + 64u * v), f32x4{__fmaf_rn(scale, e.x, tv[v].x), __fmaf_rn(scale, e.y, tv[v].y), __fmaf_rn(scale, e.z, tv[v].z), __fmaf_rn(scale, e.w, tv[v].w)});
      }
    }
    const uint32_t k = 4u * quads + lane;      // the last one to three
    if (k < count) put(sp + k, __fmaf_rn(scale, row_noise(nz, k), theta[k]));
  };
  if (nz.mode >= 2u) {
#pragma unroll 1
    for (uint32_t d0 = 4u * lane; d0 < count; d0 += 256u) {
      float z[4];
      noise_regen4(nz.row, d0, nz.gen, nz.k0, nz.k1, nz.mode == 3u, z);
#pragma unroll
      for (uint32_t k = 0; k < 4u; ++k)
        if (d0 + k < count) put(sp + d0 + k, __fmaf_rn(scale, z[k], theta[d0 + k]));
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
// What the pieces can carry: no product of theirs and no sum on the way may overflow, or an infinity of one sign would meet one of the other where the values' own product is finite or infinite.
// With parameters and environment matrices up to P = 2^16 and normalised observations up to X = 2^40, 64 ReLU units reach 2^62, 2^84 and a linear action 2^106, and its
// product with B 2^126.  Beyond that, and with infinities and NaN among them, an individual runs on the binary32 shape (in line, chosen before its weights are read: a call there cost 90 spilled registers).  (Bits without the sign, which order like the values, infinities and NaN last.)
constexpr uint32_t P_BITS = (127u + 16u) << 23, X_BITS = (127u + 40u) << 23;
__device__ __forceinline__ uint32_t magnitude(float v) { return __float_as_uint(v) & 0x7FFFFFFFu; }

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
    cut(r, val);
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
// SPLIT: binary32 products of three-piece values; Plain: the same on the binary32 shape
template <bool BF16_, int KS_, int HT_, int NAK_, bool RELU_, bool NORM_, bool SPLIT_ = !BF16_ && cols::split_fits(KS_, HT_, NAK_, NORM_)>
struct ColsShape {
  static constexpr bool BF16 = BF16_, RELU = RELU_, NORM = NORM_;
  static constexpr int KS = KS_, HT = HT_, NAK = NAK_;
  static constexpr int OT = (KS + 3) / 4;                                  // tiles of the state
  static constexpr int NA = 4;                                             // result registers of the action tile
  using SX = cols::Split<KS>; using SH = cols::Split<4 * HT>; using SA = cols::Split<NAK>;
  static constexpr bool SPLIT = SPLIT_;
  using Plain = ColsShape<BF16, KS, HT, NAK, RELU, NORM, false>;
  // operands of a product along K: bf16 a pair of tiles (four registers), split see there, else one register a K step; inputs and weights of an output tile
  static constexpr int K1 = BF16 ? (OT + 1) / 2 : SPLIT ? SX::NX : KS, KH = BF16 ? (HT + 1) / 2 : SPLIT ? SH::NX : 4 * HT, KA = BF16 ? 1 : SPLIT ? SA::NX : NAK;
  static constexpr int W1N = SPLIT ? SX::NW : K1, WHN = SPLIT ? SH::NW : KH, WAN = SPLIT ? SA::NW : KA;
  static constexpr int WREGS = (BF16 || SPLIT ? 4 : 1) * (HT * W1N + HT * WHN + WHN + OT * W1N + OT * WAN) + 8 * HT + 4;      // weights and biases of a lane
  static constexpr int WORK = SPLIT ? cols::split_work(KS, HT, NORM) : 12 * OT + 8 * HT + 40 + (NORM ? 8 * OT : 0);
  static constexpr int OCC = cols::wavefronts(WREGS + WORK);
};

// The episodes of an individual whose values are beyond what the pieces carry; its parameters are in the LDS
template <class S>
__device__ __forceinline__ void cols_beyond(const QuadArgs& a) {
  constexpr bool STAGED = true;
#include "rollout_cols_body.inc"
}

template <class S>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(S::OCC, S::OCC)))
void rollout_cols_kernel(const QuadArgs a) {
  constexpr bool STAGED = false;
#include "rollout_cols_body.inc"
}

template <class S>
int launch_cols_shape(es_ctx* ctx, QuadArgs a, float* fitness, hipStream_t st) {
  // The smallest class, up to 16 observations and units, has some fifteen products a step, few for what the cuts cost: with four wavefronts on a compute unit the binary32 shape is as fast or faster where
  // statistics or more than eight actions add to the vector work; with fewer the pieces are, and with more, since there vector and matrix instructions of two wavefronts overlap.  300 steps,
  // pieces / 16x16x4: 16-13-9 700 x 16 177 / 189 us, 800 193 / 189, 1024 197 / 189, 1100 283 / 332; 10-16-4 with statistics 700 x 16 169 / 173, 800 184 / 174, 1024 186 / 174, 1100 282 / 302
  // (without: 161 / 170, 164 / 170, 166 / 170, 258 / 295); ReLU, 900 x 16: 16-13-9 160 / 162, with statistics 174 / 170, 10-16-4 with statistics 157 / 154.
  if constexpr (S::SPLIT && S::KS == 4 && S::HT == 1 && (S::NORM || S::NAK == 4)) {
    const uint64_t wavefronts = (uint64_t)a.N * ((a.E + 15u) / 16u), cus = (uint64_t)std::max(1, ctx->num_cus);
    if (wavefronts > 3 * cus && wavefronts <= 4 * cus) return launch_cols_shape<typename S::Plain>(ctx, a, fitness, st);
  }
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
