// es_rollout in passes of FOUR environment copies on the 4x4 matrix-core shapes, binary32 or bf16 operands.
//
// Paper Sec. 3.2 / 5.1: population x environment-copy evaluation of a deterministic MLP policy with m hidden layers,
// fitness = mean undiscounted return.  One v_mfma_f32_4x4x4_16b_bf16 (binary32: 4x4x1) is sixteen independent 4x4
// products: lane 4b + x supplies A_b[row x] (four, or one, K values) and B_b[column x] of block b and holds
// D_b[rows 0..3][column x] in its four result registers; cbsz / abid broadcast the A values of one block to a group of
// blocks.  The activations are the A operand (row = copy, broadcast from the block that holds them) and the weights the
// B operand (column = the lane's own unit), so
//   * a lane owns ONE unit of a layer and accumulates it for the four copies in its four result registers: there are no
//     padded columns (a 16-column tile would be a quarter full) and the activation functions run on full lanes;
//   * the whole state of four copies, as an operand, is one 8-byte value per lane for every 64 elements;
//   * after the activation "unit per lane, copy per register" becomes the next operand, "copy per lane, unit per register", by the write to and the read from the LDS where
//     there are several wavefronts, else (and for the action layer) by a 4x4 transpose inside each lane quad.  (A transpose in front of the LDS as well, with one write of four units:
//     244-256-256-17, 4096 x 4 copies, 22.8 ms against 22.0; 200-256-256-8 128 x 1, 200 steps, 291 us against 271; binary32 12-100-100-8 256 x 8 298 against 289.)
// A workgroup of NW wavefronts (64 units of every hidden layer each) evaluates one individual; its perturbed weights and
// the environment matrices stay in registers for all T steps.
//   * NW > 1: a hidden layer's outputs cross the LDS as operands (one barrier per layer but the last); the action layer
//     is split along K - each wavefront multiplies the units it has just produced - and its binary32 partial sums cross
//     the LDS (one barrier).  Up to 64 state elements every wavefront steps the whole environment for itself from the
//     same operands in the same order (bit-identical, no exchange); beyond that the state rows are spread over the
//     wavefronts and cross the LDS as well (one more barrier).
//   * NW = 1: nothing leaves the wavefront; no barriers.
//   * bf16, NW > 1: a product whose input has crossed the LDS runs on a larger shape, v_smfmac_f32_16x16x64_bf16, at twice the weights per cycle (pair_mac).
// Returns are accumulated per lane and added up once after the last step.
// Bound: the dependent chain of a step when a few individuals are evaluated; with a full chip, matrix-core issue
// (8.5 cycles per 4x4 instruction, measured) plus the vector work of the activations (5.8 cycles per instruction of a
// lone wavefront).
// Measured, whole rollout, T = 1000 unless noted: bf16 8-256-256-2, 128 individuals x 1 copy 1.23 ms (padded 16-column kernel) -> 0.77 ms -> 0.74 with
// the books and the two branches of a step's end behind the loop; bf16 27-100-100-8, 128 x 5 copies, T = 400: 8.05 ms (LDS kernel) -> 0.34 ms -> 0.27 with
// passes of two copies on SIMDs of their own; 244-256-256-17, 1024 x 4 copies, T = 1000: 6.3 ms (16-column kernel with compacted columns) -> 5.7.  Paired products (below),
// 200 steps: 8-256-256-2 128 x 1 166 -> 142, 1024 x 4 551 -> 494; 20-100x3-6 128 x 1 246 -> 195; 27-100-100-8 128 x 1
// 128 -> 111, 1024 x 4 256 -> 248.
#pragma once

#include <type_traits>

#include "es_internal.hpp"
#include "rollout_stage.hpp"

namespace es {

struct QuadArgs {
  const float* theta;
  const void* noise;
  const uint32_t* noise_offs;   // shared noise table: start of every row, else null
  const float* A;
  const float* B;
  const float* obs_mean;        // frozen observation statistics (paper App. B), or null
  const float* obs_inv;
  float* returns;
  int32_t* ep_len;
  float* fitness;               // null when the passes of an individual run in several workgroups
  uint32_t N, E, T, no, nh, na, ld;
  uint32_t oW1, ob1, oW2, ob2, oW3, ob3;
  uint32_t gen, k0, k1;
  uint32_t antithetic, out_tanh, noise_mode;
  uint32_t split;               // workgroups per individual: workgroup s of them takes passes s, s + split, ...
  float sigma, done_thresh, act_cost;
};

namespace quad {

typedef short s16x4 __attribute__((ext_vector_type(4)));

// compile-time loop: body(std::integral_constant<int, I>) for I = 0 .. N - 1 (the broadcast block is an immediate)
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& body) {
  if constexpr (I < N) {
    body(std::integral_constant<int, I>{});
    static_for<I + 1, N>(body);
  }
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// Four consecutive K values of a weight row / of a copy, in the operand type.
template <bool BF16> struct Oper;
template <> struct Oper<true> {
  using Elem = uint16_t;
  using V4 = u32x2;
  static constexpr int PAD_H = 32, PITCH = 64 + 4;      // elements: see the LDS map below
  // acc += A values of block ABID (broadcast to 2^CB blocks) x w; G: number of the K group (two accumulators alternate)
  template <int CB, int ABID, int G>
  static __device__ __forceinline__ void mac(V4 act, V4 w, f32x4 (&acc)[2]) {
    acc[G % 2] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, act), __builtin_bit_cast(s16x4, w), acc[G % 2], CB, ABID, 0);
  }
  // unit per lane, copy per register -> copy per lane, four units packed (p, q: bits 0 and 1 of the lane; sel: byte selector of its bit 0)
  static __device__ __forceinline__ V4 transpose(f32x4 v, bool, bool q, uint32_t sel) {
    const u32x2 r = pack_bf16x4(v.x, v.y, v.z, v.w);
    const uint32_t recv = dpp_u<0x4E>(q ? r.x : r.y);                // quad_perm [2, 3, 0, 1]: the other pair's units
    const uint32_t u = q ? recv : r.x, w = q ? r.y : recv;           // units 0/1 and 2/3 of the quad, copies 2q and 2q + 1
    return V4{__builtin_amdgcn_perm(dpp_u<0xB1>(u), u, sel), __builtin_amdgcn_perm(dpp_u<0xB1>(w), w, sel)};
  }
  // two copies: unit per lane -> copy x & 1 per lane, four units packed (lanes 2 and 3 of a quad, whose rows nobody reads, repeat two units)
  static __device__ __forceinline__ V4 transpose2(float a, float b, bool, uint32_t sel) {
    const uint32_t r = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
    const uint32_t u = __builtin_amdgcn_perm(dpp_u<0xB1>(r), r, sel);      // units 0/1 in lanes 0 and 1, 2/3 in lanes 2 and 3
    return V4{u, dpp_u<0xEE>(u)};                                          // quad_perm [2, 3, 2, 3]
  }
  // one copy: unit per lane -> four units of the lane's quad
  static __device__ __forceinline__ V4 gather(float v) { return pack_bf16x4(dpp_f<0x00>(v), dpp_f<0x55>(v), dpp_f<0xAA>(v), dpp_f<0xFF>(v)); }
  // action rows R b .. of copy x in lane 4 b + x -> four rows of the copy in every (4 / R)-th block
  template <int R>
  static __device__ __forceinline__ V4 collect(const float (&v)[R]) {
    if constexpr (R == 1) return pack_bf16x4(v[0], dpp_f<0x104>(v[0]), dpp_f<0x108>(v[0]), dpp_f<0x10C>(v[0]));
    else {
      const uint32_t pk = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v[0], v[1]}, bf16x2));
      return V4{pk, dpp_u<0x104>(pk)};
    }
  }
  static __device__ __forceinline__ V4 zero() { return V4{0u, 0u}; }
};
template <> struct Oper<false> {
  using Elem = float;
  using V4 = f32x4;
  static constexpr int PAD_H = 16, PITCH = 32 + 4;
  template <int CB, int ABID, int G>
  static __device__ __forceinline__ void mac(V4 act, V4 w, f32x4 (&acc)[2]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j % 2] = __builtin_amdgcn_mfma_f32_4x4x1f32(act[j], w[j], acc[j % 2], CB, ABID, 0);
  }
  static __device__ __forceinline__ V4 transpose(f32x4 v, bool p, bool q, uint32_t) {
    const float s01 = dpp_f<0xB1>(p ? v.x : v.y), s23 = dpp_f<0xB1>(p ? v.z : v.w);      // quad_perm [1, 0, 3, 2]
    const f32x4 u = f32x4{p ? s01 : v.x, p ? v.y : s01, p ? s23 : v.z, p ? v.w : s23};
    const float s02 = dpp_f<0x4E>(q ? u.x : u.z), s13 = dpp_f<0x4E>(q ? u.y : u.w);      // quad_perm [2, 3, 0, 1]
    return f32x4{q ? s02 : u.x, q ? s13 : u.y, q ? u.z : s02, q ? u.w : s13};
  }
  static __device__ __forceinline__ V4 gather(float v) { return V4{dpp_f<0x00>(v), dpp_f<0x55>(v), dpp_f<0xAA>(v), dpp_f<0xFF>(v)}; }
  template <int R>
  static __device__ __forceinline__ V4 collect(const float (&v)[R]) {
    static_assert(R == 1, "one action row per lane");
    return V4{v[0], dpp_f<0x104>(v[0]), dpp_f<0x108>(v[0]), dpp_f<0x10C>(v[0])};
  }
  static __device__ __forceinline__ V4 zero() { return V4{0.f, 0.f, 0.f, 0.f}; }
};

// Paired products, v_smfmac_f32_16x16x64_bf16: sixteen units x 64 K values of weights an instruction in the time of a dense 16x16x32 product (16.6 cycles
// measured, dependent or not; a vector instruction behind it waits 13 of them), so twice the weights per cycle of it or of the 4x4 shapes (8.9 cycles for 256 weights).  The instruction skips half of every four K values of its first operand, row by row; here
// a copy is TWO rows, one that takes the first two values of every four and one that takes the other two, and the sum of the two rows
// is the whole product.  The weights are the dense operand.  What is doubled is the rows, of which one to four copies leave most idle.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x4 pair_mac(u32x4 act, u32x8 w, f32x4 acc, int which) {
  return __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8, act), __builtin_bit_cast(bf16x16, w), acc, which, 0, 0);
}
// Rows of the product: row 4 g + i stands in result register i of lane group g.  One copy: its first half in even groups, its second in odd ones.  Two: copy 0 in
// even groups, 1 in odd ones, the halves in registers 0 and 1.  Four: copies 0 and 1 in even groups, 2 and 3 in odd ones, halves in registers 2 k and 2 k + 1.
// (Groups 2 and 3 repeat 0 and 1: see pair_units.)
template <int NC> __device__ __forceinline__ int pair_copy(int row) {
  const int odd = (row >> 2) & 1;
  return NC == 1 ? 0 : NC == 2 ? odd : 2 * odd + ((row >> 1) & 1);
}
template <int NC> __device__ __forceinline__ int pair_half(int row) { return NC == 1 ? (row >> 2) & 1 : row & 1; }
// The four tiles' products -> a unit per lane (lane group g: tile g), a register per copy.
template <int NC>
__device__ __forceinline__ void pair_units(const f32x4 (&d)[4], bool upper, float (&z)[NC]) {
  auto swap = [](float& x, float& y) {      // odd lane groups of x against even ones of y
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
    x = __builtin_bit_cast(float, (unsigned)r[0]); y = __builtin_bit_cast(float, (unsigned)r[1]);
  };
  if constexpr (NC == 1) {
    float x = upper ? d[2][0] : d[0][0], y = upper ? d[3][0] : d[1][0];
    swap(x, y);
    z[0] = x + y;
  } else {
#pragma unroll
    for (int k = 0; k < NC / 2; ++k) {
      float v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = d[t][2 * k] + d[t][2 * k + 1];
      float x = upper ? v[2] : v[0], y = upper ? v[3] : v[1];
      swap(x, y);
      z[k] = x; z[k + NC / 2] = y;
    }
  }
}
// One row (unit) per lane, a register per copy -> rows of an exchange buffer, one per copy: `to` is the lane's place in the first.
template <bool BF16, int NC, int PITCH>
__device__ __forceinline__ void put_units(unsigned char* to, const float (&v)[NC]) {
  if constexpr (!BF16) {
#pragma unroll
    for (int c = 0; c < NC; ++c) *reinterpret_cast<float*>(to + 4 * c * PITCH) = v[c];
    return;
  }
#pragma unroll
  for (int c = 0; c < NC; c += 2) {
    const uint32_t r = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v[c], v[c + 1 < NC ? c + 1 : c]}, bf16x2));
    *reinterpret_cast<uint16_t*>(to + 2 * c * PITCH) = (uint16_t)r;
    if (c + 1 < NC) *reinterpret_cast<uint16_t*>(to + 2 * (c + 1) * PITCH) = (uint16_t)(r >> 16);
  }
}
// Place of unit u of 64 in a row of an exchange buffer: the first operand's share of lane (q, half), values 4 j + 2 half and 4 j + 2 half + 1 of q's sixteen, is contiguous.
__device__ __forceinline__ int pair_place(int u) { return (u & 48) + 8 * ((u >> 1) & 1) + 2 * ((u & 15) >> 2) + (u & 1); }
// registers of a tile's product that count
template <int NC> __device__ __forceinline__ void pair_zero(f32x4 (&d)[4]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i < (NC == 4 ? 4 : NC)) d[t][i] = 0.0f;
      else { float any; asm volatile("" : "=v"(any)); d[t][i] = any; }
    }
  }
}

// A value known to be the same in every lane, as a scalar.
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ float uniform(float v) { return __builtin_bit_cast(float, uniform(__builtin_bit_cast(uint32_t, v))); }

__device__ __forceinline__ void pin_sgpr(float& v) { asm volatile("" : "+s"(v)); }      // ... and kept in a scalar register

// Keeps a weight in the accumulation half of the unified register file, where an MFMA can read it directly.
__device__ __forceinline__ void pin_agpr(u32x2& v) { asm volatile("" : "+a"(v)); }
__device__ __forceinline__ void pin_agpr(f32x4& v) {
#pragma unroll
  for (int j = 0; j < 4; ++j) { float t = v[j]; asm volatile("" : "+a"(t)); v[j] = t; }
}
__device__ __forceinline__ void pin_agpr(u32x8& v) { asm volatile("" : "+a"(v)); }

// tanh(x + b) as 1 - 2 / (2^{c (x + b)} + 1) with cb = c b, c = 2 log2 e: the bias costs no instruction of its own
constexpr float TANH_C = 2.88539008f;
template <bool NEAR>
__device__ __forceinline__ float tanh_b(float x, float cb) {
  if (NEAR) return tanh_near(__fmaf_rn(x, TANH_C, cb));
  const float ex = __builtin_amdgcn_exp2f(__fmaf_rn(x, TANH_C, cb));
  return __fmaf_rn(-2.0f, __builtin_amdgcn_rcpf(ex + 1.0f), 1.0f);
}

}  // namespace quad

// BF16: operand type.  NW: wavefronts (hidden width <= 64 NW).  KG: observation width in groups of four (<= 16: every
// wavefront holds the whole state; else the rows are spread, 64 NW >= 4 KG).  M: hidden layers.  NC: copies a pass serves
// (4; 2 or 1: the activations of the idle copies and most of the transposes drop out).  RELU / NORM: hidden
// activation, observation statistics (compile-time: a taken branch costs a single wavefront some sixty cycles).
// NEAR: the tanh that is accurate near zero (bf16 policies of fewer than 128 units).
template <bool BF16_, int NW_, int KG_, int M_, int NC_, bool RELU_, bool NORM_, bool NEAR_>
struct QuadShape {
  using O = quad::Oper<BF16_>;
  using Elem = typename O::Elem;
  static constexpr bool BF16 = BF16_, RELU = RELU_, NORM = NORM_, NEAR = NEAR_;
  static constexpr int NW = NW_, KG = KG_, M = M_, NC = NC_;
  static constexpr int NT = 64 * NW, HID = 64 * NW, HG = 16 * NW;        // threads, padded hidden width, its K groups
  static constexpr bool SPREAD = KG > 16;                                // state rows over the wavefronts
  static constexpr int NR = (KG + 15) / 16;                              // operand registers of the state
  // products whose input comes through the LDS run as paired ones (pair_mac): the layers behind the first one, and A s and the first where rows are spread
  // (Not where four wavefronts share the rows, 129 to 256 units and more than 64 observations, although 244-256-256-17, 4096 x 4 copies, would take 20.0 ms instead of 22.0: sums
  // in another order round a few operands the other way, of which some individuals' loops there settle elsewhere - in one seed of 24, a rank by 1224 of 4096 places.)
  // (Nor for four layers in the class of 64 observations, which statistics take at any width: paired products need their operands beside the weights, seven of which are then reloaded from scratch
  // memory in every step.  100 steps, 4x4 / paired: 62-256x4-8 128 x 1 207 / 293 us, 1000 x 1 813 / 1140, with statistics 27-256x4-8 128 x 1 217 / 303, 512 x 4 701 / 754.)
  static constexpr bool PAIRS = BF16 && NW > 1 && !(SPREAD && NW > 2) && !(M == 4 && KG > 8), PAIRS_H = PAIRS && M > 1, PAIRS_X = PAIRS && SPREAD;
  using WX = std::conditional_t<PAIRS_X, quad::u32x8[NR][4], typename O::V4[KG]>;                 // a lane's weights of the first layer, its elements of A
  using WH = std::conditional_t<PAIRS_H, quad::u32x8[NW][4], typename O::V4[M > 1 ? HG : 1]>;     // ... of a layer behind it
  static constexpr int KGA = SPREAD ? 8 : 4;                             // action width in groups of four
  static constexpr int NA = 4 * KGA;                                     // padded action width
  static constexpr int ENV_ROWS = SPREAD ? 64 * NW : 64;
  // The two accumulators' sum of a copy stands right in front of its activation: with all four sums first a one-layer step of four copies is 2 to 3 % longer, binary32 34-156-8, 462 x 12, 401 steps
  // 2301 / 2371 us - but in bf16, in the class of 64 observations, up to 4 % shorter (50-200-5, 256 x 4, 400 steps 235 / 224 us; 25-113-5 with statistics, 300 x 4, 300 steps 185 / 177; 60-100-9,
  // 300 x 7, 100 steps 87 / 86; three layers 50-100x3-5 300 x 4, 200 steps 577 / 564)
  static constexpr bool SUMS_FIRST = BF16 && (M == 1 || M == 3) && NC == 4 && KG == 16;
  // One layer: where a step's loop begins in the windows in which instructions are fetched (instructions of four bytes behind a multiple of 64; -1: as it comes).  The loop is short and 1 to 5 % longer at the
  // wrong place, which code in front of it used to decide.  256 x 4 copies, 400 steps, best / worst of the eight places in 32 bytes, here: binary32 13-113-5 274 / 282, with ReLU 259 / 269; bf16 25-200-5
  // 202 / 212 and 188 / 198, 25-113-5 198 / 203; 256 x 2 154 / 160 and 150 / 158; 128 x 1 130 / 136; where the eight differ by less or by the activation, and with statistics, it is left alone.
  static constexpr int loop_at() {
    if (M != 1 || SPREAD || NORM) return -1;
    if (!BF16) return NW == 2 && NC == 4 && KG <= 8 ? (KG == 4 ? 2 : 0) : -1;
    constexpr int two[3][2] = {{6, 2}, {5, 3}, {0, -1}}, four[3][2] = {{-1, -1}, {7, 4}, {2, -1}};      // copies, observations
    return (NW == 2 ? two : four)[NC / 2][KG / 16];
  }
  static constexpr int COLS = KG < 8 ? 16 : BF16 && KG >= 16 ? 64 : 32;    // columns of a staging round
  static constexpr int GR = COLS / 4;                                    // ... in groups
  static constexpr int PWIN = PAIRS_H || PAIRS_X ? 64 + 8 : O::PITCH;                                  // window pitch: vector reads of consecutive rows hit distinct banks
  static constexpr int PW3 = HID + 4;
  static constexpr int ES = (int)sizeof(Elem);
  // LDS map (bytes).  Exchange buffers: rows of HID elements, one per copy; the pad puts the four copies' rows 64 bytes apart
  // modulo the banks' 256, so that lane (block, copy) reads without conflicts.
  static constexpr int PH = HID + O::PAD_H;
  static constexpr int HB = 4 * PH * ES;                                 // one exchange buffer
  // the action: one or two rows of one copy per lane (ROWS_COPY), or one row per lane for all copies
  static constexpr bool ROWS_COPY = NC > 1 ? (NW > 1 || !BF16) : (NW == 1 && !BF16);
  static constexpr int RPL = NA / 16;                                    // rows per lane of the former
  static constexpr int PP = NC == 1 ? 64 : NA + 4;                       // pitch (floats) of a copy's action partials
  static constexpr int PB = 4 * (BF16 ? 2 : 1) * NW * NC * PP;
  static constexpr bool P_TWICE = M == 1 && !SPREAD;                     // one barrier per step only: alternate the partials' buffer
  static constexpr int PX = 4 * KG + O::PAD_H;                           // state row of a copy (SPREAD only)
  static constexpr int XB = SPREAD ? 4 * PX * ES : 0;
  static constexpr int OFF_H = 0;
  static constexpr int OFF_P = OFF_H + (NW > 1 && M > 1 ? 2 * HB : 0);
  static constexpr int OFF_X = OFF_P + (NW > 1 ? (P_TWICE ? 2 : 1) * PB : 0);
  static constexpr int OFF_XP = OFF_X + XB;
  static constexpr int OFF_FLAG = OFF_XP + (NORM ? XB : 0);
  static constexpr int OFF_RED = OFF_FLAG + 16;
  // [copy][thread]: a lane's share of the return of a copy that has ended
  static constexpr int OFF_END = OFF_RED + 4 * 4 * NW;
  static constexpr int RUN_BYTES = OFF_END + (NC > 1 ? 4 * NC * NT : 0);
  static constexpr int WIN_ROWS = HID > ENV_ROWS ? HID : ENV_ROWS;
  static constexpr int WIN_BYTES = WIN_ROWS * PWIN * ES > NA * PW3 * ES ? WIN_ROWS * PWIN * ES : NA * PW3 * ES;
  // More than 128 observations: the initial states of the last pass, [copy][thread] binary32; most individuals of a workgroup start from the same ones
  // (244-256-256-17, 4096 x 4 copies: 8 steps 750 -> 735 us, 200 steps 4980 -> 4936; up to 128 observations 3 % slower)
  static constexpr bool KEEP_S0 = SPREAD && KG > 32;
  // registers of a lane's weights, and the wavefronts per SIMD that leaves room for
  static constexpr int VR = BF16 ? 2 : 4;
  // action layer, the wavefront's sixteen K groups: GROUPED (binary32; four layers, for the registers) four K values per instruction in groups of four
  // blocks, then a sum over the groups; HALVES (bf16, several wavefronts) two K groups per instruction, each for 32 rows,
  // the two sums of a row crossing the LDS as partials of their own; else every K group to every block, row = lane
  static constexpr bool GROUPED = !BF16 || M == 4, HALVES = !GROUPED && NW > 1;
  static constexpr int W3N = GROUPED ? 4 : HALVES ? 8 : 16;
  static constexpr int NP = HALVES ? 2 * NW : NW;                        // partial sums of an action row
  static constexpr int WREGS = VR * (2 * KG + (M - 1) * HG + W3N + KGA);
  static constexpr int OCC = WREGS + 72 <= 168 ? 3 : WREGS + 72 <= 256 ? 2 : 1;
  // Four wavefronts, up to two workgroups on a CU: two staging windows, so that a round's loads are requested while other wavefronts still read the round
  // before (one barrier a round).  Three workgroups would not fit the LDS: one layer, 1000 x 4 copies of 27-256-8, 200 steps 237 us, two windows 289
  static constexpr bool TWO_WIN = NW == 4 && OCC < 3;
  static constexpr int OFF_S0 = RUN_BYTES > (TWO_WIN ? 2 : 1) * WIN_BYTES ? RUN_BYTES : (TWO_WIN ? 2 : 1) * WIN_BYTES;
  static constexpr int LDS_BYTES = OFF_S0 + (KEEP_S0 ? 4 * NC * NT : 0);
  // Registers beside the weights while they are staged.  Where they are short, a batch of loads, or what the compiler derives from the lane's number once for
  // all individuals, is spilled, and the reloads are waited for one after the other between the loads: FRESH computes the lane's number anew
  // (lane_now), BATCH halves a batch where a second workgroup fills the waits.  4096 x 4 copies, 2 steps, neither / FRESH / both: 244-256-256-17 (96 registers) 567 / 560 / 692 us, 100-256-256-17 (224)
  // 388 / 416 / 521; 512 x 2 of 27-256-256-8 (72) 42 / 52 / 35
  static constexpr int SLACK = (OCC == 3 ? 168 : OCC == 2 ? 256 : 512) - WREGS;
  // Few registers beside the weights: the next layer's operand in a ring of two reads (200 steps of 8-256-256-2, 256 x 4 copies: all four reads at once 247 us, sixteen
  // registers reloaded from scratch memory every step; 198; four layers of 256 128 x 1 copy 355 / 317)
  static constexpr bool TIGHT = PAIRS_H && SLACK <= 80 && (NC > 1 || M == 4);
  static constexpr bool FRESH = SLACK <= 112 && M < 4;      // (41-74-74-3, 104 registers, 182 x 6 copies, 34 steps: 63.5 us without, 58.8 with; four layers: 65 us of 2 steps without, 70 with)
  static constexpr int BATCH = OCC == 2 && SLACK < 80 ? STAGE_BATCH / 2 : STAGE_BATCH;
  static constexpr bool PLACED = NW == 2 && OCC > 1;                     // may be launched with four wavefronts, two of which leave (wavefront_place)
  // first K group of portion k of A s: in the first activation, after the first exchange, in the second activation, after
  // the action's exchange, with the action's tanh
  static constexpr int env_at(int k) {
    constexpr bool two = M > 1;
    if (PAIRS_X && two) {      // between a write and its barrier and between a read and its use, at both exchanges (other splits: within 1 % at four copies, 5 % slower with nothing before the barriers at one)
      constexpr int n = 4 * NR, at[6] = {0, n / 4, n / 2, n * 3 / 4, n, n};
      return at[k];
    }
    if (PAIRS_X) {
      constexpr int n = 4 * NR, at[6] = {0, n * 3 / 8, n * 3 / 8, n * 3 / 8, n, n};
      return at[k];
    }
    // (244-256-256-17: 3 470 cycles a step with the split below, 3 330 with more of it behind the barriers, 3 220 since the transposes in front of the LDS are gone.  One copy a pass, 400 steps, 7/8 / 3/4 of it before the action's tanh: 244-256-256-17
    // 128 x 1 500 / 494 us, 100-256-256-17 405 / 398; four copies, 1024 x 4, 600 steps: 3 320 / 3 390)
    if (SPREAD && two) {
      constexpr int at[6] = {0, KG / 8, KG * 3 / 8, KG / 2, NC == 1 ? KG * 3 / 4 : KG * 7 / 8, KG};
      return at[k];
    }
    constexpr int at[6] = {0, KG * 3 / 8, NW > 1 && two ? KG / 2 : KG * 3 / 8, two ? KG * 13 / 16 : (NW > 1 && two ? KG / 2 : KG * 3 / 8), NW > 1 ? KG * 15 / 16 : (two ? KG * 13 / 16 : KG * 3 / 8), KG};
    return at[k];
  }
  static_assert(!(GROUPED && NA > 16), "grouped action layer: sixteen rows");
  static_assert(!SPREAD || 64 * NW >= 4 * KG, "the wavefronts must cover the padded state");
  static_assert(KG % GR == 0 && HG % GR == 0 && LDS_BYTES <= 160 * 1024, "staging rounds, LDS budget");
  static_assert(WREGS <= 490 && (NC == 1 || NC == 4 || (NC == 2 && HALVES)), "register budget, copies");
};

// Two wavefronts, two workgroups on a CU: the hardware starts a workgroup one SIMD after the last one's start, so that the second would put a wavefront
// beside one of the first and leave a SIMD idle.  Such workgroups are launched with four wavefronts, one per SIMD, of which two stay: those of
// SIMDs 0 and 1 in the workgroup whose LDS starts at 0, of SIMDs 2 and 3 in the other.  Only the speed depends on it: of any four the two with the
// smallest keys stay.  Returns the place among those that stay; NW or more: not one of them.
template <int NW>
__device__ __forceinline__ int wavefront_place(uint32_t* slots) {
  if (NW != 2 || blockDim.x == 64u * NW) return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  constexpr int HW_SIMD_ID = 4 | (4 << 6) | (1 << 11), LDS_BASE = 6 | (0 << 6) | (11 << 11);      // hardware registers: HW_ID bits 4..5, LDS_ALLOC bits 0..11
  const uint32_t i = threadIdx.x >> 6, simd = (uint32_t)__builtin_amdgcn_s_getreg(HW_SIMD_ID), half = __builtin_amdgcn_s_getreg(LDS_BASE) != 0 ? 1u : 0u;
  const uint32_t key = 4u * ((simd >> 1) ^ half) + i;
  if ((threadIdx.x & 63u) == 0u) slots[i] = key;
  __syncthreads();
  int place = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) place += slots[k] < key ? 1 : 0;
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(place);
}

template <class S>
__global__ __launch_bounds__(S::PLACED ? 256 : S::NT) __attribute__((amdgpu_waves_per_eu(S::OCC, S::OCC)))
void rollout_quad_kernel(const QuadArgs a) {
  using namespace quad;
  using O = typename S::O;
  using V4 = typename O::V4;
  using Elem = typename S::Elem;
  constexpr bool BF16 = S::BF16, NORM = S::NORM, SPREAD = S::SPREAD;
  constexpr int NW = S::NW, NT = S::NT, KG = S::KG, M = S::M, HID = S::HID, HG = S::HG, KGA = S::KGA, NR = S::NR, GR = S::GR, COLS = S::COLS;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int w = NW == 1 ? 0 : S::PLACED ? wavefront_place<NW>(reinterpret_cast<uint32_t*>(lds)) : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (S::PLACED && w >= NW) return;
  const int tid = S::PLACED ? 64 * w + lane : (int)threadIdx.x;
  int threads = S::PLACED ? NT : (int)blockDim.x;
  if constexpr (S::PLACED) asm volatile("" : "+s"(threads));      // (kept from the compiler, which would unroll the staging loops: 25 us of instruction misses)
  const int blk = lane >> 2, x = lane & 3;
  const bool p = (x & 1) != 0, q = (x & 2) != 0;
  const uint32_t psel = p ? 0x03020706u : 0x05040100u;
  const int no = (int)a.no, nh = (int)a.nh, na = (int)a.na;
  const int unit = 64 * w + lane;                      // this lane's unit of every hidden layer
  const int erow = SPREAD ? unit : lane;               // ... and its row of the state
  Elem* win = reinterpret_cast<Elem*>(lds);
  auto sync = [] { if constexpr (NW > 1) __syncthreads(); };
  auto stage_sync = [] { __syncthreads(); };
  auto window = [&](int round) { return win + (S::TWO_WIN && (round & 1) ? S::WIN_BYTES / S::ES : 0); };
  auto window_read = [&] { if constexpr (!S::TWO_WIN) stage_sync(); };
  auto win_group = [&](int round, int row, int pitch, int g) { return *reinterpret_cast<const V4*>(window(round) + row * pitch + 4 * g); };
  // Columns COLS r .. of a matrix from the window of `round` -> registers: K groups r GR .. of row l, or, for paired products, of lane l's rows 64 w + 16 t + (l & 15) of the
  // four tiles, of which lane (q, n) supplies K values 8 q .. and 32 + 8 q .. of every 64.
  auto take = [&](auto& W, auto rc, int round, int l) {
    constexpr int r = decltype(rc)::value;
    if constexpr (std::is_same_v<std::remove_reference_t<decltype(W[0])>, V4>) {
#pragma unroll
      for (int g = 0; g < GR; ++g) W[GR * r + g] = win_group(round, l, S::PWIN, g);
    } else {
#pragma unroll
      for (int k = 0; k < COLS / 32; ++k) {
        constexpr int per = 64 / COLS;      // rounds of 64 K values
        const int j = 4 * (per == 2 ? r & 1 : k);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const u32x4 v = *reinterpret_cast<const u32x4*>(window(round) + (64 * w + 16 * t + (l & 15)) * S::PWIN + 32 * k + 8 * (l >> 4));
          u32x8& d = W[r / per][t];
          d[j] = v.x; d[j + 1] = v.y; d[j + 2] = v.z; d[j + 3] = v.w;
        }
      }
    }
  };

  // FRESH: the lane and thread number, computed where they are needed.  What the compiler derives from the ones above and keeps from one individual to
  // the next does not fit the registers beside the weights there, and its reloads are waited for one after the other
  auto lane_now = [&] {
    if constexpr (!S::FRESH) return lane;
    int zero = 0;
    asm volatile("" : "+v"(zero));
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, (uint32_t)zero));
  };
  auto tid_now = [&] { return S::FRESH ? 64 * w + lane_now() : tid; };

  // ---- environment matrices -> registers: Ae[g] = A[erow][4g .. 4g+3] (paired: see take), Be[g] = B[erow][4g .. 4g+3] ----
  typename S::WX Ae;
  V4 Be[KGA];
  static_for<0, KG / GR>([&](auto rc) {
    constexpr int r = decltype(rc)::value;
    stage_cols<COLS, false>(window(r), S::PWIN, S::ENV_ROWS, no, no, COLS * r, a.A, NoiseRow{}, 0.0f, 0u, tid, threads);
    stage_sync();
    take(Ae, rc, r, S::PAIRS_X ? lane : erow);
    window_read();
  });
  stage_cols<4 * KGA, false>(window(KG / GR), S::PWIN, S::ENV_ROWS, no, na, 0, a.B, NoiseRow{}, 0.0f, 0u, tid, threads);
  stage_sync();
#pragma unroll
  for (int g = 0; g < KGA; ++g) Be[g] = win_group(KG / GR, erow, S::PWIN, g);
  float mu = 0.f, iv = 0.f;                            // observation statistics of this row (padded rows: scale 0)
  if (NORM && erow < no) { mu = a.obs_mean[erow]; iv = a.obs_inv[erow]; }

  constexpr int NC = S::NC;
  const uint32_t nblk = (a.E + (uint32_t)NC - 1u) / (uint32_t)NC;
  const float inv_no = 1.0f / (float)no;
  const bool squash = a.out_tanh != 0u;
  const uint32_t items = a.N * a.split;
  uint32_t s0_pass = ~0u;                              // KEEP_S0: the pass whose initial states are kept
  float* s0s = reinterpret_cast<float*>(lds + S::OFF_S0);

  for (uint32_t item = blockIdx.x; item < items; item += gridDim.x) {
    const uint32_t i = item / a.split, pass0 = item - i * a.split;
    const uint32_t row = a.antithetic ? i >> 1 : i;
    const float scale = (a.antithetic && (i & 1u)) ? -a.sigma : a.sigma;
    NoiseRow nz;
    nz.mode = a.noise_mode; nz.row = row; nz.gen = a.gen; nz.k0 = a.k0; nz.k1 = a.k1; nz.ptr = nullptr;
    if (a.noise_offs) nz.ptr = table_row_base(a.noise_mode, a.noise, a.noise_offs, row);
    else if (a.noise_mode == 1u) nz.ptr = static_cast<const uint16_t*>(a.noise) + (size_t)row * a.ld;
    else if (a.noise_mode == 0u) nz.ptr = static_cast<const float*>(a.noise) + (size_t)row * a.ld;

    // ---- perturbed parameters -> LDS window -> registers ----
    typename S::WX W1;
    typename S::WH Wh[M > 1 ? M - 1 : 1];
    V4 W3[S::W3N];
    // A lane's own biases, requested together before anything else (a load behind a bounds test would be waited for by itself: three latencies an
    // individual).  hb: as the activation takes them, c b for tanh, b for ReLU; b3: of this lane's action rows
    constexpr int RPL = S::RPL, NB = M + RPL;
    const int lane_i = lane_now(), unit_i = 64 * w + lane_i;
    float hb[M], b3[RPL];
    uint32_t bix[NB];
    bool bok[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int c = S::ROWS_COPY ? RPL * (lane_i >> 2) + k - M : (k == M ? lane_i : S::NA);
      bok[k] = k < M ? unit_i < nh : c < na;
      bix[k] = !bok[k] ? 0u : k < M ? (k == 0 ? a.ob1 : a.ob2 + (uint32_t)(k - 1) * (uint32_t)(nh * nh + nh)) + (uint32_t)unit_i : a.ob3 + (uint32_t)c;
    }
    row_values<NB>(a.theta, nz, scale, bix, [&](int k, float v) {
      if (BF16) v = bf16_round(v);
      if (!bok[k]) v = 0.0f;
      if (k < M) hb[k < M ? k : 0] = S::RELU ? v : TANH_C * v;
      else b3[k < M ? 0 : k - M] = v;
    });
    stage_sync();                // the previous individual's last reads of LDS are done
    static_for<0, KG / GR>([&](auto rc) {
      constexpr int r = decltype(rc)::value;
      stage_cols<COLS, true, S::BATCH>(window(r), S::PWIN, HID, nh, no, COLS * r, a.theta, nz, scale, a.oW1, tid_now(), threads);
      stage_sync();
      take(W1, rc, r, S::PAIRS_X ? lane_now() : tid_now());
      window_read();
    });
    static_for<0, M - 1>([&](auto lc) {
      constexpr int l = decltype(lc)::value;
      static_for<0, HG / GR>([&](auto rc) {
        constexpr int r = decltype(rc)::value, round = KG / GR + l * (HG / GR) + r;
        stage_cols<COLS, true, S::BATCH>(window(round), S::PWIN, HID, nh, nh, COLS * r, a.theta, nz, scale, a.oW2 + (uint32_t)l * (uint32_t)(nh * nh + nh), tid_now(), threads);
        stage_sync();
        take(Wh[l], rc, round, S::PAIRS_H ? lane_now() : tid_now());
        window_read();
      });
    });
    constexpr int last = KG / GR + (M - 1) * (HG / GR);
    stage_cols<HID, true, S::BATCH>(window(last), S::PW3, S::NA, na, nh, 0, a.theta, nz, scale, a.oW3, tid_now(), threads);
    stage_sync();
    const int lw = lane_now();
    if constexpr (S::HALVES) {   // lane = action row, and a half of the wavefront's K groups in either half of the lanes
#pragma unroll
      for (int g = 0; g < S::W3N; ++g) {
        W3[g] = O::zero();
        if ((lw & 31) < S::NA) W3[g] = win_group(last, lw & 31, S::PW3, 16 * w + 8 * (lw >> 5) + g);
      }
    } else if constexpr (!S::GROUPED) { // lane = action row; K group g of this wavefront's 64 units
#pragma unroll
      for (int g = 0; g < S::W3N; ++g) {
        W3[g] = O::zero();
        if (lw < S::NA) W3[g] = win_group(last, lw, S::PW3, 16 * w + g);
      }
    } else {                     // lane (group gq of 16 lanes, n) = action row n; units 64 w + 16 gq ..
#pragma unroll
      for (int g = 0; g < S::W3N; ++g) W3[g] = win_group(last, lw & 15, S::PW3, 16 * w + 4 * (lw >> 4) + g);
    }
    stage_sync();
    float sel_c[NC];             // binary32: columns of the selector that sums the four lane groups and transposes
#pragma unroll
    for (int c = 0; c < NC; ++c) sel_c[c] = (NC == 1 || x == c) ? 1.0f : 0.0f;
    float* part = reinterpret_cast<float*>(lds + S::OFF_P);
    if constexpr (NW > 1) {      // action partials past the rows that are written read as zero
      for (int k = tid_now(); k < (S::P_TWICE ? 2 : 1) * S::NP * NC * S::PP; k += NT) part[k] = 0.0f;
      stage_sync();
    }

    float fit_sum = 0.0f;
    for (uint32_t pass = pass0; pass < nblk; pass += a.split) {
      // ---- initial states ----
      uint32_t alive = 0u;       // bit c: copy c of this pass still runs (uniform)
      float ninv[NC], ncost[NC], thr[NC];   // per copy while it runs: -1 / obs, -cost, threshold; 0, 0, +inf after its end
      int len[NC];
      const int tid_p = tid_now(), erow_p = SPREAD ? tid_p : tid_p - 64 * w;
      float s[NC];               // state row of this lane, one register per copy (binary32)
      const bool mine = SPREAD || w == 0;      // the wavefront that adds up the state's share of the reward
      float* ends = reinterpret_cast<float*>(lds + S::OFF_END);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const uint32_t e = (uint32_t)NC * pass + (uint32_t)c;
        const bool on = e < a.E;
        alive |= on ? 1u << c : 0u;
        ninv[c] = uniform(on && mine ? -inv_no : 0.0f);
        ncost[c] = uniform(on && w == 0 ? -a.act_cost : 0.0f);
        thr[c] = uniform(on ? a.done_thresh : __builtin_inff());
        len[c] = (int)a.T;
        if (!S::KEEP_S0 || s0_pass != pass) {
          s[c] = 0.0f;
          if (on && erow_p < no) s[c] = reset_value((uint32_t)erow_p, e, a.gen, a.k0, a.k1);
          if constexpr (S::KEEP_S0) s0s[c * NT + tid_p] = s[c];
        } else {
          s[c] = s0s[c * NT + tid_p];      // (written by this thread)
        }
      }
      if constexpr (S::KEEP_S0) s0_pass = pass;
      float xcost = (w == 0 && ((alive >> x) & 1u)) ? -a.act_cost : 0.0f;      // -cost of this lane's copy (ROWS_COPY)
      float Rs[NC];              // per-lane shares of the returns: rows of the state (and action rows, where row = lane)
      float Rx = 0.0f;           // ... of copy x: action rows (ROWS_COPY)
#pragma unroll
      for (int c = 0; c < NC; ++c) Rs[c] = 0.0f;
      // a lane's part of paired products' first operand: elements from a row of an exchange buffer
      const int prow = lane & 15, phalf = pair_half<NC>(prow), pcopy = pair_copy<NC>(prow), pat = 16 * (lane >> 4) + 8 * phalf, pwhich = phalf ? (int)0xEEEEEEEEu : 0x44444444;
      const int pplace = pair_place(lane), copy_x = x & (NC - 1);      // (rows past the last copy are nobody's)
      const bool upper = lane >= 32;
      using SOp = std::conditional_t<S::PAIRS_X, u32x4, V4>;
      SOp sop[NR], pop[NORM ? NR : 1];          // the state as an operand: raw for A s, normalised for the policy
      // one row (unit) per lane, a register per copy -> operand
      auto operand = [&](const float (&v)[NC]) {
        if constexpr (NC == 1) return O::gather(v[0]);
        else if constexpr (NC == 2) return O::transpose2(v[0], v[1], p, psel);
        else return O::transpose(f32x4{v[0], v[1], v[2], v[3]}, p, q, psel);
      };
      auto publish = [&] {       // s -> operand (own registers, or the exchange buffer)
        if constexpr (S::PAIRS_X) {
          if (NW * 64 == 4 * KG || 64 * w < 4 * KG) {
            put_units<BF16, NC, S::PX>(lds + S::OFF_X + 2 * (64 * w + pplace), s);
            if constexpr (NORM) {
              float sn[NC];
#pragma unroll
              for (int c = 0; c < NC; ++c) sn[c] = (s[c] - mu) * iv;
              put_units<BF16, NC, S::PX>(lds + S::OFF_XP + 2 * (64 * w + pplace), sn);
            }
          }
          return;
        }
        if constexpr (SPREAD) {
          if (NW * 64 == 4 * KG || 64 * w < 4 * KG) {      // (KG: 64 rows a wavefront, or none)
            put_units<BF16, NC, S::PX>(lds + S::OFF_X + (64 * w + lane) * S::ES, s);
            if constexpr (NORM) {
              float sn[NC];
#pragma unroll
              for (int c = 0; c < NC; ++c) sn[c] = (s[c] - mu) * iv;
              put_units<BF16, NC, S::PX>(lds + S::OFF_XP + (64 * w + lane) * S::ES, sn);
            }
          }
        } else {
          sop[0] = operand(s);
          if constexpr (NORM) {
            float sn[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) sn[c] = (s[c] - mu) * iv;
            pop[0] = operand(sn);
          }
        }
      };
      auto fetch_state = [&] {
        if constexpr (S::PAIRS_X) {
#pragma unroll
          for (int r = 0; r < NR; ++r) {
            sop[r] = *reinterpret_cast<const u32x4*>(lds + S::OFF_X + (pcopy * S::PX + 64 * r + pat) * S::ES);
            if (NORM) pop[r] = *reinterpret_cast<const u32x4*>(lds + S::OFF_XP + (pcopy * S::PX + 64 * r + pat) * S::ES);
          }
        } else if constexpr (SPREAD) {
#pragma unroll
          for (int r = 0; r < NR; ++r) {
            sop[r] = *reinterpret_cast<const V4*>(lds + S::OFF_X + (copy_x * S::PX + 64 * r + 4 * blk) * S::ES);
            if (NORM) pop[r] = *reinterpret_cast<const V4*>(lds + S::OFF_XP + (copy_x * S::PX + 64 * r + 4 * blk) * S::ES);
          }
        }
      };
      // SPREAD: bits of the copies that rows of any wavefront have ended so far
      uint32_t* flags = reinterpret_cast<uint32_t*>(lds + S::OFF_FLAG);
      publish();
      if constexpr (SPREAD) {
        if (tid == 0) *flags = 0u;
        sync();
        fetch_state();
      }

      const f32x4 zero4 = f32x4{0.f, 0.f, 0.f, 0.f};
      // One branch per step, the loop's own: a taken one costs a lone wavefront some seventy cycles of instruction fetch, and its condition is one scalar
      // (the end of a copy, or of the horizon); what follows from it stands behind the loop, which is entered again while copies run.
      uint32_t t = 0u, stop, seen = 0u;      // seen: SPREAD, copies ended by any row so far
      unsigned long long over[NC];
      if constexpr (S::loop_at() >= 0) asm volatile(".p2align 6\n\t.rept %0\n\ts_nop 0\n\t.endr" ::"i"(S::loop_at() < 0 ? 0 : S::loop_at()));
      while (true) {
      do {
#pragma unroll
        for (int c = 0; c < NC; ++c)
          if constexpr (NC > 1 || !SPREAD) {      // (one copy with spread rows: constants, which the compiler keeps where it likes)
            pin_sgpr(ninv[c]); pin_sgpr(thr[c]);
            if (!S::ROWS_COPY) pin_sgpr(ncost[c]);
          }
        // (two wait states must lie between instructions on one accumulator: two accumulators alternate)
        f32x4 accE[2] = {zero4, zero4}, pairE[4];
        if constexpr (S::PAIRS_X) pair_zero<NC>(pairE);
        // A s is off the chain of dependent layers: its K groups are issued in five portions, between the vector
        // instructions of the activations and where the chain waits for the LDS
        auto env_done = [&] {      // (what has been issued so far stays in front of what follows)
          if constexpr (S::PAIRS_X) {
#pragma unroll
            for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(pairE[k]));
          }
        };
        auto env_part = [&](auto from, auto to) {
          static_for<S::env_at(decltype(from)::value), S::env_at(decltype(to)::value)>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            if constexpr (S::PAIRS_X) pairE[g % 4] = pair_mac(sop[g / 4], Ae[g / 4][g % 4], pairE[g % 4], pwhich);
            else O::template mac<4, g % 16, g>(sop[g / 16], Ae[g], accE);
          });
        };
        auto bar = [] { __builtin_amdgcn_sched_barrier(0); };
        // an activation with a portion of A s between its vector instructions
        auto mix = [&](auto from, auto to) {
          constexpr int n = (S::env_at(decltype(to)::value) - S::env_at(decltype(from)::value)) * (BF16 ? 1 : 4);
#pragma unroll
          for (int k = 0; k < n; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, S::PAIRS_X ? 3 : 1, 0);
          }
          env_done();
          bar();
        };
        // (v: two accumulators of the 4x4 shapes, or the four tiles of paired products)
        auto act = [&](const auto& v, float b, float (&h)[NC]) {
          auto squash = [&](float z) { return S::RELU ? fmaxf(z + b, 0.f) : tanh_b<S::NEAR>(z, b); };
          if constexpr (sizeof(v) == 4 * sizeof(f32x4)) {
            float z[NC];
            pair_units<NC>(v, upper, z);
#pragma unroll
            for (int c = 0; c < NC; ++c) h[c] = squash(z[c]);
          } else if constexpr (S::SUMS_FIRST) {
            float z[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) z[c] = v[0][c] + v[1][c];
#pragma unroll
            for (int c = 0; c < NC; ++c) h[c] = squash(z[c]);
          } else {
#pragma unroll
            for (int c = 0; c < NC; ++c) h[c] = squash(v[0][c] + v[1][c]);
          }
        };
        using I0 = std::integral_constant<int, 0>; using I1 = std::integral_constant<int, 1>; using I2 = std::integral_constant<int, 2>;
        using I3 = std::integral_constant<int, 3>; using I4 = std::integral_constant<int, 4>; using I5 = std::integral_constant<int, 5>;
        // ---- layer 1 ----
        bar();
        f32x4 acc[S::PAIRS_X ? 4 : 2];
        if constexpr (S::PAIRS_X) {
          pair_zero<NC>(acc);
          static_for<0, 4 * NR>([&](auto gc) {
            constexpr int m = decltype(gc)::value / 4, k = decltype(gc)::value % 4;
            if (S::OCC == 1) pin_agpr(W1[m][k]);
            acc[k] = pair_mac(NORM ? pop[NORM ? m : 0] : sop[m], W1[m][k], acc[k], pwhich);
          });
        } else {
          acc[0] = acc[1] = zero4;
          static_for<0, KG>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            if (S::OCC == 1 && KG > 16) pin_agpr(W1[g]);
            O::template mac<4, g % 16, g>(NORM ? pop[NORM ? g / 16 : 0] : sop[g / 16], W1[g], acc);
          });
        }
        // the reward's state term, from the pre-step state
#pragma unroll
        for (int c = 0; c < NC; ++c) Rs[c] = __fmaf_rn(s[c] * s[c], ninv[c], Rs[c]);
        bar();
        float hv[NC];
        if constexpr (!S::PAIRS_X || M == 1) env_part(I0{}, I1{});
        act(acc, hb[0], hv);
        V4 h;                    // this wavefront's 64 units, as an operand
        if constexpr (NW > 1 && M > 1) put_units<BF16, NC, S::PH>(lds + S::OFF_H + S::ES * (64 * w + (S::PAIRS_H ? pplace : lane)), hv);
        else h = operand(hv);
        if constexpr (S::PAIRS_X && M > 1) { bar(); env_part(I0{}, I1{}); env_done(); bar(); }      // (while the writes are under way)
        else mix(I0{}, I1{});
        // ---- further hidden layers ----
        static_for<0, M - 1>([&](auto lc) {
          constexpr int l = decltype(lc)::value;
          constexpr int RING = S::PAIRS_H && S::TIGHT ? 2 : NW;
          std::conditional_t<S::PAIRS_H, u32x4, V4> hf[RING];
          f32x4 acch[S::PAIRS_H ? 4 : 2];
          if constexpr (S::PAIRS_H) pair_zero<NC>(acch);
          else acch[0] = acch[1] = zero4;
          if constexpr (NW > 1) {
            unsigned char* hbuf = lds + S::OFF_H + (l & 1) * S::HB;
            sync();
#pragma unroll
            for (int r = 0; r < RING; ++r) {
              if constexpr (S::PAIRS_H) hf[r] = *reinterpret_cast<const u32x4*>(hbuf + (pcopy * S::PH + 64 * r + pat) * S::ES);
              else hf[r] = *reinterpret_cast<const V4*>(hbuf + (copy_x * S::PH + 64 * r + 4 * blk) * S::ES);
            }
            bar();
            if constexpr (l == 0) { env_part(I1{}, I2{}); env_done(); }
            bar();
          } else {
            hf[0] = h;
          }
          if constexpr (S::PAIRS_H) {
            static_for<0, 4 * NW>([&](auto gc) {
              constexpr int m = decltype(gc)::value / 4, k = decltype(gc)::value % 4;
              if (S::OCC == 1 && l < 2) pin_agpr(Wh[l][m][k]);
              acch[k] = pair_mac(hf[m % RING], Wh[l][m][k], acch[k], pwhich);
              if constexpr (k == 3 && m + RING < NW) {
                hf[m % RING] = *reinterpret_cast<const u32x4*>(lds + S::OFF_H + (l & 1) * S::HB + (pcopy * S::PH + 64 * (m + RING) + pat) * S::ES);
                bar();
              }
            });
          } else {
            static_for<0, HG>([&](auto gc) {
              constexpr int g = decltype(gc)::value;
              if (S::OCC == 1 && l < (BF16 ? 2 : 1)) pin_agpr(Wh[l][g]);
              O::template mac<4, g % 16, g>(hf[g / 16], Wh[l][g], acch);
            });
          }
          bar();
          if constexpr (l == 0 && !S::PAIRS_X) env_part(I2{}, I3{});
          act(acch, hb[l + 1], hv);
          if constexpr (NW > 1 && l < M - 2) put_units<BF16, NC, S::PH>(lds + S::OFF_H + ((l + 1) & 1) * S::HB + S::ES * (64 * w + (S::PAIRS_H ? pplace : lane)), hv);
          else h = operand(hv);
          if constexpr (l == 0 && !S::PAIRS_X) mix(I2{}, I3{}); else bar();
        });
        // ---- action layer: this wavefront's K slice ----
        f32x4 pa, pq[2] = {zero4, zero4};
        if constexpr (S::HALVES) {
          static_for<0, 8>([&](auto gc) { constexpr int g = decltype(gc)::value; O::template mac<3, g, g>(h, W3[g], pq); });
          pa = pq[0] + pq[1];
        } else if constexpr (!S::GROUPED) {
          static_for<0, 16>([&](auto gc) { constexpr int g = decltype(gc)::value; O::template mac<4, g, g>(h, W3[g], pq); });
          pa = pq[0] + pq[1];
        } else {
          // groups of four blocks: one instruction multiplies four K values with sixteen action rows
          static_for<0, 4>([&](auto gc) { constexpr int g = decltype(gc)::value; O::template mac<2, g, g>(h, W3[g], pq); });
          // add the four lane groups' sums and transpose: D[action][copy] += sum over groups of pa_c x [column's copy is c]
          f32x4 d = zero4;
#pragma unroll
          for (int c = 0; c < NC; ++c) d = __builtin_amdgcn_mfma_f32_16x16x4f32(pq[0][c] + pq[1][c], sel_c[c], d, 0, 0, 0);
          pa = d;                // lane (group gq, n): rows 4 gq .. 4 gq + 3 of copy n % 4
        }
        float av[S::ROWS_COPY ? RPL : NC];
        if constexpr (NW > 1) {
          float* pb = part + (S::P_TWICE ? (t & 1u) * (S::NP * NC * S::PP) : 0);
          if constexpr (S::HALVES) {
            if (S::NA == 32 || (lane & 31) < S::NA) {
#pragma unroll
              for (int c = 0; c < NC; ++c) pb[((2 * w + (lane >> 5)) * NC + c) * S::PP + (lane & 31)] = pa[c];
            }
          } else {
            if ((lane & (NC == 1 ? 15 : 12)) == 0) *reinterpret_cast<f32x4*>(pb + (w * NC + (NC == 1 ? 0 : x)) * S::PP + 4 * (lane >> 4)) = pa;
          }
          if constexpr (S::PAIRS_X) { bar(); env_part(I2{}, I3{}); env_done(); bar(); }
          sync();
          float pv[S::NP][RPL];
          const float* src = pb + (S::ROWS_COPY ? (x & (NC - 1)) * S::PP + RPL * blk : lane);
#pragma unroll
          for (int ww = 0; ww < S::NP; ++ww) {
            if constexpr (S::ROWS_COPY && RPL == 2) { const f32x2 v2 = *reinterpret_cast<const f32x2*>(src + ww * NC * S::PP); pv[ww][0] = v2.x; pv[ww][1] = v2.y; }
            else pv[ww][0] = src[ww * NC * S::PP];
          }
          bar();
          env_part(I3{}, I4{});
          env_done();
          bar();
          constexpr int NV = S::ROWS_COPY ? RPL : 1;
#pragma unroll
          for (int r = 0; r < NV; ++r) {
            float sum[2] = {pv[0][r], pv[S::NP / 2][r]};
#pragma unroll
            for (int ww = 1; ww < S::NP / 2; ++ww) { sum[0] += pv[ww][r]; sum[1] += pv[S::NP / 2 + ww][r]; }
            av[r] = sum[0] + sum[1];
          }
        } else if constexpr (S::ROWS_COPY) {
          // sixteen lanes hold rows 4 gq .. 4 gq + 3 of their copy: each takes one, row = block
          const int j = blk & 3;
          av[0] = j == 0 ? pa.x : j == 1 ? pa.y : j == 2 ? pa.z : pa.w;
          env_part(I3{}, I4{});
        } else {
#pragma unroll
          for (int c = 0; c < NC; ++c) av[c] = pa[c];
          env_part(I3{}, I4{});
        }
        // ---- the action, its cost, B a ----
        env_part(I4{}, I5{});
        V4 aop;
        if constexpr (S::ROWS_COPY) {
          float sq = 0.0f;
#pragma unroll
          for (int r = 0; r < RPL; ++r) {
            const float z = av[r] + b3[r], tz = tanh_b<S::NEAR>(z, 0.0f);
            av[r] = squash ? tz : z;
            sq = r == 0 ? av[0] * av[0] : __fmaf_rn(av[r], av[r], sq);
          }
          Rx = __fmaf_rn(sq, xcost, Rx);
          aop = O::template collect<RPL>(av);
        } else {
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const float z = av[c] + b3[0], tz = tanh_b<S::NEAR>(z, 0.0f);
            av[c] = squash ? tz : z;
            Rs[c] = __fmaf_rn(av[c] * av[c], ncost[c], Rs[c]);
          }
          aop = operand(av);
        }
        if constexpr (S::PAIRS_X) {
          float ea[NC];
          pair_units<NC>(pairE, upper, ea);
#pragma unroll
          for (int c = 0; c < NC; ++c) accE[0][c] = ea[c];
        }
        mix(I4{}, I5{});
        static_for<0, KGA>([&](auto gc) {
          constexpr int g = decltype(gc)::value;
          constexpr int from = S::ROWS_COPY ? (RPL == 2 ? 2 * g : 4 * g) : g;
          O::template mac<4, from, g>(aop, Be[g], accE);
        });
#pragma unroll
        for (int c = 0; c < NC; ++c) s[c] = tanh_b<S::NEAR>(accE[0][c] + accE[1][c], 0.0f);       // padded rows: tanh(0) = 0
        // ---- termination: max |s| > threshold ends a copy after this step ----
        unsigned long long any = 0ull;
#pragma unroll
        for (int c = 0; c < NC; ++c) { over[c] = __ballot(fabsf(s[c]) > thr[c]); any |= over[c]; }
        if constexpr (SPREAD) {
          if (__builtin_expect(any != 0ull, 0)) {
            uint32_t f = 0u;
#pragma unroll
            for (int c = 0; c < NC; ++c) f |= over[c] != 0ull ? 1u << c : 0u;
            if (lane == 0) atomicOr(flags, f);
          }
        }
        publish();
        if constexpr (SPREAD) {
          sync();
          fetch_state();
          seen = uniform(*flags) & alive;
        }
        ++t;
        asm volatile("s_cmp_eq_u32 %1, %2\n\ts_cselect_b32 %0, 1, 0" : "=s"(stop) : "s"(t), "s"(a.T) : "scc");      // (scalar: the compiler makes masks of it)
        stop |= SPREAD ? seen : (uint32_t)any | (uint32_t)(any >> 32);
      } while (stop == 0u);
        // ---- some copy ended, or all with the horizon ----
        uint32_t ended = seen;
        if constexpr (!SPREAD) {
#pragma unroll
          for (int c = 0; c < NC; ++c) ended |= over[c] != 0ull ? 1u << c : 0u;
          ended = uniform(ended & alive);
        }
        if (t == a.T) ended = alive;
        // (a copy that has ended goes on with the others and may run into infinities, so its share is put aside here: a factor of zero does not keep them out)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const bool end = (ended >> c & 1u) != 0u;
          if (NC > 1 && end) ends[c * NT + tid_now()] = Rs[c] + (x == c ? Rx : 0.0f);
          len[c] = (int)uniform(end ? t : (uint32_t)len[c]);
          ninv[c] = uniform(end ? 0.0f : ninv[c]);
          ncost[c] = uniform(end ? 0.0f : ncost[c]);
          thr[c] = uniform(end ? __builtin_inff() : thr[c]);
        }
        alive &= ~ended;
        if (((alive >> x) & 1u) == 0u) xcost = 0.0f;
        if (alive == 0u) break;
      }
      // ---- outputs of this pass: return = length + the lanes' shares ----
      const uint32_t cnt = min((uint32_t)NC, a.E - (uint32_t)NC * pass);
      float R[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) R[c] = wave_sum(NC == 1 ? Rs[0] + Rx : ends[c * NT + tid_now()]);      // (written by this thread)
      if constexpr (SPREAD) {
        float* red = reinterpret_cast<float*>(lds + S::OFF_RED);
        if (lane == 0) {
#pragma unroll
          for (int c = 0; c < NC; ++c) red[w * NC + c] = R[c];
        }
        sync();
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          R[c] = red[c];
#pragma unroll
          for (int ww = 1; ww < NW; ++ww) R[c] += red[ww * NC + c];
        }
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const float total = (float)len[c] + R[c];
        if ((uint32_t)c < cnt) {
          fit_sum += total;
          if (tid == 0) {
            a.returns[(size_t)i * a.E + (uint32_t)NC * pass + (uint32_t)c] = total;
            a.ep_len[(size_t)i * a.E + (uint32_t)NC * pass + (uint32_t)c] = len[c];
          }
        }
      }
      if constexpr (NW > 1) sync();            // the exchange buffers are free before the next pass writes them
    }
    if (a.fitness && tid == 0) a.fitness[i] = fit_sum / (float)a.E;
  }
}

// How many workgroups share an individual's passes: all of them apart while that still fits the chip at once, because
// a pass is a chain of T dependent steps; one workgroup for all passes once individuals alone fill it (staging once).
inline uint32_t quad_split(uint32_t pop, uint32_t nblk, uint32_t slots) {
  if (pop >= slots || nblk == 1u) return 1u;
  return std::min(nblk, std::max(1u, slots / pop));
}

template <class S>
int launch_quad_shape(es_ctx* ctx, QuadArgs a, float* fitness, hipStream_t st) {
  const void* fn = reinterpret_cast<const void*>(rollout_quad_kernel<S>);
  hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_BYTES);
  if (err != hipSuccess) return fail(ctx, ES_EHIP, std::string("hipFuncSetAttribute: ") + hipGetErrorString(err));
  const uint32_t per_cu = (uint32_t)std::max(1, std::min(4 * S::OCC / S::NW, ctx->lds_limit / S::LDS_BYTES));
  const uint32_t slots = (uint32_t)std::max(1, ctx->num_cus) * per_cu;
  a.split = quad_split(a.N, (a.E + (uint32_t)S::NC - 1u) / (uint32_t)S::NC, slots);
  a.fitness = a.split == 1u ? fitness : nullptr;
  const uint32_t grid = std::min<uint32_t>(a.N * a.split, slots);
  const uint32_t cus = (uint32_t)std::max(1, ctx->num_cus);
  const bool place = S::PLACED && grid > cus && grid <= 2u * cus;
  hipLaunchKernelGGL(rollout_quad_kernel<S>, dim3(grid), dim3(place ? 256 : S::NT), S::LDS_BYTES, st, a);
  int rc = check_launch(ctx, "es_rollout (passes of four copies)");
  if (rc != ES_OK || a.split == 1u) return rc;
  return launch_fitness(ctx, a.returns, fitness, st);
}

// Activation and observation statistics chosen at compile time; statistics only where WITH_NORM.
template <bool BF16, int NW, int KG, int M, int NC, bool WITH_NORM, bool NEAR>
int launch_quad_options(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  const bool relu = ctx->cfg.hidden_act == 1;
  if constexpr (WITH_NORM) {
    if (a.obs_mean)
      return relu ? launch_quad_shape<QuadShape<BF16, NW, KG, M, NC, true, true, NEAR>>(ctx, a, fitness, st)
                  : launch_quad_shape<QuadShape<BF16, NW, KG, M, NC, false, true, NEAR>>(ctx, a, fitness, st);
  }
  return relu ? launch_quad_shape<QuadShape<BF16, NW, KG, M, NC, true, false, NEAR>>(ctx, a, fitness, st)
              : launch_quad_shape<QuadShape<BF16, NW, KG, M, NC, false, false, NEAR>>(ctx, a, fitness, st);
}
// Copies of a pass: as few as the chip can take side by side, one wavefront per SIMD, since the activations of a copy are on the chain of a step.
// Per 100 steps of bf16 27-100-100-8, four copies a pass / as chosen: 128 individuals x 2 copies 97 / 75 us (one), 128 x 3 97 / 84 (one), 128 x 5 100 / 87
// (two), 512 x 2 127 / 85 (two; 42 us of it wavefront_place), 8-256-256-2 64 x 8 129 / 118 (two); three layers per 200 steps, 27-100x3-6 128 x 4
// 321 / 270 (two), 8-256x3-6 512 x 2 614 / 535 (two).  An individual is then staged by several workgroups, which very few steps do not bring back: 27-256-256-8
// 128 x 2 2 steps 32 / 34, 244-256-256-17 64 x 4 44 / 49.  (Four layers split the action layer by lane groups, which needs all four rows or one.)
template <bool BF16, int NW, int KG, int M, bool WITH_NORM, bool NEAR>
int launch_quad_copies(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  auto apart = [&](uint32_t nc) { return (uint64_t)a.N * ((a.E + nc - 1u) / nc) * NW <= 4u * (uint64_t)ctx->num_cus; };
  if (a.E == 1u || apart(1u)) return launch_quad_options<BF16, NW, KG, M, 1, WITH_NORM, NEAR>(ctx, a, fitness, st);
  if constexpr (BF16 && M <= 3) {
    if (a.E == 2u || apart(2u)) return launch_quad_options<BF16, NW, KG, M, 2, WITH_NORM, NEAR>(ctx, a, fitness, st);
  }
  return launch_quad_options<BF16, NW, KG, M, 4, WITH_NORM, NEAR>(ctx, a, fitness, st);
}
// obs <= 64: the width class (in binary32, where a group of four costs four instructions twice a step, one more class;
// observation statistics only in the widest)
template <bool BF16, int NW, int M, bool NEAR>
int launch_quad_obs64(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st) {
  if constexpr (!BF16) {
    if (a.no <= 16 && !a.obs_mean) return launch_quad_copies<BF16, NW, 4, M, false, NEAR>(ctx, a, fitness, st);
  }
  if (a.no <= 32 && !a.obs_mean) return launch_quad_copies<BF16, NW, 8, M, false, NEAR>(ctx, a, fitness, st);
  if constexpr (BF16 && M == 4) {      // (wide observations of several copies: quad_fits)
    if (a.E > 1u && !a.obs_mean) return fail(ctx, ES_EUNSUPPORTED, "es_rollout: no four-copy variant for four layers and more than 32 observations");
    if (a.E > 1u)
      return ctx->cfg.hidden_act == 1 ? launch_quad_shape<QuadShape<BF16, NW, 16, M, 4, true, true, NEAR>>(ctx, a, fitness, st)
                                      : launch_quad_shape<QuadShape<BF16, NW, 16, M, 4, false, true, NEAR>>(ctx, a, fitness, st);
    return launch_quad_options<BF16, NW, 16, M, 1, true, NEAR>(ctx, a, fitness, st);
  }
  return launch_quad_copies<BF16, NW, 16, M, true, NEAR>(ctx, a, fitness, st);
}

// one source file each (compile time); M = hidden layers of the context
int launch_quad_bf16_mid(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);     // two wavefronts, one or two layers
int launch_quad_bf16_wide(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);    // four wavefronts, one or two layers
int launch_quad_bf16_mid3(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);    // four wavefronts, three layers, fewer than 128 units
int launch_quad_bf16_mid4(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);    // ... four layers
int launch_quad_bf16_deep3(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);   // four wavefronts, three layers
int launch_quad_bf16_deep4(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);   // ... four layers
int launch_quad_f32_mid(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);      // two wavefronts, one to three layers
int launch_quad_f32_wide(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);     // four wavefronts, one or two layers
int launch_quad_narrow(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);       // one wavefront, two layers
int launch_quad_obs128(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);       // four wavefronts, bf16, two layers, obs <= 128, act <= 32
int launch_quad_obs192(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);       // ... <= 192
int launch_quad_obs256(es_ctx* ctx, const QuadArgs& a, float* fitness, hipStream_t st);       // ... <= 256

}  // namespace es
