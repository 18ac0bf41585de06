// es_rollout, register-resident MFMA variant for bf16 policies with a wide hidden layer.
//
// Paper Sec. 3.2 (population x environment-copy evaluation) and Sec. 5.1/5.2 (two hidden
// layers of 256 units, fitness = mean undiscounted return).  One workgroup of four
// wavefronts evaluates one individual at a time on up to 16 environment copies per pass:
//
//   * The individual's perturbed bf16 weights never touch HBM: theta + sign*sigma*eps is
//     computed while staging, and the result is parked in the VGPR/AGPR file as MFMA
//     A-operands (16x16x32 bf16 tiles) for all T steps.  A 256-wide policy is 130-270 KB in
//     bf16, more than the 160 KB of LDS, but fits the 512 KB register file of a CU.  The
//     environment matrices A and B (shared by all individuals) are register-resident too.
//   * Each wavefront owns 64 output units (four 16-row tiles) of every wide layer; the
//     environment copies are the 16 columns of the MFMA.  Activations travel between
//     wavefronts as bf16 through LDS ([column][unit], padded pitch, 16-byte reads).
//   * The narrow 256 -> act layer is split along K: any K order is as good as another as long
//     as both MFMA operands agree, so every wavefront multiplies the 64 units of the last
//     hidden layer it has just produced - still in its registers - with its slice of the
//     action-layer weights, and only the binary32 partial sums cross the LDS.
//   * Books are kept off the chain of a step: every lane holds its share of |s'|^2 and |a|^2 back and adds
//     them up under the next step's layer-1 stream (per-wavefront partials through the LDS, added in the same
//     fixed order everywhere, so reruns are bit-identical); a column that ends sets a bit in an LDS word that
//     is read with the next state, and everything that follows from it sits behind one branch that is not
//     taken.  (obs 27, 1024 individuals x 16 copies x 300 steps: 1.28 -> 1.19 ms together with the roles of the
//     wavefronts below; before, the norms, their maxima and the bookkeeping were on the chain of every step.)
//   * The grid is persistent: workgroup b handles individuals b, b + grid, ...
// Bound: the dependent chain of a step (MFMA streams, activation epilogues on the vector ALU,
// three LDS hand-overs) in one in-order wavefront per SIMD; two where the register file allows.
#include <type_traits>

#include "es_internal.hpp"
#include "rollout_stage.hpp"

namespace es {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct MfmaArgs {
  const float* theta;
  const void* noise;
  const uint32_t* noise_offs;   // shared noise table: start of every row, else null
  const float* A;
  const float* B;
  const float* obs_mean;     // frozen observation statistics (paper App. B), or null
  const float* obs_inv;
  float* returns;
  int32_t* ep_len;
  float* fitness;
  uint32_t N, E, T, no, nh, na, ld;
  uint32_t oW1, ob1, oW2, ob2, oW3, ob3;
  uint32_t gen, k0, k1;
  uint32_t antithetic, out_tanh, noise_mode;
  float sigma, done_thresh, act_cost;
  unsigned long long* prof;     // phase-timing build only (ES_PHASE_PROF): cycle totals per wavefront and phase
};

// A kernel argument read afresh from the kernel-argument segment (the one by-value argument starts at its offset 0),
// through a pointer the compiler cannot see through.  The staging code takes its arguments this way once per
// individual: read from the by-value copy they would be loaded once and then held in scalar registers across the
// step loop, which already spills scalar registers to vector lanes and reloads them every step.
template <class T>
__device__ __forceinline__ T kernarg_field(size_t byte_off) {
  const __attribute__((address_space(4))) char* p =
      (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *reinterpret_cast<const __attribute__((address_space(4))) T*>(p + byte_off);
}
#define KARG(field) kernarg_field<decltype(MfmaArgs::field)>(offsetof(MfmaArgs, field))

// Phase timing for tuning (compiled in with -DES_PHASE_PROF only): shader-clock cycles between consecutive stamps,
// summed over all steps of the individuals of workgroup 0, one row of 16 slots per wavefront.
#ifdef ES_PHASE_PROF
#define PSTAMP(k) do { const unsigned long long now_ = __builtin_readcyclecounter(); prof_acc[k] += now_ - prof_last; prof_last = now_; } while (0)
#else
#define PSTAMP(k) do {} while (0)
#endif

constexpr int NHP = 256;          // padded hidden width handled by this kernel
constexpr int KT_H = NHP / 32;    // 32-deep K tiles over the hidden width
constexpr int PH = NHP + 8;       // LDS pitch (bf16 elements) of a hidden activation row

constexpr int KC = 2;             // K tiles staged per round
constexpr int PW = 32 * KC + 8;   // LDS pitch of the staging window

template <int KT1_, int MT3_, int MTE_, int KTAR_, int NW_, int OCC_ = 1, int ME_ = 0, bool ENVF_ = false, bool NEAR_ = false>
struct Variant {
  static constexpr bool NEAR = NEAR_;          // the tanh that is accurate near zero
  static constexpr bool ENVF = ENVF_;          // the environment's products A s + B a stay binary32 (fp32 16x16x4 MFMAs, its own
                                              // binary32 copy of the state in LDS); the policy keeps its bf16 operands
  static constexpr int ME = ME_;              // hidden layers beyond the second (depth m = 2 + ME), each 256 x 256 in registers;
                                              // -1: a single hidden layer (the second layer's phase is skipped)
  static constexpr int OCC = OCC_;            // workgroups per CU the register budget is sized for (1 or 2)
  static constexpr int NW = NW_;              // wavefronts per workgroup: one per SIMD
  static constexpr int NT = 64 * NW;          // threads per workgroup
  static constexpr int MT_H = NHP / (16 * NW);   // 16-row tiles of a wide layer per wavefront
  static constexpr int ENV_ROWS = 16 * NW * MTE_;   // padded rows of the next-state vector covered by the workgroup
  static constexpr int NC = 16;               // environment copies per pass
  static constexpr int KT1 = KT1_;            // K tiles over the (padded) observation width
  static constexpr int MT3 = MT3_;            // 16-row tiles of the action layer
  static constexpr int MTE = MTE_;            // 16-row tiles of the next-state vector per wavefront
  static constexpr int KTAR = KTAR_;          // K tiles of the env matrix A held in registers ...
  static constexpr int KTAL = KT1 - KTAR;     // ... and in LDS (when the register file is full)
  static constexpr int KTA = (16 * MT3 + 31) / 32;   // K tiles over the (padded) action width
  static constexpr int NOP = 32 * KT1;        // padded observation width
  static constexpr int NAP = 32 * KTA;        // padded action width as a K dimension
  static constexpr int PX = NOP + 8;          // LDS pitch of a state row
  static constexpr int PA = NAP + 8;          // LDS pitch of an action row
  static constexpr int PAL = 32 * KTAL + 8;   // LDS pitch of the LDS-resident part of A
  // LDS map (bytes).  [0, REGION0) is the staging window, aliased by the rollout buffers.
  static constexpr int OFF_X = 0;
  static constexpr int OFF_H1 = OFF_X + 2 * NC * PX;
  static constexpr int OFF_H2 = OFF_H1 + 2 * NC * PH;
  static constexpr int OFF_SSP = OFF_H2 + 2 * NC * PH;      // |s'|^2 partials [column][wavefront]
  static constexpr int OFF_FLAG = OFF_SSP + 4 * 16 * NW;    // bits of the columns that rows of a wavefront have ended, one word per wavefront
  static constexpr int OFF_SCR = OFF_FLAG + 4 * NW;         // scratch for the initial-state norms; lanes without a partial to write write here
  static constexpr int ROLL_END = OFF_SCR + 4 * NT;
  static constexpr int WIN_BYTES = 2 * 256 * PW;
  static constexpr int REGION0 = ROLL_END > WIN_BYTES ? ROLL_END : WIN_BYTES;
  static constexpr int OFF_AL = REGION0;
  static constexpr int OFF_W3 = OFF_AL + (KTAL ? 2 * ENV_ROWS * PAL : 0);   // action-layer weights [16*MT3][PH]
  static constexpr int OFF_B1 = OFF_W3 + 2 * 16 * MT3 * PH;
  static constexpr int OFF_B2 = OFF_B1 + 4 * NHP;
  static constexpr int OFF_B3 = OFF_B2 + 4 * NHP;
  static constexpr int OFF_X0 = OFF_B3 + 4 * 16 * MT3;
  static constexpr int OFF_SS0 = OFF_X0 + 2 * NC * PX;
  // only used with observation statistics: the normalised state (the policy's operand), its cached
  // initial value, and the statistics themselves
  static constexpr int OFF_BX = OFF_SS0 + 4 * 16;              // biases of the extra hidden layers [ME][NHP]
  static constexpr int OFF_XP = OFF_BX + 4 * NHP * (ME > 0 ? ME : 0);
  static constexpr int OFF_X0P = OFF_XP + 2 * NC * PX;
  static constexpr int OFF_MU = OFF_X0P + 2 * NC * PX;
  static constexpr int OFF_IV = OFF_MU + 4 * NOP;
  // binary32 partial sums of the action layer, which is split along K: [wavefront][copy][PP3 rows]
  static constexpr int OFF_P3 = OFF_IV + 4 * NOP;
  // binary32 environment: the state as binary32 [copy][state index] (pitch PXF floats: 16-byte reads of 16 lanes hit
  // distinct banks), working buffer and cached initial value
  static constexpr int KPL = NOP / 4;          // state elements per lane group of the fp32 MFMA's K dimension
  static constexpr int PXF = NOP + 4;
  static constexpr int PP3 = 16 * MT3_ + 4;    // pitch (floats) of a copy's partial rows: 16-byte accesses of 16 lanes spread over the banks
  static constexpr int OFF_XF = OFF_P3 + 4 * NW * NC * PP3;
  static constexpr int OFF_X0F = OFF_XF + (ENVF ? 4 * NC * PXF : 0);
  static constexpr int OFF_BL = OFF_X0F + (ENVF ? 4 * NC * PXF : 0);      // B [ENV_ROWS][PA] bf16
  // four hidden layers leave four registers too few for everything: B then stays in LDS
  static constexpr bool B_LDS = ME_ == 2;
  static constexpr int LDS_BYTES = OFF_BL + (B_LDS ? 2 * ENV_ROWS * PA : 0);
  static_assert(!ENVF || (ME == 0 && MT3 == 1 && KT1 <= 2), "binary32 environment: passes of 16 copies, two hidden layers, obs <= 64, act <= 16");
  static_assert(ENV_ROWS >= NOP, "the wavefronts must cover the padded state");
  static_assert(ENV_ROWS <= 256, "staging window rows");
  static_assert(NW == 4, "one wavefront per SIMD (two per SIMD, each with half of the rows, measured slower at every shape)");
  static_assert(MT_H >= 1 && MT_H <= 4, "wide-layer tiles per wavefront");
  static_assert(NAP >= 16 * MT3 && KTA <= KC, "action K padding");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
  static_assert(ME <= 0 || (OCC == 1 && KTAL == 0), "deeper policies need the whole register file of the CU");
  static_assert(ME >= 0 || KTAL == 0, "the single-layer variant keeps all of A in registers");
  static_assert(MT3 <= 2 && MT3 <= 4, "action tiles: one wavefront each, partial layout holds two");
};

__device__ __forceinline__ bf16x8 lds_tile(const unsigned char* base, int byte_off) {
  const u32x4 raw = *reinterpret_cast<const u32x4*>(base + byte_off);
  return __builtin_bit_cast(bf16x8, raw);
}

// Keeps a weight tile in the accumulation-register half of the unified register file: an
// empty asm that "updates" the tile in place pins its register class right at the use, so
// the MFMA reads its A operand from there directly instead of through copies.
__device__ __forceinline__ void pin_agpr(bf16x8& v) { asm volatile("" : "+a"(v)); }
// ... and the tiles for which that half has no room in the architectural one.
__device__ __forceinline__ void pin_vgpr(bf16x8& v) { asm volatile("" : "+v"(v)); }

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// binary32 16x16x4: lane (g, n) supplies A[row n][k = g] and B[k = g][column n]
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <bool NEAR>
__device__ __forceinline__ f32x4 tanh4(f32x4 v) {
  if (NEAR) {
    const f32x4 t = v * 2.88539008f;
    return f32x4{tanh_near(t.x), tanh_near(t.y), tanh_near(t.z), tanh_near(t.w)};
  }
  return f32x4{tanh_fast(v.x), tanh_fast(v.y), tanh_fast(v.z), tanh_fast(v.w)};
}
// hidden-layer activation: tanh, or ReLU (the paper's EA experiments, App. B) - a compile-time choice,
// so that the MFMA / vector-ALU interleaving below stays one straight-line region
template <bool RELU, bool NEAR>
__device__ __forceinline__ f32x4 hidden4(f32x4 v) {
  if (RELU) return f32x4{fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f)};
  return tanh4<NEAR>(v);
}

// Sum over the four 16-lane rows of the wavefront (lanes l, l+16, l+32, l+48), result in
// every row, by the row-swap instructions of gfx950 (vector ALU speed, no LDS round trip).
__device__ __forceinline__ float rows_sum(float v) {
  const unsigned b = __builtin_bit_cast(unsigned, v);
  const auto p = __builtin_amdgcn_permlane16_swap(b, b, false, false);     // (r0,r0,r2,r2) and (r1,r1,r3,r3)
  const float t = __builtin_bit_cast(float, (unsigned)p[0]) + __builtin_bit_cast(float, (unsigned)p[1]);
  const unsigned c = __builtin_bit_cast(unsigned, t);
  const auto r = __builtin_amdgcn_permlane32_swap(c, c, false, false);     // (lo,lo) and (hi,hi)
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
// some |v[k]| above the threshold, as a mask of lanes
__device__ __forceinline__ unsigned long long exceeds(f32x4 v, float thr) {
  return __ballot(fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))) > thr);
}

// ORDERED: wavefront priorities by phase (passes of sixteen copies, two workgroups per CU)
template <class V, bool RELU, bool NORM, bool ORDERED>
__global__ __launch_bounds__(V::NT) __attribute__((amdgpu_waves_per_eu(V::OCC * V::NW / 4, V::OCC * V::NW / 4)))
void rollout_mfma_kernel(const MfmaArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int KT1 = V::KT1, MT3 = V::MT3, MTE = V::MTE, KTA = V::KTA, PX = V::PX;
  constexpr int NW = V::NW, NT = V::NT, MT_H = V::MT_H;
  constexpr bool ENV_ALL = (V::ENV_ROWS == V::NOP);   // every wavefront's next-state tiles are inside the padded state
  constexpr int NC = V::NC;
  constexpr int LDS_BASE_REG = 6 | (0 << 6) | (11 << 11);      // hardware register LDS_ALLOC, bits 0..11: where the workgroup's LDS starts

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  // wavefront index, known uniform.  Where only two of the wavefronts have next-state tiles (obs <= 32) the second workgroup of
  // a CU - the one whose LDS does not start at 0 - turns the roles by three: the hardware deals wavefronts to the SIMDs in the cyclic
  // order 0 2 1 3 and starts the second workgroup one place after the first (read back from the hardware registers on all 256 CUs,
  // profiles/wavefront_dealing.md), so that each SIMD then carries one wavefront of each kind.  Only the speed depends on it.
  int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  if constexpr (!ENV_ALL && V::OCC == 2) w = (w + ((__builtin_amdgcn_s_getreg(LDS_BASE_REG) != 0) ? NW - 1 : 0)) % NW;
  const bool env_wave = ENV_ALL || 16 * w * MTE < V::NOP;      // has next-state tiles
  const int g = lane >> 4, n = lane & 15;
  uint16_t* stage = reinterpret_cast<uint16_t*>(lds);
  float* b1s = reinterpret_cast<float*>(lds + V::OFF_B1);
  float* b2s = reinterpret_cast<float*>(lds + V::OFF_B2);
  float* b3s = reinterpret_cast<float*>(lds + V::OFF_B3);
  float* bxs = reinterpret_cast<float*>(lds + V::OFF_BX);
  constexpr int ME = V::ME;
  uint16_t* x0s = reinterpret_cast<uint16_t*>(lds + V::OFF_X0);
  float* ss0s = reinterpret_cast<float*>(lds + V::OFF_SS0);
  uint32_t* flags = reinterpret_cast<uint32_t*>(lds + V::OFF_FLAG);
  uint16_t* x0ps = reinterpret_cast<uint16_t*>(lds + V::OFF_X0P);
  float* mus = reinterpret_cast<float*>(lds + V::OFF_MU);
  float* ivs = reinterpret_cast<float*>(lds + V::OFF_IV);
  const int no = (int)a.no, nh = (int)a.nh, na = (int)a.na;

  if (NORM) {     // padded rows get scale 0: their normalised value stays 0
    for (int k = tid; k < V::NOP; k += NT) {
      mus[k] = k < no ? a.obs_mean[k] : 0.0f;
      ivs[k] = k < no ? a.obs_inv[k] : 0.0f;
    }
  }
  // ---------------- environment matrices -> registers / LDS (once per workgroup) ----------------
  constexpr int KTAR = V::KTAR, KTAL = V::KTAL, PAL = V::PAL;
  constexpr bool ENVF = V::ENVF;
  constexpr int KPL = V::KPL, PXF = V::PXF;
  bf16x8 Ar[MTE][KTAR > 0 ? KTAR : 1], Br[MTE][KTA];
  // binary32 environment: A and B as fp32 MFMA A operands.  K slot (kk, g) of the state product stands for state
  // element KPL g + kk (so a lane's KPL operands are contiguous in the binary32 state buffer), K slot (kk, g) of the
  // action product for action row 4 g + kk (what the lane holds after the action layer): Af[tt][kk] = A[row][KPL g + kk],
  // Bf[tt][kk] = B[row][4 g + kk], row = 16 (w MTE + tt) + n.
  float Af[ENVF ? MTE : 1][ENVF ? KPL : 1], Bf[ENVF ? MTE : 1][4];
  if constexpr (ENVF) {
#pragma unroll
    for (int t = 0; t < MTE; ++t) {
      const int row = 16 * (w * MTE + t) + n;
#pragma unroll
      for (int kk = 0; kk < KPL; ++kk) { const int k = KPL * g + kk; Af[t][kk] = (row < no && k < no) ? a.A[row * no + k] : 0.0f; }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) { const int c = 4 * g + kk; Bf[t][kk] = (row < no && c < na) ? a.B[row * na + c] : 0.0f; }
    }
  }
#pragma unroll
  for (int kr = 0; kr < (ENVF ? 0 : (KTAR + KC - 1) / KC); ++kr) {
    stage_cols<32 * KC, false>(stage, PW, V::ENV_ROWS, no, no, 32 * KC * kr, a.A, NoiseRow{}, 0.0f, 0u);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < MTE; ++t)
#pragma unroll
      for (int kk = 0; kk < KC; ++kk)
        if (kr * KC + kk < KTAR)
          Ar[t][kr * KC + kk] = lds_tile(lds, 2 * ((16 * (w * MTE + t) + n) * PW + 32 * kk + 8 * g));
    __syncthreads();
  }
  if (KTAL > 0)
    stage_cols<32 * (KTAL > 0 ? KTAL : 1), false>(reinterpret_cast<uint16_t*>(lds + V::OFF_AL), PAL, V::ENV_ROWS, no, no,
                                                    32 * KTAR, a.A, NoiseRow{}, 0.0f, 0u);
  auto b_slots = [](const unsigned char* src) {
    const u32x2 lo = *reinterpret_cast<const u32x2*>(src);
    u32x2 hi = u32x2{0u, 0u};                                   // second action tile: rows 16 + 4g + (j - 4) in slots 4..7
    if (MT3 > 1) hi = *reinterpret_cast<const u32x2*>(src + 2 * 16);
    return __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
  };
  if constexpr (V::B_LDS) {
    stage_cols<V::NAP, false>(reinterpret_cast<uint16_t*>(lds + V::OFF_BL), V::PA, V::ENV_ROWS, no, na, 0, a.B, NoiseRow{}, 0.0f, 0u);
  } else if constexpr (!ENVF) {
    stage_cols<32 * KC, false>(stage, PW, V::ENV_ROWS, no, na, 0, a.B, NoiseRow{}, 0.0f, 0u);
    __syncthreads();
    // K slot j < 4 of lane group g stands for action row 4g + j, slot j >= 4 for row 16 + 4g + (j - 4) of the second
    // action tile (padding when there is one tile) - the rows whose sums the lane holds after the action layer: the
    // action goes from those registers into the MFMA
#pragma unroll
    for (int t = 0; t < MTE; ++t) Br[t][0] = b_slots(lds + 2 * ((16 * (w * MTE + t) + n) * PW + 4 * g));
    __syncthreads();
  }

  const uint32_t per_unit = a.antithetic ? 2u : 1u;
  const uint32_t nblk = (a.E + (uint32_t)NC - 1u) / (uint32_t)NC;
  int x0_block = -1;

  // the grid is persistent over individuals (not over mirrored pairs: a small population then still fills the chip;
  // the noise row is fetched once per individual either way)
  for (uint32_t i = blockIdx.x; i < a.N; i += gridDim.x) {
    {
      struct { const float* theta; const void* noise; const uint32_t* noise_offs;
               uint32_t ld, oW1, ob1, oW2, ob2, oW3, ob3, gen, k0, k1, noise_mode; float sigma; } sa;
      sa.theta = KARG(theta); sa.noise = KARG(noise); sa.noise_offs = KARG(noise_offs); sa.ld = KARG(ld);
      sa.oW1 = KARG(oW1); sa.ob1 = KARG(ob1); sa.oW2 = KARG(oW2); sa.ob2 = KARG(ob2); sa.oW3 = KARG(oW3); sa.ob3 = KARG(ob3);
      sa.gen = KARG(gen); sa.k0 = KARG(k0); sa.k1 = KARG(k1); sa.noise_mode = KARG(noise_mode); sa.sigma = KARG(sigma);
      const uint32_t unit = i / per_unit, sub = i - unit * per_unit;
      const float scale = sub ? -sa.sigma : sa.sigma;
      NoiseRow nz;
      nz.mode = sa.noise_mode; nz.row = unit; nz.gen = sa.gen; nz.k0 = sa.k0; nz.k1 = sa.k1;
      nz.ptr = nullptr;           // regenerated noise has no buffer
      if (sa.noise_offs) nz.ptr = table_row_base(sa.noise_mode, sa.noise, sa.noise_offs, unit);
      else if (sa.noise_mode == 1u) nz.ptr = static_cast<const uint16_t*>(sa.noise) + (size_t)unit * sa.ld;
      else if (sa.noise_mode == 0u) nz.ptr = static_cast<const float*>(sa.noise) + (size_t)unit * sa.ld;

      // ---------------- perturbed policy weights -> registers ----------------
      bf16x8 W1r[MT_H][KT1], W2r[MT_H][KT_H], Wxr[ME > 0 ? ME : 1][MT_H][KT_H];
      for (int u = tid; u < NHP; u += NT) {     // biases: perturbed, bf16-rounded, kept as binary32
        float v1 = 0.0f, v2 = 0.0f;
        if (u < nh) {
          const uint32_t i1 = sa.ob1 + u, i2 = sa.ob2 + u;
          v1 = bf16_round(__fmaf_rn(scale, row_noise(nz, i1), sa.theta[i1]));
          if (ME >= 0) v2 = bf16_round(__fmaf_rn(scale, row_noise(nz, i2), sa.theta[i2]));      // a single hidden layer has no second one
        }
        b1s[u] = v1;
        b2s[u] = v2;
#pragma unroll
        for (int j = 0; j < ME; ++j) {          // hidden layer 3 + j: matrix, then bias, after layer 2's
          float vx = 0.0f;
          if (u < nh) {
            const uint32_t ix = sa.ob2 + (uint32_t)(j + 1) * (uint32_t)(nh * nh + nh) + u;
            vx = bf16_round(__fmaf_rn(scale, row_noise(nz, ix), sa.theta[ix]));
          }
          bxs[j * NHP + u] = vx;
        }
      }
      for (int c = tid; c < 16 * MT3; c += NT) {
        float v3 = 0.0f;
        if (c < na) {
          const uint32_t i3 = sa.ob3 + c;
          const float e3 = row_noise(nz, i3);
          v3 = bf16_round(__fmaf_rn(scale, e3, sa.theta[i3]));
        }
        b3s[c] = v3;
      }
      // action-layer weights stay in LDS (read by one wavefront per tile each step)
      stage_cols<NHP, true>(reinterpret_cast<uint16_t*>(lds + V::OFF_W3), PH, 16 * MT3, na, nh, 0, sa.theta, nz, scale, sa.oW3);
#pragma unroll
      for (int kr = 0; kr < (KT1 + KC - 1) / KC; ++kr) {
        stage_cols<32 * KC, true>(stage, PW, NHP, nh, no, 32 * KC * kr, sa.theta, nz, scale, sa.oW1);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < MT_H; ++t)
#pragma unroll
          for (int kk = 0; kk < KC; ++kk)
            if (kr * KC + kk < KT1)
              W1r[t][kr * KC + kk] = lds_tile(lds, 2 * ((16 * (w * MT_H + t) + n) * PW + 32 * kk + 8 * g));
        __syncthreads();
      }
#pragma unroll
      for (int kr = 0; kr < (ME >= 0 ? KT_H / KC : 0); ++kr) {
        stage_cols<32 * KC, true>(stage, PW, NHP, nh, nh, 32 * KC * kr, sa.theta, nz, scale, sa.oW2);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < MT_H; ++t)
#pragma unroll
          for (int kk = 0; kk < KC; ++kk)
            W2r[t][kr * KC + kk] = lds_tile(lds, 2 * ((16 * (w * MT_H + t) + n) * PW + 32 * kk + 8 * g));
        __syncthreads();
      }

      auto stage_deeper = [&](auto jc) {
        constexpr int j = decltype(jc)::value;
#pragma unroll
        for (int kr = 0; kr < KT_H / KC; ++kr) {
          stage_cols<32 * KC, true>(stage, PW, NHP, nh, nh, 32 * KC * kr, sa.theta, nz, scale,
                                    sa.oW2 + (uint32_t)(j + 1) * (uint32_t)(nh * nh + nh));
          __syncthreads();
#pragma unroll
          for (int t = 0; t < MT_H; ++t)
#pragma unroll
            for (int kk = 0; kk < KC; ++kk)
              Wxr[j][t][kr * KC + kk] = lds_tile(lds, 2 * ((16 * (w * MT_H + t) + n) * PW + 32 * kk + 8 * g));
          __syncthreads();
        }
      };
      if constexpr (ME > 0) stage_deeper(std::integral_constant<int, 0>());
      if constexpr (ME > 1) stage_deeper(std::integral_constant<int, 1>());

      // This wavefront's K slice (its own 64 hidden units) of the action-layer weights, as MFMA A operands.  The K
      // order inside a tile follows the order in which the lane holds h2 after the layer-2 epilogue: slots 0..3 = units
      // 4g..4g+3 of the even 16-unit tile, slots 4..7 = the same rows of the odd tile (any K order is as good as another
      // as long as both operands agree), so h2 goes from the epilogue's registers into the MFMA with no exchange.
      bf16x8 W3k[MT3][2];
      auto w3k_tile = [&](int mt, int kk) {
        const unsigned char* src = lds + V::OFF_W3 + 2 * ((16 * mt + n) * PH + 64 * w + 32 * kk + 4 * g);
        const u32x2 lo = *reinterpret_cast<const u32x2*>(src), hi = *reinterpret_cast<const u32x2*>(src + 2 * 16);
        return __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
      };
      // ... held in registers where the file has room for them; fetched from LDS at their use otherwise (all of A in
      // registers, two workgroups per CU, more than two hidden layers)
      constexpr bool W3K_REGS = ME < 2;
      if constexpr (W3K_REGS) {
#pragma unroll
        for (int mt = 0; mt < MT3; ++mt)
#pragma unroll
          for (int kk = 0; kk < 2; ++kk) W3k[mt][kk] = w3k_tile(mt, kk);
      }

      float fit_sum = 0.0f;
      for (uint32_t cb = 0; cb < nblk; ++cb) {
        // ---------------- initial states of this block of environment copies ----------------
        if (x0_block != (int)cb) {
          // thread -> (column n0, row group kq): s0[k] for k = kq, kq + 16, ...
          constexpr int KG = NT / NC;                // row groups
          const int n0 = tid % NC, kq = tid / NC;
          const uint32_t x_gen = KARG(gen), x_k0 = KARG(k0), x_k1 = KARG(k1);
          const uint32_t e0 = cb * (uint32_t)NC + (uint32_t)n0;
          float part = 0.0f;
          for (int k = kq; k < V::NOP; k += KG) {
            float v = 0.0f;
            if (k < no && e0 < a.E) v = reset_value((uint32_t)k, e0, x_gen, x_k0, x_k1);
            part = __fmaf_rn(v, v, part);
            x0s[n0 * PX + k] = (uint16_t)bf16_bits(v);
            if (ENVF) reinterpret_cast<float*>(lds + V::OFF_X0F)[n0 * PXF + k] = v;
            if (NORM) x0ps[n0 * PX + k] = (uint16_t)bf16_bits((v - mus[k]) * ivs[k]);
          }
          float* scratch = reinterpret_cast<float*>(lds + V::OFF_SCR);   // KG x NC partial norms
          scratch[kq * NC + n0] = part;
          __syncthreads();
          if (tid < NC) {
            float s = 0.0f;
            for (int r = 0; r < KG; ++r) s += scratch[r * NC + tid];
            ss0s[tid] = s;
          }
          x0_block = (int)cb;
          __syncthreads();
        }
        {
          // copy the cached initial state into the working buffer; no column has ended
          const uint32_t* src = reinterpret_cast<const uint32_t*>(x0s);
          uint32_t* dst = reinterpret_cast<uint32_t*>(lds + V::OFF_X);
          for (int r = tid; r < NC * PX / 2; r += NT) dst[r] = src[r];
          if (ENVF) {
            const float* srcf = reinterpret_cast<const float*>(lds + V::OFF_X0F);
            float* dstf = reinterpret_cast<float*>(lds + V::OFF_XF);
            for (int r = tid; r < NC * PXF; r += NT) dstf[r] = srcf[r];
          }
          if (NORM) {
            const uint32_t* srcp = reinterpret_cast<const uint32_t*>(x0ps);
            uint32_t* dstp = reinterpret_cast<uint32_t*>(lds + V::OFF_XP);
            for (int r = tid; r < NC * PX / 2; r += NT) dstp[r] = srcp[r];
          }
          if (tid < NW) flags[tid] = 0u;
        }
        __syncthreads();

        const uint32_t e = cb * (uint32_t)NC + (uint32_t)n;
        uint32_t alive_cols = (1u << min((uint32_t)NC, a.E - cb * (uint32_t)NC)) - 1u;      // columns still running, the same in all wavefronts
        bool add = false;        // the previous step counts for this lane's column
        float Rn = 0.0f;
        int32_t Ln = 0;
        const float inv_no = 1.0f / (float)no;
        constexpr int KA1 = ENVF ? 0 : (ME < 0 ? KT1 : (KT1 + 1) / 2);       // K tiles of A x done beside layer 1; the rest beside layer 2
        f32x4 av = f32x4{0.f, 0.f, 0.f, 0.f};     // binary32 environment: the action (rows 4g..4g+3 of column n), kept in registers

        f32x4 acc[MT_H], accE[MTE];
#pragma unroll
        for (int tt = 0; tt < MT_H; ++tt) acc[tt] = *reinterpret_cast<const f32x4*>(b1s + 16 * (w * MT_H + tt) + 4 * g);
        // Books of a step ride under the next step's layer-1 stream: every lane keeps its share of |s'|^2 and |a|^2 until then.
        // (the share of |s_0|^2: all of it in one lane of the first wavefront)
        float ssp = (w == 0 && lane < NC) ? ss0s[lane] : 0.0f;
        float part = 0.0f;
        float ss_cur = 0.0f;      // |s_{t-1}|^2 while step t starts; the reward of step t-1 is booked in step t
        // lanes that write a partial (one per column) write it to its place, the others to the scratch: no branch
        float* const ss_out = reinterpret_cast<float*>(lds + (lane < NC ? V::OFF_SSP + 4 * (lane * NW + w) : V::OFF_SCR + 4 * tid));
        // shares -> the wavefront's partial of |s_t|^2: while the layer-1 stream waits for its first tiles
        auto books_norm = [&] { *ss_out = rows_sum(ssp); };
        // the reward of step t - 1: between the instructions of the stream's second stage
        auto books_reward = [&] {
          const float aa = rows_sum(part);
          const float r = __fmaf_rn(-ss_cur, inv_no, 1.0f) - a.act_cost * aa;
          Rn += add ? r : 0.0f;
#pragma unroll
          for (int k = 0; k < MT_H; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
          }
        };
        // every lane combines the four wavefronts' partials of |s_t|^2 of its column in the same fixed order
        auto norm_total = [&](f32x4 sp4) { ss_cur = (sp4.x + sp4.y) + (sp4.z + sp4.w); };
        // the columns that ended with step t - 1, by the flags of the four wavefronts
        auto flagged = [&](u32x4 fl) { return __builtin_amdgcn_readfirstlane((fl.x | fl.y) | (fl.z | fl.w)) & alive_cols; };
        uint32_t stop = 0u;      // the step before which to look whatever the flags say: the first one, then the end
        // (rare) these columns end with t steps, all of them after the last step
        auto end_columns = [&](uint32_t seen, uint32_t t) {
          const uint32_t ended = t == a.T ? alive_cols : seen;
          Ln = (ended >> n & 1u) ? (int32_t)t : Ln;
          alive_cols &= ~ended;
          add = (alive_cols >> n & 1u) != 0u;
          stop = a.T;
        };
        *ss_out = 0.0f;           // (wavefronts without next-state tiles write no partial)
        // some lanes' state is above the threshold (rare): their columns into this wavefront's flags
        auto flag_ended = [&](unsigned long long over) {
          if (__builtin_expect(over != 0ull, 0)) {
            uint32_t m = (uint32_t)(over | over >> 32);
            m |= m >> 16;
            if (lane == 0) flags[w] |= m;
          }
        };
        __syncthreads();

#ifdef ES_PHASE_PROF
        unsigned long long prof_acc[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        unsigned long long prof_last = __builtin_readcyclecounter();
#endif
        // After the last hidden layer: it stays in registers - the lane's values of tiles 0, 1 and of tiles 2, 3 are
        // the two K tiles of this wavefront's slice of the action layer - and only the binary32 partial sums cross the LDS
        auto last_hidden_ksplit = [&](const f32x4 (&accs)[MT_H]) {
          static_assert(MT_H == 4, "four hidden tiles per wavefront");
          if constexpr (!W3K_REGS) {      // requested ahead of the activation, which hides the latency
#pragma unroll
            for (int mt = 0; mt < MT3; ++mt)
#pragma unroll
              for (int kk = 0; kk < 2; ++kk) W3k[mt][kk] = w3k_tile(mt, kk);
          }
          u32x2 hp[MT_H];
#pragma unroll
          for (int tt = 0; tt < MT_H; ++tt) {
            const f32x4 h = hidden4<RELU, V::NEAR>(accs[tt]);
            hp[tt] = pack_bf16x4(h.x, h.y, h.z, h.w);
          }
          const bf16x8 bk0 = __builtin_bit_cast(bf16x8, u32x4{hp[0].x, hp[0].y, hp[1 % MT_H].x, hp[1 % MT_H].y});
          const bf16x8 bk1 = __builtin_bit_cast(bf16x8, u32x4{hp[2 % MT_H].x, hp[2 % MT_H].y, hp[3 % MT_H].x, hp[3 % MT_H].y});
          f32x4 p3[MT3];
#pragma unroll
          for (int mt = 0; mt < MT3; ++mt) p3[mt] = mfma16(W3k[mt][0], bk0, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
          for (int mt = 0; mt < MT3; ++mt) p3[mt] = mfma16(W3k[mt][1], bk1, p3[mt]);
#pragma unroll
          for (int mt = 0; mt < MT3; ++mt)
            *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(lds + V::OFF_P3) + (w * 16 + n) * V::PP3 + 16 * mt + 4 * g) = p3[mt];
        };
        // Two workgroups on a CU: the wavefronts of a SIMD compete for its issue slots, and left alone they fall into step, vector phase on vector
        // phase.  The short serial part of a step (sums of the partials, environment, first layer: few instructions and two hand-overs) goes before the
        // long ones, the first activation before the second layer's stream: whoever is late catches up, and the other's products and tanh fill
        // the gaps.  27-256-256-8, 1024 x 16 copies x 300 steps: 1.20 -> 1.08 ms, ReLU 0.91 -> 0.83 (of sixteen orders the streams first 1.16 to 1.22).
        auto prio = [](auto p) { if constexpr (ORDERED) __builtin_amdgcn_s_setprio(decltype(p)::value); };
        using P0 = std::integral_constant<int, 0>; using P1 = std::integral_constant<int, 1>; using P2 = std::integral_constant<int, 2>; using P3 = std::integral_constant<int, 3>;
        for (uint32_t t = 0; t <= a.T; ++t) {
          prio(P2{});
          // ---- phase A: h1 = tanh(W1 x + b1); first half of A x; books of the previous step ----
          float xf[ENVF ? KPL : 1];                 // binary32 environment: this lane's state operands, elements KPL g .. of column n
          if constexpr (ENVF) {
#pragma unroll
            for (int j = 0; j < KPL / 4; ++j) {
              const f32x4 v4 = *reinterpret_cast<const f32x4*>(lds + V::OFF_XF + 4 * (n * PXF + KPL * g + 4 * j));
              xf[4 * j] = v4.x; xf[4 * j + 1] = v4.y; xf[4 * j + 2] = v4.z; xf[4 * j + 3] = v4.w;
            }
          }
          // W1 stream: the B operand (state tiles) runs two stages ahead of the MFMAs
          bf16x8 bx[KA1 > 0 ? KA1 : 1], bxr[3];     // tiles < KA1 are kept for A x below; the rest pass through a ring
          auto xload = [&](int kt) { return lds_tile(lds, V::OFF_X + 2 * (n * PX + 32 * kt + 8 * g)); };
          // with observation statistics the policy reads the normalised state and A x the raw one
          auto xfetch = [&](int kt) {
            if (NORM) {
              bxr[kt % 3] = lds_tile(lds, V::OFF_XP + 2 * (n * PX + 32 * kt + 8 * g));
              if (kt < KA1) bx[kt < KA1 ? kt : 0] = xload(kt);
            } else if (kt < KA1) {
              bx[kt < KA1 ? kt : 0] = xload(kt);
            } else {
              bxr[kt % 3] = xload(kt);
            }
          };
#pragma unroll
          for (int kt = 0; kt < 2 && kt < KT1; ++kt) xfetch(kt);
          u32x4 fl;
          if (KT1 == 1) fl = *reinterpret_cast<const u32x4*>(flags);
          uint32_t seen = 0u;
          __builtin_amdgcn_sched_barrier(0);
          if (env_wave) books_norm();
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int kt = 0; kt < KT1; ++kt) {
            if (kt + 2 < KT1) xfetch(kt + 2);
#pragma unroll
            for (int tt = 0; tt < MT_H; ++tt) {
              if (V::OCC == 1 && ME == 0) pin_agpr(W1r[tt][kt]);    // with two workgroups per CU, or deeper policies, the accumulation half belongs to the 256x256 layers
              acc[tt] = mfma16(W1r[tt][kt], (!NORM && kt < KA1) ? bx[kt < KA1 ? kt : 0] : bxr[kt % 3], acc[tt]);
            }
            if (KT1 > 1 && kt == 0) fl = *reinterpret_cast<const u32x4*>(flags);
            if (kt == (KT1 > 1 ? 1 : 0)) books_reward();      // (of the returns only the first wavefront's are read)
            if (kt == (KT1 > 2 ? 2 : KT1 - 1)) seen = flagged(fl);
            __builtin_amdgcn_sched_barrier(0);
          }
          PSTAMP(0);
          prio(P1{});
          if (__builtin_expect((seen | ((t ^ stop) - 1u) >> 31) != 0u, 0)) {      // (t == stop, in scalar arithmetic) identical in all four wavefronts
            end_columns(seen, t);
            if (alive_cols == 0u) break;
          }
          PSTAMP(1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int tt = 0; tt < MTE; ++tt) accE[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
          // first half of A x (register tiles first) interleaved with the layer-1 epilogue
#pragma unroll
          for (int kt = 0; kt < KA1; ++kt) {
#pragma unroll
            for (int tt = 0; tt < MTE; ++tt)
              if (ENV_ALL || 16 * (w * MTE + tt) < V::NOP) {
                if (kt < KTAR) accE[tt] = mfma16(Ar[tt][kt], bx[kt], accE[tt]);
                else accE[tt] = mfma16(lds_tile(lds, V::OFF_AL + 2 * ((16 * (w * MTE + tt) + n) * PAL + 32 * (kt - KTAR) + 8 * g)), bx[kt], accE[tt]);
              }
          }
          if constexpr (ENVF) {          // A s in binary32, under the layer-1 epilogue like the bf16 tiles above
#pragma unroll
            for (int kk = 0; kk < KPL; ++kk)
#pragma unroll
              for (int tt = 0; tt < MTE; ++tt)
                if (ENV_ALL || 16 * (w * MTE + tt) < V::NOP) accE[tt] = mfma4(Af[tt][kk], xf[kk], accE[tt]);
          }
          if constexpr (ME < 0) {
            last_hidden_ksplit(acc);
          } else {
#pragma unroll
            for (int tt = 0; tt < MT_H; ++tt) {
              const f32x4 h = hidden4<RELU, V::NEAR>(acc[tt]);
              *reinterpret_cast<u32x2*>(lds + V::OFF_H1 + 2 * (n * PH + 16 * (w * MT_H + tt) + 4 * g)) = pack_bf16x4(h.x, h.y, h.z, h.w);
            }
          }
#pragma unroll
          for (int r = 0; r < (ENVF ? KPL * MTE : KA1 * MTE); ++r) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
          }
          // ---- phase B: h2 = tanh(W2 h1 + b2); second half of A x ----
          PSTAMP(2);
          if constexpr (ME >= 0) {
#pragma unroll
            for (int tt = 0; tt < MT_H; ++tt) acc[tt] = *reinterpret_cast<const f32x4*>(b2s + 16 * (w * MT_H + tt) + 4 * g);
            __syncthreads();
            PSTAMP(3);
            constexpr int NT2 = ENVF ? 0 : (KT1 - KA1) * MTE;      // MFMAs of the second half of A x; j = (kt - KA1) * MTE + tt
            constexpr int PS = (NT2 + KT_H - 1) / KT_H; // ... of which this many ride in each stage of the W2 stream
            bf16x8 bh[3], at[3 * (PS > 0 ? PS : 1)], bx2[KT1 - KA1 > 0 ? KT1 - KA1 : 1];
            // operands of stage kt are fetched two stages ahead: h1 tile, LDS-resident A tiles, state tiles
            auto fetch = [&](int kt) {
              bh[kt % 3] = lds_tile(lds, V::OFF_H1 + 2 * (n * PH + 32 * kt + 8 * g));
#pragma unroll
              for (int r = 0; r < PS; ++r) {
                const int j = kt * PS + r;
                if (j < NT2) {
                  const int ka = KA1 + j / MTE, tt = j % MTE;
                  if (ka >= KTAR) at[(kt % 3) * PS + r] = lds_tile(lds, V::OFF_AL + 2 * ((16 * (w * MTE + tt) + n) * PAL + 32 * (ka - KTAR) + 8 * g));
                  if (tt == 0 || r == 0) bx2[ka - KA1] = lds_tile(lds, V::OFF_X + 2 * (n * PX + 32 * ka + 8 * g));
                }
              }
            };
            prio(P0{});
            fetch(0);
            fetch(1);
            const f32x4 sp4 = *reinterpret_cast<const f32x4*>(lds + V::OFF_SSP + 4 * NW * n);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kt = 0; kt < KT_H; ++kt) {
              if (kt + 2 < KT_H) fetch(kt + 2);
#pragma unroll
              for (int tt = 0; tt < MT_H; ++tt) { pin_agpr(W2r[tt][kt]); acc[tt] = mfma16(W2r[tt][kt], bh[kt % 3], acc[tt]); }
#pragma unroll
              for (int r = 0; r < PS; ++r) {
                const int j = kt * PS + r;
                if (j < NT2) {
                  const int ka = KA1 + j / MTE, tt = j % MTE;
                  if (ENV_ALL || 16 * (w * MTE + tt) < V::NOP) {
                    if (ka < KTAR) accE[tt] = mfma16(Ar[tt][ka < KTAR ? ka : 0], bx2[ka - KA1], accE[tt]);
                    else accE[tt] = mfma16(at[(kt % 3) * PS + r], bx2[ka - KA1], accE[tt]);
                  }
                }
              }
              if (kt == 2) norm_total(sp4);
              __builtin_amdgcn_sched_barrier(0);
            }
            PSTAMP(4);
            if constexpr (ME == 0) {
              last_hidden_ksplit(acc);
            } else {
#pragma unroll
              for (int tt = 0; tt < MT_H; ++tt) {
                const f32x4 h = hidden4<RELU, V::NEAR>(acc[tt]);
                *reinterpret_cast<u32x2*>(lds + V::OFF_H2 + 2 * (n * PH + 16 * (w * MT_H + tt) + 4 * g)) = pack_bf16x4(h.x, h.y, h.z, h.w);
              }
            }
          }
          // ---- further hidden layers (depth m > 2): the same stream, ping-ponging between the two buffers ----
          auto deeper = [&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const int off_in = (j & 1) ? V::OFF_H1 : V::OFF_H2, off_out = (j & 1) ? V::OFF_H2 : V::OFF_H1;
#pragma unroll
            for (int tt = 0; tt < MT_H; ++tt) acc[tt] = *reinterpret_cast<const f32x4*>(bxs + j * NHP + 16 * (w * MT_H + tt) + 4 * g);
            __syncthreads();
            bf16x8 bh[3];
            bh[0] = lds_tile(lds, off_in + 2 * (n * PH + 8 * g));
            bh[1] = lds_tile(lds, off_in + 2 * (n * PH + 32 + 8 * g));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kt = 0; kt < KT_H; ++kt) {
              if (kt + 2 < KT_H) bh[(kt + 2) % 3] = lds_tile(lds, off_in + 2 * (n * PH + 32 * (kt + 2) + 8 * g));
#pragma unroll
              for (int tt = 0; tt < MT_H; ++tt) {
                if (j == 0) pin_agpr(Wxr[j][tt][kt]);      // the first extra layer shares the accumulation half with layer 2
                acc[tt] = mfma16(Wxr[j][tt][kt], bh[kt % 3], acc[tt]);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (j == ME - 1) {
              last_hidden_ksplit(acc);
            } else {
#pragma unroll
              for (int tt = 0; tt < MT_H; ++tt) {
                const f32x4 h = hidden4<RELU, V::NEAR>(acc[tt]);
                *reinterpret_cast<u32x2*>(lds + off_out + 2 * (n * PH + 16 * (w * MT_H + tt) + 4 * g)) = pack_bf16x4(h.x, h.y, h.z, h.w);
              }
            }
          };
          if constexpr (ME > 0) deeper(std::integral_constant<int, 0>());
          if constexpr (ME > 1) deeper(std::integral_constant<int, 1>());
          PSTAMP(5);
          __syncthreads();
          PSTAMP(6);
          prio(P3{});
          if constexpr (ME < 0) norm_total(*reinterpret_cast<const f32x4*>(lds + V::OFF_SSP + 4 * NW * n));
          if (env_wave) {          // the others have no next-state tile
          // ---- phase C: a = tanh(sum of the partials + b3) ----
          bf16x8 ba16;             // the action as a B operand, from registers
          {
            // every lane adds the four wavefronts' partials of rows 4g..4g+3 (of every action tile) of its column, in the same order everywhere
            const float* p3s = reinterpret_cast<const float*>(lds + V::OFF_P3);
            f32x4 v[MT3], pv[MT3][NW];
            part = 0.0f;
#pragma unroll
            for (int mt = 0; mt < MT3; ++mt) {
              v[mt] = *reinterpret_cast<const f32x4*>(b3s + 16 * mt + 4 * g);
#pragma unroll
              for (int ww = 0; ww < NW; ++ww) pv[mt][ww] = *reinterpret_cast<const f32x4*>(p3s + (ww * 16 + n) * V::PP3 + 16 * mt + 4 * g);
            }
            if constexpr (V::B_LDS) {
#pragma unroll
              for (int tt = 0; tt < MTE; ++tt) Br[tt][0] = b_slots(lds + V::OFF_BL + 2 * ((16 * (w * MTE + tt) + n) * V::PA + 4 * g));
            }
            __builtin_amdgcn_sched_barrier(0);      // (all the reads before the first sum, or each would be waited for on its own)
#pragma unroll
            for (int mt = 0; mt < MT3; ++mt) {
#pragma unroll
              for (int ww = 0; ww < NW; ++ww) v[mt] += pv[mt][ww];
              {
                const f32x4 tv = tanh4<V::NEAR>(v[mt]);
                const bool squash = a.out_tanh != 0u;
                v[mt] = f32x4{squash ? tv.x : v[mt].x, squash ? tv.y : v[mt].y, squash ? tv.z : v[mt].z, squash ? tv.w : v[mt].w};
              }
              part = __fmaf_rn(v[mt].x, v[mt].x, part); part = __fmaf_rn(v[mt].y, v[mt].y, part);
              part = __fmaf_rn(v[mt].z, v[mt].z, part); part = __fmaf_rn(v[mt].w, v[mt].w, part);
            }
            if (ENVF) av = v[0];
            else {
              const u32x2 lo = pack_bf16x4(v[0].x, v[0].y, v[0].z, v[0].w);
              u32x2 hi = u32x2{0u, 0u};
              if (MT3 > 1) hi = pack_bf16x4(v[MT3 - 1].x, v[MT3 - 1].y, v[MT3 - 1].z, v[MT3 - 1].w);
              ba16 = __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
            }
          }
          // ---- phase D: s' = tanh(A x + B a); this lane's share of the norm, the termination test ----
          if constexpr (ENVF) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
#pragma unroll
              for (int tt = 0; tt < MTE; ++tt)
                if (ENV_ALL || 16 * (w * MTE + tt) < V::NOP) accE[tt] = mfma4(Bf[tt][kk], av[kk], accE[tt]);
          } else {
#pragma unroll
            for (int tt = 0; tt < MTE; ++tt)
              if (ENV_ALL || 16 * (w * MTE + tt) < V::NOP) accE[tt] = mfma16(Br[tt][0], ba16, accE[tt]);
          }
          ssp = 0.0f;
          unsigned long long over = 0ull;
#pragma unroll
          for (int tt = 0; tt < MTE; ++tt) {
            if (ENV_ALL || 16 * (w * MTE + tt) < V::NOP) {
              const f32x4 sn = tanh4<V::NEAR>(accE[tt]);
              ssp = __fmaf_rn(sn.x, sn.x, ssp); ssp = __fmaf_rn(sn.y, sn.y, ssp);
              ssp = __fmaf_rn(sn.z, sn.z, ssp); ssp = __fmaf_rn(sn.w, sn.w, ssp);
              over |= exceeds(sn, a.done_thresh);
              *reinterpret_cast<u32x2*>(lds + V::OFF_X + 2 * (n * PX + 16 * (w * MTE + tt) + 4 * g)) = pack_bf16x4(sn.x, sn.y, sn.z, sn.w);
              if (ENVF) *reinterpret_cast<f32x4*>(lds + V::OFF_XF + 4 * (n * PXF + 16 * (w * MTE + tt) + 4 * g)) = sn;
              if (NORM) {
                const int r0 = 16 * (w * MTE + tt) + 4 * g;
                const f32x4 xn = (sn - *reinterpret_cast<const f32x4*>(mus + r0)) * *reinterpret_cast<const f32x4*>(ivs + r0);
                *reinterpret_cast<u32x2*>(lds + V::OFF_XP + 2 * (n * PX + r0)) = pack_bf16x4(xn.x, xn.y, xn.z, xn.w);
              }
            }
          }
          flag_ended(over);
          }
#pragma unroll
          for (int tt = 0; tt < MT_H; ++tt) acc[tt] = *reinterpret_cast<const f32x4*>(b1s + 16 * (w * MT_H + tt) + 4 * g);
          PSTAMP(9);
          __syncthreads();
          PSTAMP(10);
        }
#ifdef ES_PHASE_PROF
        if (blockIdx.x == 0 && lane == 0 && a.prof)
          for (int k = 0; k < 12; ++k) a.prof[w * 16 + k] += prof_acc[k];
#endif
        __syncthreads();   // all reads of the rollout buffers are done before anything is restaged

        // ---------------- outputs of this block of environment copies ----------------
        if (w == 0) {
          const uint32_t cnt = min((uint32_t)NC, a.E - cb * (uint32_t)NC);
          if (g == 0 && (uint32_t)n < cnt) {
            KARG(returns)[(size_t)i * a.E + e] = Rn;
            KARG(ep_len)[(size_t)i * a.E + e] = Ln;
          }
          for (uint32_t r = 0; r < cnt; ++r) fit_sum += __shfl(Rn, (int)r, 64);
        }
      }
      if (w == 0 && lane == 0) KARG(fitness)[i] = fit_sum / (float)a.E;
    }
  }
}

constexpr int env_tiles(int nop, int nw) { return (nop / 16 + nw - 1) / nw > 0 ? (nop / 16 + nw - 1) / nw : 1; }
// The smallest-observation variant leaves half of the register file free: two workgroups (two
// individuals) share a CU and hide each other's LDS round trips and barriers (1.5x at obs 27).
// (Passes of sixteen copies: A stays in LDS - with two workgroups per CU the register file has no four registers to spare
// for its tile, and a spilled tile would be reloaded from scratch memory every step.)
template <int NW> using V32 = Variant<1, 1, env_tiles(32, NW), 0, NW, 2>;   // obs <= 32,  act <= 16
template <int NW> using V64 = Variant<2, 1, env_tiles(64, NW), 2, NW>;      // obs <= 64,  act <= 16
// the same two shapes with the environment's products in binary32 (es_config.env_dtype = 1)
template <int NW> using V32F = Variant<1, 1, env_tiles(32, NW), 1, NW, 2, 0, true>;
template <int NW> using V64F = Variant<2, 1, env_tiles(64, NW), 2, NW, 1, 0, true>;
template <int NW> using V128 = Variant<4, 2, env_tiles(128, NW), 4, NW>;    // obs <= 128, act <= 32
// Deeper policies (m = 3, 4 hidden layers) of the two narrow-observation shapes: one workgroup per CU, the
// extra 256 x 256 layers take the registers the second workgroup would have used.
// (fewer than 128 units: tanh_near, as in rollout_quad_bf16_mid.hip; 27 random shapes, three and four layers: rms error 2.2e-5 on
// the LDS kernel, 3.3e-5 with tanh_fast, 2.1e-5 with tanh_near, which costs 8 %)
template <int NW, int ME, bool NEAR> using V32D = Variant<1, 1, env_tiles(32, NW), 1, NW, 1, ME, false, NEAR>;
template <int NW, int ME, bool NEAR> using V64D = Variant<2, 1, env_tiles(64, NW), 2, NW, 1, ME, false, NEAR>;
// A single hidden layer (m = 1) of the same two shapes: the second layer's phase and weights drop out.
template <int NW> using V32S = Variant<1, 1, env_tiles(32, NW), 1, NW, 2, -1>;
template <int NW> using V64S = Variant<2, 1, env_tiles(64, NW), 2, NW, 1, -1>;
// obs <= 256, act <= 32: four of the eight K tiles of the environment matrix A sit in registers, the rest in LDS
template <int NW> using V256 = Variant<8, 2, env_tiles(256, NW), 4, NW>;

struct VariantInfo { int max_obs, max_act; const char* name; };
static const VariantInfo kVariants[] = {
    {32, 16, "rollout_mfma_reg_bf16<obs32,hid256,act16>"},
    {64, 16, "rollout_mfma_reg_bf16<obs64,hid256,act16>"},
    {128, 32, "rollout_mfma_reg_bf16<obs128,hid256,act32>"},
    {256, 32, "rollout_mfma_reg_bf16<obs256,hid256,act32>"},
};

int mfma_variant_for(const es_config& c) {
  const uint32_t m = c.num_hidden ? c.num_hidden : 2;
  if (c.dtype != 1 || c.hid_dim > (uint32_t)NHP || m < 1 || m > 4) return -1;
  // a binary32 environment is built for the two narrow-observation shapes with two hidden layers
  if (c.env_dtype == 1 && (m != 2 || c.obs_dim > 64 || c.act_dim > 16)) return -1;
  // narrow policies of one or two layers are served better by the one-wavefront-per-episode kernel when it fits; three and four
  // layers of 65 to 127 units never are (obs 27, 512 individuals x 16 copies x 40 steps, here against the LDS kernel: three layers
  // of 65 / 96 / 127 units 0.28 / 0.23 / 0.30 against 5.3 / 13.3 / 25.2 ms, four layers 0.38 / 0.30 / 0.40 against 9.2 / 25.4 / 66.8 ms)
  if (c.hid_dim < 128 && (m <= 2 || c.hid_dim <= 64) && wave_rollout_lds_bytes(c) <= 160 * 1024) return -1;
  for (int v = 0; v < 4; ++v)
    if ((int)c.obs_dim <= kVariants[v].max_obs && (int)c.act_dim <= kVariants[v].max_act)
      return (m != 2 && v > 1) ? -1 : v;      // one, three and four hidden layers: the two narrow-observation shapes only
  return -1;
}

const char* mfma_variant_name(int v) { return (v >= 0 && v < 4) ? kVariants[v].name : "none"; }

template <class V, bool RELU, bool NORM, bool ORDERED = false>
static int launch_variant_act(es_ctx* ctx, const MfmaArgs& a, uint32_t units, hipStream_t st) {
  const void* fn = reinterpret_cast<const void*>(rollout_mfma_kernel<V, RELU, NORM, ORDERED>);
  hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, V::LDS_BYTES);
  if (err != hipSuccess) return fail(ctx, ES_EHIP, std::string("hipFuncSetAttribute: ") + hipGetErrorString(err));
  // persistent grid: as many workgroups as the chip holds at once (register- and LDS-limited)
  const int per_cu = std::min(V::OCC, std::max(1, ctx->lds_limit / V::LDS_BYTES));
  const uint32_t grid = std::min<uint32_t>(units, (uint32_t)(std::max(1, ctx->num_cus) * per_cu));
  // Two workgroups per CU: priorities by phase.  They make the two equally fast, which is wrong where the last round leaves one of them an
  // individual more (a remainder of up to half the grid): without them the older one, which has it, is ahead anyway.  27-256-256-8 x 16 copies x 60
  // steps, without / with: 512 individuals 156 / 144 us, 600 220 / 233, 768 222 / 234, 800 277 / 254, 1200 328 / 355, 1600 446 / 474, 2048 552 / 504.
  if constexpr (V::OCC == 2 && !ORDERED) {
    const uint32_t rest = units % grid;
    if (per_cu == 2 && (rest == 0u || 2u * rest > grid)) return launch_variant_act<V, RELU, NORM, true>(ctx, a, units, st);
  }
  hipLaunchKernelGGL((rollout_mfma_kernel<V, RELU, NORM, ORDERED>), dim3(grid), dim3(V::NT), V::LDS_BYTES, st, a);
  return check_launch(ctx, "es_rollout (MFMA)");
}
template <class V>
static int launch_variant(es_ctx* ctx, const MfmaArgs& a, uint32_t units, hipStream_t st) {
  const bool relu = ctx->cfg.hidden_act == 1, norm = ctx->obs_mean != nullptr;
  if (relu) return norm ? launch_variant_act<V, true, true>(ctx, a, units, st) : launch_variant_act<V, true, false>(ctx, a, units, st);
  return norm ? launch_variant_act<V, false, true>(ctx, a, units, st) : launch_variant_act<V, false, false>(ctx, a, units, st);
}

int launch_rollout_mfma(es_ctx* ctx, uint32_t gen, const float* theta, const void* noise, const float* A,
                        const float* B, float* returns, int32_t* ep_len, float* fitness, void* ws,
                        hipStream_t st) {
  const Shape& s = ctx->shp;
  const es_config& c = ctx->cfg;
  MfmaArgs a;
  const NoiseView nv = noise_view(ctx, noise);
  a.theta = theta; a.noise = nv.base; a.noise_offs = nv.offs; a.A = A; a.B = B; a.obs_mean = ctx->obs_mean; a.obs_inv = ctx->obs_inv_std; a.returns = returns; a.ep_len = ep_len; a.fitness = fitness;
  a.N = s.N; a.E = s.E; a.T = s.T; a.no = s.no; a.nh = s.nh; a.na = s.na; a.ld = s.ld;
  a.oW1 = s.oW1; a.ob1 = s.ob1; a.oW2 = s.oW2; a.ob2 = s.ob2; a.oW3 = s.oW3; a.ob3 = s.ob3;
  a.gen = gen; a.k0 = (uint32_t)c.seed; a.k1 = (uint32_t)(c.seed >> 32);
  a.antithetic = c.antithetic; a.out_tanh = c.out_tanh; a.noise_mode = nv.mode;
  a.sigma = c.sigma; a.done_thresh = c.done_thresh; a.act_cost = c.act_cost;
  a.prof = static_cast<unsigned long long*>(ws);
  if ((int)V256<4>::LDS_BYTES > ctx->lds_limit)
    return fail(ctx, ES_EUNSUPPORTED, "es_rollout: this device's LDS is too small for the register-resident kernel");
  const uint32_t units = s.N;      // one work item per individual
#ifdef ES_DEV_FAST   // tuning builds only: one variant, seconds to compile
  if (c.env_dtype == 1 && ctx->mfma_variant == 0 && ctx->cfg.hidden_act == 0 && !ctx->obs_mean)
    return launch_variant_act<V32F<4>, false, false>(ctx, a, units, st);
  if (ctx->mfma_variant == 0 && s.m == 2 && ctx->cfg.hidden_act == 0 && !ctx->obs_mean)
    return launch_variant_act<V32<4>, false, false>(ctx, a, units, st);
  return fail(ctx, ES_EUNSUPPORTED, "tuning build: variant not compiled");
#else
  if (c.env_dtype == 1) {          // binary32 environment: passes of 16 copies whatever E is
    if (ctx->mfma_variant == 0) return launch_variant<V32F<4>>(ctx, a, units, st);
    if (ctx->mfma_variant == 1) return launch_variant<V64F<4>>(ctx, a, units, st);
    return fail(ctx, ES_EUNSUPPORTED, "es_rollout: no register-resident variant with a binary32 environment for this shape");
  }
  // (up to four copies, and passes of four that fit the chip at once: rollout_quad.hip)
  if (s.m == 1) {
    if (ctx->mfma_variant == 0) return launch_variant<V32S<4>>(ctx, a, units, st);
    if (ctx->mfma_variant == 1) return launch_variant<V64S<4>>(ctx, a, units, st);
  } else if (s.m == 3) {
    if (ctx->mfma_variant == 0) return s.nh < 128 ? launch_variant<V32D<4, 1, true>>(ctx, a, units, st) : launch_variant<V32D<4, 1, false>>(ctx, a, units, st);
    if (ctx->mfma_variant == 1) return s.nh < 128 ? launch_variant<V64D<4, 1, true>>(ctx, a, units, st) : launch_variant<V64D<4, 1, false>>(ctx, a, units, st);
  } else if (s.m == 4) {
    if (ctx->mfma_variant == 0) return s.nh < 128 ? launch_variant<V32D<4, 2, true>>(ctx, a, units, st) : launch_variant<V32D<4, 2, false>>(ctx, a, units, st);
    if (ctx->mfma_variant == 1) return s.nh < 128 ? launch_variant<V64D<4, 2, true>>(ctx, a, units, st) : launch_variant<V64D<4, 2, false>>(ctx, a, units, st);
  }
  if (s.m != 2) return fail(ctx, ES_EUNSUPPORTED, "es_rollout: no register-resident variant for this depth");
  switch (ctx->mfma_variant) {
    case 0: return launch_variant<V32<4>>(ctx, a, units, st);
    case 1: return launch_variant<V64<4>>(ctx, a, units, st);
    case 2: return launch_variant<V128<4>>(ctx, a, units, st);
    case 3: return launch_variant<V256<4>>(ctx, a, units, st);
    default: return fail(ctx, ES_EUNSUPPORTED, "es_rollout: no register-resident variant for this shape");
  }
#endif
}

}  // namespace es
