// Device-side building blocks for the gfx950 kernels: counter-based random words, the
// binary32 Gaussian transform, bf16 packing, tanh and wavefront reductions.
//
// The whole library is compiled with floating-point contraction off; every fused
// multiply-add below is explicit, so the bit-defined sequences (Gaussian transform,
// perturbation, reset) round exactly as written.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace es {

struct Words4 { uint32_t x, y, z, w; };

// Philox4x32 with 10 rounds (Salmon et al., SC'11).  Counter (c0..c3), key (k0,k1).
__device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;      // one 32x32->64 multiply each
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi1, c1, k0, 0x96);      // three-way exclusive or, one instruction
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi0, c3, k1, 0x96);
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return Words4{c0, c1, c2, c3};
}

// Two 32-bit words -> two standard normal variates (cosine branch, sine branch).
// Box-Muller with u1 = k1 2^-24, k1 = (xa >> 8) + 1, angle = 2 pi (xb >> 8) 2^-24.
//   -ln u1 = n ln 2 - ln m with u1 = m 2^-n, m in (sqrt(1/2), sqrt(2)],
//   ln m = 2 atanh(s), s = (m - 1)/(m + 1), odd series through s^11;
//   sine / cosine by Taylor polynomials on [0, pi/4] and octant symmetry.
// The values are DEFINED with a correctly rounded division and square root, so that any conforming machine
// reproduces them bit for bit.  The arguments here lie in a narrow range (m + 1 in (1.7, 2.42], 2 (-ln u1) in
// [0, 33.3]), so the general sequences - scaling, special values, a second Newton step: half of the transform -
// are not needed: one reciprocal (or reciprocal square root) and one multiply-add of the residual (P. W. Markstein,
// IBM J. Res. Dev. 34 (1990), pp. 111-119) round the same.  There are only 2^24 radii and 2^24 angles: tests/test_gpu_gauss.py
// compares all of them with the general sequences.
// Three more exact savings: m and n come out of one biased integer add; 4 ln m is carried scaled (num and the
// coefficients hold powers of two), so that 2 (-ln u1) needs no doubling; the octant's signs are bits of xb
// inserted into the products.  About 50 vector instructions per pair, 94 with the general sequences.
__device__ __forceinline__ void gauss_pair(uint32_t xa, uint32_t xb, float& zc, float& zs) {
  // bits of k1 as a float, offset so that the exponent steps at sqrt(2) instead of at 2
  const uint32_t ix = __float_as_uint((float)((xa >> 8) + 1u)) + 0x004AFB0Cu;
  const float n = (float)(int)(151u - (ix >> 23));
  const float m = __uint_as_float((ix & 0x007FFFFFu) + 0x3F3504F4u);
  const float num = __fmaf_rn(m, 4.0f, -4.0f), den = m + 1.0f;
  const float rc = __builtin_amdgcn_rcpf(den);
  const float q = num * rc;
  const float s = __fmaf_rn(__fmaf_rn(-den, q, num), rc, q);      // 4 (m - 1)/(m + 1)
  const float t = s * s;
  float p = 0x1.745d18p-24f;                   // 1/11 2^-20
  p = __fmaf_rn(t, p, 0x1.c71c72p-20f);        // 1/9  2^-16
  p = __fmaf_rn(t, p, 0x1.24924ap-15f);        // 1/7  2^-12
  p = __fmaf_rn(t, p, 0x1.99999ap-11f);        // 1/5  2^-8
  p = __fmaf_rn(t, p, 0x1.555556p-6f);         // 1/3  2^-4
  p = __fmaf_rn(t, p, 1.0f);
  const float x2 = __fmaf_rn(n, 2.0f * 0.693147182f, -(s * p));   // 2 (-ln u1)
  const float rs = __builtin_amdgcn_rsqf(fmaxf(x2, 1e-30f));      // u1 = 1 gives a radius of zero
  const float g = x2 * rs;
  const float rad = __fmaf_rn(__fmaf_rn(-g, g, x2), 0.5f * rs, g);

  // distance to the nearer end of the quadrant, in units of 2 pi 2^-24; the octant decides which of the two
  // series is the cosine and the signs: octant -> (cos, sin):
  // 0 (c,s) 1 (s,c) 2 (-s,c) 3 (-c,s) 4 (-c,-s) 5 (-s,-c) 6 (s,-c) 7 (c,-s)
  const uint32_t w = (xb >> 8) & 0x3FFFFFu, u = 0x400000u - w;
  const float x = (float)(w < u ? w : u) * (0.785398185f * 0x1p-21f);
  const float y = x * x;
  float sp = 0x1.71de3ap-19f;                  //  1/362880
  sp = __fmaf_rn(y, sp, -0x1.a01a02p-13f);     // -1/5040
  sp = __fmaf_rn(y, sp, 0x1.111112p-7f);       //  1/120
  sp = __fmaf_rn(y, sp, -0x1.555556p-3f);      // -1/6
  sp = __fmaf_rn(y, sp, 1.0f);
  sp = x * sp;
  float cp = -0x1.27e4fcp-22f;                 // -1/3628800
  cp = __fmaf_rn(y, cp, 0x1.a01a02p-16f);      //  1/40320
  cp = __fmaf_rn(y, cp, -0x1.6c16c2p-10f);     // -1/720
  cp = __fmaf_rn(y, cp, 0x1.555556p-5f);       //  1/24
  cp = __fmaf_rn(y, cp, -0.5f);
  cp = __fmaf_rn(y, cp, 1.0f);
  const uint32_t v = xb ^ (xb << 1);           // bit 31: sign of the cosine; bit 30: octants 1, 2, 5, 6
  const bool swap = (v & 0x40000000u) != 0u;
  const float c = swap ? sp : cp, sn = swap ? cp : sp;
  zc = __uint_as_float((__float_as_uint(rad * c) & 0x7FFFFFFFu) | (v & 0x80000000u));
  zs = __uint_as_float((__float_as_uint(rad * sn) & 0x7FFFFFFFu) | (xb & 0x80000000u));
}

// binary32 -> bf16 bit pattern, round to nearest even (finite inputs).
__device__ __forceinline__ uint32_t bf16_bits(float x) {
  uint32_t b = __float_as_uint(x);
  b += 0x7FFFu + ((b >> 16) & 1u);
  return b >> 16;
}
__device__ __forceinline__ float bf16_round(float x) { return __uint_as_float(bf16_bits(x) << 16); }
__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// Noise values recomputed from the counter stream instead of being read back (paper Sec. 5.1:
// perturbations generated on the fly; nothing is stored when the caller asks for that).
// Columns d0..d0+3 (d0 a multiple of 4) of noise row `row`: one Philox block, two transforms.
// `round` reproduces the value a bf16-stored matrix would hold.
__device__ __forceinline__ void noise_regen4(uint32_t row, uint32_t d0, uint32_t gen, uint32_t k0, uint32_t k1,
                                             bool round, float (&z)[4]) {
  const Words4 w = philox4x32_10(d0 >> 2, row, gen, 1u, k0, k1);     // stream 1 = noise
  gauss_pair(w.x, w.y, z[0], z[1]);
  gauss_pair(w.z, w.w, z[2], z[3]);
  if (round) {
#pragma unroll
    for (int k = 0; k < 4; ++k) z[k] = bf16_round(z[k]);
  }
}
// A single column (one transform; used where a thread's columns are not aligned groups of four).
__device__ __forceinline__ float noise_regen1(uint32_t row, uint32_t d, uint32_t gen, uint32_t k0, uint32_t k1, bool round) {
  const Words4 w = philox4x32_10(d >> 2, row, gen, 1u, k0, k1);
  const uint32_t xa = (d & 2u) ? w.z : w.x, xb = (d & 2u) ? w.w : w.y;
  float za, zb;
  gauss_pair(xa, xb, za, zb);
  const float z = (d & 1u) ? zb : za;
  return round ? bf16_round(z) : z;
}
// Noise element (row, d) under any of the four storage modes of es_config.noise_dtype.
__device__ __forceinline__ float noise_value(uint32_t mode, const void* base, uint32_t ld, uint32_t row, uint32_t d,
                                             uint32_t gen, uint32_t k0, uint32_t k1) {
  if (mode >= 2u) return noise_regen1(row, d, gen, k0, k1, mode == 3u);
  if (mode == 1u) return bf16_to_f32(static_cast<const uint16_t*>(base)[(size_t)row * ld + d]);
  return static_cast<const float*>(base)[(size_t)row * ld + d];
}

// With a shared noise table, row `row` starts at base + offs[row] elements; returns that row's base
// (to be indexed as row 0) for the stored element type of `mode` (0 binary32, 1 bf16).
__device__ __forceinline__ const void* table_row_base(uint32_t mode, const void* base, const uint32_t* offs, uint32_t row) {
  const uint32_t o = offs[row];
  return mode == 1u ? static_cast<const void*>(static_cast<const uint16_t*>(base) + o)
                    : static_cast<const void*>(static_cast<const float*>(base) + o);
}

// Initial state element k of environment copy e: uniform on [-0.1, 0.1).
__device__ __forceinline__ float reset_value(uint32_t k, uint32_t e, uint32_t gen, uint32_t k0, uint32_t k1) {
  const Words4 w = philox4x32_10(k >> 2, e, gen, 2u, k0, k1);
  const uint32_t q = k & 3u;
  const uint32_t word = q == 0 ? w.x : q == 1 ? w.y : q == 2 ? w.z : w.w;
  const float u = (float)(word >> 8) * 0x1p-24f;
  return __fmaf_rn(u, 0.2f, -0.1f);
}

// tanh with absolute error of a few 1e-7: odd series near zero, 1 - 2/(e^{2|x|} + 1) elsewhere.
__device__ __forceinline__ float tanh_accurate(float x) {
  const float ax = fabsf(x);
  const float x2 = x * x;
  float p = -0x1.226e36p-7f;                   // -1382/155925
  p = __fmaf_rn(x2, p, 0x1.664f48p-6f);        //  62/2835
  p = __fmaf_rn(x2, p, -0x1.ba1ba2p-5f);       // -17/315
  p = __fmaf_rn(x2, p, 0x1.111112p-3f);        //  2/15
  p = __fmaf_rn(x2, p, -0x1.555556p-2f);       // -1/3
  const float small = __fmaf_rn(x * x2, p, x);
  const float ex = __expf(ax + ax);
  const float big = copysignf(1.0f - __fdividef(2.0f, ex + 1.0f), x);
  return ax < 0.3f ? small : big;
}

// tanh as 1 - 2/(2^{c x} + 1), two transcendental issues: absolute error ~1e-7 everywhere (relative
// ~1e-6 for |x| > 1e-2; near zero the result has the absolute accuracy of 1 - (1 - 2x), which is
// what the sums it feeds need).  Used by the register-resident kernels, binary32 and bf16.
__device__ __forceinline__ float tanh_fast(float x) {
  const float ex = __builtin_amdgcn_exp2f(x * 2.88539008f);     // 2 log2(e)
  const float r = __builtin_amdgcn_rcpf(ex + 1.0f);
  return __fmaf_rn(-2.0f, r, 1.0f);
}

// tanh(x) from t = c x, c = 2 log2(e), as (1 - u) / (1 + u) with u = 2^-|t|: two instructions more than tanh_fast, but the
// numerator is exact near zero, so the absolute error stays below ~4e-8 there.  A bf16 operand of size 0.05 has neighbours 2e-4
// apart, and tanh_fast's 1.2e-7 takes one in a thousand to the wrong one.  For the bf16 kernels of shapes that are otherwise
// evaluated with tanh_accurate.
__device__ __forceinline__ float tanh_near(float t) {
  const float u = __builtin_amdgcn_exp2f(-fabsf(t));
  return __builtin_copysignf((1.0f - u) * __builtin_amdgcn_rcpf(1.0f + u), t);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

}  // namespace es
