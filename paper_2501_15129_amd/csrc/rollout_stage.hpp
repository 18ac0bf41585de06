// Staging shared by the register-resident rollout kernels: one individual's perturbed parameters
// (theta + sign * sigma * eps, one binary32 rounding, then bf16 where the kernel's operands are) written into an LDS
// window in coalesced order, from which every lane picks the weights it keeps in registers.
#pragma once

#include "es_device.hpp"

namespace es {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Staging iterations whose loads are in flight together (at 244-256-256-17 4 is 24 % slower, 16 spills; QuadShape::BATCH).
constexpr int STAGE_BATCH = 8;

// Four binary32 values -> four bf16 (round to nearest even), by the packed hardware convert.
__device__ __forceinline__ u32x2 pack_bf16x4(float a, float b, float c, float d) {
  u32x2 r;
  r.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
  r.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{c, d}, bf16x2));
  return r;
}

// One noise row under any storage mode: a pointer to the stored row, or the counters to recompute it.
struct NoiseRow {
  const void* ptr;
  uint32_t mode, row, gen, k0, k1;
};
__device__ __forceinline__ float row_noise(const NoiseRow& nz, uint32_t idx) {
  if (nz.mode >= 2u) return noise_regen1(nz.row, idx, nz.gen, nz.k0, nz.k1, nz.mode == 3u);
  return nz.mode == 1u ? bf16_to_f32(static_cast<const uint16_t*>(nz.ptr)[idx]) : static_cast<const float*>(nz.ptr)[idx];
}

// Stored noise values as binary32: binary32 as they are, bf16 widened (an int stands for "no noise").
__device__ __forceinline__ f32x4 widen4(f32x4 e) { return e; }
__device__ __forceinline__ f32x4 widen4(u32x2 raw) {
  return f32x4{__uint_as_float(raw.x << 16), __uint_as_float(raw.x & 0xFFFF0000u),
               __uint_as_float(raw.y << 16), __uint_as_float(raw.y & 0xFFFF0000u)};
}
__device__ __forceinline__ f32x4 widen4(int) { return f32x4{0.f, 0.f, 0.f, 0.f}; }
__device__ __forceinline__ float widen1(float e) { return e; }
__device__ __forceinline__ float widen1(uint16_t e) { return bf16_to_f32(e); }
__device__ __forceinline__ float widen1(int) { return 0.f; }

// Window elements: bf16 bit patterns or binary32.
__device__ __forceinline__ void put4(uint16_t* dst, f32x4 v) { *reinterpret_cast<u32x2*>(dst) = pack_bf16x4(v.x, v.y, v.z, v.w); }
__device__ __forceinline__ void put4(float* dst, f32x4 v) { *reinterpret_cast<f32x4*>(dst) = v; }
__device__ __forceinline__ void put1(uint16_t* dst, float v) { *dst = (uint16_t)bf16_bits(v); }
__device__ __forceinline__ void put1(float* dst, float v) { *dst = v; }

// put(k, value of parameter ix[k]), k < N: perturbed, the loads of all of them in flight together (each index is that of a parameter).
template <int N, class Put>
__device__ __forceinline__ void row_values(const float* __restrict__ theta, const NoiseRow nz, float scale, const uint32_t (&ix)[N], Put&& put) {
  auto batch = [&](auto fetch) {
    float tv[N];
    decltype(fetch(0u)) ev[N];
#pragma unroll
    for (int k = 0; k < N; ++k) { tv[k] = theta[ix[k]]; ev[k] = fetch(ix[k]); }
#pragma unroll
    for (int k = 0; k < N; ++k) put(k, __fmaf_rn(scale, widen1(ev[k]), tv[k]));
  };
  if (nz.mode >= 2u) batch([&](uint32_t idx) { return noise_regen1(nz.row, idx, nz.gen, nz.k0, nz.k1, nz.mode == 3u); });
  else if (nz.mode == 1u) batch([&](uint32_t idx) { return static_cast<const uint16_t*>(nz.ptr)[idx]; });
  else batch([&](uint32_t idx) { return static_cast<const float*>(nz.ptr)[idx]; });
}

// Fill dst[r * pitch + c] for r < rows_p, c < COLS with the source value of matrix element (r, kbase + c) when
// r < rows and kbase + c < cols, and zero elsewhere.
// By `step` threads, this one being `tid` of them.
// PERTURB: value = fma(scale, noise[idx], theta[idx]) with idx = off + r * cols + (kbase + c).
// The loads of U iterations are issued together and unconditionally (a masked-out element reads the
// matrix's first entries instead, which are always there), and only then consumed: a load inside the bounds test
// would be waited for in its own iteration, and the round would cost one memory latency per iteration.
template <int COLS, bool PERTURB, int U = STAGE_BATCH, class Elem>
__device__ __forceinline__ void stage_cols(Elem* dst, int pitch, int rows_p, int rows, int cols, int kbase,
                                           const float* __restrict__ src, const NoiseRow nz, float scale, uint32_t off,
                                           const int tid = (int)threadIdx.x, const int step = (int)blockDim.x) {
  if (((cols | (int)off | kbase) & 3) == 0) {
    // four consecutive columns per thread: 16-byte parameter loads, 8/16-byte noise loads, vector LDS stores
    constexpr int C4 = COLS / 4;
    const int total = rows_p * C4;
    auto batch = [&](auto fetch) {
      for (int q0 = tid; q0 < total; q0 += U * step) {
        f32x4 tv[U];
        decltype(fetch(0u)) ev[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int q = q0 + u * step;
          const int r = q / C4, k = kbase + (q % C4) * 4;
          ok[u] = q < total && r < rows && k < cols;
          const uint32_t idx = ok[u] ? off + (uint32_t)r * (uint32_t)cols + (uint32_t)k : off;
          tv[u] = *reinterpret_cast<const f32x4*>(src + idx);
          ev[u] = fetch(idx);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int q = q0 + u * step;
          if (q < total) {
            const int r = q / C4, c = (q % C4) * 4;
            f32x4 v = tv[u];
            if (PERTURB) {
              const f32x4 e = widen4(ev[u]);
              v = f32x4{__fmaf_rn(scale, e.x, v.x), __fmaf_rn(scale, e.y, v.y), __fmaf_rn(scale, e.z, v.z), __fmaf_rn(scale, e.w, v.w)};
            }
            if (!ok[u]) v = f32x4{0.f, 0.f, 0.f, 0.f};
            put4(dst + r * pitch + c, v);
          }
        }
      }
    };
    // one loop per storage mode, chosen outside it (the mode is uniform); the regenerating loop is not
    // unrolled: its body is two hundred instructions, and the staging code should stay in the instruction cache
    if (PERTURB && nz.mode >= 2u) {
#pragma unroll 1
      for (int q = tid; q < total; q += step) {
        const int r = q / C4, c = (q % C4) * 4, k = kbase + c;
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
        if (r < rows && k < cols) {
          const uint32_t idx = off + (uint32_t)r * (uint32_t)cols + (uint32_t)k;
          v = *reinterpret_cast<const f32x4*>(src + idx);
          float z[4];
          noise_regen4(nz.row, idx, nz.gen, nz.k0, nz.k1, nz.mode == 3u, z);
          v = f32x4{__fmaf_rn(scale, z[0], v.x), __fmaf_rn(scale, z[1], v.y), __fmaf_rn(scale, z[2], v.z), __fmaf_rn(scale, z[3], v.w)};
        }
        put4(dst + r * pitch + c, v);
      }
    } else if (PERTURB && nz.mode == 1u) {
      batch([&](uint32_t idx) { return *reinterpret_cast<const u32x2*>(static_cast<const uint16_t*>(nz.ptr) + idx); });
    } else if (PERTURB) {
      batch([&](uint32_t idx) { return *reinterpret_cast<const f32x4*>(static_cast<const float*>(nz.ptr) + idx); });
    } else {
      batch([&](uint32_t) { return 0; });
    }
    return;
  }
  // rows that are not multiples of four long: one column per thread
  const int total = rows_p * COLS;
  auto batch = [&](auto fetch) {
    for (int q0 = tid; q0 < total; q0 += U * step) {
      float tv[U];
      decltype(fetch(0u)) ev[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + u * step;
        const int r = q / COLS, k = kbase + q % COLS;
        ok[u] = q < total && r < rows && k < cols;
        const uint32_t idx = ok[u] ? off + (uint32_t)r * (uint32_t)cols + (uint32_t)k : off;
        tv[u] = src[idx];
        ev[u] = fetch(idx);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + u * step;
        if (q < total) {
          float v = tv[u];
          if (PERTURB) v = __fmaf_rn(scale, widen1(ev[u]), v);
          put1(dst + (q / COLS) * pitch + (q % COLS), ok[u] ? v : 0.f);
        }
      }
    }
  };
  if (PERTURB && nz.mode >= 2u) {
    // one counter block gives four consecutive parameters: per row, the aligned groups of four that cover its columns
    constexpr int G = COLS / 4 + 1;
#pragma unroll 1
    for (int q = tid; q < rows_p * G; q += step) {
      const int r = q / G;
      const uint32_t first = off + (uint32_t)r * (uint32_t)cols + (uint32_t)kbase, g0 = (first & ~3u) + 4u * (uint32_t)(q % G);
      const int k0 = (int)(g0 - first);
      float z[4] = {0.f, 0.f, 0.f, 0.f};
      const bool some = r < rows && kbase + k0 < cols && k0 < COLS;
      if (some) noise_regen4(nz.row, g0, nz.gen, nz.k0, nz.k1, nz.mode == 3u, z);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = k0 + e;
        if (k >= 0 && k < COLS) put1(dst + r * pitch + k, some && kbase + k < cols ? __fmaf_rn(scale, z[e], src[g0 + (uint32_t)e]) : 0.0f);
      }
    }
  } else if (PERTURB && nz.mode == 1u) {
    batch([&](uint32_t idx) { return static_cast<const uint16_t*>(nz.ptr)[idx]; });
  } else if (PERTURB) {
    batch([&](uint32_t idx) { return static_cast<const float*>(nz.ptr)[idx]; });
  } else {
    batch([&](uint32_t) { return 0; });
  }
}

}  // namespace es
