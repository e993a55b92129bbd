// Device-side helpers shared by the HIP kernels of the jagged HSTU attention library (gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hstu_geometry.h"

namespace hstu {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr int kNumXcd = 8;          // MI355X: 8 accelerator dies, workgroups are dealt to them round-robin
constexpr int kXcdGroup = 4;        // consecutive schedule entries kept on one die (the scheduler writes them as runs of one head)

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even fp32 -> bf16 (NaN kept quiet); inputs here are finite
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// d/dt [t sigmoid(t)]
__device__ __forceinline__ float dsilu(float t) {
  const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * t));
  return sg * (1.0f + t * (1.0f - sg));
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
  typedef float v2f __attribute__((ext_vector_type(2)));
  v2f x = {lo, hi};
  v2bf y = __builtin_convertvector(x, v2bf);                 // v_cvt_pk_bf16_f32 on gfx950 (RNE)
  return __builtin_bit_cast(uint32_t, y);
}

// Bits lo .. 31.
__device__ __forceinline__ uint32_t bits_from(int lo) { return lo > 31 ? 0u : ~0u << max(lo, 0); }

// Of a 32 x 32 block of scores (register r of a lane: streamed row 8 (r / 4) + r % 4, + 4 in the upper half-wave): `masked` where the row's bit of `vis` is 0,
// whatever stood there; a second block, if there is one, with zeros.  Three bit operations a score: a bit field, v_bfi, v_and.  (The mask is kept
// from the compiler, which makes comparisons of it: one instruction more, and a pair of scalar registers each.  Left to it, the narrow backward
// of 28 x 339, 8 heads of 64, K1 = 35 takes 65.9 us, so 64.8; of 8 x 8k-16k, 4 heads of 64, 2,443 and 2,430; the forward is the same.)
template <bool ZERO>
__device__ __forceinline__ void mask_scores(uint32_t vis, f32x16& v, float masked, f32x16& zeroed) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)vis, 8 * (r >> 2) + (r & 3), 1);
    asm volatile("" : "+v"(m));
    v[r] = __uint_as_float((__float_as_uint(v[r]) & m) | (__float_as_uint(masked) & ~m));
    if (ZERO) zeroed[r] = __uint_as_float(__float_as_uint(zeroed[r]) & m);
  }
}

}  // namespace hstu
