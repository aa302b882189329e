// Shared pieces of the kernels on the fp32 matrix instructions: storage-form loads of four elements (fp32 or bf16,
// widened exactly) and accumulator initialisation.
#pragma once

#include "mlra_internal.h"

namespace mlra {
namespace f32_tile {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr float kNegBig = -1.0e30f;   // "no token seen yet" running max (finite: no inf - inf)

// four consecutive stored elements, kept in their storage form until they are needed
struct Raw4f {
  f32x4 v;
  __device__ void zero() { v = f32x4{0.f, 0.f, 0.f, 0.f}; }
  __device__ void load(const float* p) { v = *(const f32x4*)p; }
  __device__ void set(int e, float x) { v[e] = x; }
  __device__ f32x4 get() const { return v; }
};
struct Raw4b {
  uint32_t lo, hi;
  __device__ void zero() { lo = hi = 0u; }
  __device__ void load(const bf16_t* p) { const uint2 u = *(const uint2*)p; lo = u.x; hi = u.y; }
  __device__ void set(int e, bf16_t x) {
    uint32_t& w = e < 2 ? lo : hi;
    w = (e & 1) ? (w & 0xffffu) | ((uint32_t)x << 16) : (w & 0xffff0000u) | x;
  }
  __device__ f32x4 get() const {
    return f32x4{__uint_as_float(lo << 16), __uint_as_float(lo & 0xffff0000u), __uint_as_float(hi << 16),
                 __uint_as_float(hi & 0xffff0000u)};
  }
};
template <typename T> struct RawOf;
template <> struct RawOf<float> { typedef Raw4f type; };
template <> struct RawOf<bf16_t> { typedef Raw4b type; };

// Zero that the compiler cannot fold, so that an accumulator is a register operand from its first MFMA on (the
// destination is then its accumulator input and never lies on an A / B operand).
__device__ __forceinline__ f32x4 opaque_zero4() {
  float z = 0.f;
  asm volatile("" : "+v"(z));
  return f32x4{z, z, z, z};
}

}  // namespace f32_tile
}  // namespace mlra
