// Float32 operands of the bf16 matrix cores: a value as the sum of two terms (16 significant bits) or of three (24, all of
// it), each rounded to nearest even.  An infinity, or a finite value that rounds to one, has no such terms: the lowest is a NaN.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aqt {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

// Two floats -> packed bf16 pair.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  v2f f = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, v2bf));
}

__device__ __forceinline__ v16f mfma_bf16(v4i a, v4i b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// hi = bf16(a), lo = bf16(a - hi)
__device__ __forceinline__ void split_bf16(float a, float b, uint32_t &hi, uint32_t &lo) {
  hi = pack_bf16(a, b);
  const float ha = __uint_as_float(hi << 16), hb = __uint_as_float(hi & 0xFFFF0000u);
  lo = pack_bf16(a - ha, b - hb);
}
// a = hi + mid + lo exactly
__device__ __forceinline__ void split3_bf16(float a, float b, int &hi, int &mid, int &lo) {
  const uint32_t h = pack_bf16(a, b);
  uint32_t m, l;
  split_bf16(a - __uint_as_float(h << 16), b - __uint_as_float(h & 0xFFFF0000u), m, l);
  hi = static_cast<int>(h); mid = static_cast<int>(m); lo = static_cast<int>(l);
}

}  // namespace
}  // namespace aqt
