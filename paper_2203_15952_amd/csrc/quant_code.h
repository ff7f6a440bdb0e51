// The element-wise part of the quantizer (Fig. 2): code = floor(fl(fl(v / s) + 0.5)) clamped to +-qmax, 0 where s is 0.
// The divide is IEEE and takes a dozen instructions, one of them at a quarter of the rate.  Where the scale is far from the ends
// of the exponent range u = fma(v, 1 / s, 0.5) is within 2^-15 of the exact v / s + 0.5 as long as that is below 128 (the
// reciprocal's half ulp, one rounding) and so is the defined expression (two roundings): both have the same floor unless u lies
// within 2^-13 of a whole number, and the four values of a lane of which one does are divided (one quad in a thousand).  Beyond 128 both clamp.
// With the loads that a block waits for first requested together: 65536 x 2048, both passes 205.5 -> 194.5 us; one pass of 12800 x
// 2048 26 -> 23, the normalisation's quantizer of 12800 x 512 13 -> 10.5, of 65536 x 512 39 -> 32.  The flat quantizer asks once for four quads: a
// branch at each had cost tensors of one block more than the divides (4096 elements, both passes 4.55 -> 4.77 us; so 4.3).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aqt {
namespace {

__device__ __forceinline__ float quant_floor(float v, float s, float fq) {
  const float t = (s == 0.0f) ? 0.0f : v / s;
  return fminf(fmaxf(floorf(t + 0.5f), -fq), fq);
}

// A thread's share of the largest of n words in a workgroup of T; its loads are requested together (one after the other they are a chain of
// trips to the cache at the head of every block).
template <int T>
__device__ __forceinline__ uint32_t words_max(const uint32_t *__restrict__ p, int n) {
  const int t = threadIdx.x;
  if (n <= T) return t < n ? p[t] : 0u;
  uint32_t m = 0u;
  for (int i = 0; i < n; i += 8 * T) {
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[min(i + u * T + t, n - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) m = max(m, v[u]);
  }
  return m;
}

struct Quantizer {   // uniform; fq = (float)qmax
  float s, fq, r;
  bool near_one;     // the scale allows the reciprocal
};
__device__ __forceinline__ Quantizer quantizer(float s, float fq) {
  const bool ok = s > 0x1p-60f && s < 0x1p60f;
  return Quantizer{s, fq, ok ? 1.0f / s : 0.0f, ok};
}

__device__ __forceinline__ uint32_t pack_codes(float a, float b, float c, float d) {
  const uint32_t x = static_cast<uint32_t>(static_cast<int>(a)) & 0xFFu, y = static_cast<uint32_t>(static_cast<int>(b)) & 0xFFu;
  const uint32_t z = static_cast<uint32_t>(static_cast<int>(c)) & 0xFFu, w = static_cast<uint32_t>(static_cast<int>(d));
  return x | (y << 8) | (z << 16) | (w << 24);
}
// Four codes by the reciprocal, the first in the lowest byte; false: one of the values lies too near a whole number.
__device__ __forceinline__ bool quant4_certain(float x, float y, float z, float w, const Quantizer &k, uint32_t &codes) {
  const float a = fmaf(x, k.r, 0.5f), b = fmaf(y, k.r, 0.5f), c = fmaf(z, k.r, 0.5f), d = fmaf(w, k.r, 0.5f);
  const float ea = fabsf(__builtin_amdgcn_fractf(a) - 0.5f), eb = fabsf(__builtin_amdgcn_fractf(b) - 0.5f);
  const float ec = fabsf(__builtin_amdgcn_fractf(c) - 0.5f), ed = fabsf(__builtin_amdgcn_fractf(d) - 0.5f);
  auto clamp = [&](float u) { return fminf(fmaxf(floorf(u), -k.fq), k.fq); };
  codes = pack_codes(clamp(a), clamp(b), clamp(c), clamp(d));
  return !(fmaxf(fmaxf(ea, eb), fmaxf(ec, ed)) > 0.5f - 0x1p-13f);
}
__device__ __forceinline__ uint32_t quant4_divided(float x, float y, float z, float w, const Quantizer &k) {
  return pack_codes(quant_floor(x, k.s, k.fq), quant_floor(y, k.s, k.fq), quant_floor(z, k.s, k.fq), quant_floor(w, k.s, k.fq));
}
// Four codes (apart from quant4_certain: codes packed in front of the branch cost the product that quantizes both its operands 9.5 -> 10.0 us).
__device__ __forceinline__ uint32_t quant4(float x, float y, float z, float w, const Quantizer &k) {
  if (k.near_one) {
    const float a = fmaf(x, k.r, 0.5f), b = fmaf(y, k.r, 0.5f), c = fmaf(z, k.r, 0.5f), d = fmaf(w, k.r, 0.5f);
    const float ea = fabsf(__builtin_amdgcn_fractf(a) - 0.5f), eb = fabsf(__builtin_amdgcn_fractf(b) - 0.5f);
    const float ec = fabsf(__builtin_amdgcn_fractf(c) - 0.5f), ed = fabsf(__builtin_amdgcn_fractf(d) - 0.5f);
    if (!(fmaxf(fmaxf(ea, eb), fmaxf(ec, ed)) > 0.5f - 0x1p-13f)) {
      auto clamp = [&](float u) { return fminf(fmaxf(floorf(u), -k.fq), k.fq); };
      return pack_codes(clamp(a), clamp(b), clamp(c), clamp(d));
    }
  }
  return quant4_divided(x, y, z, w, k);
}

}  // namespace
}  // namespace aqt
