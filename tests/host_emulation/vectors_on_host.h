// The short vectors of the kernels as plain structs, and the wavefront-wide instructions that the kernels for vectorised
// rows use besides those of hip_on_host.h.  Lanes exchange through tables, in step with their wavefront.
#pragma once
#include "hip_on_host.h"
#define AQT_VECTOR(name, type, n, bytes, ...)                          \
  struct alignas(bytes) name {                                         \
    type __VA_ARGS__;                                                  \
    type &operator[](int i) { return (&x)[i]; }                        \
    const type &operator[](int i) const { return (&x)[i]; }            \
  };
AQT_VECTOR(v2f, float, 2, 8, x, y)
AQT_VECTOR(v4f, float, 4, 16, x, y, z, w)
AQT_VECTOR(v2i, int, 2, 8, x, y)
AQT_VECTOR(v4i, int, 4, 16, x, y, z, w)
inline std::barrier<> &wave_meets() { return *g_wbar[threadIdx.x >> 6]; }
inline int __builtin_amdgcn_readfirstlane(int v) {
  static int table[16];
  const unsigned w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) table[w] = v;
  wave_meets().arrive_and_wait();
  v = table[w];
  wave_meets().arrive_and_wait();
  return v;
}
inline bool __any(bool p) {
  static uint8_t table[1024];
  table[threadIdx.x] = p;
  wave_meets().arrive_and_wait();
  bool any = false;
  for (unsigned l = 0; l < 64; ++l) any |= table[(threadIdx.x & ~63u) + l] != 0;
  wave_meets().arrive_and_wait();
  return any;
}
inline uint32_t bf16_bits(float f) {   // round to nearest even
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
inline uint32_t pack_bf16(float a, float b) { return bf16_bits(a) | bf16_bits(b) << 16; }
// v_mfma_f32_32x32x16_bf16: lane (lr, lk) supplies A[lr][8 lk .. 8 lk + 7] and B[8 lk .. 8 lk + 7][lr]
inline v16f mfma(v4i a, v4i b, v16f c) {
  static v4i ta[1024], tb[1024];
  const unsigned base = threadIdx.x & ~63u, lane = threadIdx.x & 63u, lr = lane & 31u, lk = lane >> 5;
  ta[threadIdx.x] = a; tb[threadIdx.x] = b;
  wave_meets().arrive_and_wait();
  for (int r = 0; r < 16; ++r) {
    const unsigned row = 8 * (r >> 2) + 4 * lk + (r & 3);
    float sum = c[r];
    for (unsigned k = 0; k < 16; ++k) {
      const uint32_t x = (uint32_t)ta[base + 32 * (k >> 3) + row][(k & 7) >> 1], y = (uint32_t)tb[base + 32 * (k >> 3) + lr][(k & 7) >> 1];
      sum = fmaf(__uint_as_float(k & 1 ? x & 0xFFFF0000u : x << 16), __uint_as_float(k & 1 ? y & 0xFFFF0000u : y << 16), sum);
    }
    c[r] = sum;
  }
  wave_meets().arrive_and_wait();
  return c;
}
// ds_read_b64_tr_b16: sixteen lanes read eight bytes each, four rows of sixteen 16-bit columns; lane i receives column i
inline v2i read_tr_b16(const uint8_t *at) {
  static uint16_t table[1024][4];
  memcpy(table[threadIdx.x], at, 8);
  wave_meets().arrive_and_wait();
  const unsigned group = threadIdx.x & ~15u, i = threadIdx.x & 15u;
  uint16_t col[4];
  for (unsigned r = 0; r < 4; ++r) col[r] = table[group + 4 * r + (i >> 2)][i & 3];
  v2i v;
  memcpy(&v, col, 8);
  wave_meets().arrive_and_wait();
  return v;
}
