// The short vectors of the kernels as plain structs, and the wavefront-wide instructions that the kernels for vectorised
// rows use besides those of hip_on_host.h.  Lanes exchange through tables, in step with their wavefront.
#pragma once
#include <atomic>
#include <type_traits>
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
AQT_VECTOR(v4d, double, 4, 32, x, y, z, w)
struct v16i { int v[16]; int &operator[](int i) { return v[i]; } const int &operator[](int i) const { return v[i]; } };
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
inline uint64_t __ballot(bool p) {
  static uint8_t table[1024];
  table[threadIdx.x] = p;
  wave_meets().arrive_and_wait();
  uint64_t r = 0;
  for (unsigned l = 0; l < 64; ++l) r |= (uint64_t)(table[(threadIdx.x & ~63u) + l] != 0) << l;
  wave_meets().arrive_and_wait();
  return r;
}
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
template <class T> inline T lane_value(T v, unsigned from) {   // of another lane of the wavefront
  static T table[1024];
  table[threadIdx.x] = v;
  wave_meets().arrive_and_wait();
  v = table[(threadIdx.x & ~63u) | (from & 63u)];
  wave_meets().arrive_and_wait();
  return v;
}
inline int __shfl(int v, int lane) { return lane_value(v, (unsigned)lane); }
inline double __shfl_xor(double v, int off) { return lane_value(v, (threadIdx.x & 63u) ^ (unsigned)off); }
inline float load_f32(const float *base, uint32_t lane_bytes, uint32_t uniform_bytes) {
  return *(const float *)((const char *)base + lane_bytes + uniform_bytes);
}
inline int anew(int v) { return v; }
inline void __builtin_amdgcn_sched_barrier(int) {}
inline uint32_t bf16_bits(float f) {   // round to nearest even
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
inline uint32_t pack_bf16(float a, float b) { return bf16_bits(a) | bf16_bits(b) << 16; }
// v_mfma_f32_32x32x16_bf16: lane (lr, lk) supplies A[lr][8 lk .. 8 lk + 7] and B[8 lk .. 8 lk + 7][lr]
inline v16f mfma_bf16(v4i a, v4i b, v16f c) {
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
// v_mfma_i32_32x32x32_i8: lane (lr, lk) supplies A[lr][16 lk .. 16 lk + 15] and B[16 lk .. 16 lk + 15][lr]
inline v16i __builtin_amdgcn_mfma_i32_32x32x32_i8(v4i a, v4i b, v16i c, int, int, int) {
  static v4i ta[1024], tb[1024];
  const unsigned base = threadIdx.x & ~63u, lane = threadIdx.x & 63u, lr = lane & 31u, lk = lane >> 5;
  ta[threadIdx.x] = a; tb[threadIdx.x] = b;
  wave_meets().arrive_and_wait();
  for (int r = 0; r < 16; ++r) {
    const unsigned row = 8 * (r >> 2) + 4 * lk + (r & 3);
    for (unsigned half = 0; half < 2; ++half) {
      int8_t x[16], y[16];
      memcpy(x, &ta[base + 32 * half + row], 16);
      memcpy(y, &tb[base + 32 * half + lr], 16);
      for (int k = 0; k < 16; ++k) c[r] += x[k] * y[k];
    }
  }
  wave_meets().arrive_and_wait();
  return c;
}
// v_mfma_i32_16x16x64_i8: lane (lc = lane % 16, lg = lane / 16) supplies A[lc][16 lg .. 16 lg + 15] and B[16 lg .. 16 lg + 15][lc];
// element r of its accumulator is row 4 lg + r, column lc
inline v4i __builtin_amdgcn_mfma_i32_16x16x64_i8(v4i a, v4i b, v4i c, int, int, int) {
  static v4i ta[1024], tb[1024];
  const unsigned base = threadIdx.x & ~63u, lane = threadIdx.x & 63u, lc = lane & 15u, lg = lane >> 4;
  ta[threadIdx.x] = a; tb[threadIdx.x] = b;
  wave_meets().arrive_and_wait();
  for (unsigned r = 0; r < 4; ++r)
    for (unsigned g = 0; g < 4; ++g) {
      int8_t x[16], y[16];
      memcpy(x, &ta[base + 16 * g + 4 * lg + r], 16);
      memcpy(y, &tb[base + 16 * g + lc], 16);
      for (int k = 0; k < 16; ++k) c[r] += x[k] * y[k];
    }
  wave_meets().arrive_and_wait();
  return c;
}
// v_mfma_f64_16x16x4_f64: lane (lc = lane % 16, lg = lane / 16) supplies A[lc][lg] and B[lg][lc]; element r of its
// accumulator is row 4 r + lg, column lc
static std::atomic<long> g_f64_products{0};
inline v4d __builtin_amdgcn_mfma_f64_16x16x4f64(double a, double b, v4d c, int, int, int) {
  static double ta[1024], tb[1024];
  if ((threadIdx.x & 63u) == 0) ++g_f64_products;
  const unsigned base = threadIdx.x & ~63u, lane = threadIdx.x & 63u, lc = lane & 15u, lg = lane >> 4;
  ta[threadIdx.x] = a; tb[threadIdx.x] = b;
  wave_meets().arrive_and_wait();
  for (unsigned r = 0; r < 4; ++r)
    for (unsigned k = 0; k < 4; ++k) c[r] = fma(ta[base + 16 * k + 4 * r + lg], tb[base + 16 * k + lc], c[r]);
  wave_meets().arrive_and_wait();
  return c;
}
// v_mfma_f32_16x16x4_f32: lanes and accumulator rows as v_mfma_i32_16x16x64_i8; the four products one after the other
inline v4f __builtin_amdgcn_mfma_f32_16x16x4f32(float a, float b, v4f c, int, int, int) {
  const unsigned base = threadIdx.x & ~63u, lane = threadIdx.x & 63u, lc = lane & 15u, lg = lane >> 4;
  g_mfa[threadIdx.x] = a; g_mfb[threadIdx.x] = b;
  wave_meets().arrive_and_wait();
  for (unsigned r = 0; r < 4; ++r)
    for (unsigned k = 0; k < 4; ++k) c[r] = fmaf(g_mfa[base + 16 * k + 4 * lg + r], g_mfb[base + 16 * k + lc], c[r]);
  wave_meets().arrive_and_wait();
  return c;
}
inline float __builtin_amdgcn_fractf(float x) { return fminf(x - floorf(x), 0x1.fffffep-1f); }
inline uint32_t __builtin_amdgcn_alignbyte(uint32_t hi, uint32_t lo, int b) { return (uint32_t)(((uint64_t)hi << 32 | lo) >> (8 * (b & 3))); }
inline uint32_t __builtin_amdgcn_perm(uint32_t hi, uint32_t lo, uint32_t sel) {   // selector bytes 0 .. 3: lo, 4 .. 7: hi
  const uint64_t v = (uint64_t)hi << 32 | lo;
  uint32_t r = 0;
  for (int e = 0; e < 4; ++e) r |= (uint32_t)(v >> (8 * (sel >> (8 * e) & 7)) & 0xFF) << (8 * e);
  return r;
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
