// Reading tensors of any shape and alignment into LDS, slice by slice of the contraction: what the kernels of
// gemm_any.hip, gemm_any_f64.hip and (its pieces, not its loop) gemm_exact.hip share.
//
// Edges: rows and columns beyond the tensors are read at clamped, valid addresses and not stored.  Contraction
// positions beyond the end are zeros: a piece that would cross the end of its row is read so that it ends there and is
// shifted down when it is staged (rows shorter than one piece are read element by element).
#pragma once
#include <type_traits>

#include "aqt_internal.h"

namespace aqt {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kSlice = 32;    // contraction positions per slice where an operand is float32

template <class T>
__device__ __forceinline__ T load_at(const void *p) {   // any byte alignment
  T v;
  __builtin_memcpy(&v, p, sizeof(T));
  return v;
}

__device__ __forceinline__ bool mask_bit(const uint32_t *__restrict__ mask, int64_t i) {
  return (mask[i >> 5] >> (i & 31)) & 1u;
}

// Up to 16 bytes at p + at, at + 16 <= end; beyond `end` zeros.
__device__ __forceinline__ v4i load16_guarded(const uint8_t *p, int64_t at, int64_t end) {
  if (at + 16 <= end) return load_at<v4i>(p + at);
  uint32_t d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 16; ++e)
    if (at + e < end) d[e >> 2] |= static_cast<uint32_t>(p[at + e]) << (8 * (e & 3));
  return v4i{static_cast<int>(d[0]), static_cast<int>(d[1]), static_cast<int>(d[2]), static_cast<int>(d[3])};
}

// 16 bytes moved down by `bytes` (0 .. 16), zeros from above.
__device__ __forceinline__ v4i shift_down(v4i v, int bytes) {
  if (bytes & 4) v = v4i{v.y, v.z, v.w, 0};
  if (bytes & 8) v = v4i{v.z, v.w, 0, 0};
  if (bytes & 16) v = v4i{0, 0, 0, 0};
  const int b = bytes & 3;
  v.x = static_cast<int>(__builtin_amdgcn_alignbyte(static_cast<uint32_t>(v.y), static_cast<uint32_t>(v.x), b));
  v.y = static_cast<int>(__builtin_amdgcn_alignbyte(static_cast<uint32_t>(v.z), static_cast<uint32_t>(v.y), b));
  v.z = static_cast<int>(__builtin_amdgcn_alignbyte(static_cast<uint32_t>(v.w), static_cast<uint32_t>(v.z), b));
  v.w = static_cast<int>(__builtin_amdgcn_alignbyte(0u, static_cast<uint32_t>(v.w), b));
  return v;
}
__device__ __forceinline__ v4f shift_down(v4f v, int elements) {   // 0 .. 4
  if (elements & 1) v = v4f{v.y, v.z, v.w, 0.0f};
  if (elements & 2) v = v4f{v.z, v.w, 0.0f, 0.0f};
  if (elements & 4) v = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  return v;
}
// how far a piece of `size` that starts at `at` was moved up to end at `end`, at most `size`
__device__ __forceinline__ int moved(int64_t at, int64_t end, int size) {
  const int64_t d = at + size - end;
  return d <= 0 ? 0 : d < size ? static_cast<int>(d) : size;
}

// Eight int4 codes in memory order (low nibble first) -> eight bytes 16 * code, in order.
__device__ __forceinline__ v2i expand16(uint32_t w) {
  const uint32_t even = (w << 4) & 0xF0F0F0F0u, odd = w & 0xF0F0F0F0u;
  v2i o;
  o.x = static_cast<int>(__builtin_amdgcn_perm(odd, even, 0x05010400u));
  o.y = static_cast<int>(__builtin_amdgcn_perm(odd, even, 0x07030602u));
  return o;
}

// What a contraction of float32 rows with rows of codes is given (dX: mask, factor, s_x; weight-only forward: bias).
struct CodesArgs {
  const float *f, *scale;
  const void *q;
  int64_t M, R, C;
  const float *s_x;
  const uint32_t *mask_x;
  const float *factor, *bias;
  float *out;
};

// What turns a sum over the rows into an element of dW.
struct DwFinish {
  const float *s_x, *s_w;
  const uint32_t *mask_w;
};

__device__ __forceinline__ float dw_value(double s, int64_t at, int64_t n, const DwFinish &fin, double sx) {
  const bool pass = fin.mask_w ? mask_bit(fin.mask_w, at) : (fin.s_w[n] != 0.0f);
  return pass ? static_cast<float>(sx * s) : 0.0f;
}

// The slice loop of a workgroup.  load(set, slice) requests a slice into register set 0 or 1, stage(set, slice, slot)
// moves it to LDS, multiply(slot) consumes it.
//   WK == 1: all wavefronts share the slices; two LDS slots, so that a slice is staged (and converted) while the one
//            before it is multiplied, one barrier per slice, loads two slices ahead.
//   WK > 1:  every wavefront has its own slices wk, wk + WK, ... and its own slot: its LDS operations are executed
//            in order, so no barrier is needed and the wavefronts overlap as they come.  The next slice is requested behind
//            wave_lds_order: in front of it the backward of 1024 x 256 layers took 1 % longer (16.8 us against 16.6).
// The loop has no branch around a load (past the end the last slice is requested again): behind a branch the compiler
// cannot count what is in flight and waits for everything, which undoes the prefetch.
template <int WK, class Load, class Stage, class Multiply>
__device__ __forceinline__ void run_slices(uint8_t *lds, int slice_bytes, int wk, int64_t slices, Load load, Stage stage,
                                           Multiply multiply) {
  constexpr std::integral_constant<int, 0> set0{};
  constexpr std::integral_constant<int, 1> set1{};
  const int64_t mine = WK > 1 ? (slices - wk + WK - 1) / WK : slices;   // this wavefront's slices
  auto at = [&](int64_t i) { return wk + WK * (i < mine ? i : mine - 1); };
  if (mine <= 0) return;   // WK > 1 only
  if (WK > 1) {
    uint8_t *const slot = lds + wk * slice_bytes;
    load(set0, at(0));
    load(set1, at(1));
    for (int64_t i = 0; i < mine; i += 2) {
      stage(set0, at(i), slot);
      wave_lds_order();
      load(set0, at(i + 2));
      multiply(slot);
      if (i + 1 >= mine) break;
      wave_lds_order();
      stage(set1, at(i + 1), slot);
      wave_lds_order();
      load(set1, at(i + 3));
      multiply(slot);
      wave_lds_order();
    }
    return;
  }
  uint8_t *const slot0 = lds, *const slot1 = lds + slice_bytes;
  load(set0, at(0));
  load(set1, at(1));
  stage(set0, at(0), slot0);
  load(set0, at(2));
  __syncthreads();
  for (int64_t s = 0; s < mine; s += 2) {
    stage(set1, at(s + 1), slot1);
    load(set1, at(s + 3));
    multiply(slot0);
    __syncthreads();
    if (s + 1 >= mine) break;
    stage(set0, at(s + 2), slot0);
    load(set0, at(s + 4));
    multiply(slot1);
    __syncthreads();
  }
}

// One slice that is loaded whole before anything else (rows shorter than a piece); WK > 1: by one wavefront alone.
template <int WK, class LoadNarrow, class Stage, class Multiply>
__device__ __forceinline__ void run_narrow(uint8_t *slot, LoadNarrow load_narrow, Stage stage, Multiply multiply) {
  constexpr std::integral_constant<int, 0> set0{};
  load_narrow(set0);
  stage(set0, 0, slot);
  if (WK > 1) wave_lds_order();
  else __syncthreads();
  multiply(slot);
  if (WK == 1) __syncthreads();
}

}  // namespace
}  // namespace aqt
