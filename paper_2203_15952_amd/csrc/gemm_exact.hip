// The float contractions off the tuned kernels' grid (see gemm_any_f64.hip) where there is enough work to fill the chip: the
// same sums, exact up to the float64 addition of six partial sums, but on the int8 matrix cores.
//
// A float32 value is 24 bits at some exponent and a code is an integer, so a row's values, scaled by one power of two so
// that the row's largest stays below 2^46, are integers of 47 bits as long as none is more than 2^22 times smaller than that
// largest.  Such an integer is six balanced base-256 digits, i.e. six int8 operands, and v_mfma_i32_16x16x64_i8 adds
// digit x code products without rounding.  One float64 fused multiply-add makes the integer (the sum with 1.5 * 2^52
// leaves it in the low mantissa bits) and adds 0x80 to every digit, so the digits are the bytes with their top bit flipped.
// In a normally distributed gradient one value in a million lies below that range; in that of a softmax most do (logits of standard
// deviation 3: a row spans thirty binades).  What the digits leave of a few such values is kept in a list as they are converted, and
// multiplied in float64, four at a time.  Where more are left than the list holds the workgroup goes through its rows again for the next plane of
// six digits, 47 binades further down, and so on; two planes do for a softmax, six for any two float32 values.
//
// An infinity or a NaN is multiplied in float64 (v_mfma_f64_16x16x4_f64), the sixty-four positions that hold it: they decide
// their row's results, whatever the rest of it adds up to.
//
// Six int8 passes are 1/10 of the matrix time of the float64 instruction, so the conversion of the float operand weighs as
// much as the products: about nine vector instructions a value, for 16 TJ products.  Hence a wavefront converts its own
// sixteen rows in registers, straight in fragment order (no LDS, no second conversion within a workgroup), and keeps 16 x 16 TJ
// results: 24 TJ accumulator registers, at TJ = 5 two wavefronts per SIMD.  The codes of a step are shared by the four
// wavefronts of a workgroup through LDS.  The order of the contraction inside a step of 64 is free: lane group g of four takes
// positions 16 i + 4 g .. + 3 (i = 0 .. 3), so that a load instruction reads whole 64-byte pieces of a row.
// At 4099 x 520 x 1000 dX takes 46 and dW 50 us, there 114 and 118; with the gradient of a softmax over the 1000 channels 74 and 81.
// (The lower planes have code of their own: in the first one's loop their conversion spilled, and cost dW 6 us with ordinary values.
// The float64 products of every step with such a value, which stood in their place, took 269 and 226.)  Error
// against float64 2.5e-8 of the result for each, as there.  A wavefront's 82 k cycles (dX, one plane) are 20 k of vector and 8 k of matrix
// instructions, 30 k waiting for the other wavefront's, 24 k waiting for loads, a third of that in the search for the extremes.
// Loads two steps ahead instead of one, for either operand, changed nothing; 96 columns a tile spill.
#include "any_shape.h"
#include "colsum.h"
#include "epilogue.h"

namespace aqt {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

#define AQT_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

constexpr int kThreads = 256;    // four wavefronts of sixteen rows (dX, weight-only) or channels (dW)
constexpr int kOwn = 64;         // rows or channels of a workgroup
constexpr int kStep = 64;        // contraction positions per step
constexpr int kDigits = 6;
constexpr int kRange = 22;       // binades below the largest that are exact in the first plane of digits
constexpr int kPlane = 47;       // binades from a plane to the next: a remainder of at most half a unit stays below 2^46
constexpr int64_t kLongest = 65536;   // 128 * 128 * 65536 < 2^31
constexpr double kMagic = 6755399441055744.0 + 141289400074368.0;   // 1.5 * 2^52 + 0x808080808080

__device__ __forceinline__ v4i mfma_i8(v4i a, v4i b, v4i c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0); }
__device__ __forceinline__ v4d mfma_f64(double a, double b, v4d c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
// base + uniform offset in scalar registers, a lane's own offset: no address arithmetic per load
__device__ __forceinline__ float load_f32(const float *base, uint32_t lane_bytes, uint32_t uniform_bytes) {
  const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, 0xFFFFFFFFu, 0x00027000);
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, lane_bytes, uniform_bytes, 0));
}
__device__ __forceinline__ int anew(int v) {   // the same value, as far as the compiler knows another one
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ double power_of_two(int e) {   // normal range
  return __builtin_bit_cast(double, static_cast<uint64_t>(1023 + e) << 52);
}

__device__ __forceinline__ bool is_finite(float v) { return (__float_as_uint(v) & 0x7FFFFFFFu) < 0x7F800000u; }

// The largest and the smallest non-zero magnitude of a row, as bit patterns.
struct Extremes {
  uint32_t top = 0u, low = 0xFFFFFFFFu;   // low: all ones where there are only zeros
  template <int N>
  __device__ __forceinline__ void note(const uint32_t (&b)[N]) {   // magnitudes; zeros cost a second look
    uint32_t least = b[0];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      top = max(top, b[i]);
      least = min(least, b[i]);
    }
    if (__any(least == 0u)) {
      least = 0xFFFFFFFFu;
#pragma unroll
      for (int i = 0; i < N; ++i) least = min(least, b[i] - 1u);   // a zero comes out on top
      if (least != 0xFFFFFFFFu) ++least;
    }
    low = min(low, least);
  }
  __device__ __forceinline__ void across_groups() {   // the four lane groups hold parts of the same row
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
      top = max(top, static_cast<uint32_t>(__shfl_xor(static_cast<int>(top), off)));
      low = min(low, static_cast<uint32_t>(__shfl_xor(static_cast<int>(low), off)));
    }
  }
  __device__ __forceinline__ bool finite() const { return top < 0x7F800000u; }
  __device__ __forceinline__ int exponent() const { return max(static_cast<int>(top >> 23), 1); }   // biased; subnormals like 1
  // every non-zero magnitude below this pattern may leave something behind planes 0 .. plane (rows that are not finite: none)
  __device__ __forceinline__ uint32_t doubtful(int plane) const {
    const int reach = kRange + kPlane * plane;
    return finite() && exponent() > reach ? static_cast<uint32_t>(exponent() - reach) << 23 : 1u;
  }
  __device__ __forceinline__ bool exact() const {
    const int least = low == 0xFFFFFFFFu ? exponent() : max(static_cast<int>(low >> 23), 1);
    return finite() && exponent() - least <= kRange;
  }
};
// value * scale_of(e) is below 2^46, its inverse undoes it
__device__ __forceinline__ double scale_of(int exponent) { return power_of_two(172 - exponent); }
__device__ __forceinline__ double unscale_of(int exponent) { return power_of_two(exponent - 172); }

// The unit of a plane's last digit is 2^(-47 plane) of the first one's.
__device__ __forceinline__ double unit_of(int plane) { return power_of_two(-kPlane * plane); }
// What a plane leaves of a value given in units of its last digit, in units of the next one's.  Exact.
__device__ __forceinline__ double next_plane(double y) { return (y - ((y + kMagic) - kMagic)) * power_of_two(kPlane); }
// What all planes down to this one leave of a finite row's value, exactly.
__device__ __forceinline__ double below_digits(float x, int exponent, int plane) {
  double y = static_cast<double>(x) * scale_of(exponent);
  for (int k = 0; k <= plane; ++k) y = next_plane(y);
  return y * (unscale_of(exponent) * unit_of(plane + 1));
}

// The few values of a wavefront's rows that reach below the digits, found while they are converted: what the digits leave of
// them, in a fixed order.  More than fit: another plane of digits.
constexpr int kFew = 16;
struct Left {
  double value;
  int row, at;   // the lane's row or channel of sixteen, the position
};
struct LeftList {
  Left *entry;   // kFew of this wavefront
  int n = 0;     // uniform
  __device__ __forceinline__ bool fits() const { return n <= kFew; }
  // four values of the lane's row, at positions at .. at + 3
  __device__ __forceinline__ void note(v4f x, uint32_t doubtful, int exponent, int plane, int row, int at) {
    uint32_t rank[4];   // of a zero: the largest
#pragma unroll
    for (int e = 0; e < 4; ++e) rank[e] = (__float_as_uint(x[e]) & 0x7FFFFFFFu) - 1u;
    if (!__any(min(min(rank[0], rank[1]), min(rank[2], rank[3])) < doubtful - 1u)) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool is = rank[e] < doubtful - 1u;
      const uint64_t lanes = __ballot(is);
      const int slot = n + static_cast<int>(__popcll(lanes & ((1ull << (threadIdx.x & 63)) - 1ull)));
      if (is && slot < kFew) entry[slot] = Left{below_digits(x[e], exponent, plane), row, at + e};
      n += static_cast<int>(__popcll(lanes));
    }
  }
  // entry k, for a lane that stands for `row`; nothing where it is another row's or behind the end
  __device__ __forceinline__ double value(int k, int row) const {
    return k < n && entry[k].row == row ? entry[k].value : 0.0;
  }
  __device__ __forceinline__ int at(int k) const { return entry[k < n ? k : n - 1].at; }
};

// Dword i of the six digit operands from the values of positions 4 i .. 4 i + 3 of the lane.
template <bool FIRST>
__device__ __forceinline__ void digits4(v4f x, double scale, int plane, int i, v4i (&d)[kDigits]) {
  uint32_t lo[4], hi[4];
  double y[4];
  if (!FIRST) {
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = static_cast<double>(x[e]) * scale;
    for (int k = 0; k < plane; ++k) {
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = next_plane(y[e]);
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint64_t u = __builtin_bit_cast(uint64_t, FIRST ? __builtin_fma(static_cast<double>(x[e]), scale, kMagic) : y[e] + kMagic);
    lo[e] = static_cast<uint32_t>(u);
    hi[e] = static_cast<uint32_t>(u >> 32);
  }
  auto pair = [](uint32_t a, uint32_t b, uint32_t sel) { return __builtin_amdgcn_perm(b, a, sel); };
  constexpr uint32_t kLow = 0x05010400u, kHigh = 0x07030602u, kFirst = 0x05040100u, kSecond = 0x07060302u;
  const uint32_t a = pair(lo[0], lo[1], kLow), b = pair(lo[2], lo[3], kLow);
  const uint32_t c = pair(lo[0], lo[1], kHigh), e = pair(lo[2], lo[3], kHigh);
  const uint32_t f = pair(hi[0], hi[1], kLow), g = pair(hi[2], hi[3], kLow);
  const uint32_t digit[kDigits] = {pair(a, b, kFirst), pair(a, b, kSecond), pair(c, e, kFirst),
                                   pair(c, e, kSecond), pair(f, g, kFirst), pair(f, g, kSecond)};
#pragma unroll
  for (int p = 0; p < kDigits; ++p) d[p][i] = static_cast<int>(digit[p] ^ 0x80808080u);
}
template <int TJ>
__device__ __forceinline__ double digits_sum(const v4i (&acc)[kDigits][TJ], int j, int r) {
  double s = static_cast<double>(acc[kDigits - 1][j][r]);
#pragma unroll
  for (int p = kDigits - 2; p >= 0; --p) s = __builtin_fma(s, 256.0, static_cast<double>(acc[p][j][r]));
  return s;
}

// LDS image of a step's codes: rows of 64 bytes, lane group g's sixteen positions in 16-byte piece g ^ turn(row), so that
// the rows of a fragment read spread over all banks.
__device__ __forceinline__ int turn(int row) { return ((row >> 1) & 3) ^ ((row >> 3) & 1); }
__device__ __forceinline__ int code_slot(int row, int group, int i) { return row * kStep + ((group ^ turn(row)) << 4) + 4 * i; }

template <int TJ, bool OWN_IS_A>
__device__ __forceinline__ void multiply(const uint8_t *codes, const v4i (&d)[kDigits], v4i (&acc)[kDigits][TJ], int lc, int lg) {
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const v4i q = *reinterpret_cast<const v4i *>(codes + code_slot(16 * j + lc, lg, 0));
#pragma unroll
    for (int p = 0; p < kDigits; ++p) acc[p][j] = OWN_IS_A ? mfma_i8(d[p], q, acc[p][j]) : mfma_i8(q, d[p], acc[p][j]);
  }
}

// Whether a condition holds in one of the workgroup's four wavefronts: set by each, asked behind a barrier, set again behind another.
__device__ __forceinline__ void set_flag(int *flag, int wave, bool mine) {
  if ((threadIdx.x & 63) == 0) flag[wave] = mine;
}
__device__ __forceinline__ bool in_some_wave(const int *flag) {
  return __builtin_amdgcn_readfirstlane(flag[0] | flag[1] | flag[2] | flag[3]) != 0;
}
__device__ __forceinline__ bool in_some_wave(int *flag, int wave, bool mine) {
  set_flag(flag, wave, mine);
  __syncthreads();
  return in_some_wave(flag);
}

// Workgroup -> (strip, tile of the strip).  A strip's tiles read the same float rows; workgroup ids eight apart run on one
// XCD, so they walk the tiles of one strip, whose rows then come from that L2.
__device__ __forceinline__ void place(int id, int strips, int tiles, int &strip, int &tile) {
  const int grp = 8 * tiles, full = strips / 8 * grp;
  if (id < full) {
    strip = id / grp * 8 + (id & 7);
    tile = id % grp >> 3;
  } else {
    strip = strips / 8 * 8 + (id - full) / tiles;
    tile = (id - full) % tiles;
  }
}

// An accumulator lane of the int8 instruction holds rows 4 g + r, one of the float64 instruction rows 4 r + g: given its
// operand's rows in this order the latter's sums fall where the former's are.
__device__ __forceinline__ int f64_row(int lc) { return 4 * (lc & 3) + (lc >> 2); }

// ---- float32 operand x codes: dX and the weight-only forward ---------------------------------
// out[m, r] = sum_c f[m, c] (* scale[c]) * q[r, c], rows of both contraction-contiguous; modes as in gemm_any_f64.hip.  A
// workgroup takes tiles_each column tiles of its rows in turn, so that a short contraction does not pay for the rows'
// extremes with each of them.  The last step's pieces that cross the end of their rows are read so that they end there and
// are moved into place (zeros from above) before they are used.
template <int TJ, bool PACKED, int MODE>
__global__ __launch_bounds__(kThreads, 2) void f32_codes_exact_kernel(
    const float *__restrict__ f, const float *__restrict__ scale, const uint8_t *__restrict__ q, int64_t M, int64_t R, int C,
    const float *__restrict__ s_x, const uint32_t *__restrict__ mask_x, const float *__restrict__ factor,
    const float *__restrict__ bias, float *__restrict__ out, int tiles_m, int tiles_r, int tiles_each) {
  constexpr bool DX = MODE == 0, GLU = MODE == 1 + AQT_EPI_GLU;
  static_assert(!GLU || TJ % 2 == 0, "a value block and its gate block side by side");
  constexpr int BQ = 16 * TJ, NQ = (BQ * 4 + kThreads - 1) / kThreads;   // pieces of sixteen codes per thread and step
  // (room for what the threads without a piece write: a branch around the writes would make the loads behind it wait)
  __shared__ __attribute__((aligned(16))) uint8_t sQ[2][NQ * kThreads * 16];
  __shared__ __attribute__((aligned(16))) float sS[2][DX ? 4 * kThreads : 4];
  const int t = threadIdx.x, lane = t & 63, lc = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int bm, group;
  place(static_cast<int>(blockIdx.x), tiles_m, static_cast<int>(cdiv(tiles_r, tiles_each)), bm, group);
  int br = group * tiles_each;
  const int br_end = min(br + tiles_each, tiles_r);
  const int64_t m0 = static_cast<int64_t>(bm) * kOwn, oc = GLU ? R / 2 : R;
  auto chan = [&](int cb) -> int64_t {
    if (GLU) return static_cast<int64_t>(br) * (BQ / 2) + (cb >> 1) * 16 + ((cb & 1) ? oc : 0);
    return static_cast<int64_t>(br) * BQ + cb * 16;
  };
  const int row_bytes = PACKED ? (C + 1) / 2 : C;
  constexpr int kPiece = PACKED ? 8 : 16;   // bytes of sixteen codes
  // rows as 32-bit offsets from a uniform base, the last row again beyond the end
  const float *const strip = f + m0 * C;
  auto row_at = [&](int row) { return static_cast<uint32_t>(min(static_cast<int64_t>(row), M - 1 - m0)) * static_cast<uint32_t>(C); };
  const uint32_t own = row_at(16 * wave + lc);
  const int steps = static_cast<int>(cdiv(C, kStep));
  auto ragged = [&](int s) { return kStep * (s + 1) > C; };
  auto piece_at = [&](const float *base, uint32_t row, int c) {
    return load_at<v4f>(reinterpret_cast<const char *>(base) + 4u * (row + static_cast<uint32_t>(min(c, C - 4))));
  };
  auto settle = [&](v4f v, int c) { return shift_down(v, min(max(c + 4 - C, 0), 4)); };
  auto clamped = [&](int s) { return s < steps ? s : steps - 1; };   // the last step again: no branch around a load

  // ---- largest and smallest of the rows ----
  // each(step, values) for all steps from `first` on, values: this lane's sixteen of its row (times their scales), element e of
  // piece i at position 64 step + 16 i + 4 lg + e
  constexpr int kAhead = 4;   // steps requested together
  auto for_all = [&](int first, auto each) {
    for (int s0 = first; s0 < steps; s0 += kAhead) {
      v4f v[kAhead][4], w[kAhead][4];
#pragma unroll
      for (int a = 0; a < kAhead; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int c = kStep * clamped(s0 + a) + 16 * i + 4 * lg;
          v[a][i] = piece_at(strip, own, c);
          if (DX) w[a][i] = piece_at(scale, 0, c);
        }
#pragma unroll
      for (int a = 0; a < kAhead; ++a) {
        const int s = clamped(s0 + a);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (DX) { v[a][i].x *= w[a][i].x; v[a][i].y *= w[a][i].y; v[a][i].z *= w[a][i].z; v[a][i].w *= w[a][i].w; }
        if (ragged(s)) {
#pragma unroll
          for (int i = 0; i < 4; ++i) v[a][i] = settle(v[a][i], kStep * s + 16 * i + 4 * lg);
        }
        each(s, v[a]);
      }
    }
  };
  Extremes x;
  int swept = 0;
  for (; kStep * (swept + kAhead) <= C; swept += kAhead) {   // whole steps: one address
    const char *const at = reinterpret_cast<const char *>(strip) + 4u * (own + kStep * swept + 4 * lg);
    const float *const sc = scale + kStep * swept + 4 * lg;
    v4f v[kAhead][4], w[kAhead][4];
#pragma unroll
    for (int a = 0; a < kAhead; ++a)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[a][i] = load_at<v4f>(at + 4 * (kStep * a + 16 * i));
        if (DX) w[a][i] = load_at<v4f>(sc + kStep * a + 16 * i);
      }
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      uint32_t bits[16];
#pragma unroll
      for (int i = 0; i < 16; ++i)
        bits[i] = __float_as_uint(DX ? fabsf(v[a][i >> 2][i & 3]) * fabsf(w[a][i >> 2][i & 3]) : fabsf(v[a][i >> 2][i & 3]));
      x.note(bits);
    }
  }
  for_all(swept, [&](int, const v4f (&v)[4]) {
    uint32_t bits[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) bits[i] = __float_as_uint(fabsf(v[i >> 2][i & 3]));
    x.note(bits);
  });
  x.across_groups();
  const int exponent = x.exponent();
  const double up = x.finite() ? scale_of(exponent) : 0.0;   // a row with an infinity: its digits are not used
  const bool finite = !__any(!x.finite()), wide = __any(!x.exact());   // uniform
  __shared__ Left few[kThreads / 64][kFew];
  __shared__ double above[4 * TJ][kThreads];   // the sums of the planes above
  __shared__ int flag[2][kThreads / 64];
  set_flag(flag[0], wave, wide);
  const bool keep = DX ? s_x[0] != 0.0f : true;

  for (; br < br_end; ++br) {
  // ---- the digits of one plane (the first in code of its own, which most rows are done with) ----
  v4i acc[kDigits][TJ];
  LeftList list{few[wave]};
  auto go_through = [&](auto first, int plane) {
  constexpr bool FIRST = decltype(first)::value;
  // the thread's place anew, unknown to the compiler: what follows from it would otherwise stay in registers over the loop
  const int tt = anew(t), lc = tt & 15, lg = tt >> 4 & 3;
  const uint8_t *pq[NQ];
#pragma unroll
  for (int u = 0; u < NQ; ++u) {
    const int piece = tt + u * kThreads, row = piece < BQ * 4 ? piece >> 2 : 0;
    const int64_t n = chan(row >> 4) + (row & 15);
    pq[u] = q + (n < R ? n : R - 1) * row_bytes;
  }
  list.n = 0;
  const uint32_t doubtful = x.doubtful(plane);
  const int zero = anew(0);
#pragma unroll
  for (int p = 0; p < kDigits; ++p)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[p][j] = v4i{zero, zero, zero, zero};
  v4f raw[4];
  v4i rq[NQ];
  v4f rs;
  auto load_f = [&](int i, int s) { raw[i] = piece_at(strip, own, kStep * s + 16 * i + 4 * lg); };
  auto load_q = [&](int s) {
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      const uint8_t *const at = pq[u] + min((4 * s + (tt & 3)) * kPiece, row_bytes - kPiece);
      if (PACKED) {
        const v2i w = load_at<v2i>(at);
        rq[u] = v4i{w.x, w.y, 0, 0};
      } else {
        rq[u] = load_at<v4i>(at);
      }
    }
    if (DX) rs = piece_at(scale, 0, kStep * s + 4 * (tt & 15));
  };
  auto store_q = [&](int slot, int s) {
    if (ragged(s)) {
      const int over = (4 * s + (tt & 3) + 1) * kPiece - row_bytes;
#pragma unroll
      for (int u = 0; u < NQ; ++u) rq[u] = shift_down(rq[u], min(max(over, 0), kPiece));
      if (DX) rs = settle(rs, kStep * s + 4 * (tt & 15));
    }
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      const int piece = tt + u * kThreads, row = piece >> 2, i = piece & 3;
      v4i w = rq[u];
      if (PACKED) {   // 16 * code; the sums are divided by 16 at the end
        const v2i a = expand16(static_cast<uint32_t>(w.x)), b = expand16(static_cast<uint32_t>(w.y));
        w = v4i{a.x, a.y, b.x, b.y};
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) *reinterpret_cast<int *>(sQ[slot] + code_slot(row, g, i)) = w[g];
    }
    if (DX) *reinterpret_cast<v4f *>(sS[slot] + 4 * tt) = rs;   // the first sixteen threads' are read
  };
  auto scaled = [&](v4f v, int i, int slot) {
    if (DX) {
      const v4f w = *reinterpret_cast<const v4f *>(sS[slot] + 16 * i + 4 * lg);
      v.x *= w.x; v.y *= w.y; v.z *= w.z; v.w *= w.w;   // rounded to float32, as a float graph has it
    }
    return v;
  };
  v4i d[kDigits];
  load_q(0);
  AQT_SCHED_FENCE();
  store_q(0, 0);
  load_q(clamped(1));
  AQT_SCHED_FENCE();
#pragma unroll
  for (int i = 0; i < 4; ++i) load_f(i, 0);
  AQT_SCHED_FENCE();
  __syncthreads();
  // Step s: its codes are in LDS slot s % 2, the next step's on their way.
  auto step = [&](auto parity, int s) {
    constexpr int P = decltype(parity)::value;
    store_q(P ^ 1, clamped(s + 1));   // a slot last read before the barrier that all have passed
    load_q(clamped(s + 2));
    AQT_SCHED_FENCE();   // the loads stay in this order: what is waited for first is requested first
    if (ragged(s)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) raw[i] = settle(raw[i], kStep * s + 16 * i + 4 * lg);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const v4f v = scaled(raw[i], i, P);
      digits4<FIRST>(v, up, plane, i, d);
      if (wide && list.fits()) list.note(v, doubtful, exponent, plane, lc, kStep * s + 16 * i + 4 * lg);
      load_f(i, clamped(s + 1));
    }
    AQT_SCHED_FENCE();
    multiply<TJ, true>(sQ[P], d, acc, lc, lg);
    __syncthreads();
  };
  for (int s = 0; s < steps; s += 2) {
    step(std::integral_constant<int, 0>{}, s);
    if (s + 1 < steps) step(std::integral_constant<int, 1>{}, s + 1);
  }

  };

  // ---- sums: the planes, then what they left ----
  v4d sum[TJ];
  auto take_sums = [&](int plane) {
    const int eg = anew(lane) >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double down = (PACKED ? 0.0625 : 1.0) * unscale_of(__shfl(exponent, 4 * eg + r)) * unit_of(plane);
      const bool fine = __shfl(static_cast<int>(x.finite()), 4 * eg + r) != 0;
#pragma unroll
      for (int j = 0; j < TJ; ++j) sum[j][r] = fine ? digits_sum<TJ>(acc, j, r) * down : 0.0;
    }
  };
  go_through(std::true_type{}, 0);
  take_sums(0);
  if (in_some_wave(flag[0])) {   // behind the sixth plane nothing is left of any value
    for (int plane = 1; in_some_wave(flag[1], wave, !list.fits()); ++plane) {
#pragma unroll
      for (int i = 0; i < 4 * TJ; ++i) above[i][t] = sum[i >> 2][i & 3];
      go_through(std::false_type{}, plane);
      take_sums(plane);
#pragma unroll
      for (int i = 0; i < 4 * TJ; ++i) sum[i >> 2][i & 3] = above[i][t] + sum[i >> 2][i & 3];
    }
  }
  const int el = anew(lane), ec = el & 15, eg = el >> 4;
  auto code_at = [&](int64_t n, int c) -> int {
    const uint8_t *const qr = q + (n < R ? n : R - 1) * row_bytes;
    if (PACKED) return static_cast<int>(static_cast<uint32_t>(qr[c >> 1]) << ((c & 1) ? 24 : 28)) >> 28;
    return static_cast<int8_t>(qr[c]);
  };
  wave_lds_order();
  for (int k = 0; k < list.n; k += 4) {   // four entries in turn as the positions of a product
    const double left = list.value(k + eg, f64_row(ec));
    const int at = list.at(k + eg);
    double code[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) code[j] = static_cast<double>(code_at(chan(j) + ec, at));
#pragma unroll
    for (int j = 0; j < TJ; ++j) sum[j] = mfma_f64(left, code[j], sum[j]);
  }
  if (!finite) {
    const int row = f64_row(ec);
    const bool fine = __shfl(static_cast<int>(x.finite()), row) != 0;
    const uint32_t fr = row_at(16 * wave + row);
    int last = -1;   // a step that is seen again is not added again
    for_all(0, [&](int s, const v4f (&seen)[4]) {
      bool some = false;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) some = some || !is_finite(seen[i][e]);
      if (s == last || !__any(some)) return;
      last = s;
      for (int c0 = kStep * s; c0 < kStep * (s + 1) && c0 < C; c0 += 16) {
        const int c = c0 + 4 * eg;
        v4f v = piece_at(strip, fr, c);
        if (DX) {
          const v4f w = piece_at(scale, 0, c);
          v.x *= w.x; v.y *= w.y; v.z *= w.z; v.w *= w.w;
        }
        v = settle(v, c);
        double code[TJ][4];
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) code[j][e] = static_cast<double>(code_at(chan(j) + ec, c + e < C ? c + e : C - 1));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double left = fine ? 0.0 : static_cast<double>(v[e]);
#pragma unroll
          for (int j = 0; j < TJ; ++j) sum[j] = mfma_f64(left, c + e < C ? code[j][e] : 0.0, sum[j]);
        }
      }
    });
  }

  constexpr int JS = GLU ? 2 : 1;
#pragma unroll
  for (int j = 0; j < TJ; j += JS) {
    const int64_t n = chan(j) + ec;
    const bool live = n < oc;
    const int64_t nc = live ? n : oc - 1, ng = nc + (GLU ? oc : 0);
    const double sc_a = DX ? 1.0 : scale[nc], sc_b = GLU ? scale[ng] : 0.0f;
    const float bias_a = bias ? bias[nc] : 0.0f, bias_b = (GLU && bias) ? bias[ng] : 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t m = m0 + 16 * wave + 4 * eg + r, at = m * oc + n;
      if (!live || m >= M) continue;
      if (DX) {
        float v = static_cast<float>(sum[j][r]);
        if (factor) v = v * factor[at];
        out[at] = (mask_x ? mask_bit(mask_x, at) : keep) ? v : 0.0f;
      } else {
        const float v = static_cast<float>(sum[j][r] * sc_a) + bias_a;
        float o = v;
        if (MODE == 1 + AQT_EPI_SWISH) o = swish_f32(v);
        else if (GLU) o = v * sigmoid_f32(static_cast<float>(sum[j + JS - 1][r] * sc_b) + bias_b);
        out[at] = o;
      }
    }
  }
  }
}

// ---- dW: contraction over the rows of both operands ---------------------------------------------
// partial[slab][k][n] = sum over the slab's rows of xq[m,k] dy[m,n].  A wavefront owns sixteen channels: its lanes load and
// convert the gradient column by column, which is fragment order as it stands.  The codes are gathered 4 positions x 8 rows
// a thread and written along the rows into LDS, position 4 g + b in LDS row b * BQ / 4 + g (neighbouring lanes write
// neighbouring rows).  Bias sums and slabs as in gemm_any_f64.hip.
template <int TJ>
__global__ __launch_bounds__(kThreads, 2) void bwd_dw_exact_kernel(const int8_t *__restrict__ xq, const float *__restrict__ dy,
                                                                   int64_t M, int64_t K, int64_t N, int64_t rows_per_slab,
                                                                   double *__restrict__ partial, float *__restrict__ dw,
                                                                   int tiles_k, int tiles_n, int slabs, DwFinish fin,
                                                                   double *__restrict__ bias_part) {
  constexpr int BQ = 16 * TJ, G = BQ / 4;   // G groups of four positions: the first 8 G threads gather 4 x 8 rows of codes each
  static_assert(8 * G <= kThreads);
  // behind the codes, 32 bytes for each thread that has none to write
  __shared__ __attribute__((aligned(16))) uint8_t sQ[2][BQ * kStep + (kThreads - 8 * G) * 32];
  const int t = threadIdx.x, lane = t & 63, lc = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int strip, kt;
  place(static_cast<int>(blockIdx.x), slabs * tiles_n, tiles_k, strip, kt);
  const int slab = strip / tiles_n;
  const int64_t k0 = static_cast<int64_t>(kt) * BQ, n0 = static_cast<int64_t>(strip % tiles_n) * kOwn;
  const int64_t m0 = slab * rows_per_slab;
  const int rows = static_cast<int>((m0 + rows_per_slab < M ? m0 + rows_per_slab : M) - m0);
  const int64_t n = n0 + 16 * wave + lc;
  const bool live = n < N;
  // uniform bases and 32-bit lane offsets; the row of element e of piece i in step s: 64 s + 16 i + 4 lg + e
  const float *const py = dy + m0 * N;
  const uint32_t own = static_cast<uint32_t>(4 * lg * N + (live ? n : N - 1)) * 4u, row_bytes = static_cast<uint32_t>(N) * 4u;
  auto dy_at = [&](int row, int more) {   // uniform rows, to which the lane adds its 4 lg; more < 64
    return load_f32(py + static_cast<int64_t>(row) * N, own, more * row_bytes);
  };
  const int8_t *const px = xq + m0 * K;
  const int whole = rows / kStep;

  auto guarded = [&](int s, int i) {
    v4f v;
    const int g4 = anew(4 * lg);   // or sixteen addresses stay in registers from plane to plane
#pragma unroll
    for (int e = 0; e < 4; ++e) {   // clamped: no branch around a load
      const int row = kStep * s + 16 * i + g4 + e;
      v[e] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(py + static_cast<int64_t>(min(row, rows - 1) - g4) * N) + own);
      if (row >= rows) v[e] = 0.0f;
    }
    return v;
  };
  constexpr int kAhead = 3;   // steps requested together
  const int steps = static_cast<int>(cdiv(rows, kStep));
  auto for_all = [&](auto each) {
    for (int s0 = 0; s0 < whole; s0 += kAhead) {
      v4f v[kAhead][4];
#pragma unroll
      for (int a = 0; a < kAhead; ++a)
#pragma unroll
        for (int i = 0; i < 16; ++i)   // the last step again: no branch around a load
          v[a][i >> 2][i & 3] = dy_at(kStep * (s0 + a < whole ? s0 + a : whole - 1), 16 * (i >> 2) + (i & 3));
#pragma unroll
      for (int a = 0; a < kAhead; ++a) each(s0 + a < whole ? s0 + a : whole - 1, v[a]);
    }
    if (whole < steps) {
      v4f v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = guarded(whole, i);
      each(whole, v);
    }
  };
  Extremes x;
  for_all([&](int, const v4f (&v)[4]) {
    uint32_t bits[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) bits[i] = __float_as_uint(fabsf(v[i >> 2][i & 3]));
    x.note(bits);
  });
  x.across_groups();
  const int exponent = x.exponent();
  const double up = x.finite() ? scale_of(exponent) : 0.0;
  const bool finite = !__any(!x.finite()), wide = __any(!x.exact());   // uniform
  __shared__ Left few[kThreads / 64][kFew];
  __shared__ double above[4 * TJ][kThreads];   // the sums of the planes above
  __shared__ int flag[2][kThreads / 64];
  set_flag(flag[0], wave, wide);

  // the digits of one plane (the first in code of its own, which most rows are done with)
  v4i acc[kDigits][TJ];
  LeftList list{few[wave]};
  double colsum = 0.0;          // of this lane's channel, over the steps that are this tile's turn
  auto go_through = [&](auto first, int plane) {
  constexpr bool FIRST = decltype(first)::value;
  const int tt = anew(t), g = tt % G, mg = tt / G;        // this thread's positions 4 g .. + 3 and rows 8 mg .. + 7 of a step
  const bool has = tt < 8 * G;
  int slot_of[4];                           // of positions 4 g + k, first four rows; the other four: 16 bytes to or fro
#pragma unroll
  for (int k = 0; k < 4; ++k) slot_of[k] = has ? code_slot(k * G + g, 2 * (mg & 1), mg >> 1) : BQ * kStep + (tt - 8 * G) * 32 + 4 * k;
  const int64_t kc = k0 + 4 * g;
  // a piece that would cross the end of its row is read so that it ends there (what lies behind the end altogether is not used)
  const int shift = 8 * (moved(kc, K, 4) & 3);
  const uint32_t at_q = static_cast<uint32_t>((has ? 8 * mg : 0) * K + (kc + 4 <= K ? kc : K - 4));
  list.n = 0;
  const uint32_t doubtful = x.doubtful(plane);
#pragma unroll
  for (int p = 0; p < kDigits; ++p)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[p][j] = v4i{0, 0, 0, 0};
  v4f raw[4];
  uint32_t rq[8];
  auto load_f = [&](int i, int s) {
#pragma unroll
    for (int e = 0; e < 4; ++e) raw[i][e] = dy_at(kStep * s, 16 * i + e);
  };
  auto load_q = [&](int s) {
#pragma unroll
    for (int i = 0; i < 8; ++i) rq[i] = load_at<uint32_t>(px + (static_cast<int64_t>(kStep) * s + i) * K + at_q);
  };
  auto store_q = [&](int slot) {
#pragma unroll
    for (int i = 0; i < 8; ++i) rq[i] >>= shift;
    auto pair = [](uint32_t a, uint32_t b, uint32_t sel) { return __builtin_amdgcn_perm(b, a, sel); };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t *const q = rq + 4 * h;
      const uint32_t a = pair(q[0], q[1], 0x05010400u), b = pair(q[2], q[3], 0x05010400u);
      const uint32_t c = pair(q[0], q[1], 0x07030602u), e = pair(q[2], q[3], 0x07030602u);
      const uint32_t along[4] = {pair(a, b, 0x05040100u), pair(a, b, 0x07060302u), pair(c, e, 0x05040100u), pair(c, e, 0x07060302u)};
#pragma unroll
      for (int k = 0; k < 4; ++k)
        *reinterpret_cast<uint32_t *>(sQ[slot] + (slot_of[k] ^ 16 * h)) = along[k];
    }
  };
  auto add_up = [&](int s, const v4f (&v)[4]) {
    if (!FIRST || !bias_part || s % tiles_k != kt) return;   // uniform
#pragma unroll
    for (int i = 0; i < 4; ++i)
      colsum += (static_cast<double>(v[i][0]) + static_cast<double>(v[i][1])) +
                (static_cast<double>(v[i][2]) + static_cast<double>(v[i][3]));
  };
  v4i d[kDigits];
  if (whole > 0) {
    auto clamped = [&](int s) { return s < whole ? s : whole - 1; };
    load_q(0);
    AQT_SCHED_FENCE();
    store_q(0);
    load_q(clamped(1));
    AQT_SCHED_FENCE();
#pragma unroll
    for (int i = 0; i < 4; ++i) load_f(i, 0);
    AQT_SCHED_FENCE();
    __syncthreads();
    // Step s: its codes are in LDS slot s % 2, the next step's on their way.
    auto step = [&](auto parity, int s) {
      constexpr int P = decltype(parity)::value;
      store_q(P ^ 1);   // a slot last read before the barrier that all have passed
      load_q(clamped(s + 2));
      AQT_SCHED_FENCE();   // the loads stay in this order: what is waited for first is requested first
      add_up(s, raw);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        digits4<FIRST>(raw[i], up, plane, i, d);
        if (wide && list.fits()) list.note(raw[i], doubtful, exponent, plane, lc, kStep * s + 16 * i + 4 * lg);
        load_f(i, clamped(s + 1));
      }
      AQT_SCHED_FENCE();
      multiply<TJ, false>(sQ[P], d, acc, lc, lg);
      __syncthreads();
    };
    for (int s = 0; s < whole; s += 2) {
      step(std::integral_constant<int, 0>{}, s);
      if (s + 1 < whole) step(std::integral_constant<int, 1>{}, s + 1);
    }
  }
  if (whole * kStep < rows) {
    const int first = anew(kStep * whole + (has ? 8 * mg : 0));
#pragma unroll
    for (int i = 0; i < 8; ++i)
      rq[i] = load_at<uint32_t>(px + static_cast<int64_t>(min(first + i, rows - 1)) * K + (kc + 4 <= K ? kc : K - 4));
    store_q(0);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      raw[i] = guarded(whole, i);
      digits4<FIRST>(raw[i], up, plane, i, d);
      if (wide && list.fits()) list.note(raw[i], doubtful, exponent, plane, lc, kStep * whole + 16 * i + 4 * lg);
    }
    add_up(whole, raw);
    multiply<TJ, false>(sQ[0], d, acc, lc, lg);
  }
  };

  // ---- sums: the planes, then what they left ----
  v4d sum[TJ];
  auto take_sums = [&](int plane) {
    const double down = unscale_of(exponent) * unit_of(plane);
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[j][r] = x.finite() ? digits_sum<TJ>(acc, j, r) * down : 0.0;
  };
  go_through(std::true_type{}, 0);
  take_sums(0);
  if (in_some_wave(flag[0])) {   // behind the sixth plane nothing is left of any value
    for (int plane = 1; in_some_wave(flag[1], wave, !list.fits()); ++plane) {
#pragma unroll
      for (int i = 0; i < 4 * TJ; ++i) above[i][t] = sum[i >> 2][i & 3];
      go_through(std::false_type{}, plane);
      take_sums(plane);
#pragma unroll
      for (int i = 0; i < 4 * TJ; ++i) sum[i >> 2][i & 3] = above[i][t] + sum[i >> 2][i & 3];
    }
  }
  if (bias_part) {
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) colsum += __shfl_xor(colsum, off);
    if (lg == 0 && live) bias_part[(static_cast<int64_t>(slab) * tiles_k + kt) * N + n] = colsum;
  }

  // tile row 16 j + x holds the position of LDS row 16 j + x
  auto position = [&](int row) { return k0 + 4 * (row % G) + row / G; };
  const int el = anew(lane), ec = el & 15, eg = el >> 4;   // the thread's place anew, as in the kernel above
  wave_lds_order();
  for (int k = 0; k < list.n; k += 4) {   // four entries in turn as the positions of a product
    const double left = list.value(k + eg, ec);
    const int8_t *const row = px + static_cast<int64_t>(list.at(k + eg)) * K;
    double code[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int64_t at = position(16 * j + f64_row(ec));
      code[j] = static_cast<double>(row[at < K ? at : K - 1]);
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) sum[j] = mfma_f64(code[j], left, sum[j]);
  }
  if (!finite) {
    int last = -1;
    for_all([&](int s, const v4f (&seen)[4]) {
      bool some = false;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) some = some || !is_finite(seen[i][e]);
      if (s == last || !__any(some)) return;
      last = s;
#pragma unroll 1
      for (int i = 0; i < 4; ++i) {
        const v4f v = guarded(s, i);   // zeros behind the slab
        double left[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) left[e] = x.finite() ? 0.0 : static_cast<double>(v[e]);
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          const int64_t k = position(16 * j + f64_row(ec));
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int row = kStep * s + 16 * i + 4 * eg + e;
            const double code = static_cast<double>(px[static_cast<int64_t>(row < rows ? row : rows - 1) * K + (k < K ? k : K - 1)]);
            sum[j] = mfma_f64(code, left[e], sum[j]);
          }
        }
      }
    });
  }
  const double sx = dw ? static_cast<double>(fin.s_x[0]) : 1.0;
#pragma unroll
  for (int j = 0; j < TJ; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t k = position(16 * j + 4 * eg + r), at = k * N + n;
      if (k >= K || !live) continue;
      if (dw) dw[at] = dw_value(sum[j][r], at, n, fin, sx);
      else partial[static_cast<int64_t>(slab) * K * N + at] = sum[j][r];
    }
}

// Tiles of at most five blocks of sixteen (four where a value block needs its gate block beside it), as even as they come; least: 4.
struct Tiling {
  int tiles, blocks;
};
Tiling tiling(int64_t blocks, int least, int unit) {
  const int64_t tiles = cdiv(blocks, unit == 2 ? 4 : 5);
  int64_t per = cdiv(cdiv(blocks, tiles), unit) * unit;
  return Tiling{static_cast<int>(cdiv(blocks, per < least ? least : per)), static_cast<int>(per < least ? least : per)};
}

template <int TJ, bool PACKED, int MODE>
aqt_status f32_codes_exact(const CodesArgs &a, int tiles_r, hipStream_t st) {
  const int64_t tm = cdiv(a.M, kOwn);
  if (tm * tiles_r > 0x7FFFFFFF) return AQT_ERR_UNSUPPORTED;
  // column tiles in turn as long as two workgroups per compute unit are left
  const int64_t each = tm * tiles_r >= 2 * 512 ? cdiv(tiles_r, cdiv(512, tm)) : 1;
  f32_codes_exact_kernel<TJ, PACKED, MODE><<<static_cast<unsigned>(tm * cdiv(tiles_r, each)), kThreads, 0, st>>>(
      a.f, a.scale, static_cast<const uint8_t *>(a.q), a.M, a.R, static_cast<int>(a.C), a.s_x, a.mask_x, a.factor, a.bias,
      a.out, static_cast<int>(tm), tiles_r, static_cast<int>(each));
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

template <bool PACKED, int MODE>
aqt_status f32_codes_sized(const CodesArgs &a, hipStream_t st) {
  if constexpr (MODE == 1 + AQT_EPI_GLU) {
    const Tiling g = tiling(2 * cdiv(a.R / 2, 16), 4, 2);
    return f32_codes_exact<4, PACKED, MODE>(a, g.tiles, st);
  } else {
    const Tiling g = tiling(cdiv(a.R, 16), 4, 1);
    return g.blocks == 4 ? f32_codes_exact<4, PACKED, MODE>(a, g.tiles, st) : f32_codes_exact<5, PACKED, MODE>(a, g.tiles, st);
  }
}

}  // namespace

// Fewer results than this leave compute units idle while a workgroup goes through the contraction, which gemm_any_f64.hip splits
// instead; below 128 positions the search for the extremes and the sums outweigh the steps.  Measured in us, there / here / here with a
// softmax's gradient (logits of standard deviation 3), which takes two planes; there the values do not matter:
//   dX M x K of N positions: 4099 x 520 of 1000 114 / 46 / 74, 4099 x 1000 of 520 103 / 54 / 90, 9000 x 520 of 2040 392 / 144 / 256,
//   5000 x 520 of 520 73 / 45 / 76, 10008 x 144 of 576 53 / 34 / 51, 10008 x 144 of 432 44 / 25 / 41, 3000 x 700 of 300 40 / 25 / 36;
//   where a second plane costs more than the first one gains: 10008 x 144 of 144 20 / 16 / 27, 10008 x 576 of 144 48 / 38 / 74,
//   1300 x 400 of 400 24 / 18 / 32, 5200 x 144 of 576 32 / 25 / 39;
//   given up on one side of the line: 1300 x 400 of 1200 47 / 42 / 68, 4000 x 1001 of 100 31 / 27 / 43, 16000 x 72 of 72 15 / 13 / 20; on the
//   other: 2600 x 288 of 288 18 / 18 / 29, 2600 x 288 of 1152 45 / 39 / 64; right of it 520 x 520 of 1000 27 / 30 / 58, 300 x 1030 of 2040
//   48 / 53 / 104, 30000 x 96 of 96 24 / 26 / 41;
//   weight-only 4099 x 1000 of 520 106 / 48 / 86, 520 x 1000 of 520 28 / 18 / 34, 4000 x 1001 of 100 30 / 25 / 40, 300 x 1030 of 2040 48 / 43 / 90.
bool f32_codes_exact_ok(int64_t M, int64_t R, int64_t C) {
  return C >= 128 && C <= kLongest && M * R >= (C > 1024 ? C * 488 : 500000);
}

aqt_status launch_bwd_dx_exact(const float *dy, const int8_t *wq_kn, const float *s_w, const float *s_x, const uint32_t *mask_x,
                               const float *factor, int64_t M, int64_t K, int64_t N, float *dx, hipStream_t st) {
  return f32_codes_sized<false, 0>(CodesArgs{dy, s_w, wq_kn, M, K, N, s_x, mask_x, factor, nullptr, dx}, st);
}

template <bool PACKED>
static aqt_status wonly(const CodesArgs &a, int epilogue, hipStream_t st) {
  return epilogue == AQT_EPI_NONE    ? f32_codes_sized<PACKED, 1 + AQT_EPI_NONE>(a, st)
         : epilogue == AQT_EPI_SWISH ? f32_codes_sized<PACKED, 1 + AQT_EPI_SWISH>(a, st)
                                     : f32_codes_sized<PACKED, 1 + AQT_EPI_GLU>(a, st);
}
aqt_status launch_dense_fwd_wonly_exact(const float *x, const void *wq_packed, const float *s_w, int64_t M, int64_t K,
                                        int64_t N, int bits_w, const float *bias, int epilogue, float *y, hipStream_t st) {
  const CodesArgs a{x, s_w, wq_packed, M, N, K, nullptr, nullptr, nullptr, bias, y};
  return packed4(bits_w) ? wonly<true>(a, epilogue, st) : wonly<false>(a, epilogue, st);
}

// Rows enough for two steps, and so many products (of whole tiles) that one launch more or less of a step does not decide.  us, as above,
// M x K x N: 10008 x 144 x 144 30 / 22 / 31, 2600 x 288 x 288 27 / 22 / 30, 800 x 400 x 400 24 / 17 / 25, 200 x 520 x 1000 25 / 20 / 28,
// 16000 x 72 x 72 26 / 18 / 26, 130 x 2000 x 2000 42 / 32 / 55, 4099 x 520 x 1000 118 / 50 / 81; below the line 128 x 520 x 1000 14 / 13 / 20,
// 64 x 2000 x 2000 23 / 24 / 34, 1024 x 144 x 576 17 / 15 / 23, 6000 x 100 x 100 16 / 15 / 23, 600 x 72 x 72 13 / 13 / 20.
bool dw_exact_ok(int64_t M, int64_t K, int64_t N, int slabs) {
  const Tiling g = tiling(cdiv(K, 16), 4, 1);
  return M >= 2 * kStep && K >= 4 && K < (1 << 24) && N < (1 << 24) &&   // 32-bit byte offsets inside a step
         M * (static_cast<int64_t>(g.tiles) * 16 * g.blocks) * (cdiv(N, kOwn) * kOwn) >= 100000000 &&
         cdiv(cdiv(M, slabs), kStep) * kStep <= kLongest;
}

// Slabs of rows so that two workgroups per compute unit have work, of at least 128 rows each.
int dw_exact_slabs(int64_t M, int64_t K, int64_t N) {
  const int64_t wish = 512 / (tiling(cdiv(K, 16), 4, 1).tiles * cdiv(N, kOwn)), fill = wish > 0 ? wish : 1;
  const int64_t most = cdiv(M, 128), least = cdiv(M, kLongest);
  const int64_t slabs = fill < most ? fill : most;
  return static_cast<int>(slabs > least ? slabs : least);
}

aqt_status launch_bwd_dw_exact(const float *dy, const int8_t *xq, const float *s_x, const float *s_w, const uint32_t *mask_w,
                               int64_t M, int64_t K, int64_t N, float *dw, double *partial, int slabs, float *dbias,
                               double *bias_part, hipStream_t st) {
  const Tiling g = tiling(cdiv(K, 16), 4, 1);
  const int64_t rows = cdiv(cdiv(M, slabs), kStep) * kStep, used = cdiv(M, rows), tiles_n = cdiv(N, kOwn);
  if (g.tiles * tiles_n * used > 0x7FFFFFFF) return AQT_ERR_UNSUPPORTED;
  const DwFinish fin{s_x, s_w, mask_w};
  const bool one = used == 1;
  auto kern = g.blocks == 4 ? bwd_dw_exact_kernel<4> : bwd_dw_exact_kernel<5>;
  kern<<<static_cast<unsigned>(g.tiles * tiles_n * used), kThreads, 0, st>>>(
      xq, dy, M, K, N, rows, partial, one ? dw : nullptr, g.tiles, static_cast<int>(tiles_n), static_cast<int>(used), fin,
      dbias ? bias_part : nullptr);
  AQT_HIP(hipGetLastError());
  return launch_dw_f64_fold(partial, static_cast<int>(used), K, N, s_x, s_w, mask_w, one ? nullptr : dw, bias_part,
                            static_cast<int>(used) * g.tiles, dbias, st);
}

}  // namespace aqt
