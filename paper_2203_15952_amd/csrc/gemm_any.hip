// The contractions of the quantized dense layer straight from the caller's tensors, without a re-ordered operand or a
// pre-pass (arxiv 2203.15952, Sec. 1 and Sec. 2.2; the straight-through backward; Sec. 4.1 for the weight-only modes):
//   the forward, integer sums, for any shape that no tile of the tuned kernel in gemm_fwd.hip divides, and for problems
//   too small to fill the chip with its tiles;
//   dX, dW and the weight-only forward for problems on the grid of the tuned kernels in gemm_bwd.hip (which checks
//   it: whole column tiles, 16-byte aligned tensors) that are too small for their tiles.  Off that grid gemm_any_f64.hip.
//
// A workgroup is WM x WN wavefronts side by side, times WK groups of them that share one output tile and take turns
// along the contraction.  Each group brings a slice of its tile's rows through registers into LDS, whole 64- or
// 128-byte row pieces at a time, converts what has to be converted there once for all its wavefronts, and multiplies
// while the next two slices' loads are in flight.  (Fragments fetched straight from memory, one row per lane, were
// tried first: rows a power of two apart share a cache set and every access misses; dX 40 x 2048 -> 512 took 20 us
// that way, 11 us this way.)  Small problems (WK = 8, one wavefront per group) are bound by the latency of a trip to
// memory, so eight slices are in flight at a time; the sums are added up through LDS.
// Measured against the one-thread-per-output kernels these replace: forward 4099 x 520 x 1000, int8 codes, 17 us (7902);
// 40 x 512 -> 2048 3.5 us (about 170).
#include "any_shape.h"
#include "bf16_terms.h"
#include "colsum.h"
#include "epilogue.h"
#include "quant_code.h"

namespace aqt {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

// LDS rows are CH chunks of 16 bytes without padding; the chunk index is XORed with row bits so that the rows
// of a fragment read spread over all banks.
template <int CH>
__device__ __forceinline__ int swz(int row) {
  return CH >= 8 ? (row & 7) : CH == 4 ? ((row >> 1) & 3) : ((row >> 2) & 1);
}
template <int CH>
__device__ __forceinline__ int chunk_at(int row, int chunk) { return row * (CH * 16) + ((chunk ^ swz<CH>(row)) << 4); }

// ---- forward: int8 codes x int8 / int4 codes, int32 sums -----------------------------------
// A wavefront owns TM x TN blocks of 32 x 32; a GLU tile pairs value (even) and gate (odd) column blocks.
// BK: fan-in positions per slice.
// FILL: where a tile's codes come from when they are not in xq: fill(lds, slice bytes, tile row, tile column, scales) makes them from
// float32 rows, at most one slice to each of the WK wavefronts, at the place of each slice's A rows, and returns the scale; with
// kWeights those of the tile's B rows too, as bytes, and their scales.
struct FromCodes {
  static constexpr bool kFills = false, kWeights = false;
};
template <int TM, int TN, int WM, int WN, int WK, int BK, bool PACKED, int EPI, class FILL>
__device__ __forceinline__ void dense_fwd_any_body(
    const int8_t *__restrict__ xq, const float *__restrict__ s_x, const uint8_t *__restrict__ wq,
    const float *__restrict__ s_w, int64_t M, int64_t K, int64_t N, const float *__restrict__ bias,
    float *__restrict__ y, int32_t *__restrict__ acc_out, uint32_t *__restrict__ y_absmax, float *__restrict__ dact,
    int tiles_n, const FILL &fill) {
  static_assert(16 % WK == 0 && (EPI != AQT_EPI_GLU || TN % 2 == 0), "the epilogue is shared out by registers");
  constexpr bool GLU = EPI == AQT_EPI_GLU;
  constexpr int G = 64 * WM * WN;                       // threads of a group
  constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
  constexpr int CHA = BK / 16, CHB = PACKED ? BK / 32 : BK / 16;   // 16-byte chunks per row
  constexpr int NA = BM * CHA / G, NB = BN * CHB / G;   // chunks per thread and slice
  static_assert(NA * G == BM * CHA && NB * G == BN * CHB && NA > 0 && NB > 0, "whole chunks per thread");
  constexpr int kSliceBytes = BM * CHA * 16 + BN * CHB * 16;
  constexpr int kRedBytes = WK > 1 ? WK * TM * TN * 16 * 64 * 4 : 0;
  constexpr int kBuffers = WK == 1 ? 2 : WK;            // two slots for a shared slice, one per private one
  constexpr int kLds = kBuffers * kSliceBytes > kRedBytes ? kBuffers * kSliceBytes : kRedBytes;
  __shared__ __attribute__((aligned(16))) uint8_t lds[kLds];
  const int t = threadIdx.x, lane = t & 63, lr = lane & 31, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wk = wave / (WM * WN), wn = wave % WN, wm = (wave / WN) % WM, gt = t - wk * G;
  const int64_t bm = blockIdx.x / tiles_n, bn = blockIdx.x % tiles_n;
  const int64_t oc = GLU ? N / 2 : N;
  // first channel of the tile's column block cb
  auto chan = [&](int cb) -> int64_t {
    if (GLU) return bn * (BN / 2) + (cb >> 1) * 32 + ((cb & 1) ? oc : 0);
    return bn * BN + cb * 32;
  };
  const int64_t row_bytes = PACKED ? (K + 1) / 2 : K;
  const uint8_t *pa[NA], *pb[NB];
#pragma unroll
  for (int u = 0; u < NA; ++u) {
    const int64_t m = bm * BM + (gt + u * G) / CHA;
    pa[u] = FILL::kFills ? nullptr : reinterpret_cast<const uint8_t *>(xq) + (m < M ? m : M - 1) * K;
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int r = (gt + u * G) / CHB;
    const int64_t n = chan(r >> 5) + (r & 31);
    pb[u] = FILL::kWeights ? nullptr : wq + (n < N ? n : N - 1) * row_bytes;
  }
  // G is a multiple of the chunks per row: a thread's chunks sit at the same place of their rows
  const int ca = gt % CHA, cb = gt % CHB;
  v4i ra[2][NA], rb[2][NB];
  constexpr int kRowSlice = PACKED ? BK / 2 : BK;   // bytes of a weight row per slice
  const bool narrow = K < 16 || row_bytes < 16;     // uniform
  auto load = [&](auto set, int64_t slice) {
    constexpr int S = decltype(set)::value;
    const int64_t a0 = slice * BK + 16 * ca, b0 = slice * kRowSlice + 16 * cb;
    const int64_t at = a0 + 16 <= K ? a0 : K - 16, bt = b0 + 16 <= row_bytes ? b0 : row_bytes - 16;
    if constexpr (!FILL::kFills) {
#pragma unroll
      for (int u = 0; u < NA; ++u) ra[S][u] = load_at<v4i>(pa[u] + at);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) rb[S][u] = load_at<v4i>(pb[u] + bt);
  };
  auto load_narrow = [&](auto set) {   // fewer than 32 positions: part of the first slice
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int u = 0; u < NA; ++u) ra[S][u] = load16_guarded(pa[u], 16 * ca, K);
#pragma unroll
    for (int u = 0; u < NB; ++u) rb[S][u] = load16_guarded(pb[u], 16 * cb, row_bytes);
  };
  v16i acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
  // slot: where a slice lives in LDS (its A rows, then its B rows)
  auto stage = [&](auto set, int64_t slice, uint8_t *slot) {
    constexpr int S = decltype(set)::value;
    if ((slice + 1) * BK > K && !narrow) {
      const int da = moved(slice * BK + 16 * ca, K, 16), db = moved(slice * kRowSlice + 16 * cb, row_bytes, 16);
      if constexpr (!FILL::kFills) {
#pragma unroll
        for (int u = 0; u < NA; ++u) ra[S][u] = shift_down(ra[S][u], da);
      }
#pragma unroll
      for (int u = 0; u < NB; ++u) rb[S][u] = shift_down(rb[S][u], db);
    }
    if constexpr (!FILL::kFills) {
#pragma unroll
      for (int u = 0; u < NA; ++u) *reinterpret_cast<v4i *>(slot + chunk_at<CHA>((gt + u * G) / CHA, ca)) = ra[S][u];
    }
#pragma unroll
    for (int u = 0; u < NB; ++u)
      *reinterpret_cast<v4i *>(slot + BM * CHA * 16 + chunk_at<CHB>((gt + u * G) / CHB, cb)) = rb[S][u];
  };
  auto multiply = [&](const uint8_t *slot) {
    const uint8_t *const sA = slot, *const sB = slot + BM * CHA * 16;
#pragma unroll
    for (int kk = 0; kk < BK / 32; ++kk) {
      v4i a[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        a[i] = *reinterpret_cast<const v4i *>(sA + chunk_at<CHA>((wm * TM + i) * 32 + lr, 2 * kk + lk));
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        v4i b;
        if (PACKED) {
          const v2i w = *reinterpret_cast<const v2i *>(sB + chunk_at<CHB>((wn * TN + j) * 32 + lr, kk) + 8 * lk);
          const v2i lo = expand16(static_cast<uint32_t>(w.x)), hi = expand16(static_cast<uint32_t>(w.y));
          b = v4i{lo.x, lo.y, hi.x, hi.y};
        } else {
          b = *reinterpret_cast<const v4i *>(sB + chunk_at<CHB>((wn * TN + j) * 32 + lr, 2 * kk + lk));
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b, acc[i][j], 0, 0, 0);
      }
    }
  };
  float sx;
  __shared__ float scales[FILL::kWeights ? BN : 1];
  static_assert(!FILL::kWeights || (TN == 1 && WN == 1 && !PACKED), "one block of byte rows");
  if constexpr (FILL::kFills) {
    static_assert(WM * WN * TM == 1 && BK == 64, "32 rows, one slice to a wavefront");
    constexpr std::integral_constant<int, 0> set0{};
    const bool mine = wk < cdiv(K, BK);   // uniform
    if (!FILL::kWeights && mine) load(set0, wk);
    sx = fill(lds, kSliceBytes, bm, bn, scales);
    __syncthreads();
    if (mine) {
      if constexpr (!FILL::kWeights) {
        stage(set0, wk, lds + wk * kSliceBytes);
        wave_lds_order();
      }
      multiply(lds + wk * kSliceBytes);
    }
  } else {
    if (!narrow) run_slices<WK>(lds, kSliceBytes, wk, cdiv(K, BK), load, stage, multiply);
    else if (wk == 0) run_narrow<WK>(lds, load_narrow, stage, multiply);
    sx = s_x[0];
  }

  // The groups of a tile add their sums (integers: any order) and share the epilogue: each takes 16 / WK of the
  // accumulator registers.
  constexpr int RW = 16 / WK;
  int *const red = reinterpret_cast<int *>(lds);
  static_assert(WK == 1 || WM * WN == 1, "the sums of a split contraction are kept per wavefront");
  if (WK > 1) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) red[(((wk * TM + i) * TN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
    __syncthreads();
  }
  auto sum_of = [&](int i, int j, int rr) -> int {   // register wk * RW + rr
    int v;
    if (WK > 1) {
      v = 0;
#pragma unroll
      for (int w = 0; w < WK; ++w) v += red[(((w * TM + i) * TN + j) * 16 + wk * RW + rr) * 64 + lane];
    } else {
      v = acc[i][j][rr];
    }
    return PACKED ? (v >> 4) : v;
  };
  uint32_t amax = 0u;
  constexpr int JS = GLU ? 2 : 1;
  const int64_t m_lane = bm * BM + wm * 32 * TM + 4 * lk;   // this lane's first row
#pragma unroll
  for (int j = 0; j < TN; j += JS) {
    const int64_t n = chan(wn * TN + j) + lr;
    const bool live = n < oc;
    const int64_t nc = live ? n : oc - 1, ng = nc + (GLU ? oc : 0);
    const float sc_a = sx * (FILL::kWeights ? scales[nc - bn * BN] : s_w[nc]), bias_a = bias ? bias[nc] : 0.0f;
    const float sc_b = GLU ? sx * s_w[ng] : 0.0f, bias_b = (GLU && bias) ? bias[ng] : 0.0f;
    const int rows = live ? static_cast<int>(M - m_lane < BM ? M - m_lane : BM) : 0;   // rows of this lane's column in the tensor
    float *const yl = y + m_lane * oc + n, *const dl = dact + m_lane * N + n;
    int32_t *const al = acc_out + m_lane * N + n;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int rr = 0; rr < RW; ++rr) {
        const int r = wk * RW + rr, row = i * 32 + 8 * (r >> 2) + (r & 3);   // the same in every lane
        const int a0 = sum_of(i, j, rr);
        const int a1 = GLU ? sum_of(i, j + JS - 1, rr) : 0;
        if (row >= rows) continue;
        if (acc_out) {
          al[row * N] = a0;
          if (GLU) al[row * N + oc] = a1;
        }
        const float v = dequant_f32(a0, sc_a) + bias_a;
        float out = v;
        if (EPI == AQT_EPI_SWISH) {
          const float sg = sigmoid_f32(v);
          out = v * sg;
          if (dact) dl[row * N] = swish_dact_f32(v, sg);
        } else if (GLU) {
          const float sg = sigmoid_f32(dequant_f32(a1, sc_b) + bias_b);
          out = v * sg;
          if (dact) {
            dl[row * N] = sg;
            dl[row * N + oc] = glu_gate_dact_f32(v, sg);
          }
        }
        yl[row * oc] = out;
        amax = max(amax, __float_as_uint(out) & 0x7FFFFFFFu);
      }
  }
  // Uniform: one atomic per workgroup, and only if it can raise the word (it only grows).  The workgroups of a first round all
  // find it at zero and queue at it: 40 x 512 -> 2048 with Swish 8.5 us with one per wavefront, 5.3; 1302 x 144 -> 576 12.3, 9.3.
  if (y_absmax) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) amax = max(amax, static_cast<uint32_t>(__shfl_xor(static_cast<int>(amax), off)));
    constexpr int kWaves = WM * WN * WK;
    __shared__ uint32_t wave_max[kWaves];
    if (lane == 0) wave_max[wave] = amax;
    __syncthreads();
    if (t == 0) {
#pragma unroll
      for (int w = 1; w < kWaves; ++w) amax = max(amax, wave_max[w]);
      if (amax > *reinterpret_cast<volatile uint32_t *>(y_absmax)) atomicMax(y_absmax, amax);
    }
  }
}

template <int TM, int TN, int WM, int WN, int WK, int BK, bool PACKED, int EPI>
__global__ __launch_bounds__(64 * WM * WN * WK, WM * WN == 8 ? 4 : 2) void dense_fwd_any_kernel(
    const int8_t *__restrict__ xq, const float *__restrict__ s_x, const uint8_t *__restrict__ wq,
    const float *__restrict__ s_w, int64_t M, int64_t K, int64_t N, const float *__restrict__ bias,
    float *__restrict__ y, int32_t *__restrict__ acc_out, uint32_t *__restrict__ y_absmax, float *__restrict__ dact,
    int tiles_n) {
  dense_fwd_any_body<TM, TN, WM, WN, WK, BK, PACKED, EPI>(xq, s_x, wq, s_w, M, K, N, bias, y, acc_out, y_absmax, dact, tiles_n,
                                                          FromCodes{});
}

// ---- float32 operand x codes ------------------------------------------------------------------
// Codes are exact in bf16; the float operand is carried whole, as three bf16 terms of 8 significant bits each
// (a = hi + mid + lo exactly), and three v_mfma_f32_32x32x16_bf16 passes form products that are exact in
// float32.  Sums run in float32 over at most kChain contraction positions and are added up in float64.  (The tuned
// kernels that would otherwise take these shapes carry two terms and one float32 sum: error against float64 2.4e-6 of
// the result at 1024 x 256 x 1024, here 1.1e-7 for dX, 8e-8 for dW.)  An infinity, or a finite value above bf16's
// largest, gives NaN, as it does in the tuned kernels.
constexpr int kChain = 512;
constexpr int kCh = 4;        // 16-byte chunks of an LDS row: kSlice bf16 values

// four floats -> their four bf16 pieces of each of the three images
__device__ __forceinline__ void store_split(uint8_t *at, int image, v4f v) {
  v2i h, m, l;
  int x, y, z;
  split3_bf16(v.x, v.y, x, y, z); h.x = x; m.x = y; l.x = z;
  split3_bf16(v.z, v.w, x, y, z); h.y = x; m.y = y; l.y = z;
  *reinterpret_cast<v2i *>(at) = h;
  *reinterpret_cast<v2i *>(at + image) = m;
  *reinterpret_cast<v2i *>(at + 2 * image) = l;
}
__device__ __forceinline__ v4i codes8_bf16(uint32_t x, uint32_t y) {   // eight int8 codes in order
  float f[8];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[e] = static_cast<float>(static_cast<int8_t>(x >> (8 * e)));
    f[4 + e] = static_cast<float>(static_cast<int8_t>(y >> (8 * e)));
  }
  return v4i{static_cast<int>(pack_bf16(f[0], f[1])), static_cast<int>(pack_bf16(f[2], f[3])),
             static_cast<int>(pack_bf16(f[4], f[5])), static_cast<int>(pack_bf16(f[6], f[7]))};
}
__device__ __forceinline__ v4i nibbles8_bf16(uint32_t w) {   // eight int4 codes, low nibble first
  float f[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = static_cast<float>(static_cast<int>(w << (28 - 4 * e)) >> 28);
  return v4i{static_cast<int>(pack_bf16(f[0], f[1])), static_cast<int>(pack_bf16(f[2], f[3])),
             static_cast<int>(pack_bf16(f[4], f[5])), static_cast<int>(pack_bf16(f[6], f[7]))};
}

// out[m, r] = sum_c f[m, c] (* scale[c]) * q[r, c]: rows of both operands contraction-contiguous.
//   MODE 0 (dX):   f = dy [M,N], scale = s_w, q = wq_kn [K,N]; out times the clip mask and the factor
//   MODE 1 + e:    weight-only forward with epilogue e: f = x [M,K], q = the forward weight operand [N][K]
// Eight wavefronts share a tile of 32 rows x 32 TN columns and take turns along the contraction.
// LONG: a wavefront's share of the contraction exceeds kChain, so float32 sums are moved to float64 on the way.
template <int TN, bool LONG>
constexpr int codes_lds_bytes() {
  constexpr int slices = 8 * (3 * 32 + 32 * TN) * 64, sums = 8 * TN * 16 * 64 * (LONG ? 8 : 4);
  return slices > sums ? slices : sums;
}
template <int TN, bool PACKED, int MODE, bool LONG>
__device__ __forceinline__ void f32_codes_tile(
    uint8_t *lds, unsigned block, const float *__restrict__ f, const float *__restrict__ scale, const uint8_t *__restrict__ q,
    int64_t M, int64_t R, int64_t C, const float *__restrict__ s_x, const uint32_t *__restrict__ mask_x,
    const float *__restrict__ factor, const float *__restrict__ bias, float *__restrict__ out, int tiles_r) {
  static_assert(MODE != 1 + AQT_EPI_GLU || TN % 2 == 0, "a GLU tile pairs value and gate blocks");
  constexpr bool DX = MODE == 0, GLU = MODE == 1 + AQT_EPI_GLU;
  constexpr int WK = 8, G = 64, BM = 32, BN = 32 * TN;
  constexpr int NA = BM * 8 / G, NB = BN * 2 / G;   // pieces of four floats, of sixteen codes, per thread and slice
  constexpr int kImage = BM * 64;
  constexpr int kSliceBytes = 3 * kImage + BN * 64;
  const int lane = threadIdx.x & 63, lr = lane & 31, lk = lane >> 5;
  const int wk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t bm = block / tiles_r, br = block % tiles_r;
  const int64_t oc = GLU ? R / 2 : R;
  auto chan = [&](int cb) -> int64_t {
    if (GLU) return br * (BN / 2) + (cb >> 1) * 32 + ((cb & 1) ? oc : 0);
    return br * BN + cb * 32;
  };
  const int64_t row_bytes = PACKED ? C / 2 : C;
  const float *pf[NA];
  const uint8_t *pq[NB];
  const int piece = lane & 7;   // a thread's pieces sit at the same place of their rows
#pragma unroll
  for (int u = 0; u < NA; ++u) {
    const int64_t m = bm * BM + ((lane + u * G) >> 3);
    pf[u] = f + (m < M ? m : M - 1) * C;
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int r = (lane + u * G) >> 1;
    const int64_t n = chan(r >> 5) + (r & 31);
    pq[u] = q + n * row_bytes;
  }
  v4f ra[2][NA], rs[2] = {{1.0f, 1.0f, 1.0f, 1.0f}, {1.0f, 1.0f, 1.0f, 1.0f}};
  v4i rb[2][NB];
  constexpr int kPiece = PACKED ? 8 : 16;   // bytes of sixteen codes
  auto load = [&](auto set, int64_t slice) {
    constexpr int S = decltype(set)::value;
    const int64_t c = slice * kSlice + 4 * piece, at = slice * (2 * kPiece) + kPiece * (lane & 1);
#pragma unroll
    for (int u = 0; u < NA; ++u) ra[S][u] = load_at<v4f>(pf[u] + c);
    if (DX) rs[S] = load_at<v4f>(scale + c);
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      if (PACKED) {
        const v2i w = load_at<v2i>(pq[u] + at);
        rb[S][u] = v4i{w.x, w.y, 0, 0};
      } else {
        rb[S][u] = load_at<v4i>(pq[u] + at);
      }
    }
  };
  v16f acc[TN];
  double sum[LONG ? TN : 1][16];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc[j][r] = 0.0f;
      if (LONG) sum[LONG ? j : 0][r] = 0.0;
    }
  auto fold = [&]() {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sum[LONG ? j : 0][r] += static_cast<double>(acc[j][r]);
        acc[j][r] = 0.0f;
      }
  };
  int since = 0;
  auto stage = [&](auto set, int64_t slice, uint8_t *slot) {
    constexpr int S = decltype(set)::value;
    uint8_t *const sA = slot, *const sB = slot + 3 * kImage;
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      v4f v = ra[S][u];
      if (DX) { v.x *= rs[S].x; v.y *= rs[S].y; v.z *= rs[S].z; v.w *= rs[S].w; }
      store_split(sA + chunk_at<kCh>((lane + u * G) >> 3, piece >> 1) + 8 * (piece & 1), kImage, v);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int r = (lane + u * G) >> 1, c0 = 2 * (lane & 1);
      const v4i w = rb[S][u];
      const uint32_t w0 = static_cast<uint32_t>(w.x), w1 = static_cast<uint32_t>(w.y), w2 = static_cast<uint32_t>(w.z),
                     w3 = static_cast<uint32_t>(w.w);
      *reinterpret_cast<v4i *>(sB + chunk_at<kCh>(r, c0)) = PACKED ? nibbles8_bf16(w0) : codes8_bf16(w0, w1);
      *reinterpret_cast<v4i *>(sB + chunk_at<kCh>(r, c0 + 1)) = PACKED ? nibbles8_bf16(w1) : codes8_bf16(w2, w3);
    }
  };
  auto multiply = [&](const uint8_t *slot) {
    const uint8_t *const sA = slot, *const sB = slot + 3 * kImage;
#pragma unroll
    for (int kk = 0; kk < kSlice / 16; ++kk) {
      v4i b[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const v4i *>(sB + chunk_at<kCh>(j * 32 + lr, 2 * kk + lk));
#pragma unroll
      for (int img = 2; img >= 0; --img) {   // smallest terms first
        const v4i a = *reinterpret_cast<const v4i *>(sA + img * kImage + chunk_at<kCh>(lr, 2 * kk + lk));
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[j] = mfma_bf16(a, b[j], acc[j]);
      }
    }
    if (LONG && ++since == kChain / kSlice) {
      fold();
      since = 0;
    }
  };
  run_slices<WK>(lds, kSliceBytes, wk, C / kSlice, load, stage, multiply);
  if (LONG) fold();
  constexpr int RW = 16 / WK;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int at = ((wk * TN + j) * 16 + r) * 64 + lane;
      if (LONG) reinterpret_cast<double *>(lds)[at] = sum[LONG ? j : 0][r];
      else reinterpret_cast<float *>(lds)[at] = acc[j][r];
    }
  __syncthreads();
  auto sum_of = [&](int j, int rr) -> double {   // register wk * RW + rr, the wavefronts' shares in order
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      const int at = ((w * TN + j) * 16 + wk * RW + rr) * 64 + lane;
      v += LONG ? reinterpret_cast<const double *>(lds)[at] : static_cast<double>(reinterpret_cast<const float *>(lds)[at]);
    }
    return v;
  };
  const int64_t m_lane = bm * BM + 4 * lk;   // this lane's first row
  if (DX) {
    const bool keep = s_x[0] != 0.0f;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t n = chan(j) + lr, at0 = m_lane * R + n;
      const int rows = static_cast<int>(M - m_lane < BM ? M - m_lane : BM);
#pragma unroll
        for (int rr = 0; rr < RW; ++rr) {
          const int r = wk * RW + rr, row = 8 * (r >> 2) + (r & 3);   // the same in every lane
          float v = static_cast<float>(sum_of(j, rr));
          if (row >= rows) continue;
          const int64_t at = at0 + row * R;
          if (factor) v = v * factor[at];
          out[at] = (mask_x ? mask_bit(mask_x, at) : keep) ? v : 0.0f;
        }
    }
    return;
  }
  constexpr int JS = GLU ? 2 : 1;
#pragma unroll
  for (int j = 0; j < TN; j += JS) {
    const int64_t n = chan(j) + lr, ng = n + (GLU ? oc : 0);
    const double sc_a = scale[n], sc_b = GLU ? scale[ng] : 0.0f;
    const float bias_a = bias ? bias[n] : 0.0f, bias_b = (GLU && bias) ? bias[ng] : 0.0f;
    const int rows = static_cast<int>(M - m_lane < BM ? M - m_lane : BM);
    float *const ol = out + m_lane * oc + n;
#pragma unroll
      for (int rr = 0; rr < RW; ++rr) {
        const int r = wk * RW + rr, row = 8 * (r >> 2) + (r & 3);
        const float v = static_cast<float>(sum_of(j, rr) * sc_a) + bias_a;
        const float gate = GLU ? static_cast<float>(sum_of(j + JS - 1, rr) * sc_b) + bias_b : 0.0f;
        if (row >= rows) continue;
        float o = v;
        if (MODE == 1 + AQT_EPI_SWISH) o = swish_f32(v);
        else if (GLU) o = v * sigmoid_f32(gate);
        ol[row * oc] = o;
      }
  }
}

template <int TN, bool PACKED, int MODE, bool LONG>
__global__ __launch_bounds__(512, 2) void f32_codes_any_kernel(
    const float *__restrict__ f, const float *__restrict__ scale, const uint8_t *__restrict__ q, int64_t M, int64_t R,
    int64_t C, const float *__restrict__ s_x, const uint32_t *__restrict__ mask_x, const float *__restrict__ factor,
    const float *__restrict__ bias, float *__restrict__ out, int tiles_r) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[codes_lds_bytes<TN, LONG>()];
  f32_codes_tile<TN, PACKED, MODE, LONG>(lds, blockIdx.x, f, scale, q, M, R, C, s_x, mask_x, factor, bias, out, tiles_r);
}

// ---- dW: contraction over the rows of both operands ---------------------------------------------
// partial[slab][k][n] = sum over the slab's rows of xq[m,k] dy[m,n].  A workgroup of four wavefronts owns 128
// fan-in positions x 128 channels and one slab of rows, 32 rows per slice.  Neither operand is
// contraction-contiguous, so a thread gathers 4 positions x 4 rows of each with row-wise loads and writes pieces
// along the rows into LDS; tile column 4 g + b lives in LDS row 32 b + g, so that the lanes of a write spread over
// the banks.  With a single slab the result is finished here; otherwise dw_any_fold_kernel adds the slabs in
// order, in float64.  The bias gradient's column sums are taken on the way, in float64: the row tiles of a column stage the
// same gradient, so tile kt adds up the slices s with s % (number of row tiles) == kt and leaves one partial row.
// Eight layers of a 10008-token, 144-wide encoder layer: 131 us for passes of their own, 11 us here.
constexpr int kDwThreads = kColsumThreads;
static_assert(kDwThreads == 256);
constexpr int kDwTile = 128;

__global__ __launch_bounds__(kDwThreads, 2) void bwd_dw_any_kernel(const int8_t *__restrict__ xq, const float *__restrict__ dy,
                                                                   int64_t M, int64_t K, int64_t N, int64_t rows_per_slab,
                                                                   float *__restrict__ out, int tiles_n, int tiles, int finish,
                                                                   DwFinish fin, double *__restrict__ bias_part) {
  constexpr int kImage = kDwTile * 64;
  constexpr int kSliceBytes = 4 * kImage;             // codes; dy hi, mid, lo
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kSliceBytes];
  const int t = threadIdx.x, lane = t & 63, lr = lane & 31, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int slab = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  const int64_t k0 = (tile / tiles_n) * static_cast<int64_t>(kDwTile), n0 = (tile % tiles_n) * static_cast<int64_t>(kDwTile);
  const int64_t m0 = slab * rows_per_slab, m1 = m0 + rows_per_slab < M ? m0 + rows_per_slab : M;
  const int g = t & 31, mg = t >> 5;          // this thread's column group and its four rows 4 mg .. + 3 of a slice
  const int64_t kc = k0 + 4 * g, nc = n0 + 4 * g;
  const int64_t slices = cdiv(m1 - m0, kSlice);
  const int last_rows = static_cast<int>(m1 - m0 - (slices - 1) * kSlice);
  // byte offsets of this thread's rows in a slice (K, N below 2^24), so that a load is one scalar base and a fixed lane
  // offset; in the last slice, rows beyond the end are its last
  uint32_t xo[4], yo[4], xl[4], yl[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = 4 * mg + i, l = r < last_rows ? r : last_rows - 1;
    xo[i] = static_cast<uint32_t>(r * K + kc);
    yo[i] = static_cast<uint32_t>((r * N + nc) * 4);
    xl[i] = static_cast<uint32_t>(l * K + kc);
    yl[i] = static_cast<uint32_t>((l * N + nc) * 4);
  }
  uint32_t rc[2][4];
  v4f rg[2][4];
  auto load = [&](auto set, int64_t slice) {
    constexpr int S = decltype(set)::value;
    const int64_t m = m0 + slice * kSlice;
    const bool last = slice == slices - 1;
    const char *x = reinterpret_cast<const char *>(xq) + m * K, *y = reinterpret_cast<const char *>(dy + m * N);
#pragma unroll
    for (int i = 0; i < 4; ++i) rc[S][i] = load_at<uint32_t>(x + (last ? xl[i] : xo[i]));
#pragma unroll
    for (int i = 0; i < 4; ++i) rg[S][i] = load_at<v4f>(y + (last ? yl[i] : yo[i]));
  };
  // a wavefront multiplies all four codes blocks with one block of the gradient (seven fragment reads per twelve products)
  v16f acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.0f;
  double colsum[4] = {0.0, 0.0, 0.0, 0.0};          // of this thread's columns, over the slices that are this tile's turn
  const int kt = tile / tiles_n, tiles_k = tiles / tiles_n;
  int64_t staged = 0, turn = bias_part ? kt : slices;
  auto stage = [&](auto set, int64_t slice, uint8_t *slot) {
    constexpr int S = decltype(set)::value;
    if (slice == slices - 1 && last_rows < kSlice) {   // rows beyond the slab contribute nothing
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * mg + i >= last_rows) {
          rc[S][i] = 0u;
          rg[S][i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
    if (staged == turn && staged < slices) {   // the loop stages the last slice more than once
      turn += tiles_k;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        colsum[b] += (static_cast<double>(rg[S][0][b]) + static_cast<double>(rg[S][1][b])) +
                     (static_cast<double>(rg[S][2][b]) + static_cast<double>(rg[S][3][b]));
    }
    ++staged;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      uint8_t *const at = slot + chunk_at<kCh>(32 * b + g, mg >> 1) + 8 * (mg & 1);
      v2i a;
      a.x = static_cast<int>(pack_bf16(static_cast<float>(static_cast<int8_t>(rc[S][0] >> (8 * b))),
                                       static_cast<float>(static_cast<int8_t>(rc[S][1] >> (8 * b)))));
      a.y = static_cast<int>(pack_bf16(static_cast<float>(static_cast<int8_t>(rc[S][2] >> (8 * b))),
                                       static_cast<float>(static_cast<int8_t>(rc[S][3] >> (8 * b)))));
      *reinterpret_cast<v2i *>(at) = a;
      store_split(at + kImage, kImage, v4f{rg[S][0][b], rg[S][1][b], rg[S][2][b], rg[S][3][b]});
    }
  };
  auto multiply = [&](const uint8_t *slot) {
#pragma unroll
    for (int kk = 0; kk < kSlice / 16; ++kk) {
      v4i a[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = *reinterpret_cast<const v4i *>(slot + chunk_at<kCh>(i * 32 + lr, 2 * kk + lk));
#pragma unroll
      for (int img = 2; img >= 0; --img) {
        const v4i d = *reinterpret_cast<const v4i *>(slot + (1 + img) * kImage + chunk_at<kCh>(wave * 32 + lr, 2 * kk + lk));
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = mfma_bf16(a[i], d, acc[i]);
      }
    }
  };
  run_slices<1>(lds, kSliceBytes, 0, slices, load, stage, multiply);
  if (bias_part) {   // the eight row groups of a column, in order
    double *const sums = reinterpret_cast<double *>(lds);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 4; ++b) sums[b * kDwThreads + t] = colsum[b];
    __syncthreads();
    if (t < kDwTile) {
      const double *const p = sums + (t & 3) * kDwThreads + (t >> 2);
      double sum = p[0];
#pragma unroll
      for (int i = 1; i < 8; ++i) sum += p[32 * i];
      bias_part[(static_cast<int64_t>(slab) * tiles_k + kt) * N + n0 + t] = sum;
    }
  }
  // Out through LDS as whole rows, 32 tile rows 4 q + p at a time: they are codes block p, and tile column 4 g + b is
  // gradient block b = wave, column g.
  constexpr int kRow = kDwTile + 4;
  static_assert(32 * kRow * 4 <= 2 * kSliceBytes, "the output image must fit");
  float *const img = reinterpret_cast<float *>(lds);
  const double sx = finish ? fin.s_x[0] : 1.0;
  bool nz[4];                       // channels whose scale is not zero (what a missing clip mask stands for)
#pragma unroll
  for (int e = 0; e < 4; ++e) nz[e] = finish && fin.s_w[nc + e] != 0.0f;
  float *const o = out + (finish ? 0 : static_cast<int64_t>(slab) * K * N);
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) img[(8 * (r >> 2) + 4 * lk + (r & 3)) * kRow + 4 * lr + wave] = acc[p][r];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = (t >> 5) + 8 * u;
      const int64_t k = k0 + 4 * q + p, at = k * N + nc;
      v4f v = *reinterpret_cast<const v4f *>(img + q * kRow + 4 * g);
      if (finish) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (fin.mask_w ? mask_bit(fin.mask_w, at + e) : nz[e]) ? static_cast<float>(sx * v[e]) : 0.0f;
      }
      *reinterpret_cast<v4f *>(o + at) = v;
    }
  }
}

// The same for few rows: eight wavefronts share a tile of 32 fan-in positions x 32 channels and take turns along the rows, 32 at
// a time, each with a slot of its own, so that there are tiles enough without slabs, no partial result goes through memory and nothing
// is left to fold.  Sums of 64 rows in float32, then float64.  The tiles of the first 32 positions add up the bias gradient.
// Bound by the latency of its few trips to memory and the conversions: 1024 x 256 x 1024 10.2 us, 20.9 with slabs of 64 rows and a
// fold; error of the result against float64 8.2e-8 of its norm either way (1300 x 512 x 512 8.0e-8 and 8.2e-8).  At most 128 registers
// for two workgroups per compute unit: 56 spilled, 15.3 us.
constexpr int kDwSplitTile = 32;
constexpr int kDwSplitImage = kDwSplitTile * 64, kDwSplitSlice = 4 * kDwSplitImage;   // codes; dy hi, mid, lo
constexpr int kDwSplitLds = 8 * kDwSplitSlice;
static_assert(kDwSplitLds >= 8 * 16 * 64 * 8, "the wavefronts' sums must fit");

__device__ __forceinline__ void dw_split_tile(uint8_t *lds, unsigned block, const int8_t *__restrict__ xq, const float *__restrict__ dy,
                                              int64_t M, int64_t K, int64_t N, DwFinish fin, float *__restrict__ dw,
                                              float *__restrict__ dbias) {
  constexpr int WK = 8;
  const int lane = threadIdx.x & 63, lr = lane & 31, lk = lane >> 5;
  const int wk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned tiles_n = static_cast<unsigned>(N / kDwSplitTile), kt = block / tiles_n;
  const int64_t k0 = static_cast<int64_t>(kt) * kDwSplitTile, n0 = static_cast<int64_t>(block % tiles_n) * kDwSplitTile;
  const int g = lane & 7, mg = lane >> 3;   // this thread's four columns 4 g .. and four rows 4 mg .. of a slice
  const int64_t slices = cdiv(M, kSlice);
  uint32_t rc[2][4];
  v4f rg[2][4];
  auto load = [&](auto set, int64_t slice) {
    constexpr int S = decltype(set)::value;
    const int64_t m = slice * kSlice + 4 * mg;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t r = m + i < M ? m + i : M - 1;
      rc[S][i] = load_at<uint32_t>(xq + r * K + k0 + 4 * g);
      rg[S][i] = load_at<v4f>(dy + r * N + n0 + 4 * g);
    }
  };
  v16f acc;
  double sum[16], colsum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    acc[r] = 0.0f;
    sum[r] = 0.0;
  }
  auto fold = [&]() {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sum[r] += static_cast<double>(acc[r]);
      acc[r] = 0.0f;
    }
  };
  const bool bias = dbias && kt == 0;
  auto stage = [&](auto set, int64_t slice, uint8_t *slot) {
    constexpr int S = decltype(set)::value;
    if ((slice + 1) * kSlice > M) {   // rows beyond the end contribute nothing
      const int64_t m = slice * kSlice + 4 * mg;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (m + i >= M) {
          rc[S][i] = 0u;
          rg[S][i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
    if (bias) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
        colsum[b] += (static_cast<double>(rg[S][0][b]) + static_cast<double>(rg[S][1][b])) +
                     (static_cast<double>(rg[S][2][b]) + static_cast<double>(rg[S][3][b]));
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {   // tile column 4 g + b lives in LDS row 8 b + g
      uint8_t *const at = slot + chunk_at<kCh>(8 * b + g, mg >> 1) + 8 * (mg & 1);
      v2i a;
      a.x = static_cast<int>(pack_bf16(static_cast<float>(static_cast<int8_t>(rc[S][0] >> (8 * b))),
                                       static_cast<float>(static_cast<int8_t>(rc[S][1] >> (8 * b)))));
      a.y = static_cast<int>(pack_bf16(static_cast<float>(static_cast<int8_t>(rc[S][2] >> (8 * b))),
                                       static_cast<float>(static_cast<int8_t>(rc[S][3] >> (8 * b)))));
      *reinterpret_cast<v2i *>(at) = a;
      store_split(at + kDwSplitImage, kDwSplitImage, v4f{rg[S][0][b], rg[S][1][b], rg[S][2][b], rg[S][3][b]});
    }
  };
  int since = 0;
  auto multiply = [&](const uint8_t *slot) {
#pragma unroll
    for (int kk = 0; kk < kSlice / 16; ++kk) {
      const int at = chunk_at<kCh>(lr, 2 * kk + lk);
      const v4i a = *reinterpret_cast<const v4i *>(slot + at);
#pragma unroll
      for (int img = 3; img >= 1; --img)   // smallest terms first
        acc = mfma_bf16(a, *reinterpret_cast<const v4i *>(slot + img * kDwSplitImage + at), acc);
    }
    if (++since == 2) {
      fold();
      since = 0;
    }
  };
  run_slices<WK>(lds, kDwSplitSlice, wk, slices, load, stage, multiply);
  fold();
  double *const red = reinterpret_cast<double *>(lds);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) red[(wk * 16 + r) * 64 + lane] = sum[r];
  __syncthreads();
  const double sx = fin.s_x[0];
#pragma unroll
  for (int rr = 0; rr < 2; ++rr) {   // the wavefronts' shares in order
    const int r = 2 * wk + rr, row = 8 * (r >> 2) + 4 * lk + (r & 3);
    double v = red[r * 64 + lane];
#pragma unroll
    for (int w = 1; w < WK; ++w) v += red[(w * 16 + r) * 64 + lane];
    const int64_t k = k0 + 4 * (row & 7) + (row >> 3), n = n0 + 4 * (lr & 7) + (lr >> 3), at = k * N + n;
    dw[at] = dw_value(v, at, n, fin, sx);
  }
  if (bias) {   // uniform: the row groups of every wavefront, in order
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 4; ++b) red[(wk * 8 + mg) * 32 + 4 * g + b] = colsum[b];
    __syncthreads();
    if (threadIdx.x < kDwSplitTile) {
      double v = red[threadIdx.x];
      for (int i = 1; i < 8 * WK; ++i) v += red[i * 32 + threadIdx.x];
      dbias[n0 + threadIdx.x] = static_cast<float>(v);
    }
  }
}
__global__ __launch_bounds__(512, 2) void bwd_dw_split_kernel(const int8_t *__restrict__ xq, const float *__restrict__ dy, int64_t M,
                                                              int64_t K, int64_t N, DwFinish fin, float *__restrict__ dw,
                                                              float *__restrict__ dbias) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kDwSplitLds];
  dw_split_tile(lds, blockIdx.x, xq, dy, M, K, N, fin, dw, dbias);
}

// Both gradients of a small problem in one launch: the first dw_blocks workgroups take the tiles of dW, the others those of dX, each with the
// sums of its own kernel.  Two launches -> one: 128 x 256 x 256 9.1 -> 5.6 us, 1024 x 256 x 256 14.2 -> 10.0, 1024 x 256 x 1024
// 18.8 -> 16.9, 2048 x 256 x 1024 25.7 -> 23.9, 2560 x 512 x 512 30.0 -> 30.3.
template <int TN>
__global__ __launch_bounds__(512, 2) void bwd_small_kernel(CodesArgs a, int tiles_r, const int8_t *__restrict__ xq, int64_t K, int64_t N,
                                                           DwFinish fin, float *__restrict__ dw, float *__restrict__ dbias,
                                                           unsigned dw_blocks) {
  constexpr int kDx = codes_lds_bytes<TN, false>();
  __shared__ __attribute__((aligned(16))) uint8_t lds[kDx > kDwSplitLds ? kDx : kDwSplitLds];
  if (blockIdx.x < dw_blocks) {
    dw_split_tile(lds, blockIdx.x, xq, a.f, a.M, K, N, fin, dw, dbias);
  } else {
    f32_codes_tile<TN, false, 0, false>(lds, blockIdx.x - dw_blocks, a.f, a.scale, static_cast<const uint8_t *>(a.q), a.M, a.R, a.C, a.s_x,
                                        a.mask_x, a.factor, nullptr, a.out, tiles_r);
  }
}

// 64 elements x 4 groups of slabs per workgroup, eight loads in flight per thread; the order of the sums is fixed.
// The first bias_blocks workgroups fold the column sums instead.
__global__ __launch_bounds__(kDwThreads) void dw_any_fold_kernel(const float *__restrict__ partial, int slabs, int64_t K,
                                                                 int64_t N, DwFinish fin, float *__restrict__ dw,
                                                                 const double *__restrict__ bias_part, int bias_rows,
                                                                 unsigned bias_blocks, float *__restrict__ dbias) {
  if (blockIdx.x < bias_blocks) {
    fold_column_sums(bias_part, bias_rows, N, blockIdx.x, dbias);
    return;
  }
  __shared__ double sm[4][64];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int64_t KN = K * N, at = static_cast<int64_t>(blockIdx.x - bias_blocks) * 64 + lane, ac = at < KN ? at : KN - 1;
  double s = 0.0;
  for (int j = grp * 8; j < slabs; j += 32) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = partial[(j + u < slabs ? j + u : slabs - 1) * KN + ac];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += j + u < slabs ? static_cast<double>(v[u]) : 0.0;
  }
  sm[grp][lane] = s;
  __syncthreads();
  if (grp == 0 && at < KN)
    dw[at] = dw_value((sm[0][lane] + sm[1][lane]) + (sm[2][lane] + sm[3][lane]), at, at % N, fin, fin.s_x[0]);
}

// Which workgroup arrangement of the forward.  The lines were drawn from sweeps over all of them, every epilogue and both widths of
// the weights (us):
//   the split contraction (32 columns to a tile, all eight wavefronts on it) while that makes fewer than 800 workgroups: 2604 x 144 -> 144
//   (410) 3.9 against 5.3 in 64 x 128 tiles, 700 x 520 -> 1000 (704) 6.3 and 7.0, 1280 x 2048 -> 512 (640) 9.2 and 12.2;
//   1302 x 520 -> 1000 (1312) 9.5 and 7.7;
//   from there 64 x 128 tiles, eight wavefronts, but
//   128 x 128 with int4 weights and long contractions, where the expansion of the codes is shared by twice the rows, if their
//   rounds over the compute units are as full as those of 64 x 128: 10008 x 2040 -> 2040 90 against 97, 6500 x 2040 -> 1000 39 and 43, 13000 x
//   4100 -> 400 64 and 73, 30000 x 2040 -> 200 41 and 44; not 1000 positions (0.96 - 1.02), nor with int8 weights (646 against 467
//   at 50000 x 4100 -> 1000), nor where a round is left half empty, 4099 x 2040 -> 1100 37 and 33;
//   128 x 64, four wavefronts, where it saves such rounds because 64 x 128 would compute padding: 6500 x 2040 -> 288 int8 18.5 against 24.4,
//   17000 x 288 -> 288 15.1 and 17.1, 10008 x 144 -> 576 with Swish 16.9 and 18.6, 13000 x 144 -> 288 int4 11.2 and 12.5; with as many rounds it
//   is behind by 8 to 20 %, 10008 x 520 -> 288 14.3 and 13.2, with Swish 17.9 and 15.0; a tile's few wavefronts work longest with Swish (4099 x 520 -> 400, one
//   round against a little more than one, 13.8 and 11.8; 4099 x 4100 -> 400 33.9 and 38.3; without it 4351 x 1000 -> 400 13.7 and 16.3); and for long contractions with int8 weights, where
//   fewer bytes through LDS per product count (50000 x 4100 -> 1000 467 and 526, 17000 x 2040 -> 1100 0.90 of the time, 5000 x 1000 -> 1000 0.97;
//   with int4 weights 1.05 to 1.20 times the time).
enum class Tile { kRows, kLarge, kNarrow, kSmall, kSmallest };   // 64 x 128, 128 x 128, 128 x 64; split contraction: 32 x 64 (the GLU's pairs), 32 x 32
Tile pick_tile(int64_t M, int64_t cols, int64_t contraction, int epilogue, bool packed) {
  if (cdiv(M, 32) * cdiv(cols, 32) < 800) return epilogue == AQT_EPI_GLU ? Tile::kSmall : Tile::kSmallest;
  constexpr int64_t kUnits = 256;
  const int64_t rows = cdiv(M, 64) * cdiv(cols, 128), large = cdiv(M, 128) * cdiv(cols, 128), narrow = cdiv(M, 128) * cdiv(cols, 64);
  const int64_t rounds = cdiv(rows, kUnits), narrow_rounds = cdiv(narrow, kUnits);
  if (packed && contraction >= 1500 && large > kUnits && 2 * cdiv(large, kUnits) <= rounds) return Tile::kLarge;
  if (cols >= 640) return !packed && contraction >= 1000 && rows > 512 ? Tile::kNarrow : Tile::kRows;
  const bool swish = epilogue == AQT_EPI_SWISH, light = packed && epilogue == AQT_EPI_NONE;
  if (narrow_rounds == 1) return contraction >= (rows < 272 ? 1500 : swish ? 1000 : 0) && rounds > 1 ? Tile::kNarrow : Tile::kRows;
  if (light ? 3 * narrow_rounds <= 2 * rounds : 4 * narrow_rounds <= 3 * rounds) return Tile::kNarrow;
  // half of the last 128-wide tile would be padding, and a short contraction hides no wavefront's epilogue
  return cdiv(cols, 64) % 2 && contraction <= 256 && rows > 512 && !light ? Tile::kNarrow : Tile::kRows;
}

// ---- forward from float32 rows: the one-pass quantizer in the product's launch ----
// A launch in a chain takes 4 us whatever it does, and the quantizer of a small tensor is one.  Where its producer has left the largest
// |value|, every workgroup of the product makes the codes of its 32 rows itself, in the quantizer's own arithmetic, under
// the trip of its weights from memory, and those of the first column tile write them out.  40 x 512 -> 512 the quantizer 3.6 and the
// product 4.0 us -> 5.8 in one, 1302 x 144 -> 144 4.2 and 4.1 -> 5.2, 1024 x 256 -> 256 3.9 and 4.0 -> 5.9, and a launch's
// gap less.  With the normalisation in front of the quantizer as well it took 10 - 16 us against 4 and 5 (gamma and beta spill).
struct FillRows {
  static constexpr bool kFills = true, kWeights = false;
  RowSource s;
  int64_t M;
  int K;
  __device__ __forceinline__ float operator()(uint8_t *lds, int slice_bytes, int64_t bm, int64_t bn, float *) const {
    constexpr int kSlices = 8;
    const bool first = bn == 0;
    const int t = threadIdx.x, row = t >> 4, c = t & 15;   // sixteen threads a row, four positions of every slice each
    const bool live = bm * 32 + row < M;
    const int64_t m = live ? bm * 32 + row : M - 1;
    const float *const x = s.x + m * K;
    v4f v[kSlices];
#pragma unroll
    for (int k = 0; k < kSlices; ++k) {   // clamped: no branch around a load
      const int at = 64 * k + 4 * c;
      v[k] = *reinterpret_cast<const v4f *>(x + (at < K ? at : 0));
    }
    const uint32_t mx = s.absmax[0];
    const float fq = static_cast<float>(s.qmax), scale = __uint_as_float(mx) / fq;
    const Quantizer qz = quantizer(scale, fq);
    if (blockIdx.x == 0 && t == 0) {
      s.scale[0] = scale;
      if (mx >= 0x7F800000u && s.dev_status) *s.dev_status = AQT_ERR_NONFINITE;
    }
#pragma unroll
    for (int k = 0; k < kSlices; ++k) {
      const int at = 64 * k + 4 * c;
      if (64 * k < K) {   // uniform
        const uint32_t code = at < K ? quant4(v[k].x, v[k].y, v[k].z, v[k].w, qz) : 0u;
        *reinterpret_cast<uint32_t *>(lds + k * slice_bytes + chunk_at<4>(row, c >> 2) + 4 * (c & 3)) = code;
        if (first && live && at < K) *reinterpret_cast<uint32_t *>(s.q + m * K + at) = code;
      }
    }
    return scale;
  }
};
template <bool PACKED>
__global__ __launch_bounds__(512, 4) void dense_fwd_rows_kernel(const RowSource src, const uint8_t *__restrict__ wq,
                                                                const float *__restrict__ s_w, int64_t M, int64_t K, int64_t N,
                                                                const float *__restrict__ bias, float *__restrict__ y, int tiles_n) {
  dense_fwd_any_body<1, 1, 1, 1, 8, 64, PACKED, AQT_EPI_NONE>(nullptr, nullptr, wq, s_w, M, K, N, bias, y, nullptr, nullptr, nullptr,
                                                              tiles_n, FillRows{src, M, static_cast<int>(K)});
}

// ---- forward of a small dense layer from its float32 tensors, behind the pass that takes the maxima ----
// Both quantizers in the product's launch: a workgroup makes the codes of its 32 rows and of its 32 channels (four positions x four
// channels a thread); the first column tile writes the activations' codes, the first
// row tile everything the weights leave behind.
struct FillDense {
  static constexpr bool kFills = true, kWeights = true;
  DenseSource s;
  int64_t M, N;
  int K;
  __device__ __forceinline__ float operator()(uint8_t *lds, int slice_bytes, int64_t bm, int64_t bn, float *scales) const {
    constexpr int T = 512, kSlices = 4;
    __shared__ uint32_t most[T / 64];
    __shared__ __attribute__((aligned(16))) uint32_t top[kWeightSlabs][32];
    const int t = threadIdx.x, row = t >> 4, c = t & 15, nb = t & 7, kq = t >> 3;
    const bool live = bm * 32 + row < M, channels = bn * 32 + 4 * nb < N;   // four channels at once: N is a multiple of four
    const int64_t m = live ? bm * 32 + row : M - 1, n = bn * 32 + 4 * nb, nc = channels ? n : N - 4;
    const float *const x = s.x + m * K;
    v4f v[kSlices], wv[4];
#pragma unroll
    for (int k = 0; k < kSlices; ++k) {   // clamped: no branch around a load
      const int at = 64 * k + 4 * c;
      v[k] = *reinterpret_cast<const v4f *>(x + (at < K ? at : 0));
    }
    const int kw = 4 * kq;   // this thread's positions of its channels
#pragma unroll
    for (int i = 0; i < 4; ++i) wv[i] = *reinterpret_cast<const v4f *>(s.w + static_cast<int64_t>(kw + i < K ? kw + i : K - 1) * N + nc);
    uint32_t mx = words_max<T>(s.partial, s.nparts);
    if (t < 8 * kWeightSlabs) {
      const int slab = t >> 3;
      *reinterpret_cast<v4i *>(&top[slab][4 * nb]) =
          *reinterpret_cast<const v4i *>(s.part + static_cast<int64_t>(slab < s.slabs ? slab : s.slabs - 1) * N + nc);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = max(mx, static_cast<uint32_t>(__shfl_xor(static_cast<int>(mx), off)));
    if ((t & 63) == 0) most[t >> 6] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < T / 64; ++w) mx = max(mx, most[w]);
    const float fq = static_cast<float>(s.qmax_x), scale = __uint_as_float(mx) / fq, fw = static_cast<float>(s.qmax_w);
    const Quantizer qz = quantizer(scale, fq);
    if (blockIdx.x == 0 && t == 0) {
      s.s_x[0] = scale;
      if (mx >= 0x7F800000u && s.dev_status) *s.dev_status = AQT_ERR_NONFINITE;
    }
    uint32_t wm[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int slab = 0; slab < kWeightSlabs; ++slab) {
      const v4i a = *reinterpret_cast<const v4i *>(&top[slab][4 * nb]);
#pragma unroll
      for (int e = 0; e < 4; ++e) wm[e] = max(wm[e], static_cast<uint32_t>(a[e]));
    }
#pragma unroll
    for (int k = 0; k < kSlices; ++k) {
      const int at = 64 * k + 4 * c;
      if (64 * k < K) {   // uniform
        const uint32_t code = at < K ? quant4(v[k].x, v[k].y, v[k].z, v[k].w, qz) : 0u;
        *reinterpret_cast<uint32_t *>(lds + k * slice_bytes + chunk_at<4>(row, c >> 2) + 4 * (c & 3)) = code;
        if (bn == 0 && live && at < K) *reinterpret_cast<uint32_t *>(s.xq + m * K + at) = code;
      }
    }
    uint32_t codes[4];   // channel 4 nb + e
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float ws = __uint_as_float(wm[e]) / fw;
      if (kq == 0) scales[4 * nb + e] = ws;
      if (bm == 0 && kq == 0 && channels) {
        s.s_w[n + e] = ws;
        if (!(fabsf(ws) < INFINITY) && s.dev_status) *s.dev_status = AQT_ERR_NONFINITE;
      }
      const Quantizer qw = quantizer(ws, fw);
      codes[e] = quant4(wv[0][e], wv[1][e], wv[2][e], wv[3][e], qw);
      if (kw < K) *reinterpret_cast<uint32_t *>(lds + (kw >> 6) * slice_bytes + 32 * 64 + chunk_at<4>(4 * nb + e, (kw & 63) >> 4) + (kw & 15)) = codes[e];
    }
    if (bm == 0 && channels && kw < K) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t w = codes[e];
        if (s.packed) {
          const uint32_t b = (w & 0xFu) | ((w >> 4) & 0xF0u) | ((w >> 8) & 0xF00u) | ((w >> 12) & 0xF000u);
          *reinterpret_cast<uint16_t *>(s.wq_packed + (n + e) * (K / 2) + kw / 2) = static_cast<uint16_t>(b);
        } else {
          *reinterpret_cast<uint32_t *>(s.wq_packed + (n + e) * K + kw) = w;
        }
      }
      if (s.wq_kn) {   // four channels of a position
        auto pair = [](uint32_t a, uint32_t b, uint32_t sel) { return __builtin_amdgcn_perm(b, a, sel); };
        const uint32_t a = pair(codes[0], codes[1], 0x05010400u), b = pair(codes[2], codes[3], 0x05010400u);
        const uint32_t d = pair(codes[0], codes[1], 0x07030602u), f = pair(codes[2], codes[3], 0x07030602u);
        const uint32_t at[4] = {pair(a, b, 0x05040100u), pair(a, b, 0x07060302u), pair(d, f, 0x05040100u), pair(d, f, 0x07060302u)};
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<uint32_t *>(s.wq_kn + static_cast<int64_t>(kw + i) * N + n) = at[i];
      }
    }
    return scale;
  }
};
template <int EPI>
__global__ __launch_bounds__(512, 4) void dense_fwd_raw_kernel(const DenseSource src, int64_t M, int64_t K, int64_t N,
                                                               const float *__restrict__ bias, float *__restrict__ y,
                                                               float *__restrict__ dact, int tiles_n) {
  dense_fwd_any_body<1, 1, 1, 1, 8, 64, false, EPI>(nullptr, nullptr, nullptr, nullptr, M, K, N, bias, y, nullptr, nullptr, dact, tiles_n,
                                                    FillDense{src, M, N, static_cast<int>(K)});
}

template <int TM, int TN, int WM, int WN, int WK, int BK, bool PACKED>
aqt_status fwd_any(const int8_t *xq, const float *s_x, const void *wq, const float *s_w, int64_t M, int64_t K, int64_t N,
                   const float *bias, int epilogue, float *y, int32_t *acc_out, uint32_t *y_absmax, float *dact,
                   hipStream_t st) {
  const int64_t oc = epilogue == AQT_EPI_GLU ? N / 2 : N;
  const int64_t tn = cdiv(oc, (epilogue == AQT_EPI_GLU ? 16 : 32) * TN * WN), tm = cdiv(M, 32 * TM * WM);
  if (tn * tm > 0x7FFFFFFF) return AQT_ERR_UNSUPPORTED;
  constexpr int kGlu = TN % 2 ? AQT_EPI_NONE : AQT_EPI_GLU;   // tiles of one column block are not picked for GLU
  auto kern = epilogue == AQT_EPI_NONE    ? dense_fwd_any_kernel<TM, TN, WM, WN, WK, BK, PACKED, AQT_EPI_NONE>
              : epilogue == AQT_EPI_SWISH ? dense_fwd_any_kernel<TM, TN, WM, WN, WK, BK, PACKED, AQT_EPI_SWISH>
                                          : dense_fwd_any_kernel<TM, TN, WM, WN, WK, BK, PACKED, kGlu>;
  kern<<<static_cast<unsigned>(tn * tm), 64 * WM * WN * WK, 0, st>>>(xq, s_x, static_cast<const uint8_t *>(wq), s_w, M, K, N,
                                                                     bias, y, acc_out, y_absmax, dact, static_cast<int>(tn));
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

template <bool PACKED>
aqt_status fwd_any_sized(const int8_t *xq, const float *s_x, const void *wq, const float *s_w, int64_t M, int64_t K, int64_t N,
                         const float *bias, int epilogue, float *y, int32_t *acc_out, uint32_t *y_absmax, float *dact,
                         hipStream_t st) {
  switch (pick_tile(M, N, K, epilogue, PACKED)) {
    case Tile::kLarge:
      if constexpr (PACKED) return fwd_any<1, 2, 4, 2, 1, 128, true>(xq, s_x, wq, s_w, M, K, N, bias, epilogue, y, acc_out, y_absmax, dact, st);
      else return AQT_ERR_UNSUPPORTED;   // not picked
    case Tile::kRows:
      if (epilogue != AQT_EPI_GLU) return fwd_any<1, 1, 2, 4, 1, 128, PACKED>(xq, s_x, wq, s_w, M, K, N, bias, epilogue, y, acc_out, y_absmax, dact, st);
      return fwd_any<1, 2, 2, 2, 1, 128, PACKED>(xq, s_x, wq, s_w, M, K, N, bias, epilogue, y, acc_out, y_absmax, dact, st);
    case Tile::kNarrow: return fwd_any<1, 2, 4, 1, 1, 128, PACKED>(xq, s_x, wq, s_w, M, K, N, bias, epilogue, y, acc_out, y_absmax, dact, st);
    case Tile::kSmallest: return fwd_any<1, 1, 1, 1, 8, 64, PACKED>(xq, s_x, wq, s_w, M, K, N, bias, epilogue, y, acc_out, y_absmax, dact, st);
    default: return fwd_any<1, 2, 1, 1, 8, 64, PACKED>(xq, s_x, wq, s_w, M, K, N, bias, epilogue, y, acc_out, y_absmax, dact, st);
  }
}

template <int TN, bool PACKED, int MODE, bool LONG>
aqt_status f32_codes_any(const CodesArgs &a, hipStream_t st) {
  const int64_t tr = a.R / (32 * TN), tm = cdiv(a.M, 32);
  f32_codes_any_kernel<TN, PACKED, MODE, LONG><<<static_cast<unsigned>(tr * tm), 512, 0, st>>>(
      a.f, a.scale, static_cast<const uint8_t *>(a.q), a.M, a.R, a.C, a.s_x, a.mask_x, a.factor, a.bias, a.out, static_cast<int>(tr));
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

// Tiles of 32 x 64 halve the conversions of the float operand where there are enough of them; the float64 sums of long
// contractions need registers they do not leave.  (us: dX 3200 x 512 -> 128, 50 tiles of 64 x 128, 14.1 as such, 6.9 split.)
static bool codes_any_wide(int64_t M, int64_t R) { return cdiv(M, 32) * (R / 64) >= 128; }
template <bool PACKED, int MODE>
aqt_status f32_codes_any_sized(const CodesArgs &a, hipStream_t st) {
  const bool lng = a.C > 8 * kChain;
  if constexpr (MODE == 1 + AQT_EPI_GLU) {
    return lng ? f32_codes_any<2, PACKED, MODE, true>(a, st) : f32_codes_any<2, PACKED, MODE, false>(a, st);
  } else {
    if (lng) return f32_codes_any<1, PACKED, MODE, true>(a, st);
    return codes_any_wide(a.M, a.R) ? f32_codes_any<2, PACKED, MODE, false>(a, st) : f32_codes_any<1, PACKED, MODE, false>(a, st);
  }
}

template <bool PACKED>
aqt_status wonly_any(const CodesArgs &a, int epilogue, hipStream_t st) {
  return epilogue == AQT_EPI_NONE    ? f32_codes_any_sized<PACKED, 1 + AQT_EPI_NONE>(a, st)
         : epilogue == AQT_EPI_SWISH ? f32_codes_any_sized<PACKED, 1 + AQT_EPI_SWISH>(a, st)
                                     : f32_codes_any_sized<PACKED, 1 + AQT_EPI_GLU>(a, st);
}

}  // namespace

aqt_status launch_dense_fwd_any(const int8_t *xq, const float *s_x, const void *wq_packed, const float *s_w, int64_t M,
                                int64_t K, int64_t N, int bits_w, const float *bias, int epilogue, float *y,
                                int32_t *acc_out, uint32_t *y_absmax, float *dact, hipStream_t st) {
  return packed4(bits_w) ? fwd_any_sized<true>(xq, s_x, wq_packed, s_w, M, K, N, bias, epilogue, y, acc_out, y_absmax, dact, st)
                         : fwd_any_sized<false>(xq, s_x, wq_packed, s_w, M, K, N, bias, epilogue, y, acc_out, y_absmax, dact, st);
}

// Rows of whole 16-byte pieces that the eight wavefronts hold as one slice each, and where the split contraction is picked anyhow.  Above six
// slices the conversions pay while every workgroup has a compute unit to itself, and two to a unit where many column tiles find the
// rows in their cache.  A module, quantizer and product apart -> in one launch, us: convolution, 5000 x 144 (785 workgroups) 36.5 -> 34.3, 2600 x 256
// (656) 31.9 -> 31.6, 2600 x 320 (820) 37.6 -> 37.3, 600 x 400 (247) 26.0 -> 24.7, 200 x 512 (112) 23.5 -> 22.3, 800 x 448 (350) 30.0 -> 29.5,
// 1200 x 400 (494) 34.3 -> 33.9, but 600 x 512 (304) 29.2 -> 29.8, 1302 x 512 (656) 35.6 -> 37.2, 1580 x 400 (650) 36.6 -> 37.6; feed-forward,
// fan-in 384 -> 96, 6000 rows (564) 34.3 -> 33.6, 512 -> 128, 1302 (164) 25.0 -> 23.9, but 2600 (328) 26.6 -> 28.5, 480 -> 120, 4000 (500)
// 29.5 -> 32.6, 400 -> 100, 4000 (500) 28.9 -> 30.7.
bool dense_fwd_rows_ok(int64_t M, int64_t K, int64_t N) {
  const int64_t tiles = cdiv(M, 32) * cdiv(N, 32);
  return K >= 64 && K <= 512 && K % 4 == 0 && pick_tile(M, N, K, AQT_EPI_NONE, false) == Tile::kSmallest &&
         (K <= 384 || tiles <= 256 || (K <= 480 && tiles <= 512 && 2 * N >= K));
}
aqt_status launch_dense_fwd_rows(const RowSource &src, const void *wq_packed, const float *s_w, int64_t M, int64_t K, int64_t N,
                                 int bits_w, const float *bias, float *y, hipStream_t st) {
  const int64_t tn = cdiv(N, 32), tm = cdiv(M, 32);
  auto kern = packed4(bits_w) ? dense_fwd_rows_kernel<true> : dense_fwd_rows_kernel<false>;
  kern<<<static_cast<unsigned>(tn * tm), 512, 0, st>>>(src, static_cast<const uint8_t *>(wq_packed), s_w, M, K, N, bias, y,
                                                       static_cast<int>(tn));
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

// While every workgroup has a compute unit to itself.  The two launches apart -> in one (chained launches of a whole layer, us), at 256
// workgroups: 256 x 64 -> 1024 10.2 -> 8.9, 256 x 128 10.5 -> 9.5, 256 x 256 10.7 -> 10.3, 2048 x 256 -> 128 10.9 -> 10.1; at 32: 40 x 256 -> 512 10.1 -> 9.5;
// the call of three launches, which the host bounds, becomes one of two: 15.4 -> 12.2 us at 256 x 256 -> 1024 from Python.  Two to a compute
// unit: at 512, fan-ins of 64 10.8 -> 10.8 and 128 11.0 -> 11.1, but 192 11.1 -> 11.7 and 256 11.4 -> 12.0; at 259, 64 10.8 -> 10.2, 128
// 10.9 -> 10.9, 256 11.5 -> 11.9; 700 x 252 -> 1000 (704) 13.2 -> 16.5.  Fan-ins of up to 512 spill (256 x 512 -> 1024 10.6 -> 18.7).
bool dense_fwd_raw_ok(int64_t M, int64_t K, int64_t N, int epilogue) {
  return epilogue != AQT_EPI_GLU && N % 4 == 0 && K <= 256 && cdiv(M, 32) * cdiv(N, 32) <= 256 && dense_fwd_rows_ok(M, K, N);
}
aqt_status launch_dense_fwd_raw(const DenseSource &src, int64_t M, int64_t K, int64_t N, const float *bias, int epilogue, float *y,
                                float *dact, hipStream_t st) {
  const int64_t tn = cdiv(N, 32), tm = cdiv(M, 32);
  auto kern = epilogue == AQT_EPI_SWISH ? dense_fwd_raw_kernel<AQT_EPI_SWISH> : dense_fwd_raw_kernel<AQT_EPI_NONE>;
  kern<<<static_cast<unsigned>(tn * tm), 512, 0, st>>>(src, M, K, N, bias, y, dact, static_cast<int>(tn));
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

aqt_status launch_bwd_dx_any(const float *dy, const int8_t *wq_kn, const float *s_w, const float *s_x, const uint32_t *mask_x,
                             const float *factor, int64_t M, int64_t K, int64_t N, float *dx, hipStream_t st) {
  return f32_codes_any_sized<false, 0>(CodesArgs{dy, s_w, wq_kn, M, K, N, s_x, mask_x, factor, nullptr, dx}, st);
}

aqt_status launch_dense_fwd_wonly_any(const float *x, const void *wq_packed, const float *s_w, int64_t M, int64_t K,
                                      int64_t N, int bits_w, const float *bias, int epilogue, float *y, hipStream_t st) {
  const CodesArgs a{x, s_w, wq_packed, M, N, K, nullptr, nullptr, nullptr, bias, y};
  return packed4(bits_w) ? wonly_any<true>(a, epilogue, st) : wonly_any<false>(a, epilogue, st);
}

// Slabs of at most kChain rows, so that a float32 sum is never longer; shorter slabs while the launch does not fill the
// chip, of at least 64 rows each.
int dw_any_slabs(int64_t M, int64_t K, int64_t N) {
  const int64_t slabs = cdiv(M, kChain), fill = cdiv(512, (K / kDwTile) * (N / kDwTile)), most = cdiv(M, 64);
  return static_cast<int>(slabs >= fill ? slabs : fill < most ? fill : most);
}

// The split kernel while its tiles, with their four times as many conversions and reads, cost less than partial results through memory
// and a fold, and while there are tiles enough.  us with the bias gradient, slabs and split: 1024 x 256 x 1024 20.9 and 10.2, 2000 x 256 x 256
// 15.2 and 14.9, 2500 x 512 x 512 24.7 and 18.0, 100 x 2048 x 2048 54 and 46, 16 x 512 x 2048 13.5 and 13.2; behind it
//   in rows, 2000 x 256 x 128 12.8 and 14.6, 3000 x 256 x 128 14.3 and 19.0, 3000 x 256 x 256 18.3 and 19.3, 4000 x 512 x 256 23.9 and 24.3 (in one
//   launch with dX later: 2000 x 256 x 128 17.3 and 15.4, 3000 x 256 x 128 22.0 and 20.3, 4000 x 256 x 256 27.4 and 24.9; the line is one for both,
//   so that dW has the same bits with dX and without);
//   in products, the fewer the more tiles: 2500 x 512 x 1024 27.5 and 30.9, 1400 x 1024 x 1024 31.4 and 35.8, 768 x 1024 x 2048 41 and 47,
//   200 x 2048 x 2048 with dX 62 and 69;
//   where a slab of rows is all there are and the other kernel finishes by itself: 64 x 1024 x 2048 15 and 24, 64 x 2048 x 2048 16 and 44,
//   100 x 4096 x 2048 23 and 88 (up to 1024 tiles 64 x 1024 x 1024 14.3 and 13.4, 32 x 512 x 512 13.1 and 6.1).
static bool dw_any_splits(int64_t M, int64_t K, int64_t N) {
  const int64_t tiles = (K / kDwSplitTile) * (N / kDwSplitTile);
  if (tiles > 1024 && dw_any_slabs(M, K, N) == 1) return false;
  return M <= (tiles < 64 ? 2048 : 3072) && M * K * N <= 1000000000 - 100000 * tiles;
}

aqt_status launch_bwd_dw_any(const float *dy, const int8_t *xq, const float *s_x, const float *s_w, const uint32_t *mask_w,
                             int64_t M, int64_t K, int64_t N, float *dw, float *partial, float *dbias, double *bias_part,
                             hipStream_t st) {
  const DwFinish fin{s_x, s_w, mask_w};
  if (dw_any_splits(M, K, N)) {
    bwd_dw_split_kernel<<<static_cast<unsigned>((K / kDwSplitTile) * (N / kDwSplitTile)), 512, 0, st>>>(xq, dy, M, K, N, fin, dw, dbias);
    AQT_HIP(hipGetLastError());
    return AQT_OK;
  }
  const int64_t tiles_n = N / kDwTile, tiles = (K / kDwTile) * tiles_n;
  const int64_t rows = cdiv(cdiv(M, dw_any_slabs(M, K, N)), kSlice) * kSlice, slabs = cdiv(M, rows);
  if (tiles * slabs > 0x7FFFFFFF) return AQT_ERR_UNSUPPORTED;
  const bool one = slabs == 1;
  bwd_dw_any_kernel<<<static_cast<unsigned>(tiles * slabs), kDwThreads, 0, st>>>(
      xq, dy, M, K, N, rows, one ? dw : partial, static_cast<int>(tiles_n), static_cast<int>(tiles), one ? 1 : 0, fin,
      dbias ? bias_part : nullptr);
  AQT_HIP(hipGetLastError());
  const unsigned bias_blocks = dbias ? static_cast<unsigned>(cdiv(N, kColsumCols)) : 0;
  const unsigned dw_blocks = one ? 0 : static_cast<unsigned>(cdiv(K * N, 64));
  if (bias_blocks + dw_blocks == 0) return AQT_OK;
  dw_any_fold_kernel<<<bias_blocks + dw_blocks, kDwThreads, 0, st>>>(partial, static_cast<int>(slabs), K, N, fin, dw, bias_part,
                                                                    static_cast<int>(slabs * (tiles / tiles_n)), bias_blocks, dbias);
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

// dX and dW (and the bias gradient) in one launch: where dW takes the split kernel and dX no float64 sums.
bool bwd_small_ok(int64_t M, int64_t K, int64_t N) { return N <= 8 * kChain && dw_any_splits(M, K, N); }
aqt_status launch_bwd_small_any(const float *dy, const int8_t *wq_kn, const float *s_w, const float *s_x, const uint32_t *mask_x,
                                const float *factor, const int8_t *xq, const uint32_t *mask_w, int64_t M, int64_t K, int64_t N,
                                float *dx, float *dw, float *dbias, hipStream_t st) {
  const CodesArgs a{dy, s_w, wq_kn, M, K, N, s_x, mask_x, factor, nullptr, dx};
  const DwFinish fin{s_x, s_w, mask_w};
  const int64_t tm = cdiv(M, 32);
  const bool wide = codes_any_wide(M, K);
  const int64_t tr = K / (wide ? 64 : 32);
  const unsigned dwb = static_cast<unsigned>((K / kDwSplitTile) * (N / kDwSplitTile)), blocks = dwb + static_cast<unsigned>(tr * tm);
  auto kern = wide ? bwd_small_kernel<2> : bwd_small_kernel<1>;
  kern<<<blocks, 512, 0, st>>>(a, static_cast<int>(tr), xq, K, N, fin, dw, dbias, dwb);
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

}  // namespace aqt
