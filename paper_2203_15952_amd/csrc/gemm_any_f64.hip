// The float contractions of the quantized dense layer off the tuned kernels' grid (sizes that no tile divides, fewer
// than 128 rows, tensors that are not 16-byte aligned): dX, dW and the weight-only forward with every product and sum
// in float64 on v_mfma_f64_16x16x4_f64, rounded to float32 once.  Where there is enough work gemm_exact.hip forms the same
// sums on the int8 matrix cores (its rules say where); what is left here are small problems and short contractions.
//
// Nothing is split and nothing overflows or is lost on the way: a float32 value times a code is exact, infinities and
// the largest finite values behave as in a float64 loop, and a sum of any length is as good as one.  Float32 sums of 512 products on the
// bf16 matrix cores (three bf16 terms per value) took half the time, but their error against float64 was 2.1e-7 (dX),
// 1.7e-7 (dW) and 2.1e-7 (weight-only) of the result at 4099 x 520 x 1000; here it is 3.6e-8, 2.5e-8 and 2.5e-8, the last rounding
// (in dX also the float32 product dy * s_w).
//
// The instruction itself allows 46 TFLOP/s on the whole chip (independent ones on registers, two or more wavefronts per SIMD; 35 with
// one), and 4099 x 520 x 1000, which gemm_exact.hip takes now, reached 41 in dX and 38 in dW.  What is left here is bound by how
// few wavefronts it makes: dX 1300 x 400 of 1200 positions 47 us (27 TFLOP/s, padding not counted), 300 x 1030 of 2040 48 (26), 520 x 520
// of 1000 27 (20), 2600 x 144 of 576 20 (22), 800 x 400 of 400 18 (14); dW 64 x 520 x 1000 11 (6), 1024 x 144 x 576 17 (10).  So everything
// else is kept small rather than clever: float32 values and int8 codes go through LDS as they are and are converted when a
// fragment is read (one instruction per value, a small part of the products' clocks), and tiles are small so that a launch
// fills 256 compute units evenly.
//
// A lane of the instruction holds one element of A (row lane % 16) and of B (column lane % 16) at contraction index
// lane / 16.  Which positions those are is free as long as both operands agree: lane group g takes positions
// 4 g .. 4 g + 3 of sixteen in four steps, so that it reads four values with one access.
#include "any_shape.h"
#include "colsum.h"
#include "epilogue.h"

namespace aqt {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4d mfma_f64(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ double code_f64(uint32_t codes, int e) {
  return static_cast<double>(static_cast<int>(static_cast<int8_t>(codes >> (8 * e))));
}

// ---- float32 operand x codes: dX and the weight-only forward ---------------------------------
// out[m, r] = sum_c f[m, c] (* scale[c]) * q[r, c]: rows of both operands contraction-contiguous.
//   MODE 0 (dX):   f = dy [M,N], scale = s_w, q = wq_kn [K,N]; out times the clip mask and the factor
//   MODE 1 + e:    weight-only forward with epilogue e: f = x [M,K], q = the forward weight operand [N][K]
// A workgroup is WN wavefronts side by side, times WK groups of them (of one wavefront) that share one output tile and
// take turns along the contraction.  A wavefront owns 32 rows x 16 TN columns; a GLU tile pairs value (even) and gate
// (odd) column blocks.
constexpr int kRows = 32;            // rows of a tile
constexpr int kRowF = 4 * kSlice + 16, kRowQ = kSlice + 16;   // LDS row strides in bytes: fragment reads spread over all banks

template <int TN, int WN, int WK, bool PACKED, int MODE>
__global__ __launch_bounds__(64 * WN * WK, 2) void f32_codes_f64_kernel(
    const float *__restrict__ f, const float *__restrict__ scale, const uint8_t *__restrict__ q, int64_t M, int64_t R,
    int64_t C, const float *__restrict__ s_x, const uint32_t *__restrict__ mask_x, const float *__restrict__ factor,
    const float *__restrict__ bias, float *__restrict__ out, int tiles_r) {
  constexpr bool DX = MODE == 0, GLU = MODE == 1 + AQT_EPI_GLU;
  static_assert((WK == 1 || (WN == 1 && WK == 8)) && (!GLU || TN % 2 == 0), "the epilogue is shared out by row groups");
  constexpr int G = 64 * WN, BN = 16 * TN * WN;
  // pieces of four floats, of sixteen codes, per thread and slice; a narrow tile leaves some threads without codes
  constexpr int NA = kRows * 8 / G, NB = BN * 2 >= G ? BN * 2 / G : 1;
  static_assert(NA * G == kRows * 8 && NA > 0 && (NB * G == BN * 2 || BN * 2 < G), "whole pieces per thread");
  constexpr int kSliceBytes = kRows * kRowF + BN * kRowQ;
  constexpr int kRedBytes = WK > 1 ? WK * 2 * TN * 4 * 64 * 8 : 0;
  constexpr int kBuffers = WK == 1 ? 2 : WK;
  constexpr int kLds = kBuffers * kSliceBytes > kRedBytes ? kBuffers * kSliceBytes : kRedBytes;
  __shared__ __attribute__((aligned(16))) uint8_t lds[kLds];
  const int t = threadIdx.x, lane = t & 63, lc = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wk = wave / WN, wn = wave % WN, gt = t - wk * G;
  const int64_t bm = blockIdx.x / tiles_r, br = blockIdx.x % tiles_r;
  const int64_t oc = GLU ? R / 2 : R;
  // first column of the tile's block cb
  auto chan = [&](int cb) -> int64_t {
    if (GLU) return br * (BN / 2) + (cb >> 1) * 16 + ((cb & 1) ? oc : 0);
    return br * BN + cb * 16;
  };
  const int64_t row_bytes = PACKED ? (C + 1) / 2 : C;
  const float *pf[NA];
  const uint8_t *pq[NB];
  const bool has_codes = BN * 2 >= G || gt < BN * 2;
  const int piece = gt & 7;   // G is a multiple of 8: a thread's pieces sit at the same place of their rows
#pragma unroll
  for (int u = 0; u < NA; ++u) {
    const int64_t m = bm * kRows + ((gt + u * G) >> 3);
    pf[u] = f + (m < M ? m : M - 1) * C;
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int r = has_codes ? (gt + u * G) >> 1 : 0;
    const int64_t n = chan(r >> 4) + (r & 15);
    pq[u] = q + (n < R ? n : R - 1) * row_bytes;
  }
  v4f ra[2][NA], rs[2] = {{1.0f, 1.0f, 1.0f, 1.0f}, {1.0f, 1.0f, 1.0f, 1.0f}};
  v4i rb[2][NB];
  constexpr int kPiece = PACKED ? 8 : 16;   // bytes of sixteen codes
  const bool narrow = C < 4 || row_bytes < kPiece;   // uniform
  auto load = [&](auto set, int64_t slice) {
    constexpr int S = decltype(set)::value;
    const int64_t c0 = slice * kSlice + 4 * piece, a0 = slice * (2 * kPiece) + kPiece * (gt & 1);
    const int64_t c = c0 + 4 <= C ? c0 : C - 4, at = a0 + kPiece <= row_bytes ? a0 : row_bytes - kPiece;
#pragma unroll
    for (int u = 0; u < NA; ++u) ra[S][u] = load_at<v4f>(pf[u] + c);
    if (DX) rs[S] = load_at<v4f>(scale + c);
#pragma unroll
    for (int u = 0; u < NB; ++u) {   // a thread without codes reads what it will not use
      if (PACKED) {
        const v2i w = load_at<v2i>(pq[u] + at);
        rb[S][u] = v4i{w.x, w.y, 0, 0};
      } else {
        rb[S][u] = load_at<v4i>(pq[u] + at);
      }
    }
  };
  auto load_narrow = [&](auto set) {   // fewer than 16 positions
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      ra[S][u] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * piece + e < C) ra[S][u][e] = pf[u][4 * piece + e];
    }
    if (DX) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * piece + e < C) rs[S][e] = scale[4 * piece + e];
    }
#pragma unroll
    for (int u = 0; u < NB; ++u)
      rb[S][u] = load16_guarded(pq[u], kPiece * (gt & 1), (gt & 1) ? kPiece : row_bytes);   // all in the first piece
  };
  auto stage = [&](auto set, int64_t slice, uint8_t *slot) {
    constexpr int S = decltype(set)::value;
    uint8_t *const sA = slot, *const sB = slot + kRows * kRowF;
    if ((slice + 1) * kSlice > C && !narrow) {
      const int df = moved(slice * kSlice + 4 * piece, C, 4), dq = moved(slice * (2 * kPiece) + kPiece * (gt & 1), row_bytes, kPiece);
#pragma unroll
      for (int u = 0; u < NA; ++u) ra[S][u] = shift_down(ra[S][u], df);
      if (DX) rs[S] = shift_down(rs[S], df);
#pragma unroll
      for (int u = 0; u < NB; ++u) rb[S][u] = shift_down(rb[S][u], dq);
    }
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      v4f v = ra[S][u];
      if (DX) { v.x *= rs[S].x; v.y *= rs[S].y; v.z *= rs[S].z; v.w *= rs[S].w; }   // rounded to float32, as a float graph has it
      *reinterpret_cast<v4f *>(sA + ((gt + u * G) >> 3) * kRowF + 16 * piece) = v;
    }
    if (has_codes) {
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        v4i w = rb[S][u];
        if (PACKED) {   // 16 * code; the sums are divided by 16 at the end
          const v2i a = expand16(static_cast<uint32_t>(w.x)), b = expand16(static_cast<uint32_t>(w.y));
          w = v4i{a.x, a.y, b.x, b.y};
        }
        *reinterpret_cast<v4i *>(sB + ((gt + u * G) >> 1) * kRowQ + 16 * (gt & 1)) = w;
      }
    }
  };
  v4d acc[2][TN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  auto multiply = [&](const uint8_t *slot) {
    const uint8_t *const sA = slot, *const sB = slot + kRows * kRowF;
#pragma unroll
    for (int h = 0; h < kSlice / 16; ++h) {
      v4f a[2];
      uint32_t b[TN];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const v4f *>(sA + (16 * i + lc) * kRowF + 64 * h + 16 * lg);
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const uint32_t *>(sB + ((wn * TN + j) * 16 + lc) * kRowQ + 16 * h + 4 * lg);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const double c = code_f64(b[j], e);
#pragma unroll
          for (int i = 0; i < 2; ++i) acc[i][j] = mfma_f64(static_cast<double>(a[i][e]), c, acc[i][j]);
        }
    }
  };
  if (!narrow) run_slices<WK>(lds, kSliceBytes, wk, cdiv(C, kSlice), load, stage, multiply);
  else if (wk == 0) run_narrow<WK>(lds, load_narrow, stage, multiply);
  // The groups of a tile add their sums in order and share the epilogue: each takes one of the eight (i, r).
  double *const red = reinterpret_cast<double *>(lds);
  if (WK > 1) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(((wk * 2 + i) * TN + j) * 4 + r) * 64 + lane] = acc[i][j][r];
    __syncthreads();
  }
  constexpr int kMine = WK > 1 ? 1 : 8;   // (i, r) pairs of a wavefront
  auto sum_of = [&](int ir, int j) -> double {
    double v = 0.0;
    if (WK > 1) {
#pragma unroll
      for (int w = 0; w < WK; ++w) v += red[(((w * 2 + (wk >> 2)) * TN + j) * 4 + (wk & 3)) * 64 + lane];
    } else {
      v = acc[ir >> 2][j][ir & 3];
    }
    return PACKED ? v * 0.0625 : v;
  };
  constexpr int JS = GLU ? 2 : 1;
  const bool keep = DX ? s_x[0] != 0.0f : true;
#pragma unroll
  for (int j = 0; j < TN; j += JS) {
    const int64_t n = chan(wn * TN + j) + lc;
    const bool live = n < oc;
    const int64_t nc = live ? n : oc - 1, ng = nc + (GLU ? oc : 0);
    const double sc_a = DX ? 1.0 : scale[nc], sc_b = GLU ? scale[ng] : 0.0f;
    const float bias_a = bias ? bias[nc] : 0.0f, bias_b = (GLU && bias) ? bias[ng] : 0.0f;
#pragma unroll
    for (int p = 0; p < kMine; ++p) {
      const int ir = WK > 1 ? wk : p;
      const int64_t m = bm * kRows + 16 * (ir >> 2) + 4 * (ir & 3) + lg, at = m * oc + n;
      const double s = sum_of(ir, j), s2 = GLU ? sum_of(ir, j + JS - 1) : 0.0;
      if (!live || m >= M) continue;
      if (DX) {
        float v = static_cast<float>(s);
        if (factor) v = v * factor[at];
        out[at] = (mask_x ? mask_bit(mask_x, at) : keep) ? v : 0.0f;
      } else {
        const float v = static_cast<float>(s * sc_a) + bias_a;
        float o = v;
        if (MODE == 1 + AQT_EPI_SWISH) o = swish_f32(v);
        else if (GLU) o = v * sigmoid_f32(static_cast<float>(s2 * sc_b) + bias_b);
        out[at] = o;
      }
    }
  }
}

// ---- dW: contraction over the rows of both operands ---------------------------------------------
// partial[slab][k][n] = sum over the slab's rows of xq[m,k] dy[m,n].  A workgroup of four wavefronts owns 64 fan-in
// positions x 64 channels and one slab of rows, 64 rows per slice.  Neither operand is contraction-contiguous, so a
// thread gathers 4 positions x 4 rows of each with row-wise loads and writes pieces along the rows into LDS; tile
// column 4 g + b lives in LDS row 16 b + g, so that the lanes of a write spread over the banks and an accumulator lane holds
// four neighbouring channels.  With a single slab the result is finished here; otherwise dw_f64_fold_kernel adds the slabs
// in order.  The bias gradient's column sums are taken on the way: the row tiles of a column stage the same gradient, so
// tile kt adds up the slices s with s % (number of row tiles) == kt and leaves one partial row.
constexpr int kDwThreads = kColsumThreads;
static_assert(kDwThreads == 256);
constexpr int kDwTile = 64, kDwSlice = 64;
constexpr int kDwRowQ = kDwSlice + 4, kDwRowF = 4 * kDwSlice + 16;   // LDS row strides in bytes

__global__ __launch_bounds__(kDwThreads, 3) void bwd_dw_f64_kernel(const int8_t *__restrict__ xq, const float *__restrict__ dy,
                                                                   int64_t M, int64_t K, int64_t N, int64_t rows_per_slab,
                                                                   double *__restrict__ partial, float *__restrict__ dw,
                                                                   int tiles_n, int tiles, DwFinish fin,
                                                                   double *__restrict__ bias_part) {
  constexpr int kCodesBytes = kDwTile * kDwRowQ, kSliceBytes = kCodesBytes + kDwTile * kDwRowF;
  static_assert(kCodesBytes % 16 == 0 && kSliceBytes % 16 == 0);
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kSliceBytes];
  const int t = threadIdx.x, lane = t & 63, lc = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int slab = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  const int64_t k0 = (tile / tiles_n) * static_cast<int64_t>(kDwTile), n0 = (tile % tiles_n) * static_cast<int64_t>(kDwTile);
  const int64_t m0 = slab * rows_per_slab, rows = (m0 + rows_per_slab < M ? m0 + rows_per_slab : M) - m0;
  const int g = t & 15, mg = t >> 4;          // this thread's column group and its four rows 4 mg .. + 3 of a slice
  const int64_t kc = k0 + 4 * g, nc = n0 + 4 * g;
  const bool narrow = K < 4 || N < 4, edge = k0 + kDwTile > K || n0 + kDwTile > N;   // uniform
  const int64_t kr = narrow || kc + 4 <= K ? kc : K - 4, nr = narrow || nc + 4 <= N ? nc : N - 4;
  const int dk = moved(kc, K, 4), dn = moved(nc, N, 4);
  const int64_t slices = cdiv(rows, kDwSlice);
  const int8_t *const px = xq + m0 * K + kr;
  const float *const py = dy + m0 * N + nr;
  uint32_t rc[2][4];
  v4f rg[2][4];
  auto load = [&](auto set, int64_t slice) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t r = slice * kDwSlice + 4 * mg + i, rr = r < rows ? r : rows - 1;
      rc[S][i] = load_at<uint32_t>(px + rr * K);
      rg[S][i] = load_at<v4f>(py + rr * N);
    }
  };
  int64_t narrow_slice = 0;
  auto load_narrow = [&](auto set) {   // fewer than four columns of an operand: element by element
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t r = narrow_slice * kDwSlice + 4 * mg + i;
      rc[S][i] = 0u;
      rg[S][i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (r < rows && kc + e < K) rc[S][i] |= static_cast<uint32_t>(static_cast<uint8_t>(px[r * K + e])) << (8 * e);
        if (r < rows && nc + e < N) rg[S][i][e] = py[r * N + e];
      }
    }
  };
  double colsum[4] = {0.0, 0.0, 0.0, 0.0};          // of this thread's columns, over the slices that are this tile's turn
  const int kt = tile / tiles_n, tiles_k = tiles / tiles_n;
  int64_t staged = 0, turn = bias_part ? kt : slices;
  auto stage = [&](auto set, int64_t slice, uint8_t *slot) {
    constexpr int S = decltype(set)::value;
    if (edge && !narrow) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        rc[S][i] = dk < 4 ? rc[S][i] >> (8 * dk) : 0u;
        rg[S][i] = shift_down(rg[S][i], dn);
      }
    }
    if ((slice + 1) * kDwSlice > rows) {   // rows beyond the slab contribute nothing
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (slice * kDwSlice + 4 * mg + i >= rows) {
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
      const uint32_t sel = static_cast<uint32_t>(b) | (static_cast<uint32_t>(4 + b) << 8);   // byte b of two rows
      const uint32_t lo = __builtin_amdgcn_perm(rc[S][1], rc[S][0], sel), hi = __builtin_amdgcn_perm(rc[S][3], rc[S][2], sel);
      *reinterpret_cast<uint32_t *>(slot + (16 * b + g) * kDwRowQ + 4 * mg) = (lo & 0xFFFFu) | (hi << 16);
      *reinterpret_cast<v4f *>(slot + kCodesBytes + (16 * b + g) * kDwRowF + 16 * mg) = v4f{rg[S][0][b], rg[S][1][b], rg[S][2][b], rg[S][3][b]};
    }
  };
  // wavefront w multiplies the fan-in positions 4 x + w (x = 0 .. 15) with all channels; block j: channels 4 x + j
  v4d acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = v4d{0.0, 0.0, 0.0, 0.0};
  auto multiply = [&](const uint8_t *slot) {
#pragma unroll
    for (int h = 0; h < kDwSlice / 16; ++h) {
      const uint32_t a = *reinterpret_cast<const uint32_t *>(slot + (16 * wave + lc) * kDwRowQ + 16 * h + 4 * lg);
      v4f d[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) d[j] = *reinterpret_cast<const v4f *>(slot + kCodesBytes + (16 * j + lc) * kDwRowF + 64 * h + 16 * lg);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double c = code_f64(a, e);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = mfma_f64(c, static_cast<double>(d[j][e]), acc[j]);
      }
    }
  };
  if (!narrow) run_slices<1>(lds, kSliceBytes, 0, slices, load, stage, multiply);
  else
    for (; narrow_slice < slices; ++narrow_slice) run_narrow<1>(lds, load_narrow, stage, multiply);
  if (bias_part) {   // the sixteen row groups of a column, in order
    double *const sums = reinterpret_cast<double *>(lds);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 4; ++b) sums[b * kDwThreads + t] = colsum[b];
    __syncthreads();
    if (t < kDwTile && n0 + t < N) {
      const double *const p = sums + (t & 3) * kDwThreads + (t >> 2);
      double sum = p[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) sum += p[16 * i];
      bias_part[(static_cast<int64_t>(slab) * tiles_k + kt) * N + n0 + t] = sum;
    }
  }
  const double sx = dw ? static_cast<double>(fin.s_x[0]) : 1.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t k = k0 + 4 * (4 * r + lg) + wave, n = n0 + 4 * lc, at = k * N + n;
    if (k >= K) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (n + j < N) {
        if (dw) dw[at + j] = dw_value(acc[j][r], at + j, n + j, fin, sx);
        else partial[static_cast<int64_t>(slab) * K * N + at + j] = acc[j][r];
      }
  }
}

// 64 elements x 4 groups of slabs per workgroup; the order of the sums is fixed.  The first bias_blocks workgroups
// fold the column sums instead.
__global__ __launch_bounds__(kDwThreads) void dw_f64_fold_kernel(const double *__restrict__ partial, int slabs, int64_t K,
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
  for (int j = grp * 4; j < slabs; j += 16) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = partial[(j + u < slabs ? j + u : slabs - 1) * KN + ac];
#pragma unroll
    for (int u = 0; u < 4; ++u) s += j + u < slabs ? v[u] : 0.0;
  }
  sm[grp][lane] = s;
  __syncthreads();
  if (grp == 0 && at < KN)
    dw[at] = dw_value((sm[0][lane] + sm[1][lane]) + (sm[2][lane] + sm[3][lane]), at, at % N, fin, fin.s_x[0]);
}

template <int TN, int WN, int WK, bool PACKED, int MODE>
aqt_status f32_codes_f64(const CodesArgs &a, hipStream_t st) {
  constexpr bool GLU = MODE == 1 + AQT_EPI_GLU;
  const int64_t tr = cdiv(GLU ? a.R / 2 : a.R, (GLU ? 8 : 16) * TN * WN), tm = cdiv(a.M, kRows);
  if (tr * tm > 0x7FFFFFFF) return AQT_ERR_UNSUPPORTED;
  f32_codes_f64_kernel<TN, WN, WK, PACKED, MODE><<<static_cast<unsigned>(tr * tm), 64 * WN * WK, 0, st>>>(
      a.f, a.scale, static_cast<const uint8_t *>(a.q), a.M, a.R, a.C, a.s_x, a.mask_x, a.factor, a.bias, a.out, static_cast<int>(tr));
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

// 32 x 64 tiles of four wavefronts (32 outputs of a GLU: two wavefronts) where there are enough of them for 256 compute
// units, else 32 x 32 tiles (32 x 16 if even those are few) with the contraction shared out over eight wavefronts, which also evens out a last
// round of long tiles.  Measured in us, 32 x 64 / split: 171 tiles, contraction 1000, 30.6 / 25.9; 150 of 384 long 9.3 / 9.6;
// 304 of 520 27.4 / 26.5; 376 of 800 38.1 / 33.7; 315 of 2000 92 / 69; 369 of 144 12.0 / 16.1; 1008 of 520 47.8 / 68.9.
template <bool PACKED, int MODE>
aqt_status f32_codes_f64_sized(const CodesArgs &a, hipStream_t st) {
  constexpr bool GLU = MODE == 1 + AQT_EPI_GLU;
  const int64_t rows = cdiv(a.M, kRows), tiles = rows * cdiv(a.R, 64);
  if constexpr (!GLU)
    if (rows * cdiv(a.R, 32) <= 128) return f32_codes_f64<1, 1, 8, PACKED, MODE>(a, st);
  if (tiles < 256 || (tiles < 512 && a.C >= 768)) return f32_codes_f64<2, 1, 8, PACKED, MODE>(a, st);
  if constexpr (GLU) return f32_codes_f64<2, 2, 1, PACKED, MODE>(a, st);
  else return f32_codes_f64<1, 4, 1, PACKED, MODE>(a, st);
}

template <bool PACKED>
aqt_status wonly_f64(const CodesArgs &a, int epilogue, hipStream_t st) {
  return epilogue == AQT_EPI_NONE    ? f32_codes_f64_sized<PACKED, 1 + AQT_EPI_NONE>(a, st)
         : epilogue == AQT_EPI_SWISH ? f32_codes_f64_sized<PACKED, 1 + AQT_EPI_SWISH>(a, st)
                                     : f32_codes_f64_sized<PACKED, 1 + AQT_EPI_GLU>(a, st);
}

}  // namespace

aqt_status launch_bwd_dx_f64(const float *dy, const int8_t *wq_kn, const float *s_w, const float *s_x, const uint32_t *mask_x,
                             const float *factor, int64_t M, int64_t K, int64_t N, float *dx, hipStream_t st) {
  if (f32_codes_exact_ok(M, K, N)) return launch_bwd_dx_exact(dy, wq_kn, s_w, s_x, mask_x, factor, M, K, N, dx, st);
  return f32_codes_f64_sized<false, 0>(CodesArgs{dy, s_w, wq_kn, M, K, N, s_x, mask_x, factor, nullptr, dx}, st);
}

aqt_status launch_dense_fwd_wonly_f64(const float *x, const void *wq_packed, const float *s_w, int64_t M, int64_t K,
                                      int64_t N, int bits_w, const float *bias, int epilogue, float *y, hipStream_t st) {
  if (f32_codes_exact_ok(M, N, K)) return launch_dense_fwd_wonly_exact(x, wq_packed, s_w, M, K, N, bits_w, bias, epilogue, y, st);
  const CodesArgs a{x, s_w, wq_packed, M, N, K, nullptr, nullptr, nullptr, bias, y};
  return packed4(bits_w) ? wonly_f64<true>(a, epilogue, st) : wonly_f64<false>(a, epilogue, st);
}

// Slabs of rows so that the launch fills the chip once (three workgroups fit a compute unit), of at least 128 rows each.
int dw_f64_slabs(int64_t M, int64_t K, int64_t N) {
  const int64_t fill = cdiv(768, cdiv(K, kDwTile) * cdiv(N, kDwTile)), most = cdiv(M, 128);
  return static_cast<int>(fill < most ? fill : most);
}

// dw or dbias null: that part is not wanted.
aqt_status launch_dw_f64_fold(const double *partial, int slabs, int64_t K, int64_t N, const float *s_x, const float *s_w,
                              const uint32_t *mask_w, float *dw, const double *bias_part, int bias_rows, float *dbias,
                              hipStream_t st) {
  const unsigned bias_blocks = dbias ? static_cast<unsigned>(cdiv(N, kColsumCols)) : 0;
  const unsigned dw_blocks = dw ? static_cast<unsigned>(cdiv(K * N, 64)) : 0;
  if (bias_blocks + dw_blocks == 0) return AQT_OK;
  dw_f64_fold_kernel<<<bias_blocks + dw_blocks, kDwThreads, 0, st>>>(partial, slabs, K, N, DwFinish{s_x, s_w, mask_w}, dw,
                                                                    bias_part, bias_rows, bias_blocks, dbias);
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

aqt_status launch_bwd_dw_f64(const float *dy, const int8_t *xq, const float *s_x, const float *s_w, const uint32_t *mask_w,
                             int64_t M, int64_t K, int64_t N, float *dw, double *partial, int max_slabs, float *dbias,
                             double *bias_part, hipStream_t st) {
  const int digits = dw_exact_slabs(M, K, N) < max_slabs ? dw_exact_slabs(M, K, N) : max_slabs;
  if (dw_exact_ok(M, K, N, digits))
    return launch_bwd_dw_exact(dy, xq, s_x, s_w, mask_w, M, K, N, dw, partial, digits, dbias, bias_part, st);
  const int64_t tiles_n = cdiv(N, kDwTile), tiles = cdiv(K, kDwTile) * tiles_n;
  const int wish = dw_f64_slabs(M, K, N);
  const int64_t rows = cdiv(cdiv(M, wish < max_slabs ? wish : max_slabs), kDwSlice) * kDwSlice, slabs = cdiv(M, rows);
  if (tiles * slabs > 0x7FFFFFFF) return AQT_ERR_UNSUPPORTED;
  const DwFinish fin{s_x, s_w, mask_w};
  const bool one = slabs == 1;
  bwd_dw_f64_kernel<<<static_cast<unsigned>(tiles * slabs), kDwThreads, 0, st>>>(
      xq, dy, M, K, N, rows, partial, one ? dw : nullptr, static_cast<int>(tiles_n), static_cast<int>(tiles), fin,
      dbias ? bias_part : nullptr);
  AQT_HIP(hipGetLastError());
  return launch_dw_f64_fold(partial, static_cast<int>(slabs), K, N, s_x, s_w, mask_w, one ? nullptr : dw, bias_part,
                            static_cast<int>(slabs * (tiles / tiles_n)), dbias, st);
}

}  // namespace aqt
