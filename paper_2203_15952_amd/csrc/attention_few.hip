// Forward of the float attention core where attention_fwd.hip's tiles of 128 queries are too few to fill the chip: a short
// utterance, a small batch, few heads.  There a launch takes what one wavefront takes to walk the keys, 8200 cycles of matrix
// instructions per 64 keys for its 32 queries; here a workgroup owns 16 queries and its four wavefronts share each
// step: wavefront w forms the scores of keys 16 w .. + 15 and the result's head columns 16 w .. + 15, 1000 cycles a step, with
// scores' maxima and probabilities through LDS between them.
// The same bits as attention_fwd.hip: v_mfma_f32_16x16x4_f32 adds its four products one after the other, as two
// v_mfma_f32_32x32x2_f32 do (both equal a chain of fmaf, measured on 2^18 dot products of 64), and the order of every sum
// is kept: scores along the head; the result over keys k, k + 4, k + 1, k + 5, ..; the normaliser as two shares, keys with bit 2
// clear and set.  (Finite values; a key that a window hides has the probability zero, and where zero times an infinite value is formed at
// all follows the tiles: here those of 16 queries, there of 32.)
#include "attention_tiles.h"

namespace aqt {
namespace {

constexpr int kQf = 16;          // queries a workgroup owns
constexpr int kK = 64;           // key frames per step
constexpr int kLdK = 64 + 4;     // LDS row strides in floats: rows of keys start four banks apart,
constexpr int kLdV = 64 + 16;    // those of values sixteen
constexpr int kLdP = 64 + 4;
constexpr int kSlotFloats = kK * (kLdK + kLdV);

// Row of a value tile that holds key k: the keys k, k + 4, k + 1, k + 5 of a matrix instruction lie next to each other.
__device__ __forceinline__ int value_row(int k) { return (k & ~7) + 4 * ((k >> 1) & 1) + 2 * (k & 1) + ((k >> 2) & 1); }

// KS: steps of 16 head positions (head widths up to 16 KS)
template <int KS>
__global__ __launch_bounds__(kThreads) void attention_fwd_few_kernel(const float *__restrict__ qkv, AttnShape g, int tiles,
                                                                     float *__restrict__ ctx, uint32_t *__restrict__ absmax,
                                                                     float *__restrict__ lse) {
  __shared__ __attribute__((aligned(16))) float slots[2 * kSlotFloats];
  __shared__ __attribute__((aligned(16))) float P[kQf * kLdP];   // [query][4 lg + i / 4][i % 4]: lane group lg's 16 probabilities
  __shared__ float most[4][kQf];                                 // a wavefront's largest score per query
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63, lc = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int id = static_cast<int>(blockIdx.x), tile = id % tiles, bh = id / tiles, h = bh % g.heads;
  const int64_t b = bh / g.heads, ld = 3 * g.D;
  const int T = g.T, t0 = tile * kQf, t = t0 + lc;
  const float *const base = qkv + b * T * ld + static_cast<int64_t>(h) * g.dh;   // queries; keys + D, values + 2 D

  float q[4 * KS];   // this lane's query, positions 4 i + lg
  {
    const float *row = base + static_cast<int64_t>(t < T ? t : T - 1) * ld;
#pragma unroll
    for (int i = 0; i < 4 * KS; ++i) {
      const float x = row[4 * i < g.dh ? 4 * i + lg : 0];
      q[i] = 4 * i < g.dh ? x : 0.0f;
    }
  }
  const int lo = g.left < 0 ? 0 : t - g.left, hi = g.right < 0 || t + g.right > T - 1 ? T - 1 : t + g.right;   // this query's window
  const int jmin = g.left < 0 || t0 - g.left < 0 ? 0 : t0 - g.left;                                            // any query's
  const int tlast = t0 + kQf - 1 < T ? t0 + kQf - 1 : T - 1;
  const int jmax = g.right < 0 || tlast + g.right > T - 1 ? T - 1 : tlast + g.right;

  // this thread's sixteen positions of a key and of a value
  const int row = tid >> 2, piece = tid & 3;
  v4f kn[4], vn[4];
  auto load = [&](int j0) {
    const int j = j0 + row < T ? j0 + row : T - 1;   // clamped: no branch around a load
    const float *p = base + static_cast<int64_t>(j) * ld + g.D;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int d = 16 * piece + 4 * c, at = d < g.dh ? d : 0;
      kn[c] = *reinterpret_cast<const v4f *>(p + at);
      vn[c] = *reinterpret_cast<const v4f *>(p + g.D + at);
    }
  };
  auto store = [&](float *slot, int j0) {
    if (piece >= KS) return;   // beyond what the products read
    const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const bool ok = 16 * piece + 4 * c < g.dh && j0 + row < T;
      kn[c] = ok ? kn[c] : zero;
      vn[c] = ok ? vn[c] : zero;
    }
    float *const k = slot + row * kLdK + 4 * piece, *const v = slot + kK * kLdK + value_row(row) * kLdV + 16 * piece;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      *reinterpret_cast<v4f *>(k + 16 * c) = v4f{kn[0][c], kn[1][c], kn[2][c], kn[3][c]};   // positions 4 i + c, i = 4 piece ..
      *reinterpret_cast<v4f *>(v + 4 * c) = vn[c];
    }
  };

  float m = -1e30f, l = 0.0f;             // running maximum (exponent domain of exp2); the share of keys with bit 2 = lg & 1
  v4f o = {0.0f, 0.0f, 0.0f, 0.0f};       // head columns 16 wave + 4 lg + r of query lc
  const int jfirst = jmin / kK * kK;
  float *cur = slots, *nxt = slots + kSlotFloats;
  load(jfirst);
  store(cur, jfirst);
  load(jfirst + kK);
  __syncthreads();
  for (int j0 = jfirst; j0 <= jmax; j0 += kK) {
    v4f s = {0.0f, 0.0f, 0.0f, 0.0f};     // keys j0 + 16 wave + 4 lg + r
    {
      const float *k = cur + (16 * wave + lc) * kLdK + 16 * lg;
#pragma unroll
      for (int i4 = 0; i4 < KS; ++i4) {
        const v4f x = *reinterpret_cast<const v4f *>(k + 4 * i4);
#pragma unroll
        for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], q[4 * i4 + e], s, 0, 0, 0);
      }
    }
    float mx = -1e30f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = j0 + 16 * wave + 4 * lg + r;
      s[r] = j >= lo && j <= hi ? s[r] * g.scale_log2e : -1e30f;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (lg == 0) most[wave][lc] = mx;
    __syncthreads();   // the maxima are there; everyone is past the last step's probabilities and values
    const float mnew = fmaxf(fmaxf(fmaxf(most[0][lc], most[1][lc]), fmaxf(most[2][lc], most[3][lc])), m);
    const float alpha = __builtin_amdgcn_exp2f(m - mnew);
    m = mnew;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float p = __builtin_amdgcn_exp2f(s[r] - m);
      s[r] = s[r] > -1e29f ? p : 0.0f;
    }
    {
      // key 16 wave + 4 lg + r: lane group 2 (r % 2) + lg % 2, instruction 4 wave + 2 (lg / 2) + r / 2
      typedef float v2f __attribute__((ext_vector_type(2)));
      float *p = P + lc * kLdP + 16 * (lg & 1) + 4 * wave + 2 * (lg >> 1);
      *reinterpret_cast<v2f *>(p) = v2f{s[0], s[2]};
      *reinterpret_cast<v2f *>(p + 32) = v2f{s[1], s[3]};
    }
    if (j0 + kK <= jmax) store(nxt, j0 + kK);
    __syncthreads();
    load(j0 + 2 * kK);
    l *= alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] *= alpha;
    float sum = 0.0f;
    const float *const pe = P + lc * kLdP + 16 * (lg & 1);   // even keys of this share, odd ones at + 32
    const float *const v = cur + kK * kLdK + lg * kLdV + 16 * wave + lc;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (j0 + 32 * half > jmax || j0 + 32 * half + 31 < jmin) continue;   // zeros (and values nobody sees)
#pragma unroll
      for (int i4 = 2 * half; i4 < 2 * half + 2; ++i4) {
        const v4f x = *reinterpret_cast<const v4f *>(pe + 4 * i4), y = *reinterpret_cast<const v4f *>(pe + 32 + 4 * i4);
        float vv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) vv[e] = 16 * wave < 16 * KS ? v[4 * (4 * i4 + e) * kLdV] : 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[e], lg < 2 ? x[e] : y[e], o, 0, 0, 0);
          sum += x[e];
          sum += y[e];
        }
      }
    }
    l += sum;
    float *const other = cur; cur = nxt; nxt = other;
  }
  const float lt = l + __shfl_xor(l, 16, 64);
  const float inv = lt > 0.0f ? 1.0f / lt : 0.0f;
  // what the backward needs to form the probabilities again: p = exp2(score - lse)
  if (lse && wave == 0 && lg == 0 && t < T) lse[(b * T + t) * g.heads + h] = m + log2f(lt);
  uint32_t amax = 0u;
  const int d = 16 * wave + 4 * lg;
  if (t < T && d < g.dh) {
    const v4f x = {o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv};
    *reinterpret_cast<v4f *>(ctx + (b * T + t) * g.D + static_cast<int64_t>(h) * g.dh + d) = x;
#pragma unroll
    for (int r = 0; r < 4; ++r) amax = max(amax, __float_as_uint(x[r]) & 0x7FFFFFFFu);
  }
  if (absmax) {   // uniform; one atomic per workgroup, and only if it can raise the word (it only grows)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) amax = max(amax, static_cast<uint32_t>(__shfl_xor(static_cast<int>(amax), off)));
    __syncthreads();   // the maxima of the scores are no longer read
    if (lane == 0) most[wave][0] = __uint_as_float(amax);
    __syncthreads();
    if (tid == 0) {
#pragma unroll
      for (int w = 1; w < 4; ++w) amax = max(amax, __float_as_uint(most[w][0]));
      if (amax > *reinterpret_cast<volatile uint32_t *>(absmax)) atomicMax(absmax, amax);
    }
  }
}

}  // namespace

// As long as all of its workgroups run at once, two to a compute unit (80 KB of LDS each).  In us, tiles of 128 -> here: 6 x 217
// frames, 4 heads of 36 (336 workgroups) 20.9 -> 12; 8 x 128, 4 heads of 64 (256) 15.4 -> 9.3, what a launch from Python takes;
// 8 x 128, 8 heads (512) 15.6 -> 14.8; 2 x 1000, 4 heads (504) 85 -> 53; 8 x 217, 8 heads (896) 24 -> 34.
// Where two share a compute unit and an utterance is one step of keys, it is behind in two places.  Up to 32 frames one wavefront of the other
// kernel does an utterance: 25 x 32 ... 63 x 32 frames, 4 heads of 24 7.1 -> 8.4, of 64 8.7 -> 10.4, of 4 6.7 -> 7.0, and 13 to 16 frames
// where a head fills its steps of 16 positions, of 24 8.0 -> 8.3, of 48 9.4 -> 9.7 (of 36 0.97 - 1.00 of the time, of 64 0.96).  64 frames that all see
// each other are a tile without masks there: heads of 24 8.4 -> 9.1, of 32 8.4 -> 8.8, of 44 10.2 -> 10.6, of 48 10.4 -> 10.7 (of 36 0.97, of 64 0.97, of 16 0.93).
// Between them, 33 to 63 frames, 0.87 to 1.04 of the time, most of it below 1; one to a compute unit it is ahead everywhere (31 x
// 17, 4 heads of 4 6.6 -> 6.0).
bool attention_few_ok(const AttnShape &g) {
  const int64_t groups = cdiv(g.T, kQf) * g.heads;
  if (groups > 512 / g.B) return false;
  if (groups <= 256 / g.B) return true;
  const bool fills = g.dh > 16 && (g.dh <= 32 || (g.dh > 40 && g.dh <= 48));
  const bool whole = g.T == 64 && (g.left < 0 || g.left >= 63) && (g.right < 0 || g.right >= 63);
  return g.T <= (fills ? 12 : 16) || (g.T > 32 && !(whole && fills));
}

aqt_status launch_attention_few(const float *qkv, const AttnShape &g, float *ctx, uint32_t *absmax, float *lse, hipStream_t st) {
  const int tiles = static_cast<int>(cdiv(g.T, kQf));
  const unsigned blocks = static_cast<unsigned>(tiles * static_cast<int64_t>(g.heads) * g.B);
  auto kern = g.dh <= 16   ? attention_fwd_few_kernel<1>
              : g.dh <= 32 ? attention_fwd_few_kernel<2>
              : g.dh <= 48 ? attention_fwd_few_kernel<3>
                           : attention_fwd_few_kernel<4>;
  kern<<<blocks, kThreads, 0, st>>>(qkv, g, tiles, ctx, absmax, lse);
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

}  // namespace aqt
