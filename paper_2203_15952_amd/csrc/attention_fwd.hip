// Forward of the float attention core for heads of a multiple of four positions on 16-byte aligned tensors: the method and
// the arithmetic of attention.hip (float32 matrix instructions, the same products in the same order, the same bits: the
// quantizer behind it turns a last bit into a whole code now and then), with the time around the products taken out:
//   loads of 16 bytes, split parity-major on the way into LDS (keys) or transposed 4 x 4 in registers (values), so that
//     both products read their LDS operand 16 bytes at a time: 32 reads per step instead of 80;
//   contractions as long as the head (KS steps of 16 positions), not 64; key halves that no query of the wavefront sees
//     are left out (their probabilities are zeros);
//   the window test only in tiles that a window cuts, the rescaling of the accumulator only when the maximum moved
//     (it multiplies by one otherwise), frame indices in 32 bits;
// Measured in us, before -> here: 32 utterances of 400 frames, 8 heads of 64: 172 -> 144; 128 of 512: 702 -> 619 (the float32
// matrix instructions alone take 440 at the full clock; inside an encoder layer the matrix pipes are busy 58 % of the
// kernel's cycles, profiles/encoder_layer_12800_tokens.txt); 24 of 417, 4 heads of 36: 84 -> 69.  Registers bound it to two
// wavefronts per SIMD; at three (16 registers spilled) 150 and 653.  The backward's six-pass bf16 products, built in full
// (three wavefronts per SIMD), take 90 and 401 and are closer to float64 (3.8e-7 of the result's norm against 4.7e-7), but they
// change last bits, and with them a code in every few thousand rows of the layers behind: an int8 layer of 32 x 400
// frames then differs by 1.2e-2 of its gradients' norm.
// Small batches: attention_few.hip, the same bits.
#include "attention_tiles.h"

namespace aqt {
namespace {

constexpr int kK = 64;         // key frames per step
constexpr int kLd = 64 + 4;    // LDS row stride in floats

template <int KS>
struct Rows {   // a lane's query: positions 2 i + lk
  float v[8 * KS];
};

// One step of 64 keys against the wavefront's queries.  NB0 .. NB1 - 1: the 32-key halves that hold a visible key.
template <int KS, int NB0, int NB1>
__device__ __forceinline__ void attend(const float *Ks, const float *Vt, const Rows<KS> &q, int j0, const Window &w, bool whole,
                                       float scale_log2e, float &m, float &l, v16f (&o)[(KS + 1) / 2], int lr, int lk) {
  constexpr int DB = (KS + 1) / 2;
  v16f s[2];   // s[nb][r]: score of key j0 + 32 nb + 8 (r / 4) + 4 lk + r % 4 against this lane's query
#pragma unroll
  for (int nb = NB0; nb < NB1; ++nb) s[nb] = zero16();
#pragma unroll
  for (int i4 = 0; i4 < 2 * KS; ++i4) {
    v4f k[2];
#pragma unroll
    for (int nb = NB0; nb < NB1; ++nb) k[nb] = *reinterpret_cast<const v4f *>(Ks + (nb * 32 + lr) * kLd + lk * 32 + 4 * i4);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int nb = NB0; nb < NB1; ++nb) s[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(k[nb][e], q.v[4 * i4 + e], s[nb], 0, 0, 0);
  }
  float mx = -1e30f;
  if (whole) {
#pragma unroll
    for (int nb = NB0; nb < NB1; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[nb][r] *= scale_log2e;
        mx = fmaxf(mx, s[nb][r]);
      }
  } else {
#pragma unroll
    for (int nb = NB0; nb < NB1; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int j = j0 + 32 * nb + 8 * (r >> 2) + 4 * lk + (r & 3);
        s[nb][r] = (j >= w.lo && j <= w.hi) ? s[nb][r] * scale_log2e : -1e30f;
        mx = fmaxf(mx, s[nb][r]);
      }
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  if (__any(mx > m)) {
    const float mnew = fmaxf(m, mx), alpha = __builtin_amdgcn_exp2f(m - mnew);
    m = mnew;
    l *= alpha;
#pragma unroll
    for (int blk = 0; blk < DB; ++blk)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[blk][r] *= alpha;
  }
  float sum = 0.0f;
#pragma unroll
  for (int nb = NB0; nb < NB1; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = __builtin_amdgcn_exp2f(s[nb][r] - m);
      s[nb][r] = s[nb][r] > -1e29f ? p : 0.0f;   // in whole tiles too: a NaN or an overflow counts as a masked key everywhere
      sum += s[nb][r];
    }
  l += sum;
  // O^T += V^T P^T: step (nb, r) contracts the keys 32 nb + 8 (r / 4) + r % 4 (lk = 0) and that + 4 (lk = 1)
#pragma unroll
  for (int nb = NB0; nb < NB1; ++nb)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      v4f v[DB];
#pragma unroll
      for (int blk = 0; blk < DB; ++blk) v[blk] = *reinterpret_cast<const v4f *>(Vt + (32 * blk + lr) * kLd + 32 * nb + 8 * r4 + 4 * lk);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int blk = 0; blk < DB; ++blk) o[blk] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[blk][e], s[nb][4 * r4 + e], o[blk], 0, 0, 0);
    }
}

// KS: steps of 16 head positions (head widths up to 16 KS)
template <int KS>
__global__ __launch_bounds__(kThreads, 2) void attention_fwd_rows_kernel(const float *__restrict__ qkv, AttnShape g,
                                                                         float *__restrict__ ctx,
                                                                         uint32_t *__restrict__ absmax,
                                                                         float *__restrict__ lse) {
  constexpr int DB = (KS + 1) / 2;
  __shared__ __attribute__((aligned(16))) float lds[2 * kK * kLd];
  float *const Ks = lds;              // [key][even positions, odd positions at + 32]
  float *const Vt = lds + kK * kLd;   // [head column][key]
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63, lr = lane & 31, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Place pl = place_of(g, static_cast<int>(blockIdx.x));
  const int T = g.T, t0 = pl.r0, tw = t0 + wave * 32, t = tw + lr;   // this wavefront's first query, this lane's query
  const bool active = tw < T;   // idle wavefronts of a ragged tile still stage and meet the barriers
  const int64_t ld = 3 * g.D;
  const float *const base = qkv + pl.b * T * ld + pl.hc;   // queries of this utterance and head; keys + D, values + 2 D

  Rows<KS> q;
  {
    const float *row = base + static_cast<int64_t>(t < T ? t : T - 1) * ld;
#pragma unroll
    for (int p = 0; p < 4 * KS; ++p) {
      v4f x = *reinterpret_cast<const v4f *>(row + (4 * p < g.dh ? 4 * p : 0));
      if (4 * p >= g.dh) x = v4f{0.0f, 0.0f, 0.0f, 0.0f};
      q.v[2 * p] = lk ? x.y : x.x;
      q.v[2 * p + 1] = lk ? x.w : x.z;
    }
  }
  const Window w = window_of(t, tw, g.left, g.right, T);
  // key frames any query of this workgroup may look at
  const int jmin = (g.left < 0 || t0 - g.left < 0) ? 0 : t0 - g.left;
  const int tlast = t0 + kQ - 1 < T ? t0 + kQ - 1 : T - 1;
  const int jmax = (g.right < 0 || tlast + g.right > T - 1) ? T - 1 : tlast + g.right;

  // this thread's block of four frames x four positions of the key and value tiles
  const int piece = tid & 15, rows = 4 * (tid >> 4);
  const bool in_head = 4 * piece < g.dh;
  const int64_t at = g.D + (in_head ? 4 * piece : 0);
  v4f kn[4], vn[4];
  auto load = [&](int j0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = j0 + rows + i;
      const float *p = base + static_cast<int64_t>(j < T ? j : T - 1) * ld + at;   // clamped: no branch around a load
      kn[i] = *reinterpret_cast<const v4f *>(p);
      vn[i] = *reinterpret_cast<const v4f *>(p + g.D);
    }
  };
  auto store = [&](int j0) {
    if (piece >= 4 * KS && piece >= 8 * DB) return;   // beyond what the products read
    const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool ok = in_head && j0 + rows + i < T;
      kn[i] = ok ? kn[i] : zero;
      vn[i] = ok ? vn[i] : zero;
      typedef float v2f __attribute__((ext_vector_type(2)));
      float *p = Ks + (rows + i) * kLd + 2 * piece;
      *reinterpret_cast<v2f *>(p) = v2f{kn[i].x, kn[i].z};
      *reinterpret_cast<v2f *>(p + 32) = v2f{kn[i].y, kn[i].w};
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
      *reinterpret_cast<v4f *>(Vt + (4 * piece + c) * kLd + rows) = v4f{vn[0][c], vn[1][c], vn[2][c], vn[3][c]};
  };

  float m = -1e30f, l = 0.0f;   // running maximum (exponent domain of exp2); this lane's share of the running sum
  v16f o[DB];                   // element r: head column 32 blk + 8 (r / 4) + 4 lk + r % 4 of this lane's query
#pragma unroll
  for (int blk = 0; blk < DB; ++blk) o[blk] = zero16();
  const int jfirst = jmin / kK * kK;
  load(jfirst);
  for (int j0 = jfirst; j0 <= jmax; j0 += kK) {
    __syncthreads();   // the previous step's reads are over
    store(j0);
    __syncthreads();
    load(j0 + kK);
    if (!active) continue;
    const bool first = j0 <= w.some_hi && j0 + 31 >= w.some_lo, second = j0 + 32 <= w.some_hi && j0 + 63 >= w.some_lo;
    if (first && second) {
      attend<KS, 0, 2>(Ks, Vt, q, j0, w, j0 >= w.all_lo && j0 + 63 <= w.all_hi, g.scale_log2e, m, l, o, lr, lk);
    } else if (first) {
      attend<KS, 0, 1>(Ks, Vt, q, j0, w, j0 >= w.all_lo && j0 + 31 <= w.all_hi, g.scale_log2e, m, l, o, lr, lk);
    } else if (second) {
      attend<KS, 1, 2>(Ks, Vt, q, j0, w, j0 + 32 >= w.all_lo && j0 + 63 <= w.all_hi, g.scale_log2e, m, l, o, lr, lk);
    }
  }
  __syncthreads();
  float *const img = lds + wave * 32 * kLd;   // [32 queries][68], this wavefront's own quarter: rows leave whole
  uint32_t amax = 0u;
  if (active) {
    const float lt = l + __shfl_xor(l, 32, 64);
    const float inv = lt > 0.0f ? 1.0f / lt : 0.0f;
    // what the backward needs to form the probabilities again: p = exp2(score - lse)
    if (lse && lk == 0 && t < T) lse[(pl.b * T + t) * g.heads + pl.h] = m + log2f(lt);
#pragma unroll
    for (int blk = 0; blk < DB; ++blk)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        *reinterpret_cast<v4f *>(img + lr * kLd + 32 * blk + 8 * r4 + 4 * lk) =
            v4f{o[blk][4 * r4] * inv, o[blk][4 * r4 + 1] * inv, o[blk][4 * r4 + 2] * inv, o[blk][4 * r4 + 3] * inv};
    wave_lds_order();
    const int d = 4 * (lane & 15);   // sixteen lanes per row, four rows at a time
    float *const out = ctx + (pl.b * T + tw) * g.D + pl.hc;
#pragma unroll
    for (int q4 = 0; q4 < 8; ++q4) {
      const int r = 4 * q4 + (lane >> 4);
      if (tw + r < T && d < g.dh) {
        const v4f v = *reinterpret_cast<const v4f *>(img + r * kLd + d);
        *reinterpret_cast<v4f *>(out + r * g.D + d) = v;
        amax = max(max(amax, __float_as_uint(v.x) & 0x7FFFFFFFu), max(__float_as_uint(v.y) & 0x7FFFFFFFu,
                   max(__float_as_uint(v.z) & 0x7FFFFFFFu, __float_as_uint(v.w) & 0x7FFFFFFFu)));
      }
    }
  }
  if (absmax) {   // uniform: the word only grows, so a stale read can only cost a redundant atomic
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) amax = max(amax, static_cast<uint32_t>(__shfl_xor(static_cast<int>(amax), off)));
    if (lane == 0 && amax > *reinterpret_cast<volatile uint32_t *>(absmax)) atomicMax(absmax, amax);
  }
}

}  // namespace

aqt_status launch_attention_rows(const float *qkv, const AttnShape &g, float *ctx, uint32_t *absmax, float *lse, hipStream_t st) {
  if (attention_few_ok(g)) return launch_attention_few(qkv, g, ctx, absmax, lse, st);
  const unsigned blocks = static_cast<unsigned>(static_cast<int64_t>(g.qtiles) * g.heads * g.B);
  auto kern = g.dh <= 16   ? attention_fwd_rows_kernel<1>
              : g.dh <= 32 ? attention_fwd_rows_kernel<2>
              : g.dh <= 48 ? attention_fwd_rows_kernel<3>
                           : attention_fwd_rows_kernel<4>;
  kern<<<blocks, kThreads, 0, st>>>(qkv, g, ctx, absmax, lse);
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

}  // namespace aqt
