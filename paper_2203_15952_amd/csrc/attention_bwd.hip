// Backward of the float attention core for heads of a multiple of four positions on 16-byte aligned tensors (the chain rule
// and the two kernels of attention.hip).  The scores are formed as in the forward, on the float32 matrix cores with the same
// products in the same order, so that a probability exp2(score - lse) is the one the forward's normaliser was made of:
// a score that differs in its last bits, even for the better, leaves rows that do not add up to one, an error that grows with
// the scores (normal queries and keys, heads of 64, 512 frames, times eight: dv off by 3.0e-5 of its norm, 4.3e-6 so).
// The other products run on the bf16 matrix cores without giving up float32: every operand is carried whole
// as three bf16 terms of 8 significant bits each (a = hi + mid + lo exactly), and a product is six
// v_mfma_f32_32x32x16_bf16 passes, hi hi, hi mid, mid hi, mid mid, hi lo, lo hi.  What is left out is at most 2^-24 (1 + 2^-10)
// of a product, one rounding of it, and mostly far less: 64-term dot products measured against float64, rms error
// 1.8e-8 of the sum of magnitudes, 2.4e-8 with v_mfma_f32_32x32x2_f32.  Six bf16 passes take 6/16 of the float32
// instruction's time; the splitting is vector work, done once per workgroup for the staged rows.
// An infinity, or a value that rounds to one in bf16, has no such terms: its lowest is a NaN, and so is every sum that it
// enters.  A wavefront that ends with a value that is not finite forms its rows again with every product in float32
// (redo_dq, redo_dkv, straight from memory), so what is finite or infinite in float32 stays so: 32 utterances of 400 frames, 8 heads
// of 64, 302 us, 1321 if every wavefront does.
//
// As in attention.hip all products are formed transposed, a lane owns one query (in the key / value gradient kernel:
// one key) from start to end, and the probabilities go from the first products' accumulators into the last products'
// B operand without leaving the lane.  Tiles of 32 rows go through LDS: split images row-major, one 128-byte row per image,
// 16-byte chunks XOR-swizzled with the row, and the rows that scores are made of once more in float32, parity-major as in
// attention.hip.  Operands that contract along the head are read as 16-byte row pieces; operands
// that contract along the rows are read from the same image with ds_read_b64_tr_b16 (sixteen lanes read four rows of
// sixteen columns, each lane receives one column), whose four-row groups are exactly the rows an accumulator lane
// holds.  Two LDS slots: a tile is staged and split while the one before it is multiplied, one barrier per tile.
//
// Measured in us, all products in float32 (attention.hip) -> scores in float32, the rest here: 32 utterances of 400 frames,
// 8 heads of 64: 621 -> 295; 128 of 512: 2808 -> 1455; 24 of 417, 4 heads of 36: 310 -> 136.  What every tile pays counts:
// window tests and zeros beyond the head or the utterance stand under branches of their own, and the constant part of an LDS
// address goes into the instruction (310 -> 295, 1510 -> 1453, 146 -> 136, the same bits).  Before that, all products in bf16
// passes took 273, 1392 and 125 against 306, 1500 and 146, with the error above.  The matrix pipes are busy 52 % of the
// cycles of both kernels inside an encoder layer (profiles/encoder_layer_12800_tokens.txt).
// Small batches, whose workgroups of 128 rows leave the chip idle: FEW, 32 rows to a workgroup and the tiles shared out among
// its wavefronts (attention_bwd_few_ok).
#include <type_traits>

#include "attention_tiles.h"
#include "bf16_terms.h"

namespace aqt {
namespace {

constexpr int kStep = 32;            // rows per staged tile
constexpr int kRowBytes = 128;       // an LDS row: 64 bf16
constexpr int kImage = kStep * kRowBytes;
constexpr int kTensor = 3 * kImage;  // hi, mid, lo
constexpr int kLd = 68;              // row stride in floats of the float32 rows and of the output image
constexpr int kSlot = 2 * kTensor + kStep * kLd * 4;   // two tensors per tile, and the float32 rows of the first

typedef short v4s __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));

struct Split {   // one operand fragment: eight values of a lane as three bf16 terms
  v4i hi, mid, lo;
};

__device__ __forceinline__ Split split8(float a, float b, float c, float d, float e, float f, float g, float h) {
  Split s;
  int x, y, z;
  split3_bf16(a, b, x, y, z); s.hi.x = x; s.mid.x = y; s.lo.x = z;
  split3_bf16(c, d, x, y, z); s.hi.y = x; s.mid.y = y; s.lo.y = z;
  split3_bf16(e, f, x, y, z); s.hi.z = x; s.mid.z = y; s.lo.z = z;
  split3_bf16(g, h, x, y, z); s.hi.w = x; s.mid.w = y; s.lo.w = z;
  return s;
}

__device__ __forceinline__ v16f mfma6(const Split &a, const Split &b, v16f c) {   // smallest terms first
  c = mfma_bf16(a.lo, b.hi, c);
  c = mfma_bf16(a.hi, b.lo, c);
  c = mfma_bf16(a.mid, b.mid, c);
  c = mfma_bf16(a.mid, b.hi, c);
  c = mfma_bf16(a.hi, b.mid, c);
  return mfma_bf16(a.hi, b.hi, c);
}
// Rows lr of an image set, head positions 16 s + 8 lk .. + 7: contraction along the head.
__device__ __forceinline__ Split read_rows(const uint8_t *tensor, int s, int lr, int lk) {
  const uint8_t *p = tensor + lr * kRowBytes + (((2 * s + lk) ^ (lr & 7)) << 4);
  return Split{*reinterpret_cast<const v4i *>(p), *reinterpret_cast<const v4i *>(p + kImage),
               *reinterpret_cast<const v4i *>(p + 2 * kImage)};
}
// Head columns 32 blk + lr, the eight rows 16 s + 8 (e / 4) + 4 lk + e % 4: contraction along the rows, in the order
// in which elements 8 s .. 8 s + 7 of an accumulator lane hold them.
template <int AT>
__device__ __forceinline__ v4i read_tr8(uint32_t at) {   // LDS addresses at + AT and eight rows on: the constant goes into the instruction
  typedef __attribute__((address_space(3))) v4s *lds_v4s;
  const v2i a = __builtin_bit_cast(v2i, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_v4s>(at + AT)));
  const v2i b = __builtin_bit_cast(v2i, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_v4s>(at + AT + 8 * kRowBytes)));
  return v4i{a.x, a.y, b.x, b.y};
}
template <int S>
__device__ __forceinline__ Split read_cols(const uint8_t *tensor, int blk, int lane) {
  const int i = lane & 15, c = i & 3, chunk = 4 * blk + 2 * ((lane >> 4) & 1) + (c >> 1);
  const int row = 4 * (lane >> 5) + (i >> 2);   // the first of eight, the same modulo 8 in every group of sixteen
  const uint32_t at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(tensor)) + row * kRowBytes + ((chunk ^ (row & 7)) << 4) + 8 * (c & 1);
  constexpr int kAt = 16 * S * kRowBytes;
  return Split{read_tr8<kAt>(at), read_tr8<kAt + kImage>(at), read_tr8<kAt + 2 * kImage>(at)};
}

// A thread's share of a tile: eight head positions of one row (rows beyond the utterance are read from its last one).
struct Raw {
  v4f a, b;
};
__device__ __forceinline__ Raw load_piece(const float *__restrict__ src, int64_t ld, const AttnShape &g, int64_t b, int row0,
                                          int64_t col0, int thread) {
  const int piece = thread & 7;
  const int t = row0 + (thread >> 3), tc = t < g.T ? t : g.T - 1;
  const float *p = src + (b * g.T + tc) * ld + col0;
  const int d = 8 * piece, d0 = d < g.dh ? d : g.dh - 4, d1 = d + 4 < g.dh ? d + 4 : g.dh - 4;
  return Raw{*reinterpret_cast<const v4f *>(p + d0), *reinterpret_cast<const v4f *>(p + d1)};
}
// ... split into the three images; zeros beyond the head and, where `rows` says so, beyond the utterance
// (`floats`: the same rows in float32, even positions, then odd ones).
template <int PIECES>
__device__ __forceinline__ void stage_piece(uint8_t *tensor, Raw v, const AttnShape &g, int row0, bool rows, int thread,
                                            float *floats = nullptr) {
  const int piece = thread & 7, row = thread >> 3;
  const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
  if (8 * PIECES > g.dh) {   // uniform, as the next: most tiles pay for neither
    if (8 * piece >= g.dh) v.a = zero;
    if (8 * piece + 4 >= g.dh) v.b = zero;
  }
  if (rows && row0 + kStep > g.T && row0 + row >= g.T) v.a = v.b = zero;
  if (PIECES == 8 || piece < PIECES) {
    const Split s = split8(v.a.x, v.a.y, v.a.z, v.a.w, v.b.x, v.b.y, v.b.z, v.b.w);
    uint8_t *p = tensor + row * kRowBytes + ((piece ^ (row & 7)) << 4);
    *reinterpret_cast<v4i *>(p) = s.hi;
    *reinterpret_cast<v4i *>(p + kImage) = s.mid;
    *reinterpret_cast<v4i *>(p + 2 * kImage) = s.lo;
    if (floats) {
      *reinterpret_cast<v4f *>(floats + row * kLd + 4 * piece) = v4f{v.a.x, v.a.z, v.b.x, v.b.z};
      *reinterpret_cast<v4f *>(floats + row * kLd + 32 + 4 * piece) = v4f{v.a.y, v.a.w, v.b.y, v.b.w};
    }
  }
}

// A lane's own row as a B operand of the scores: positions 2 i + lk.
template <int KS>
struct Own {
  float v[8 * KS];
};
template <int KS>
__device__ __forceinline__ Own<KS> own_floats(const float *row, int lk, int dh) {
  Own<KS> q;
#pragma unroll
  for (int p = 0; p < 4 * KS; ++p) {
    v4f x = *reinterpret_cast<const v4f *>(row + (4 * p < dh ? 4 * p : 0));
    if (4 * p >= dh) x = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    q.v[2 * p] = lk ? x.y : x.x;
    q.v[2 * p + 1] = lk ? x.w : x.z;
  }
  return q;
}
// ... as a split operand: positions 16 s + 8 lk .. + 7.
__device__ __forceinline__ void load_own(v4f &x, v4f &y, const float *row, int s, int lk, int dh) {
  const int d = 16 * s + 8 * lk;
  const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
  x = d < dh ? *reinterpret_cast<const v4f *>(row + d) : zero;
  y = d + 4 < dh ? *reinterpret_cast<const v4f *>(row + d + 4) : zero;
}
__device__ __forceinline__ Split split_own(v4f x, v4f y) { return split8(x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w); }

// Scores (staged rows x own row, the forward's bits) and the second product of a tile, in one loop so that either's
// chain of matrix instructions runs under the other's operand reads.
template <int KS>
__device__ __forceinline__ void first_products(const uint8_t *slot, const Own<KS> &own, const Split (&second)[KS], v16f &s, v16f &dp,
                                               int lr, int lk) {
  const float *const rows = reinterpret_cast<const float *>(slot + 2 * kTensor) + lr * kLd + lk * 32;
  s = zero16();
  dp = zero16();
#pragma unroll
  for (int k = 0; k < KS; ++k) {
#pragma unroll
    for (int i4 = 2 * k; i4 < 2 * k + 2; ++i4) {
      const v4f x = *reinterpret_cast<const v4f *>(rows + 4 * i4);
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], own.v[4 * i4 + e], s, 0, 0, 0);
    }
    dp = mfma6(read_rows(slot + kTensor, k, lr, lk), second[k], dp);
  }
}
__device__ __forceinline__ float dot8(v4f a, v4f b, v4f c, v4f d) {
  return ((a.x * c.x + a.y * c.y) + (a.z * c.z + a.w * c.w)) + ((b.x * d.x + b.y * d.y) + (b.z * d.z + b.w * d.w));
}

// a wavefront's transposed result (head positions x 32 rows) out through its own part of LDS as whole rows
template <int DB>
__device__ __forceinline__ void store_rows(float *img, const v16f (&acc)[DB], float mul, float *__restrict__ out, int64_t ld,
                                               int rows_left, int dh, int lane) {
  const int lr = lane & 31, lk = lane >> 5;
#pragma unroll
  for (int blk = 0; blk < DB; ++blk)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const v4f v = {acc[blk][4 * r4] * mul, acc[blk][4 * r4 + 1] * mul, acc[blk][4 * r4 + 2] * mul, acc[blk][4 * r4 + 3] * mul};
      *reinterpret_cast<v4f *>(img + lr * kLd + 32 * blk + 8 * r4 + 4 * lk) = v;
    }
  wave_lds_order();
  // sixteen lanes per row, four rows at a time
  const int d = 4 * (lane & 15);
#pragma unroll
  for (int q4 = 0; q4 < 8; ++q4) {
    const int q = 4 * q4 + (lane >> 4);
    if (q < rows_left && d < dh) *reinterpret_cast<v4f *>(out + q * ld + d) = *reinterpret_cast<const v4f *>(img + q * kLd + d);
  }
  wave_lds_order();
}

template <int DB>
__device__ __forceinline__ bool any_nonfinite(const v16f (&acc)[DB]) {
  uint32_t most = 0u;
#pragma unroll
  for (int blk = 0; blk < DB; ++blk)
#pragma unroll
    for (int r = 0; r < 16; ++r) most = max(most, __float_as_uint(acc[blk][r]) & 0x7FFFFFFFu);
  return __any(most >= 0x7F800000u);
}

// The tile loop: rows first, first + 32, ... <= last, two tensors per tile; compute(slot, row0) between.
template <class Load, class Stage, class Compute>
__device__ __forceinline__ void run_tiles(uint8_t *lds, int first, int last, Load load, Stage stage, Compute compute) {
  uint8_t *cur = lds, *nxt = lds + kSlot;
  load(first);
  stage(cur, first);
  load(first + kStep);   // rows beyond the utterance are clamped: no branch around a load
  __syncthreads();
  for (int r0 = first; r0 <= last; r0 += kStep) {
    if (r0 + kStep <= last) stage(nxt, r0 + kStep);
    load(r0 + 2 * kStep);
    compute(cur, r0);
    __syncthreads();
    uint8_t *const t = cur; cur = nxt; nxt = t;
  }
}

// FEW: a workgroup owns 32 rows, and its wavefronts take the tiles in turn, each with a slot of its own, loaded and split by
// itself: no barrier on the way.  bring(slot, row0) requests and stages a tile.
template <class Bring, class Compute>
__device__ __forceinline__ void run_tiles_apart(uint8_t *slot, int wave, int first, int last, Bring bring, Compute compute) {
  for (int r0 = first + wave * kStep; r0 <= last; r0 += 4 * kStep) {
    bring(slot, r0);
    wave_lds_order();
    compute(slot, r0);
    wave_lds_order();
  }
}
// The four wavefronts' shares of 32 rows, in order, into v (row tid / 8, positions 8 (tid % 8) .. + 7); lds: 4 x 32 x kLd floats.
// True in every thread if one of the sums is not finite.
template <int DB>
__device__ __forceinline__ bool add_shares(float *lds, const v16f (&acc)[DB], int wave, int lane, v4f (&v)[2]) {
  const int lr = lane & 31, lk = lane >> 5, row = static_cast<int>(threadIdx.x >> 3), at = 8 * static_cast<int>(threadIdx.x & 7);
  __syncthreads();   // the tiles, or the shares before these, are no longer read
  float *const img = lds + wave * 32 * kLd;
#pragma unroll
  for (int blk = 0; blk < DB; ++blk)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4)
      *reinterpret_cast<v4f *>(img + lr * kLd + 32 * blk + 8 * r4 + 4 * lk) =
          v4f{acc[blk][4 * r4], acc[blk][4 * r4 + 1], acc[blk][4 * r4 + 2], acc[blk][4 * r4 + 3]};
  __syncthreads();
  bool bad = false;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    v[c] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    if (at >= 32 * DB) continue;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const v4f x = *reinterpret_cast<const v4f *>(lds + (w * 32 + row) * kLd + at + 4 * c);
      v[c].x += x.x; v[c].y += x.y; v[c].z += x.z; v[c].w += x.w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) bad = bad || (__float_as_uint(v[c][e]) & 0x7FFFFFFFu) >= 0x7F800000u;
  }
  return __syncthreads_or(bad) != 0;
}
__device__ __forceinline__ void store_shares(const v4f (&v)[2], float mul, float *__restrict__ out, int64_t ld, int rows_left, int dh) {
  const int row = static_cast<int>(threadIdx.x >> 3), at = 8 * static_cast<int>(threadIdx.x & 7);
#pragma unroll
  for (int c = 0; c < 2; ++c)
    if (row < rows_left && at + 4 * c < dh)
      *reinterpret_cast<v4f *>(out + row * ld + at + 4 * c) = v4f{v[c].x * mul, v[c].y * mul, v[c].z * mul, v[c].w * mul};
}

// ---- the same sums with every product in float32, a wavefront by itself --------------------------------
// (Only where it is needed: everything is formed anew from the workgroup's number, so that nothing has to be kept for it.)
// A's 32 rows (zeros beyond the utterance) times each lane's own row, along the head, in the order of first_products.
__device__ __forceinline__ v16f float_product(const float *__restrict__ row, bool in, const float *__restrict__ own, int lk, int dh) {
  v16f s = zero16();
#pragma unroll 1
  for (int d = 0; d < dh; d += 4) {
    v4f x = *reinterpret_cast<const v4f *>(row + d);
    const v4f y = *reinterpret_cast<const v4f *>(own + d);
    if (!in) x = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    s = __builtin_amdgcn_mfma_f32_32x32x2f32(lk ? x.y : x.x, lk ? y.y : y.x, s, 0, 0, 0);
    s = __builtin_amdgcn_mfma_f32_32x32x2f32(lk ? x.w : x.z, lk ? y.w : y.z, s, 0, 0, 0);
  }
  return s;
}
// acc += rows^T x: step r contracts the rows r0 + 8 (r / 4) + r % 4 (lk = 0) and that + 4 (lk = 1)
template <int DB>
__device__ __forceinline__ void float_product_rows(v16f (&acc)[DB], const float *__restrict__ src, int64_t ld, const AttnShape &g,
                                                   int r0, const v16f &x, int lr, int lk) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int at = r0 + 8 * (r >> 2) + 4 * lk + (r & 3);
#pragma unroll
    for (int blk = 0; blk < DB; ++blk) {
      const int d = 32 * blk + lr;
      const float v = src[(at < g.T ? at : g.T - 1) * ld + (d < g.dh ? d : 0)];
      acc[blk] = __builtin_amdgcn_mfma_f32_32x32x2f32(at < g.T && d < g.dh ? v : 0.0f, x[r], acc[blk], 0, 0, 0);
    }
  }
}
// What a wavefront of either kernel walks: its lane's own row t of the utterance, and the rows first .. last, of which
// the lane's row meets lo .. hi; back / ahead: how far that reaches from its own row (negative: no limit).
struct Redo {
  int64_t base, hc;   // the utterance's first token, the head's first column
  int tw, t, tc, first, last, lo, hi, h, lr, lk;
};
template <int ROWS>
__device__ __forceinline__ Redo redo_place(const AttnShape &g, int back, int ahead) {
  int id = static_cast<int>(blockIdx.x), thread = static_cast<int>(threadIdx.x);
  asm volatile("" : "+s"(id));
  asm volatile("" : "+v"(thread));
  const Place pl = place_of<ROWS>(g, id);
  const int lr = thread & 31, tw = pl.r0 + (__builtin_amdgcn_readfirstlane(thread) >> 6) * 32, t = tw + lr;
  const Window w = window_of(t, tw, back, ahead, g.T);
  return Redo{pl.b * g.T, pl.hc, tw, t, t < g.T ? t : g.T - 1, w.some_lo > 0 ? w.some_lo / kStep * kStep : 0, w.some_hi, w.lo, w.hi,
              pl.h, lr, (thread >> 5) & 1};
}
template <int DB, int ROWS>
__device__ __forceinline__ void redo_dq(v16f (&dq)[DB], const float *__restrict__ qkv, const float *__restrict__ dctx,
                                        const float *__restrict__ lse, const float *dsum, const AttnShape &g) {
  const Redo w = redo_place<ROWS>(g, g.left, g.right);
  const int64_t ld = 3 * g.D;
  const float *const q = qkv + (w.base + w.tc) * ld + w.hc, *const go = dctx + (w.base + w.tc) * g.D + w.hc;
  const float *const keys = qkv + w.base * ld + g.D + w.hc;
  const float L = lse[(w.base + w.tc) * g.heads + w.h], D = dsum[(w.base + w.tc) * g.heads + w.h];
#pragma unroll
  for (int blk = 0; blk < DB; ++blk) dq[blk] = zero16();
#pragma unroll 1
  for (int j0 = w.first; j0 <= w.last; j0 += kStep) {
    const bool in = j0 + w.lr < g.T;
    const float *const key = keys + (in ? j0 + w.lr : g.T - 1) * ld;
    v16f s = float_product(key, in, q, w.lk, g.dh);
    const v16f dp = float_product(key + g.D, in, go, w.lk, g.dh);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + 8 * (r >> 2) + 4 * w.lk + (r & 3);
      const float p = (j >= w.lo && j <= w.hi) ? __builtin_amdgcn_exp2f(s[r] * g.scale_log2e - L) : 0.0f;
      s[r] = p * (dp[r] - D);
    }
    float_product_rows(dq, keys, ld, g, j0, s, w.lr, w.lk);
  }
}
template <int DB, int ROWS>
__device__ __forceinline__ void redo_dkv(v16f (&dk)[DB], v16f (&dv)[DB], const float *__restrict__ qkv, const float *__restrict__ dctx,
                                         const float *__restrict__ lse, const float *__restrict__ dsum, const AttnShape &g) {
  const Redo w = redo_place<ROWS>(g, g.right, g.left);
  const int64_t ld = 3 * g.D;
  const float *const k = qkv + (w.base + w.tc) * ld + g.D + w.hc;
  const float *const queries = qkv + w.base * ld + w.hc, *const grads = dctx + w.base * g.D + w.hc;
#pragma unroll
  for (int blk = 0; blk < DB; ++blk) {
    dk[blk] = zero16();
    dv[blk] = zero16();
  }
#pragma unroll 1
  for (int t0 = w.first; t0 <= w.last; t0 += kStep) {
    const bool in = t0 + w.lr < g.T;
    const int64_t at = in ? t0 + w.lr : g.T - 1;
    v16f s = float_product(queries + at * ld, in, k, w.lk, g.dh);
    v16f dp = float_product(grads + at * g.D, in, k + g.D, w.lk, g.dh);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int t = t0 + 8 * (r >> 2) + 4 * w.lk + (r & 3);
      const int64_t row = (w.base + (t < g.T ? t : g.T - 1)) * g.heads + w.h;
      const float p = (w.t < g.T && t >= w.lo && t <= w.hi) ? __builtin_amdgcn_exp2f(s[r] * g.scale_log2e - lse[row]) : 0.0f;
      s[r] = p;
      dp[r] = p * (dp[r] - dsum[row]);
    }
    float_product_rows(dv, grads, g.D, g, t0, s, w.lr, w.lk);
    float_product_rows(dk, queries, ld, g, t0, dp, w.lr, w.lk);
  }
}

// ---- backward: the chain rule and the two kernels of attention.hip ---------------------------------
// dq: a lane owns a query.  Also forms D_t = dO_t . O_t of its queries (the lane reads dO_t anyway) and leaves it in
// dsum for the dk / dv kernel.
template <int KS, bool FEW = false>
__global__ __launch_bounds__(kThreads, FEW ? 1 : 2) void attention_bwd_dq_rows_kernel(const float *__restrict__ qkv,
                                                                             const float *__restrict__ ctx,
                                                                             const float *__restrict__ dctx,
                                                                             const float *__restrict__ lse,
                                                                             float *__restrict__ dsum, AttnShape g,
                                                                             float *__restrict__ dqkv) {
  constexpr int DB = (KS + 1) / 2, kRows = FEW ? 32 : kQ;
  __shared__ __attribute__((aligned(16))) uint8_t lds[(FEW ? 4 : 2) * kSlot];
  const int lane = threadIdx.x & 63, lr = lane & 31, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Place pl = place_of<kRows>(g, static_cast<int>(blockIdx.x));
  const int64_t b = pl.b, hc = pl.hc;
  const int t0 = pl.r0;
  const int tw = FEW ? t0 : t0 + wave * 32, t = tw + lr, tc = t < g.T ? t : g.T - 1;
  const bool active = tw < g.T;
  const float *const qrow = qkv + (b * g.T + tc) * 3 * g.D + hc, *const grow = dctx + (b * g.T + tc) * g.D + hc;
  const Own<KS> q = own_floats<KS>(qrow, lk, g.dh);
  Split go[KS];
  float D = 0.0f;
  {
    const float *orow = ctx + (b * g.T + tc) * g.D + hc;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      v4f gx, gy, ox, oy;
      load_own(gx, gy, grow, s, lk, g.dh);
      load_own(ox, oy, orow, s, lk, g.dh);
      go[s] = split_own(gx, gy);
      D += dot8(gx, gy, ox, oy);
    }
  }
  D += __shfl_xor(D, 32, 64);
  const float L = lse[(b * g.T + tc) * g.heads + pl.h];
  if ((!FEW || wave == 0) && lk == 0 && t < g.T) dsum[(b * g.T + t) * g.heads + pl.h] = D;
  const int tlast = t0 + kRows - 1 < g.T ? t0 + kRows - 1 : g.T - 1;
  const int jmin = (g.left < 0 || t0 - g.left < 0) ? 0 : t0 - g.left;
  const int jmax = (g.right < 0 || tlast + g.right > g.T - 1) ? g.T - 1 : tlast + g.right;
  const int wlo = g.left < 0 ? 0 : t - g.left;
  const int whi = (g.right < 0 || t + g.right > g.T - 1) ? g.T - 1 : t + g.right;
  const int some_lo = g.left < 0 ? 0 : tw - g.left, all_lo = g.left < 0 ? 0 : tw + 31 - g.left;
  const int some_hi = (g.right < 0 || tw + 31 + g.right > g.T - 1) ? g.T - 1 : tw + 31 + g.right;
  const int all_hi = (g.right < 0 || tw + g.right > g.T - 1) ? g.T - 1 : tw + g.right;
  v16f dq[DB];
#pragma unroll
  for (int blk = 0; blk < DB; ++blk) dq[blk] = zero16();
  constexpr int P = FEW ? 4 : 1;   // pieces of a thread
  Raw kr[P], vr[P];
  auto thread = [&](int i) { return FEW ? lane + 64 * i : static_cast<int>(threadIdx.x); };
  auto load = [&](int j0) {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      kr[i] = load_piece(qkv, 3 * g.D, g, b, j0, g.D + hc, thread(i));
      vr[i] = load_piece(qkv, 3 * g.D, g, b, j0, 2 * g.D + hc, thread(i));
    }
  };
  auto stage = [&](uint8_t *slot, int j0) {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      stage_piece<4 * DB>(slot, kr[i], g, j0, true, thread(i), reinterpret_cast<float *>(slot + 2 * kTensor));
      stage_piece<2 * KS>(slot + kTensor, vr[i], g, j0, false, thread(i));
    }
  };
  auto compute = [&](const uint8_t *slot, int j0) {
    if (!active || j0 > some_hi || j0 + kStep - 1 < some_lo) return;
    v16f s, dp;
    first_products<KS>(slot, q, go, s, dp, lr, lk);   // S^T: keys x this lane's query; dP^T
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(s[r] * g.scale_log2e - L) * (dp[r] - D);
    if (j0 < all_lo || j0 + kStep - 1 > all_hi) {   // cut by a window: a loop of its own, or every tile pays for the test
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int j = j0 + 8 * (r >> 2) + 4 * lk + (r & 3);
        s[r] = j >= wlo && j <= whi ? s[r] : 0.0f;
      }
    }
    auto add_half = [&](auto half) {
      constexpr int k = decltype(half)::value;
      const Split d = split8(s[8 * k], s[8 * k + 1], s[8 * k + 2], s[8 * k + 3], s[8 * k + 4], s[8 * k + 5], s[8 * k + 6], s[8 * k + 7]);
#pragma unroll
      for (int blk = 0; blk < DB; ++blk) dq[blk] = mfma6(read_cols<k>(slot, blk, lane), d, dq[blk]);   // dQ^T += K^T dS^T
    };
    add_half(std::integral_constant<int, 0>{});
    add_half(std::integral_constant<int, 1>{});
  };
  float *const out = dqkv + (b * g.T + tw) * 3 * g.D + hc;
  if constexpr (FEW) {
    run_tiles_apart(lds + wave * kSlot, wave, jmin / kStep * kStep, jmax, [&](uint8_t *slot, int j0) { load(j0); stage(slot, j0); }, compute);
    v4f v[2];
    if (!add_shares<DB>(reinterpret_cast<float *>(lds), dq, wave, lane, v)) {
      store_shares(v, g.scale, out, 3 * g.D, g.T - tw, g.dh);
      return;
    }
    if (wave != 0) return;
    redo_dq<DB, kRows>(dq, qkv, dctx, lse, dsum, g);
  } else {
    run_tiles(lds, jmin / kStep * kStep, jmax, load, stage, compute);
    if (!active) return;
    if (any_nonfinite(dq)) redo_dq<DB, kRows>(dq, qkv, dctx, lse, dsum, g);
  }
  store_rows<DB>(reinterpret_cast<float *>(lds) + wave * 32 * kLd, dq, g.scale, out, 3 * g.D, g.T - tw, g.dh, lane);
}

// dk / dv: a lane owns a key, the tiles are queries and upstream gradient rows.
template <int KS, bool FEW = false>
__global__ __launch_bounds__(kThreads, FEW ? 1 : 2) void attention_bwd_dkv_rows_kernel(const float *__restrict__ qkv,
                                                                              const float *__restrict__ dctx,
                                                                              const float *__restrict__ lse,
                                                                              const float *__restrict__ dsum, AttnShape g,
                                                                              float *__restrict__ dqkv) {
  constexpr int DB = (KS + 1) / 2, kRows = FEW ? 32 : kQ;
  __shared__ __attribute__((aligned(16))) uint8_t lds[(FEW ? 4 : 2) * kSlot];
  __shared__ __attribute__((aligned(16))) float Ls[FEW ? 4 : 2][kStep], Ds[FEW ? 4 : 2][kStep];
  const int lane = threadIdx.x & 63, lr = lane & 31, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Place pl = place_of<kRows>(g, static_cast<int>(blockIdx.x));
  const int64_t b = pl.b, hc = pl.hc;
  const int j0t = pl.r0;
  const int jw = FEW ? j0t : j0t + wave * 32, j = jw + lr, jc = j < g.T ? j : g.T - 1;
  const bool active = jw < g.T;
  const float *const krow = qkv + (b * g.T + jc) * 3 * g.D + g.D + hc;
  const Own<KS> kk = own_floats<KS>(krow, lk, g.dh);
  Split vv[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    v4f x, y;
    load_own(x, y, krow + g.D, s, lk, g.dh);
    vv[s] = split_own(x, y);
  }
  // query frames that may look at a key of this workgroup / of this wavefront: t - left <= j <= t + right
  const int jlast = j0t + kRows - 1 < g.T ? j0t + kRows - 1 : g.T - 1;
  const int tmin = (g.right < 0 || j0t - g.right < 0) ? 0 : j0t - g.right;
  const int tmax = (g.left < 0 || jlast + g.left > g.T - 1) ? g.T - 1 : jlast + g.left;
  const int qlo = g.right < 0 ? 0 : j - g.right;
  const int qhi = (g.left < 0 || j + g.left > g.T - 1) ? g.T - 1 : j + g.left;
  const int some_lo = g.right < 0 ? 0 : jw - g.right, all_lo = g.right < 0 ? 0 : jw + 31 - g.right;
  const int some_hi = (g.left < 0 || jw + 31 + g.left > g.T - 1) ? g.T - 1 : jw + 31 + g.left;
  const int all_hi = (g.left < 0 || jw + g.left > g.T - 1) ? g.T - 1 : jw + g.left;
  v16f dk[DB], dv[DB];
#pragma unroll
  for (int blk = 0; blk < DB; ++blk) {
    dk[blk] = zero16();
    dv[blk] = zero16();
  }
  constexpr int P = FEW ? 4 : 1;   // pieces of a thread
  Raw qr[P], gr[P];
  float Lr, Dr;
  const int row = static_cast<int>(threadIdx.x & 31);
  auto thread = [&](int i) { return FEW ? lane + 64 * i : static_cast<int>(threadIdx.x); };
  auto load = [&](int t0) {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      qr[i] = load_piece(qkv, 3 * g.D, g, b, t0, hc, thread(i));
      gr[i] = load_piece(dctx, g.D, g, b, t0, hc, thread(i));
    }
    const int tt = t0 + row < g.T ? t0 + row : g.T - 1;
    Lr = lse[(b * g.T + tt) * g.heads + pl.h];
    Dr = dsum[(b * g.T + tt) * g.heads + pl.h];
  };
  auto slot_no = [&](const uint8_t *slot) { return FEW ? wave : slot == lds ? 0 : 1; };
  auto stage = [&](uint8_t *slot, int t0) {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      stage_piece<4 * DB>(slot, qr[i], g, t0, true, thread(i), reinterpret_cast<float *>(slot + 2 * kTensor));
      stage_piece<4 * DB>(slot + kTensor, gr[i], g, t0, true, thread(i));
    }
    if ((FEW ? lane : static_cast<int>(threadIdx.x)) < kStep) {
      const int at = slot_no(slot);
      Ls[at][row] = Lr;
      Ds[at][row] = Dr;
    }
  };
  auto compute = [&](const uint8_t *slot, int t0) {
    if (!active || t0 > some_hi || t0 + kStep - 1 < some_lo) return;
    const int at = slot_no(slot);
    v16f s, dp;
    first_products<KS>(slot, kk, vv, s, dp, lr, lk);   // S: queries x this lane's key; dP
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const v4f L4 = *reinterpret_cast<const v4f *>(&Ls[at][8 * r4 + 4 * lk]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        s[4 * r4 + e] = __builtin_amdgcn_exp2f(s[4 * r4 + e] * g.scale_log2e - L4[e]);
    }
    if (t0 < all_lo || t0 + kStep - 1 > all_hi || jw + 31 >= g.T) {   // cut by a window or the end of the utterance
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int tt = t0 + 8 * (r >> 2) + 4 * lk + (r & 3);
        s[r] = j < g.T && tt >= qlo && tt <= qhi ? s[r] : 0.0f;
      }
    }
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const v4f D4 = *reinterpret_cast<const v4f *>(&Ds[at][8 * r4 + 4 * lk]);
#pragma unroll
      for (int e = 0; e < 4; ++e) dp[4 * r4 + e] = s[4 * r4 + e] * (dp[4 * r4 + e] - D4[e]);
    }
    auto add_half = [&](auto half) {
      constexpr int k = decltype(half)::value;
      const Split p = split8(s[8 * k], s[8 * k + 1], s[8 * k + 2], s[8 * k + 3], s[8 * k + 4], s[8 * k + 5], s[8 * k + 6], s[8 * k + 7]);
#pragma unroll
      for (int blk = 0; blk < DB; ++blk) dv[blk] = mfma6(read_cols<k>(slot + kTensor, blk, lane), p, dv[blk]);   // dV^T += dO^T P
      const Split d = split8(dp[8 * k], dp[8 * k + 1], dp[8 * k + 2], dp[8 * k + 3], dp[8 * k + 4], dp[8 * k + 5], dp[8 * k + 6], dp[8 * k + 7]);
#pragma unroll
      for (int blk = 0; blk < DB; ++blk) dk[blk] = mfma6(read_cols<k>(slot, blk, lane), d, dk[blk]);             // dK^T += Q^T dS
    };
    add_half(std::integral_constant<int, 0>{});
    add_half(std::integral_constant<int, 1>{});
  };
  float *const out = dqkv + (b * g.T + jw) * 3 * g.D + g.D + hc;
  if constexpr (FEW) {
    run_tiles_apart(lds + wave * kSlot, wave, tmin / kStep * kStep, tmax, [&](uint8_t *slot, int t0) { load(t0); stage(slot, t0); }, compute);
    v4f k[2], v[2];
    const bool bad_k = add_shares<DB>(reinterpret_cast<float *>(lds), dk, wave, lane, k);
    const bool bad_v = add_shares<DB>(reinterpret_cast<float *>(lds), dv, wave, lane, v);
    if (!bad_k && !bad_v) {
      store_shares(k, g.scale, out, 3 * g.D, g.T - jw, g.dh);
      store_shares(v, 1.0f, out + g.D, 3 * g.D, g.T - jw, g.dh);
      return;
    }
    if (wave != 0) return;
    redo_dkv<DB, kRows>(dk, dv, qkv, dctx, lse, dsum, g);
  } else {
    run_tiles(lds, tmin / kStep * kStep, tmax, load, stage, compute);
    if (!active) return;
    if (any_nonfinite(dk) || any_nonfinite(dv)) redo_dkv<DB, kRows>(dk, dv, qkv, dctx, lse, dsum, g);
  }
  float *const img = reinterpret_cast<float *>(lds) + wave * 32 * kLd;
  store_rows<DB>(img, dk, g.scale, out, 3 * g.D, g.T - jw, g.dh, lane);
  store_rows<DB>(img, dv, 1.0f, out + g.D, 3 * g.D, g.T - jw, g.dh, lane);
}

}  // namespace

bool attention_rows_ok(const AttnShape &g, const void *a, const void *b, const void *c, const void *d) {
  auto aligned = [](const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
  return g.T <= 1 << 30 && g.dh % 4 == 0 && g.D % 4 == 0 && aligned(a) && aligned(b) && aligned(c) && aligned(d);
}

template <bool FEW>
static aqt_status bwd_rows(const float *qkv, const float *ctx, const float *dctx, const float *lse, const AttnShape &g, float *dqkv,
                           float *dsum, hipStream_t st) {
  const unsigned blocks = static_cast<unsigned>(static_cast<int64_t>(g.qtiles) * g.heads * g.B);
  auto dq = g.dh <= 16   ? attention_bwd_dq_rows_kernel<1, FEW>
            : g.dh <= 32 ? attention_bwd_dq_rows_kernel<2, FEW>
            : g.dh <= 48 ? attention_bwd_dq_rows_kernel<3, FEW>
                         : attention_bwd_dq_rows_kernel<4, FEW>;
  dq<<<blocks, kThreads, 0, st>>>(qkv, ctx, dctx, lse, dsum, g, dqkv);
  AQT_HIP(hipGetLastError());
  auto dkv = g.dh <= 16   ? attention_bwd_dkv_rows_kernel<1, FEW>
             : g.dh <= 32 ? attention_bwd_dkv_rows_kernel<2, FEW>
             : g.dh <= 48 ? attention_bwd_dkv_rows_kernel<3, FEW>
                          : attention_bwd_dkv_rows_kernel<4, FEW>;
  dkv<<<blocks, kThreads, 0, st>>>(qkv, dctx, lse, dsum, g, dqkv);
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

// FEW: its workgroups take 133 KB of LDS, one to a compute unit.  Times in us or as shares of what 128 rows to a workgroup take.
// All at once (256 workgroups): ahead as soon as there is a second tile to share.  8 x 128 frames, 4 heads of 64, causal (128) 41 -> 24; 6 x
//   217, 4 of 36 (168) 50 -> 28; 2 x 1000, 4 of 64 (256) 218 -> 87; 50 x 33, 2 of 4 to 64 (200) 0.90 - 1.01; but 62 x 16, 4 of 64 18.3 -> 22.2
//   and 100 x 32, 2 of 24 13.7 -> 16.8.
// In two rounds (512): ahead where rows meet more than 400 frames and the tiles fill the steps of the four wavefronts well, the narrower the
//   head the later.  480 workgroups, no limits: heads of 64, 401 frames (13 tiles, 4 steps) 0.97, 417 0.92, 1000 0.73; of 48, 401
//   1.02, 417 0.96; of 24 and 32, 401 1.07 - 1.11, 440 1.04, 480 0.97, 512 0.91 - 0.95; of 4 and 16, 401 1.14, 480 1.03 - 1.05, 512
//   0.98, 800 (25 tiles, 7 steps) 1.00 - 1.03, 1000 0.90.  A limit makes the rows of a workgroup uneven, which costs 128 of them more: causal
//   heads of 4, 401 1.05, 480 0.89, of 36, 401 0.91; 200 frames each way, 7 x 1000, 2 of 24 0.82, but 17 x 420, 2 of 4 1.07, of 24 1.02.
//   Below 400 frames it is ahead at times (9 x 352 81 against 85, 8 x 370 79 and 93, 8 x 288 76 and 71).
// Four rounds: 8 x 1000 223 -> 315.
// Errors against float64 are no larger (four partial sums: dq at 2 x 1000 6.7e-7 -> 5.2e-7).
bool attention_bwd_few_ok(const AttnShape &g) {
  const int64_t tiles = cdiv(g.T, 32), groups = tiles * g.heads, T = g.T;
  if (T <= 32 || groups > 512 / g.B) return false;
  if (groups <= 256 / g.B) return true;
  const int64_t met = g.left < 0 || g.right < 0 ? T : static_cast<int64_t>(g.left) + g.right + 1;   // frames that a row meets, at most T
  if (met <= 400 || T <= 400) return false;
  if ((g.left < 0 || g.left >= T - 1) && (g.right < 0 || g.right >= T - 1))
    return 10 * tiles > 33 * cdiv(tiles, 4) + (g.dh <= 16 ? 21 : g.dh <= 32 ? 14 : g.dh <= 48 ? 0 : -4);
  return tiles > 14 || g.dh > (g.left < 0 || g.right < 0 ? 16 : 32);
}

aqt_status launch_attention_bwd_rows(const float *qkv, const float *ctx, const float *dctx, const float *lse, const AttnShape &g,
                                      float *dqkv, float *dsum, hipStream_t st) {
  if (attention_bwd_few_ok(g)) {
    AttnShape few = g;
    few.qtiles = static_cast<int>(cdiv(g.T, 32));
    return bwd_rows<true>(qkv, ctx, dctx, lse, few, dqkv, dsum, st);
  }
  return bwd_rows<false>(qkv, ctx, dctx, lse, g, dqkv, dsum, st);
}

}  // namespace aqt
