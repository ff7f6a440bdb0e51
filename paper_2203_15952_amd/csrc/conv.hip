// The float layers between the two pointwise convolutions of the Conformer convolution
// module (arxiv 2203.15952, Sec. 3.2: depthwise kernel size 32; Sec. 3.3: causal depthwise
// convolution of kernel size 15, and convolution kernels are left unquantized): depthwise
// convolution along time, the normalisation behind it with fixed statistics (one scale and
// one shift per channel), Swish, and the abs-max of the result for the quantizer of the
// second pointwise convolution (Fig. 2), in one pass over the tensor; the adjoint kernels
// for the backward.  Plain float32 vector arithmetic: about 32 multiply-adds per 8 bytes
// moved, so HBM time bounds these kernels, not the ALUs.
//
// Layout: x [B,T,C], C contiguous (tokens x channels, B utterances of T frames); w [kw,C].
// A workgroup owns 64 frames x 64 channels of one utterance: the frames it needs (64 + kw - 1
// rows, each a coalesced 256-byte piece per wavefront) and the taps go to LDS once, a lane
// owns a channel (LDS reads are conflict-free) and forms eight neighbouring results at a time
// from a sliding window of eight registers whose slots are compile-time numbers (eight taps per
// turn of the loop, so nothing is moved), one LDS read per tap for the values and one for the
// tap.  With windows of four, two LDS reads per four multiply-adds kept the LDS as busy as the
// ALUs.  Neighbouring tiles share their halo through L2.
// Measured in us, windows of four and four-byte loads -> here, 512 channels: 128 utterances of 512 frames, 32 taps,
// forward with slopes and input gradient 149 -> 94 on average (402 MB: 4.3 TB/s), taps and bias 184 -> 102 (4 TB/s); 32
// utterances of 400 frames, forward without slopes 49 -> 33; one of 40 frames, 15 taps, 11.9 -> 8.
// The abs-max costs one atomic per workgroup: the wavefronts of a first round all find the word at zero and queue at it
// (one atomic per wavefront: 109 instead of 94, 46 instead of 33).
#include "aqt_internal.h"
#include "epilogue.h"

namespace aqt {
namespace {

constexpr int kThreads = 256;
constexpr int kTile = 64;      // frames per workgroup tile
constexpr int kTapsMax = 32;   // largest kernel size the tiled kernels take (at most 198 LDS rows of 256 bytes)

__device__ __forceinline__ uint32_t wave_max_bits(uint32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t o = static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), off, 64));
    v = v > o ? v : o;
  }
  return v;
}

typedef float v4f __attribute__((vector_size(16)));

struct ConvGeom {
  int64_t B, T, C;
  int kw, pad_left;
  int cgroups, tgroups;   // 64-channel groups; tiles per utterance, of 64 frames (of 32 where launch_corr halves them)
};

// Stage rows [t0 - pl, t0 - pl + rows) of channel group cg of utterance b into LDS as
// xs[row][lane] (zero outside the utterance and beyond channel C), multiplied by xmul if given.
// Eight rows per wavefront are in flight at a time: every load goes to a clamped, always valid
// address and the value is zeroed afterwards, so the loads carry no branches and overlap.
__device__ __forceinline__ void stage_frames(float *__restrict__ xs, int rows, const float *__restrict__ xin,
                                             const float *__restrict__ xmul, const ConvGeom &g, int64_t b,
                                             int64_t t0, int pl, int64_t c) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t cc = c < g.C ? c : g.C - 1;
  const float *xb = xin + b * g.T * g.C + cc;
  const float *mb = xmul ? xmul + b * g.T * g.C + cc : nullptr;
  for (int r0 = wave; r0 < rows; r0 += 32) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      int64_t tt = t0 + (r0 + 4 * k) - pl;
      tt = tt < 0 ? 0 : (tt >= g.T ? g.T - 1 : tt);
      v[k] = xb[tt * g.C];
    }
    if (mb) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        int64_t tt = t0 + (r0 + 4 * k) - pl;
        tt = tt < 0 ? 0 : (tt >= g.T ? g.T - 1 : tt);
        v[k] *= mb[tt * g.C];
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int r = r0 + 4 * k;
      const int64_t tt = t0 + r - pl;
      if (r < rows) xs[r * 64 + lane] = (c < g.C && tt >= 0 && tt < g.T) ? v[k] : 0.0f;
    }
  }
}

// The same rows 16 bytes at a time, sixteen lanes to a row, for channels in fours on 16-byte aligned tensors: all of a
// tile's loads (up to 16 N rows) are in flight together, and may be requested before another tensor's are waited for.
template <int N>
struct Frames {
  v4f v[N], m[N];
};

__device__ __forceinline__ bool quads_ok(const ConvGeom &g, const float *a, const float *b, const float *c) {
  return g.C % 4 == 0 &&
         ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) | reinterpret_cast<uintptr_t>(c)) & 15) == 0;
}

template <int N>
__device__ __forceinline__ void load_frames(Frames<N> &f, int rows, const float *__restrict__ xin,
                                            const float *__restrict__ xmul, const ConvGeom &g, int64_t b, int64_t t0,
                                            int pl, int64_t c0) {
  const int r0 = threadIdx.x >> 4;
  const int64_t c = c0 + 4 * (threadIdx.x & 15), cc = c < g.C ? c : g.C - 4, base = b * g.T * g.C + cc;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int r = r0 + 16 * k < rows ? r0 + 16 * k : rows - 1;
    int64_t tt = t0 + r - pl;
    tt = tt < 0 ? 0 : (tt >= g.T ? g.T - 1 : tt);
    f.v[k] = *reinterpret_cast<const v4f *>(xin + base + tt * g.C);
    if (xmul) f.m[k] = *reinterpret_cast<const v4f *>(xmul + base + tt * g.C);
  }
}

template <int N>
__device__ __forceinline__ void put_frames(float *__restrict__ xs, const Frames<N> &f, int rows, bool mul,
                                           const ConvGeom &g, int64_t t0, int pl, int64_t c0) {
  const int r0 = threadIdx.x >> 4, q = 4 * (threadIdx.x & 15);
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int r = r0 + 16 * k;
    const int64_t tt = t0 + r - pl;
    v4f v = f.v[k];
    if (mul) v = v * f.m[k];
    if (c0 + q >= g.C || tt < 0 || tt >= g.T) v = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    if (r < rows) *reinterpret_cast<v4f *>(xs + r * 64 + q) = v;
  }
}

// out[b,t,c] = act( (bias[c] + sum_j tap_j * in[b, t + j - pl, c]) * na[c] + nb[c] ),  in = xin (* xmul)
// tap_j = w[j] (the layer itself), or w[kw - 1 - j] when rev (the gradient with respect to the
// input is the correlation of the upstream gradient with the mirrored kernel, and the caller
// passes pl = kw - 1 - pad_left).  dfac (nullable) receives d out / d (convolution result);
// absmax (nullable) the largest |out| as float bits.
// GATE, with gate [B T, 2 C] (and neither na, nb, swish, dfac nor absmax) out is [B T, 2 C]: the sum times the frame's two halves of the gate,
// the gradient through the gated unit in front of the layer (65536 x 512,
// 32 taps: 79 us and 126 for a pass of its own, 147 in one).
// GROUPS: groups of eight frames a wavefront takes in turn, 32 GROUPS frames to a workgroup.
// Dynamic LDS: (32 GROUPS + 2 kw - 1) * 256 bytes.
template <bool GATE = false, int GROUPS = kTile / 32>
__global__ __launch_bounds__(kThreads) void dwconv_kernel(const float *__restrict__ xin, const float *__restrict__ xmul,
                                                          const float *__restrict__ w, const float *__restrict__ bias,
                                                          const float *__restrict__ na, const float *__restrict__ nb,
                                                          int swish, int rev, ConvGeom g, int pl,
                                                          float *__restrict__ out, float *__restrict__ dfac,
                                                          uint32_t *__restrict__ absmax,
                                                          const float *__restrict__ gate = nullptr) {
  constexpr int kFrames = 32 * GROUPS;
  extern __shared__ float lds[];
  const int rows = kFrames + g.kw - 1;
  float *xs = lds;               // [rows][64]
  float *ws = lds + rows * 64;   // [kw][64]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t id = blockIdx.x;
  const int cg = static_cast<int>(id % g.cgroups);
  id /= g.cgroups;
  const int tg = static_cast<int>(id % g.tgroups);
  const int64_t b = id / g.tgroups;
  const int64_t c = static_cast<int64_t>(cg) * 64 + lane;
  const int64_t t0 = static_cast<int64_t>(tg) * kFrames;
  if (quads_ok(g, xin, xmul, w)) {
    const int64_t c0 = static_cast<int64_t>(cg) * 64, cq = c0 + 4 * (threadIdx.x & 15), cc = cq < g.C ? cq : g.C - 4;
    constexpr int kPieces = (kFrames + kTapsMax + 14) / 16;
    static_assert(kTapsMax <= 2 * 16);
    Frames<kPieces> f;
    load_frames(f, rows, xin, xmul, g, b, t0, pl, c0);
    v4f taps[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int j = static_cast<int>(threadIdx.x >> 4) + 16 * k, jc = j < g.kw ? j : g.kw - 1;
      taps[k] = *reinterpret_cast<const v4f *>(w + static_cast<int64_t>(rev ? g.kw - 1 - jc : jc) * g.C + cc);
    }
    put_frames(xs, f, rows, xmul != nullptr, g, t0, pl, c0);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int j = static_cast<int>(threadIdx.x >> 4) + 16 * k;
      if (j < g.kw) *reinterpret_cast<v4f *>(ws + j * 64 + 4 * (threadIdx.x & 15)) = taps[k];   // unused beyond channel C
    }
  } else {
    stage_frames(xs, rows, xin, xmul, g, b, t0, pl, c);
    for (int j = wave; j < g.kw; j += 4)
      ws[j * 64 + lane] = (c < g.C) ? w[static_cast<int64_t>(rev ? g.kw - 1 - j : j) * g.C + c] : 0.0f;
  }
  __syncthreads();
  uint32_t amax = 0u;
  if (c < g.C) {
    const float b0 = bias ? bias[c] : 0.0f;
    const float a = na ? na[c] : 1.0f, sh = nb ? nb[c] : 0.0f;
    for (int grp = 0; grp < GROUPS; ++grp) {
      const int tl = (wave * GROUPS + grp) * 8;
      if (t0 + tl >= g.T) break;
      const float *const xr = xs + tl * 64 + lane, *const wr = ws + lane;
      const int64_t first = (b * g.T + t0 + tl) * g.C + c, at2 = 2 * first - c;   // at2: in frames of 2 C
      const int frames = static_cast<int>(g.T - t0 - tl < 8 ? g.T - t0 - tl : 8);
      float ga[8], gb[8];
      if constexpr (GATE) {   // in flight under the taps
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int64_t f = at2 + 2 * (k < frames ? k : frames - 1) * g.C;
          ga[k] = gate[f];
          gb[k] = gate[f + g.C];
        }
      }
      float acc[8], x[8];   // frame tl + j + k of the window of tap j sits in x[(j + k) % 8]
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] = b0;
#pragma unroll
      for (int k = 0; k < 7; ++k) x[k] = xr[k * 64];
      int j = 0;
      for (; j + 8 <= g.kw; j += 8) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          x[(u + 7) & 7] = xr[(j + u + 7) * 64];
          const float wj = wr[(j + u) * 64];
#pragma unroll
          for (int k = 0; k < 8; ++k) acc[k] = fmaf(wj, x[(u + k) & 7], acc[k]);
        }
      }
#pragma unroll
      for (int u = 0; u < 7; ++u)
        if (j + u < g.kw) {
          x[(u + 7) & 7] = xr[(j + u + 7) * 64];
          const float wj = wr[(j + u) * 64];
#pragma unroll
          for (int k = 0; k < 8; ++k) acc[k] = fmaf(wj, x[(u + k) & 7], acc[k]);
        }
      if constexpr (GATE) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (k < frames) {
            out[at2 + 2 * k * g.C] = acc[k] * ga[k];
            out[at2 + 2 * k * g.C + g.C] = acc[k] * gb[k];
          }
        continue;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int64_t t = t0 + tl + k;
        if (t < g.T) {
          float n = acc[k];
          if (na) n = n * a;
          if (nb) n = n + sh;
          float o = n, df = a;
          if (swish) {
            const float sg = sigmoid_f32(n);
            o = n * sg;
            df = a * swish_dact_f32(n, sg);
          }
          const int64_t at = first + k * g.C;
          out[at] = o;
          if (dfac) dfac[at] = df;
          amax = max(amax, __float_as_uint(o) & 0x7FFFFFFFu);
        }
      }
    }
  }
  if (absmax) {   // uniform: the word only grows, so a stale read can only cost a redundant atomic
    amax = wave_max_bits(amax);
    __syncthreads();   // the frames are no longer read: four words of them hold the wavefronts' maxima
    if (lane == 0) lds[wave] = __uint_as_float(amax);
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int i = 1; i < 4; ++i) amax = max(amax, __float_as_uint(lds[i]));
      if (amax > *reinterpret_cast<volatile uint32_t *>(absmax)) atomicMax(absmax, amax);
    }
  }
}

// Any kernel size: one thread per output element.
__global__ __launch_bounds__(kThreads) void dwconv_any_kernel(const float *__restrict__ xin,
                                                              const float *__restrict__ xmul,
                                                              const float *__restrict__ w, const float *__restrict__ bias,
                                                              const float *__restrict__ na, const float *__restrict__ nb,
                                                              int swish, int rev, ConvGeom g, int pl,
                                                              float *__restrict__ out, float *__restrict__ dfac,
                                                              uint32_t *__restrict__ absmax) {
  const int64_t total = g.B * g.T * g.C;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
  uint32_t amax = 0u;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < total; i += stride) {
    const int64_t c = i % g.C, bt = i / g.C, t = bt % g.T, b = bt / g.T;
    float acc = bias ? bias[c] : 0.0f;
    for (int j = 0; j < g.kw; ++j) {
      const int64_t tt = t + j - pl;
      if (tt < 0 || tt >= g.T) continue;
      const int64_t at = (b * g.T + tt) * g.C + c;
      float xv = xin[at];
      if (xmul) xv *= xmul[at];
      acc = fmaf(w[static_cast<int64_t>(rev ? g.kw - 1 - j : j) * g.C + c], xv, acc);
    }
    const float a = na ? na[c] : 1.0f;
    float n = acc;
    if (na) n = n * a;
    if (nb) n = n + nb[c];
    float o = n, df = a;
    if (swish) {
      const float sg = sigmoid_f32(n);
      o = n * sg;
      df = a * swish_dact_f32(n, sg);
    }
    out[i] = o;
    if (dfac) dfac[i] = df;
    amax = max(amax, __float_as_uint(o) & 0x7FFFFFFFu);
  }
  if (absmax) {
    amax = wave_max_bits(amax);
    if ((threadIdx.x & 63) == 0 && amax > *reinterpret_cast<volatile uint32_t *>(absmax)) atomicMax(absmax, amax);
  }
}

__global__ void zero_absmax_kernel(uint32_t *p) {
  if (threadIdx.x == 0) *p = 0u;
}

// Gradient of the taps and of the bias:
//   dw[j,c] = sum_{b,t} dv[b,t,c] * x[b, t + j - pl, c],   dbias[c] = sum_{b,t} dv[b,t,c],   dv = dout (* dmul).
// Workgroup (cg, p) walks the tiles p, p + P, ... of its 64-channel group (a tile = 64 frames of
// one utterance): dv and the frames of x it meets go to LDS; a lane owns a channel, a wavefront
// TAPS neighbouring taps (four up to 16 taps, else eight), whose sums stay in its registers: a window of
// registers as in the forward, two LDS reads per TAPS multiply-adds.  Without sums in LDS four
// workgroups fit a compute unit, so the 1024 of a launch run at once instead of in two rounds.
// The workgroup leaves one partial per tap and channel; dwconv_dw_fold_kernel adds the
// P partials in order.  Same bits on every run.
// Dynamic LDS: 2 kTile + kwp - 1 rows of 256 bytes, kwp = kw rounded up to TAPS.
constexpr int dw_taps(int kw) { return kw > 16 ? 8 : 4; }

template <int TAPS>
__device__ __forceinline__ void dwconv_dw_tiles(float *__restrict__ lds, const float *__restrict__ dout,
                                                const float *__restrict__ dmul, const float *__restrict__ x,
                                                const ConvGeom &g, int P, float *__restrict__ part) {
  const int kwp = (g.kw + TAPS - 1) / TAPS * TAPS;
  const int rows = kTile + kwp - 1;             // frames of x a tile meets
  float *dvs = lds;                             // [kTile][64]
  float *xs = dvs + kTile * 64;                 // [rows][64]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cg = blockIdx.x % g.cgroups, p = blockIdx.x / g.cgroups;
  const int64_t c0 = static_cast<int64_t>(cg) * 64, c = c0 + lane;
  const int j0 = wave * TAPS;
  const bool quads = quads_ok(g, dout, dmul, x);
  float acc[TAPS], accb = 0.0f;
#pragma unroll
  for (int k = 0; k < TAPS; ++k) acc[k] = 0.0f;
  const int64_t ntile = g.B * g.tgroups;
  for (int64_t q = p; q < ntile; q += P) {
    const int64_t b = q / g.tgroups;
    const int64_t t0 = (q % g.tgroups) * kTile;
    if (quads) {
      Frames<4> fd;
      Frames<6> fx;
      load_frames(fd, kTile, dout, dmul, g, b, t0, 0, c0);
      load_frames(fx, rows, x, nullptr, g, b, t0, g.pad_left, c0);
      __syncthreads();   // the previous tile's reads are over
      put_frames(dvs, fd, kTile, dmul != nullptr, g, t0, 0, c0);
      put_frames(xs, fx, rows, false, g, t0, g.pad_left, c0);
    } else {
      __syncthreads();
      stage_frames(dvs, kTile, dout, dmul, g, b, t0, 0, c);
      stage_frames(xs, rows, x, nullptr, g, b, t0, g.pad_left, c);
    }
    __syncthreads();
    float sb = 0.0f;
    for (int t = wave * 16; t < wave * 16 + 16; ++t) sb += dvs[t * 64 + lane];
    accb += sb;
    if (j0 < g.kw) {
      const float *const xr = xs + j0 * 64 + lane, *const dr = dvs + lane;
      float a[TAPS], xw[TAPS];
#pragma unroll
      for (int k = 0; k < TAPS; ++k) a[k] = 0.0f;
#pragma unroll
      for (int k = 0; k < TAPS - 1; ++k) xw[k] = xr[k * 64];
      for (int t = 0; t < kTile; t += 8) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          xw[(u + TAPS - 1) % TAPS] = xr[(t + u + TAPS - 1) * 64];
          const float d = dr[(t + u) * 64];
#pragma unroll
          for (int k = 0; k < TAPS; ++k) a[k] = fmaf(d, xw[(u + k) % TAPS], a[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < TAPS; ++k) acc[k] += a[k];
    }
  }
  __syncthreads();
  dvs[wave * 64 + lane] = accb;
  __syncthreads();
  if (c < g.C) {
    float *o = part + static_cast<int64_t>(p) * (g.kw + 1) * g.C + c;
#pragma unroll
    for (int k = 0; k < TAPS; ++k)
      if (j0 + k < g.kw) o[static_cast<int64_t>(j0 + k) * g.C] = acc[k];
    if (wave == 0)
      o[static_cast<int64_t>(g.kw) * g.C] =
          ((dvs[lane] + dvs[64 + lane]) + dvs[128 + lane]) + dvs[192 + lane];   // the bias sum sits behind the taps
  }
}

__global__ __launch_bounds__(kThreads, 4) void dwconv_dw_kernel(const float *__restrict__ dout,
                                                                const float *__restrict__ dmul,
                                                                const float *__restrict__ x, ConvGeom g, int P,
                                                                float *__restrict__ part) {
  extern __shared__ float lds[];
  if (dw_taps(g.kw) == 8) dwconv_dw_tiles<8>(lds, dout, dmul, x, g, P, part);
  else dwconv_dw_tiles<4>(lds, dout, dmul, x, g, P, part);
}

// Any kernel size: one thread per (tap, channel), the whole sum over (b, t) in order; the
// bias sum is row kw.  P = 1.
__global__ __launch_bounds__(kThreads) void dwconv_dw_any_kernel(const float *__restrict__ dout,
                                                                 const float *__restrict__ dmul,
                                                                 const float *__restrict__ x, ConvGeom g,
                                                                 float *__restrict__ part) {
  const int64_t total = static_cast<int64_t>(g.kw + 1) * g.C;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (i >= total) return;
  const int64_t c = i % g.C;
  const int j = static_cast<int>(i / g.C);
  float acc = 0.0f;
  for (int64_t b = 0; b < g.B; ++b)
    for (int64_t t = 0; t < g.T; ++t) {
      const int64_t at = (b * g.T + t) * g.C + c;
      float v = dout[at];
      if (dmul) v *= dmul[at];
      if (j == g.kw) {
        acc += v;
      } else {
        const int64_t tt = t + j - g.pad_left;
        if (tt >= 0 && tt < g.T) acc = fmaf(v, x[(b * g.T + tt) * g.C + c], acc);
      }
    }
  part[i] = acc;
}

// 64 sums per workgroup, its four wavefronts share the partials (eight loads in flight each) and are added up in order.
// Bound by the latency of those loads: one thread per sum walking all 256 partials took 12.2 us at 512 channels and 14.7 at 144,
// 32 taps; so 4.8 and 5.2.
__global__ __launch_bounds__(kThreads) void dwconv_dw_fold_kernel(const float *__restrict__ part, int P, int kw,
                                                                  int64_t C, float *__restrict__ dw,
                                                                  float *__restrict__ dbias) {
  __shared__ float sm[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t n = static_cast<int64_t>(kw + 1) * C, i = static_cast<int64_t>(blockIdx.x) * 64 + lane, ic = i < n ? i : n - 1;
  float s = 0.0f;
  for (int p = wave * 8; p < P; p += 32) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[static_cast<int64_t>(p + u < P ? p + u : P - 1) * n + ic];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p + u < P ? v[u] : 0.0f;
    s += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
  }
  sm[wave][lane] = s;
  __syncthreads();
  if (wave || i >= n) return;
  s = (sm[0][lane] + sm[1][lane]) + (sm[2][lane] + sm[3][lane]);
  if (i < static_cast<int64_t>(kw) * C) {
    if (dw) dw[i] = s;
  } else if (dbias) {
    dbias[i - static_cast<int64_t>(kw) * C] = s;
  }
}

ConvGeom geom(int64_t B, int64_t T, int64_t C, int kw, int pad_left) {
  ConvGeom g;
  g.B = B; g.T = T; g.C = C; g.kw = kw; g.pad_left = pad_left;
  g.cgroups = static_cast<int>(cdiv(C, 64));
  g.tgroups = static_cast<int>(cdiv(T, kTile));
  return g;
}

// Partials of the tap gradient: as many workgroups per channel group as give the chip a few
// workgroups per compute unit, never more than there are tiles.
int dw_partials(const ConvGeom &g) {
  if (g.kw > kTapsMax) return 1;
  int64_t P = cdiv(1024, g.cgroups);
  const int64_t ntile = g.B * g.tgroups;
  if (P > ntile) P = ntile;
  if (P > 256) P = 256;
  return static_cast<int>(P);
}

bool corr_staged(const ConvGeom &g) {   // else the kernel for any number of taps
  return g.kw <= kTapsMax && static_cast<int64_t>(g.cgroups) * g.tgroups * g.B < (int64_t(1) << 31);
}
aqt_status launch_corr(bool rev, const float *xin, const float *xmul, const float *w, const float *bias,
                       const float *na, const float *nb, int swish, const ConvGeom &g, float *out, float *dfac,
                       uint32_t *absmax, hipStream_t st, bool absmax_is_zero = false, const float *gate = nullptr) {
  const int pl = rev ? g.kw - 1 - g.pad_left : g.pad_left;
  if (absmax && !absmax_is_zero) zero_absmax_kernel<<<1, 64, 0, st>>>(absmax);
  if (corr_staged(g)) {
    int64_t blocks = static_cast<int64_t>(g.cgroups) * g.tgroups * g.B;
    // Fewer workgroups than compute units: tiles of half the frames, so that a wavefront is done after one group.  1 x 1024 x 512, 15
    // taps (128 workgroups) 6.3 -> 4.9 us, with scale, Swish and slope 7.8 -> 5.7; 8 x 192 x 512, 32 taps (192) 7.1 -> 5.7 and 8.7 -> 6.7; with the
    // largest value as well 11.4 -> 10.4 and 12.9 -> 12.0, but at times a short last tile had spared the larger ones their atomics (1 x 1096
    // 10.0 -> 11.0).
    const bool half = blocks < 256;
    ConvGeom gt = g;
    if (half) gt.tgroups = static_cast<int>(cdiv(g.T, kTile / 2));
    blocks = static_cast<int64_t>(gt.cgroups) * gt.tgroups * gt.B;
    const size_t lds = static_cast<size_t>((half ? kTile / 2 : kTile) + 2 * g.kw - 1) * 64 * sizeof(float);
    auto kern = half ? (gate ? dwconv_kernel<true, kTile / 64> : dwconv_kernel<false, kTile / 64>)
                     : (gate ? dwconv_kernel<true> : dwconv_kernel<false>);
    kern<<<static_cast<unsigned>(blocks), kThreads, lds, st>>>(xin, xmul, w, bias, na, nb, swish, rev ? 1 : 0, gt, pl, out, dfac,
                                                               absmax, gate);
  } else {
    int64_t grid = cdiv(g.B * g.T * g.C, kThreads);
    if (grid > 8192) grid = 8192;
    dwconv_any_kernel<<<static_cast<unsigned>(grid), kThreads, 0, st>>>(xin, xmul, w, bias, na, nb, swish, rev ? 1 : 0, g,
                                                                      pl, out, dfac, absmax);
  }
  AQT_HIP(hipGetLastError());
  return AQT_OK;
}

}  // namespace

// However the frames are divided into utterances (no more tiles than frames), the staged kernel takes them.
bool dwconv_takes_gate(int64_t M, int64_t C, int kw) { return kw <= kTapsMax && M < (int64_t(1) << 31) / cdiv(C, 64); }

// Shape-only bound (the partial count never exceeds what an unlimited number of tiles gives).
size_t dwconv_bwd_ws_bytes(int64_t C, int kw) {
  ConvGeom g = geom(int64_t(1) << 20, kTile, C, kw, 0);
  return align_up(static_cast<size_t>(dw_partials(g)) * (kw + 1) * C * sizeof(float), 256);
}

aqt_status launch_dwconv_fwd(const float *x, const float *w, const float *bias, const float *na, const float *nb,
                             int swish, int64_t B, int64_t T, int64_t C, int kw, int pad_left, float *out, float *dfac,
                             uint32_t *absmax, hipStream_t st, bool absmax_is_zero) {
  return launch_corr(false, x, nullptr, w, bias, na, nb, swish, geom(B, T, C, kw, pad_left), out, dfac, absmax, st,
                     absmax_is_zero);
}

aqt_status launch_dwconv_bwd(const float *dout, const float *dmul, const float *x, const float *w, int64_t B, int64_t T,
                             int64_t C, int kw, int pad_left, float *dx, float *dw, float *dbias, void *ws,
                             hipStream_t st, const float *gate, float *dv) {
  const ConvGeom g = geom(B, T, C, kw, pad_left);
  if (gate && dwconv_takes_gate(B * T, C, kw)) {
    AQT_TRY(launch_corr(true, dout, dmul, w, nullptr, nullptr, nullptr, 0, g, dv, nullptr, nullptr, st, false, gate));
  } else if (gate) {
    AQT_TRY(launch_corr(true, dout, dmul, w, nullptr, nullptr, nullptr, 0, g, dx, nullptr, nullptr, st));
    AQT_TRY(launch_dact_mul(dx, gate, B * T, 2 * C, C, dv, st));
  } else if (dx) AQT_TRY(launch_corr(true, dout, dmul, w, nullptr, nullptr, nullptr, 0, g, dx, nullptr, nullptr, st));
  if (dw || dbias) {
    float *part = static_cast<float *>(ws);
    const int P = dw_partials(g);
    if (kw <= kTapsMax) {
      const int kwp = static_cast<int>(cdiv(kw, dw_taps(kw))) * dw_taps(kw);
      const size_t lds = static_cast<size_t>(2 * kTile + kwp - 1) * 64 * sizeof(float);
      dwconv_dw_kernel<<<static_cast<unsigned>(g.cgroups) * P, kThreads, lds, st>>>(dout, dmul, x, g, P, part);
    } else {
      dwconv_dw_any_kernel<<<static_cast<unsigned>(cdiv(static_cast<int64_t>(kw + 1) * C, kThreads)), kThreads, 0, st>>>(
          dout, dmul, x, g, part);
    }
    AQT_HIP(hipGetLastError());
    dwconv_dw_fold_kernel<<<static_cast<unsigned>(cdiv(static_cast<int64_t>(kw + 1) * C, 64)), kThreads, 0, st>>>(
        part, P, kw, C, dw, dbias);
    AQT_HIP(hipGetLastError());
  }
  return AQT_OK;
}

}  // namespace aqt
