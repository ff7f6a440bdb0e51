// What the attention kernels for vectorised rows (attention_fwd.hip, attention_bwd.hip) share.
#pragma once
#include "aqt_internal.h"

namespace aqt {
namespace {

constexpr int kThreads = 256;
constexpr int kQ = 128;   // rows a workgroup owns (32 per wavefront)

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ v16f zero16() {
  v16f z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.0f;
  return z;
}

// Workgroup -> (utterance, head, tile of 128 rows).  The tiles of one head read the same rows; workgroup ids eight apart
// run on one XCD, so with a multiple of eight heads in all they are given to one XCD, whose L2 then holds those rows
// (128 utterances of 512 frames, backward: 1358 us, against 1499 with the tile slowest).
struct Place {
  int64_t b, hc;
  int r0, h;
};
template <int ROWS = kQ>   // rows a workgroup owns; g.qtiles of them make an utterance
__device__ __forceinline__ Place place_of(const AttnShape &g, int block) {
  const int64_t id = block, heads = static_cast<int64_t>(g.heads) * g.B;
  int64_t bh, tile;
  if (heads % 8 == 0) {
    bh = id / (8 * g.qtiles) * 8 + id % 8;
    tile = id / 8 % g.qtiles;
  } else {
    bh = id / g.qtiles;
    tile = id % g.qtiles;
  }
  const int h = static_cast<int>(bh % g.heads);
  return Place{bh / g.heads, static_cast<int64_t>(h) * g.dh, static_cast<int>(tile) * ROWS, h};
}

// The frames that this wavefront's 32 rows (from tw), and this lane's row t, may look at or be seen from:
// lo frames back and hi frames ahead (negative: no limit), clipped to the utterance.
struct Window {
  int lo, hi;            // this lane's row
  int some_lo, some_hi;  // any row of the wavefront
  int all_lo, all_hi;    // every row of the wavefront
};
__device__ __forceinline__ Window window_of(int t, int tw, int back, int ahead, int T) {
  auto upto = [&](int x) { return ahead < 0 || x + ahead > T - 1 ? T - 1 : x + ahead; };
  auto from = [&](int x) { return back < 0 ? 0 : x - back; };
  return Window{from(t), upto(t), from(tw), upto(tw + 31), from(tw + 31), upto(tw)};
}

}  // namespace
}  // namespace aqt
