// Column sums of a gradient (the bias gradient, dbias[n] = sum_m dy[m,n]), taken in float64: the dW kernels add up
// what they stage anyway and leave one partial row per workgroup of a column; this folds the rows.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aqt {

constexpr int kColsumThreads = 256;
constexpr int kColsumCols = 32;      // columns per workgroup; eight groups of rows, eight loads in flight per thread

// out[n] = sum of part[row * N + n] over `rows` rows, in a fixed order; `block` counts workgroups of 32 columns.
__device__ __forceinline__ void fold_column_sums(const double *__restrict__ part, int rows, int64_t N, int64_t block,
                                                 float *__restrict__ out) {
  constexpr int G = kColsumThreads / kColsumCols, U = 8;
  __shared__ double sm[G][kColsumCols];
  const int c = threadIdx.x % kColsumCols, grp = threadIdx.x / kColsumCols;
  const int64_t n = block * kColsumCols + c, nc = n < N ? n : N - 1;
  double s = 0.0;
  for (int j = grp * U; j < rows; j += G * U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = part[static_cast<int64_t>(j + u < rows ? j + u : rows - 1) * N + nc];
#pragma unroll
    for (int u = 0; u < U; ++u) s += j + u < rows ? v[u] : 0.0;
  }
  sm[grp][c] = s;
  __syncthreads();
  if (grp == 0 && n < N) {
    double total = sm[0][c];
#pragma unroll
    for (int g = 1; g < G; ++g) total += sm[g][c];
    out[n] = static_cast<float>(total);
  }
}

}  // namespace aqt
