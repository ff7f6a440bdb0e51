// Driver of the host emulation of the attention kernels for vectorised rows: the test splices attention_tiles.h, the
// kernels of attention_fwd.hip (namespace fwd_rows), attention_few.hip (few) and attention_bwd.hip (bwd_rows) in front of this file.
// Forward, then both backward kernels, in tiles of 128 rows and in the forms for small batches (16 queries, 32 rows), on tensors
// of exactly the sizes that the kernels may touch; results are compared with plain float64 loops written here.
namespace aqt {
static int bad = 0;
template <int KS> void launch(unsigned blocks, const float *qkv, float *ctx, uint32_t *am, float *lse, const float *dctx, float *dsum,
                              float *dqkv, const AttnShape &g) {
  run(blocks, 256, 0, [&] { fwd_rows::attention_fwd_rows_kernel<KS>(qkv, g, ctx, am, lse); });
  run(blocks, 256, 0, [&] { bwd_rows::attention_bwd_dq_rows_kernel<KS>(qkv, ctx, dctx, lse, dsum, g, dqkv); });
  run(blocks, 256, 0, [&] { bwd_rows::attention_bwd_dkv_rows_kernel<KS>(qkv, dctx, lse, dsum, g, dqkv); });
}
template <int KS> void launch_few(const float *qkv, float *ctx, uint32_t *am, float *lse, const float *dctx, float *dsum, float *dqkv,
                                  AttnShape g) {
  const int tiles = (g.T + few::kQf - 1) / few::kQf;
  run((unsigned)(tiles * g.heads * g.B), 256, 0, [&] { few::attention_fwd_few_kernel<KS>(qkv, g, tiles, ctx, am, lse); });
  g.qtiles = (g.T + 31) / 32;
  const unsigned blocks = (unsigned)(g.qtiles * g.heads * g.B);
  run(blocks, 256, 0, [&] { bwd_rows::attention_bwd_dq_rows_kernel<KS, true>(qkv, ctx, dctx, lse, dsum, g, dqkv); });
  run(blocks, 256, 0, [&] { bwd_rows::attention_bwd_dkv_rows_kernel<KS, true>(qkv, dctx, lse, dsum, g, dqkv); });
}
// big: one value of dctx that is finite in float32 and an infinity in bf16, so that its rows are formed a second time
static void one(int64_t B, int T, int64_t D, int heads, int left, int right, bool big = false) {
  printf("case %ld %d %ld %d %d %d %d\n", (long)B, T, (long)D, heads, left, right, (int)big); fflush(stdout);
  const size_t n = (size_t)(B * T * D), rows = (size_t)(B * T * heads);
  float *qkv = (float *)malloc(3 * n * 4), *ctx = (float *)malloc(n * 4), *dctx = (float *)malloc(n * 4);
  float *lse = (float *)malloc(rows * 4), *dsum = (float *)malloc(rows * 4), *dqkv = (float *)malloc(3 * n * 4);
  uint32_t s = 13u, am = 0;
  for (size_t i = 0; i < 3 * n; ++i) { s = s * 1664525u + 1013904223u; qkv[i] = 2.0f * ((float)(s >> 8) / 8388608.0f - 1.0f); dqkv[i] = NAN; }
  for (size_t i = 0; i < n; ++i) { s = s * 1664525u + 1013904223u; dctx[i] = (float)(s >> 8) / 8388608.0f - 1.0f; ctx[i] = NAN; }
  if (big) { for (size_t i = 0; i < 3 * n; ++i) qkv[i] *= 0.05f; dctx[n / 2] = 3.4e38f; }
  const int dh = (int)(D / heads);
  AttnShape g{};
  g.B = B; g.D = D; g.T = T; g.heads = heads; g.dh = dh;
  g.left = std::min(left, T); g.right = std::min(right, T); g.qtiles = (T + 127) / 128;
  g.scale_log2e = (float)(1.4426950408889634 / sqrt((double)dh)); g.scale = (float)(1.0 / sqrt((double)dh));
  const unsigned blocks = (unsigned)(g.qtiles * heads * B);
  auto f = dh <= 16 ? launch<1> : dh <= 32 ? launch<2> : dh <= 48 ? launch<3> : launch<4>;
  f(blocks, qkv, ctx, &am, lse, dctx, dsum, dqkv, g);
  float *ctx2 = (float *)malloc(n * 4), *lse2 = (float *)malloc(rows * 4), *dqkv2 = (float *)malloc(3 * n * 4), *dsum2 = (float *)malloc(rows * 4);
  uint32_t am2 = 0;
  for (size_t i = 0; i < 3 * n; ++i) dqkv2[i] = NAN;
  auto f2 = dh <= 16 ? launch_few<1> : dh <= 32 ? launch_few<2> : dh <= 48 ? launch_few<3> : launch_few<4>;
  f2(qkv, ctx2, &am2, lse2, dctx, dsum2, dqkv2, g);
  if (memcmp(ctx, ctx2, n * 4) || memcmp(lse, lse2, rows * 4) || am != am2) { printf("  MISMATCH of the forward's bits\n"); bad = 1; }
  const double scale = 1.0 / sqrt((double)dh);
  std::vector<double> out(n, 0.0), omag(n, 0.0), ref(3 * n, 0.0), mag(3 * n, 0.0), p(T), dp(T);
  for (int64_t b = 0; b < B; ++b) for (int h = 0; h < heads; ++h) for (int64_t t = 0; t < T; ++t) {
    int64_t j0 = (left < 0 || t - left < 0) ? 0 : t - left, j1 = (right < 0 || t + right > T - 1) ? T - 1 : t + right;
    const size_t qo = (b * T + t) * 3 * D + h * dh, oo = (b * T + t) * D + h * dh;
    double m = -1e300, sum = 0, dd = 0, dda = 0;
    for (int64_t j = j0; j <= j1; ++j) { double a = 0; for (int d = 0; d < dh; ++d) a += (double)qkv[qo + d] * qkv[(b * T + j) * 3 * D + D + h * dh + d]; p[j] = a * scale; if (p[j] > m) m = p[j]; }
    for (int64_t j = j0; j <= j1; ++j) { p[j] = exp(p[j] - m); sum += p[j]; }
    for (int64_t j = j0; j <= j1; ++j) {
      const size_t vo = (b * T + j) * 3 * D + 2 * D + h * dh;
      double a = 0, aa = 0;
      p[j] /= sum;
      for (int d = 0; d < dh; ++d) {
        a += (double)dctx[oo + d] * qkv[vo + d]; aa += fabs((double)dctx[oo + d] * qkv[vo + d]);
        out[oo + d] += p[j] * qkv[vo + d]; omag[oo + d] += p[j] * fabs(qkv[vo + d]);
      }
      dp[j] = a; dd += p[j] * a; dda += p[j] * aa;
    }
    for (int64_t j = j0; j <= j1; ++j) {
      const size_t ko = (b * T + j) * 3 * D + D + h * dh, vo = ko + D;
      double aa = 0;
      for (int d = 0; d < dh; ++d) aa += fabs((double)dctx[oo + d] * qkv[vo + d]);
      const double ds = p[j] * (dp[j] - dd) * scale, dsa = p[j] * (aa + dda) * scale;
      for (int d = 0; d < dh; ++d) {
        ref[qo + d] += ds * qkv[ko + d]; mag[qo + d] += dsa * fabs(qkv[ko + d]);
        ref[ko + d] += ds * qkv[qo + d]; mag[ko + d] += dsa * fabs(qkv[qo + d]);
        ref[vo + d] += p[j] * dctx[oo + d]; mag[vo + d] += p[j] * fabs(dctx[oo + d]);
      }
    }
  }
  double worst = 0, worst_fwd = 0;
  float mx = 0;
  for (size_t i = 0; i < 3 * n; ++i) {
    at_least(worst, fabs((double)dqkv[i] - ref[i]) / (mag[i] + 1e-30));
    at_least(worst, fabs((double)dqkv2[i] - ref[i]) / (mag[i] + 1e-30));
  }
  for (size_t i = 0; i < n; ++i) { at_least(worst_fwd, fabs((double)ctx[i] - out[i]) / (omag[i] + 1e-30)); mx = std::max(mx, fabsf(ctx[i])); }
  printf("  worst err / sum|terms| = %.3g forward, %.3g backward\n", worst_fwd, worst);
  if (!(worst < 1e-5) || !(worst_fwd < 1e-5) || __float_as_uint(mx) != am) { printf("  MISMATCH\n"); bad = 1; }
  free(qkv); free(ctx); free(dctx); free(lse); free(dsum); free(dqkv);
  free(ctx2); free(lse2); free(dqkv2); free(dsum2);
}
}  // namespace aqt
int main() {
  using namespace aqt;
  one(1, 1, 4, 1, -1, -1); one(1, 70, 64, 1, -1, -1); one(1, 130, 36, 1, 23, 0); one(2, 65, 12, 3, 5, 7); one(1, 64, 8, 1, 0, 0);
  one(1, 97, 20, 1, -1, 3); one(1, 33, 64, 1, 40, 2); one(1, 40, 32, 2, 5, -1, true); one(1, 150, 60, 1, 20, 30, true);
  printf(bad ? "MISMATCH\n" : "ok\n"); return bad;
}
