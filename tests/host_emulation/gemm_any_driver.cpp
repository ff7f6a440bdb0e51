// Driver of the host emulation of the contractions straight from the caller's tensors: the test splices any_shape.h,
// colsum.h and epilogue.h, the kernels of gemm_any.hip (namespace any), of gemm_any_f64.hip (namespace f64) and of gemm_exact.hip
// (namespace exact) in front of this file.  Every tensor is an allocation of exactly its size; results are compared with plain loops written here.
namespace aqt {
static int bad = 0;
static uint32_t seed = 17u;
static float uniform() { seed = seed * 1664525u + 1013904223u; return (float)(seed >> 8) / 8388608.0f - 1.0f; }
static int code(int q) { return (int)lrintf(uniform() * (float)q); }
template <class T> struct Exact {   // n elements on the heap, nothing behind them
  T *p;
  explicit Exact(size_t n) : p((T *)malloc(n * sizeof(T))) { memset(p, 0x7E, n * sizeof(T)); }
  ~Exact() { free(p); }
  operator T *() const { return p; }
};
static void expect(const char *what, double worst, double limit) {
  printf("  %s: worst %.3g\n", what, worst); fflush(stdout);
  if (!(worst <= limit)) { printf("  MISMATCH\n"); bad = 1; }
}
static double sigma(double x) { return 1.0 / (1.0 + exp(-x)); }
// rows of codes [R][row bytes], and what they hold
struct Codes {
  std::vector<int> v;
  Exact<uint8_t> bytes;
  Codes(int64_t R, int64_t C, bool packed) : v(R * C), bytes(R * (packed ? (C + 1) / 2 : C)) {
    const int64_t rb = packed ? (C + 1) / 2 : C;
    for (int64_t r = 0; r < R; ++r) {
      if (packed) memset(bytes + r * rb, 0, rb);
      for (int64_t c = 0; c < C; ++c) {
        const int q = code(packed ? 7 : 127);
        v[r * C + c] = q;
        if (packed) bytes[r * rb + c / 2] |= (uint8_t)((q & 15) << (4 * (c & 1)));
        else bytes[r * rb + c] = (uint8_t)(int8_t)q;
      }
    }
  }
};

template <int TM, int TN, int WM, int WN, int WK, int BK, bool PACKED, int EPI> void forward(int64_t M, int64_t K, int64_t N) {
  printf("forward tile %d %d %d %d %d packed %d epilogue %d: %ld %ld %ld\n", TM, TN, WM, WN, WK, (int)PACKED, EPI, (long)M, (long)K, (long)N);
  constexpr bool GLU = EPI == AQT_EPI_GLU;
  const int64_t oc = GLU ? N / 2 : N;
  Codes x(M, K, false), w(N, K, PACKED);
  Exact<float> sw(N), bias(N), y(M * oc), dact(M * N), sx(1);
  Exact<int32_t> acc(M * N);
  Exact<uint32_t> am(1);
  am[0] = 0; sx[0] = 0.01f;
  for (int64_t n = 0; n < N; ++n) { sw[n] = 0.02f + 0.01f * uniform(); bias[n] = uniform(); }
  const int64_t tn = cdiv(oc, (GLU ? 16 : 32) * TN * WN), tm = cdiv(M, 32 * TM * WM);
  run((unsigned)(tn * tm), 64 * WM * WN * WK, 0, [&] {
    any::dense_fwd_any_kernel<TM, TN, WM, WN, WK, BK, PACKED, EPI>((const int8_t *)x.bytes.p, sx, w.bytes, sw, M, K, N, bias, y, acc, am, dact, (int)tn);
  });
  double worst = 0, sums = 0;
  float mx = 0;
  for (int64_t m = 0; m < M; ++m) for (int64_t n = 0; n < oc; ++n) {
    double v[2];
    for (int h = 0; h < (GLU ? 2 : 1); ++h) {
      int s = 0;
      for (int64_t k = 0; k < K; ++k) s += x.v[m * K + k] * w.v[(n + h * oc) * K + k];
      if (s != acc[m * N + n + h * oc]) ++sums;
      v[h] = (double)s * ((double)sx[0] * sw[n + h * oc]) + bias[n + h * oc];
    }
    const double ref = GLU ? v[0] * sigma(v[1]) : EPI == AQT_EPI_SWISH ? v[0] * sigma(v[0]) : v[0];
    const double e = fabs((double)y[m * oc + n] - ref) / (1.0 + fabs(ref));
    at_least(worst, e);
    mx = std::max(mx, fabsf(y[m * oc + n]));
  }
  expect("integer sums that differ", sums, 0);
  expect("outputs", worst, 1e-5);
  if (__float_as_uint(mx) != am[0]) { printf("  MISMATCH of the largest value\n"); bad = 1; }
}

// ---- the small products that make the codes themselves ----
static float scale_of(float most, int qmax) { return most / (float)qmax; }
static int code_of(float v, float s, int qmax) {
  const float t = s == 0.0f ? 0.0f : v / s, r = floorf(t + 0.5f);
  return (int)fminf(fmaxf(r, -(float)qmax), (float)qmax);
}
// values next to the lines between two codes among them, so that some are divided
static void fill(float *p, size_t n, float top, int qmax) {
  for (size_t i = 0; i < n; ++i) p[i] = i % 9 == 4 ? ((float)(int)(i % 11) - 5.0f - 0.5f) * (top / (float)qmax) : top * uniform();
}
template <bool PACKED> void from_rows(int64_t M, int64_t K, int64_t N, int bits_x) {
  printf("codes made by the product: %ld %ld %ld packed %d, %d bits\n", (long)M, (long)K, (long)N, (int)PACKED, bits_x);
  const int q = (1 << (bits_x - 1)) - 1;
  Codes w(N, K, PACKED);
  Exact<float> x(M * K), sw(N), bias(N), y(M * N), sx(1);
  Exact<int8_t> xq(M * K);
  Exact<uint32_t> most(1);
  Exact<int32_t> status(1);
  fill(x, M * K, 3.0f, q);
  uint32_t top = 0;
  for (int64_t i = 0; i < M * K; ++i) top = std::max(top, __float_as_uint(x[i]) & 0x7FFFFFFFu);
  most[0] = top; status[0] = 0;
  for (int64_t n = 0; n < N; ++n) { sw[n] = 0.02f + 0.01f * uniform(); bias[n] = uniform(); }
  const int64_t tn = cdiv(N, 32), tm = cdiv(M, 32);
  run((unsigned)(tn * tm), 512, 0, [&] { any::dense_fwd_rows_kernel<PACKED>(RowSource{x, most, q, xq, sx, status}, w.bytes, sw, M, K, N, bias, y, (int)tn); });
  const float s = scale_of(__uint_as_float(top), q);
  double wrong = sx[0] != s || status[0] != 0, worst = 0;
  for (int64_t m = 0; m < M; ++m) {
    for (int64_t k = 0; k < K; ++k) wrong += xq[m * K + k] != code_of(x[m * K + k], s, q);
    for (int64_t n = 0; n < N; ++n) {
      int64_t sum = 0;
      for (int64_t k = 0; k < K; ++k) sum += xq[m * K + k] * w.v[n * K + k];
      const double ref = (double)sum * ((double)s * sw[n]) + bias[n];
      at_least(worst, fabs((double)y[m * N + n] - ref) / (1.0 + fabs(ref)));
    }
  }
  expect("codes and scale that differ", wrong, 0);
  expect("outputs", worst, 1e-5);
}
template <int EPI> void from_dense(int64_t M, int64_t K, int64_t N, int bits_w, bool kn) {
  printf("both quantizers in the product: %ld %ld %ld, %d bits, epilogue %d\n", (long)M, (long)K, (long)N, bits_w, EPI);
  const int qx = 127, qw = (1 << (bits_w - 1)) - 1, packed = bits_w <= 4, parts = 3;
  Exact<float> x(M * K), w(K * N), sw(N), bias(N), y(M * N), dact(M * N), sx(1);
  Exact<int8_t> xq(M * K), wkn(K * N);
  Exact<uint8_t> wq(N * (packed ? K / 2 : K));
  Exact<int32_t> status(1);
  fill(x, M * K, 2.0f, qx);
  for (int64_t k = 0; k < K; ++k) for (int64_t n = 0; n < N; ++n) w[k * N + n] = n % 7 == 3 ? 0.0f : uniform() * (float)(1 + n % 5);
  for (int64_t n = 0; n < N; ++n) bias[n] = uniform();
  status[0] = 0;
  Exact<uint32_t> partial(parts);
  uint32_t top = 0;
  for (int i = 0; i < parts; ++i) partial[i] = 0;
  for (int64_t i = 0; i < M * K; ++i) { const uint32_t u = __float_as_uint(x[i]) & 0x7FFFFFFFu; partial[i % parts] = std::max(partial[i % parts], u); top = std::max(top, u); }
  int64_t slabs = std::min<int64_t>(cdiv(K, 32), kWeightSlabs);
  const int64_t rows = cdiv(K, slabs);
  slabs = cdiv(K, rows);
  uint32_t *part = (uint32_t *)aligned_alloc(16, align_up(slabs * N * 4, 16));
  for (int64_t i = 0; i < slabs * N; ++i) part[i] = 0;
  for (int64_t k = 0; k < K; ++k) for (int64_t n = 0; n < N; ++n) {
    uint32_t &u = part[k / rows * N + n];
    u = std::max(u, __float_as_uint(w[k * N + n]) & 0x7FFFFFFFu);
  }
  const int64_t tn = cdiv(N, 32), tm = cdiv(M, 32);
  const DenseSource src{x, partial, parts, qx, xq, sx, w, part, (int)slabs, qw, packed, wq, sw, kn ? wkn.p : nullptr, status};
  run((unsigned)(tn * tm), 512, 0, [&] { any::dense_fwd_raw_kernel<EPI>(src, M, K, N, bias, y, dact, (int)tn); });
  const float s = scale_of(__uint_as_float(top), qx);
  double wrong = sx[0] != s || status[0] != 0, worst = 0, worst_d = 0;
  std::vector<int> cx(M * K), cw(K * N);
  for (int64_t i = 0; i < M * K; ++i) { cx[i] = code_of(x[i], s, qx); wrong += xq[i] != cx[i]; }
  for (int64_t n = 0; n < N; ++n) {
    uint32_t u = 0;
    for (int64_t j = 0; j < slabs; ++j) u = std::max(u, part[j * N + n]);
    const float t = scale_of(__uint_as_float(u), qw);
    wrong += sw[n] != t;
    for (int64_t k = 0; k < K; ++k) {
      const int c = cw[k * N + n] = code_of(w[k * N + n], t, qw);
      const int got = packed ? (int)(int8_t)(uint8_t)(wq[n * (K / 2) + k / 2] << (k & 1 ? 0 : 4)) >> 4 : (int8_t)wq[n * K + k];
      wrong += got != c || (kn && wkn[k * N + n] != c);
    }
  }
  for (int64_t m = 0; m < M; ++m) for (int64_t n = 0; n < N; ++n) {
    int64_t sum = 0;
    for (int64_t k = 0; k < K; ++k) sum += cx[m * K + k] * cw[k * N + n];
    const double v = (double)sum * ((double)s * sw[n]) + bias[n], g = sigma(v);
    const double ref = EPI == AQT_EPI_SWISH ? v * g : v;
    at_least(worst, fabs((double)y[m * N + n] - ref) / (1.0 + fabs(ref)));
    if (EPI == AQT_EPI_SWISH) at_least(worst_d, fabs((double)dact[m * N + n] - g * (1 + v * (1 - g))));
  }
  expect("codes and scales that differ", wrong, 0);
  expect("outputs", worst, 1e-5);
  expect("slopes", worst_d, 1e-5);
  ::free(part);
}

// MODE 0: dX with a factor and a clip mask; 1 + e: weight-only forward.  kernel(f, scale, q, s_x, mask, factor, bias, out)
// `wild`: rows whose values lie further apart than the digits of gemm_exact.hip reach, and among them rows with an infinity
// (kInfinite) or that take all planes of digits (kFar)
enum Wild { kTame, kInfinite, kFar };
static void disturb(float *f, int64_t row, int64_t step, int64_t length, int64_t i, Wild wild) {   // element j of the row: f[row + j * step]
  for (int64_t j = 0; j < length; ++j) {
    float &v = f[row + j * step];
    if (i % 7 == 1) v = ldexpf(v, -(int)(j % 60));
    if (i % 7 == 2 && j % 50 == 9) v = ldexpf(v, -30);
    if (i % 7 == 3 && j % 2) v = ldexpf(v, 100);
    if (i % 7 == 4) v = ldexpf(v, -140);
    if (i % 7 == 5 && wild == kFar) v = ldexpf(v, 100 - (int)(j * 37 % 240));
    if (i % 7 == 6) v = 0.0f;
  }
  if (i % 7 == 5 && wild == kInfinite) f[row + (length - 1) * step] = i % 2 ? INFINITY : -INFINITY;
}
// Not further from the float64 loop than the last rounding and its own sums: at most 1.
static double beyond_rounding(float got, double ref, double rounded, double mag, double share) {   // rounded: what float32 held on the way
  const double wrong = INFINITY;
  if (!std::isfinite((float)ref)) return (std::isnan(ref) ? std::isnan(got) : got == (float)ref) ? 0.0 : wrong;
  if (!std::isfinite(mag) || !std::isfinite(rounded)) return got == ref ? 0.0 : wrong;   // an infinity behind a clip mask
  const double limit = share * rounded + 1e-13 * mag + 3e-45;
  return fabs((double)got - ref) / limit;
}
template <int MODE, bool PACKED, class Kernel> void float_rows(int64_t M, int64_t R, int64_t C, double limit, Kernel kernel, Wild wild = kTame) {
  constexpr bool GLU = MODE == 1 + AQT_EPI_GLU;
  printf("float rows, mode %d packed %d: %ld %ld %ld\n", MODE, (int)PACKED, (long)M, (long)R, (long)C);
  const int64_t oc = GLU ? R / 2 : R, ns = MODE ? R : C;
  Codes q(R, C, PACKED);
  Exact<float> f(M * C), scale(ns), bias(R), factor(M * R), out(M * oc), sx(1);
  Exact<uint32_t> mask(cdiv(M * R, 32));
  sx[0] = 1.0f;
  for (int64_t i = 0; i < M * C; ++i) f[i] = uniform();
  if (wild)
    for (int64_t i = 0; i < M; ++i) disturb(f, i * C, 1, C, i, wild);
  for (int64_t i = 0; i < ns; ++i) scale[i] = 0.02f + 0.01f * uniform();
  for (int64_t i = 0; i < R; ++i) bias[i] = MODE ? uniform() : 0.0f;
  for (int64_t i = 0; i < M * R; ++i) factor[i] = uniform();
  for (int64_t i = 0; i < cdiv(M * R, 32); ++i) { uniform(); mask[i] = seed | (seed << 16); }
  kernel((const float *)f, (const float *)scale, (const uint8_t *)q.bytes, (const float *)sx, (const uint32_t *)mask, (const float *)factor, (const float *)bias, (float *)out);
  double worst = 0;
  for (int64_t m = 0; m < M; ++m) for (int64_t r = 0; r < oc; ++r) {
    double v[2], mag = 0, held = 0;
    for (int h = 0; h < (GLU ? 2 : 1); ++h) {
      double s = 0;
      for (int64_t c = 0; c < C; ++c) {
        const double t = MODE ? (double)f[m * C + c] * q.v[(r + h * oc) * C + c] * scale[r + h * oc] : (double)(f[m * C + c] * scale[c]) * q.v[r * C + c];
        s += t; mag += fabs(t);
      }
      v[h] = s + bias[r + h * oc]; mag += fabs(bias[r + h * oc]);
      if (MODE) held += fabs(s) + fabs(bias[r + h * oc]);
    }
    double ref = v[0];
    if (!MODE) ref = (mask[(m * R + r) >> 5] >> ((m * R + r) & 31) & 1) ? v[0] * factor[m * R + r] : 0.0;
    else if (GLU) ref = v[0] * sigma(v[1]);
    else if (MODE == 1 + AQT_EPI_SWISH) ref = v[0] * sigma(v[0]);
    const double e = wild ? beyond_rounding(out[m * oc + r], ref, fabs(ref) + held, mag, limit) : fabs((double)out[m * oc + r] - ref) / (mag + 1e-30);
    at_least(worst, e);
  }
  expect(wild ? "error / (rounding of the result)" : "error / sum |terms|", worst, wild ? 1 : limit);
}
template <int TN, int WN, int WK, bool PACKED, int MODE> void rows_f64(int64_t M, int64_t R, int64_t C) {
  const int64_t tr = cdiv(MODE == 1 + AQT_EPI_GLU ? R / 2 : R, (MODE == 1 + AQT_EPI_GLU ? 8 : 16) * TN * WN), tm = cdiv(M, 32);
  float_rows<MODE, PACKED>(M, R, C, MODE > 1 ? 3e-6 : 1.2e-7, [&](auto f, auto scale, auto q, auto sx, auto mask, auto factor, auto bias, auto out) {
    run((unsigned)(tr * tm), 64 * WN * WK, 0, [&] {
      f64::f32_codes_f64_kernel<TN, WN, WK, PACKED, MODE>(f, scale, q, M, R, C, sx, MODE ? nullptr : mask, MODE ? nullptr : factor, MODE ? bias : nullptr, out, (int)tr);
    });
  });
}
// finite values never take the float64 instructions, an infinity those of its 64 positions only
static void expect_few_f64(Wild wild, int64_t strips, int64_t tiles, int blocks) {
  expect("float64 instructions", (double)g_f64_products, wild == kInfinite ? (double)(strips * 4 * tiles * 16 * blocks) : 0.0);
}
template <int TJ, bool PACKED, int MODE> void rows_exact(int64_t M, int64_t R, int64_t C, Wild wild, int each = 1) {
  constexpr bool GLU = MODE == 1 + AQT_EPI_GLU;
  const int64_t tr = cdiv(GLU ? R / 2 : R, (GLU ? 8 : 16) * TJ), tm = cdiv(M, 64);
  g_f64_products = 0;
  float_rows<MODE, PACKED>(M, R, C, MODE > 1 ? 3e-6 : 1.2e-7, [&](auto f, auto scale, auto q, auto sx, auto mask, auto factor, auto bias, auto out) {
    run((unsigned)(cdiv(tr, each) * tm), 256, 0, [&] {
      exact::f32_codes_exact_kernel<TJ, PACKED, MODE>(f, scale, q, M, R, (int)C, sx, MODE ? nullptr : mask, MODE ? nullptr : factor, MODE ? bias : nullptr, out, (int)tm, (int)tr, each);
    });
  }, wild);
  expect_few_f64(wild, tm, tr, TJ);
}
template <int TN, bool PACKED, int MODE, bool LONG> void rows_any(int64_t M, int64_t R, int64_t C) {
  const int64_t tr = R / (32 * TN), tm = cdiv(M, 32);
  float_rows<MODE, PACKED>(M, R, C, 3e-6, [&](auto f, auto scale, auto q, auto sx, auto mask, auto factor, auto bias, auto out) {
    run((unsigned)(tr * tm), 512, 0, [&] {
      any::f32_codes_any_kernel<TN, PACKED, MODE, LONG>(f, scale, q, M, R, C, sx, MODE ? nullptr : mask, MODE ? nullptr : factor, MODE ? bias : nullptr, out, (int)tr);
    });
  });
}

// dW in slabs of `rows` rows, with the bias gradient (rows 0: no slabs, the split kernel); T: what a slab's partial sums are kept in; TJ > 0: gemm_exact.hip
template <class T, int TJ = 0> void weights(int64_t M, int64_t K, int64_t N, int64_t rows, bool masked, Wild wild = kTame) {
  constexpr bool F64 = sizeof(T) == 8;
  const int64_t tile = F64 ? 64 : 128, tiles_n = cdiv(N, tile), tiles_k = cdiv(K, TJ ? 16 * TJ : tile), slabs = rows ? cdiv(M, rows) : 1;
  printf("dW %s: %ld %ld %ld, %ld slabs, masked %d\n", TJ ? "digits" : F64 ? "float64" : "bf16", (long)M, (long)K, (long)N, (long)slabs, (int)masked);
  Codes x(M, K, false);
  Exact<float> dy(M * N), sx(1), sw(N), dw(K * N), db(N);
  Exact<T> partial(slabs * K * N);
  Exact<double> part(slabs * tiles_k * N);
  Exact<uint32_t> mask(cdiv(K * N, 32));
  sx[0] = 0.03f;
  for (int64_t i = 0; i < M * N; ++i) dy[i] = uniform();
  if (wild)
    for (int64_t n = 0; n < N; ++n)
      for (int64_t m0 = 0; m0 < M; m0 += rows) disturb(dy, m0 * N + n, N, std::min(rows, M - m0), n + m0 / rows, wild);
  for (int64_t i = 0; i < N; ++i) sw[i] = i % 5 ? 0.5f : 0.0f;
  for (int64_t i = 0; i < cdiv(K * N, 32); ++i) { uniform(); mask[i] = seed | (seed << 16); }
  const bool one = slabs == 1;
  const unsigned grid = (unsigned)(tiles_k * tiles_n * slabs), bias_blocks = (unsigned)cdiv(N, kColsumCols), dw_blocks = one ? 0 : (unsigned)cdiv(K * N, 64);
  if constexpr (F64) {
    const DwFinish fin{sx, sw, masked ? mask.p : nullptr};
    g_f64_products = 0;
    if constexpr (TJ > 0)
      run(grid, 256, 0, [&] { exact::bwd_dw_exact_kernel<TJ>((const int8_t *)x.bytes.p, dy, M, K, N, rows, partial, one ? dw.p : nullptr, (int)tiles_k, (int)tiles_n, (int)slabs, fin, part); });
    else
    run(grid, 256, 0, [&] { f64::bwd_dw_f64_kernel((const int8_t *)x.bytes.p, dy, M, K, N, rows, partial, one ? dw.p : nullptr, (int)tiles_n, (int)(tiles_k * tiles_n), fin, part); });
    run(bias_blocks + dw_blocks, 256, 0, [&] { f64::dw_f64_fold_kernel(partial, (int)slabs, K, N, fin, dw, part, (int)(slabs * tiles_k), bias_blocks, db); });
  } else {
    const DwFinish fin{sx, sw, masked ? mask.p : nullptr};
    if (!rows) {
      run((unsigned)(K / 32 * (N / 32)), 512, 0, [&] { any::bwd_dw_split_kernel((const int8_t *)x.bytes.p, dy, M, K, N, fin, dw, db); });
    } else {
    run(grid, 256, 0, [&] { any::bwd_dw_any_kernel((const int8_t *)x.bytes.p, dy, M, K, N, rows, one ? dw.p : (float *)partial.p, (int)tiles_n, (int)(tiles_k * tiles_n), one ? 1 : 0, fin, part); });
    run(bias_blocks + dw_blocks, 256, 0, [&] { any::dw_any_fold_kernel((const float *)partial.p, (int)slabs, K, N, fin, dw, part, (int)(slabs * tiles_k), bias_blocks, db); });
    }
  }
  if (TJ) expect_few_f64(wild, tiles_n * slabs, tiles_k, TJ);
  double worst = 0, worst_b = 0;
  for (int64_t n = 0; n < N; ++n) {
    double b = 0, ba = 0;
    for (int64_t m = 0; m < M; ++m) { b += dy[m * N + n]; ba += fabs(dy[m * N + n]); }
    at_least(worst_b, wild ? beyond_rounding(db[n], b, fabs(b), ba, 6.1e-8) : fabs(db[n] - b) / (ba + 1e-30));
    for (int64_t k = 0; k < K; ++k) {
      double s = 0, mag = 0;
      for (int64_t m = 0; m < M; ++m) { const double t = (double)sx[0] * x.v[m * K + k] * dy[m * N + n]; s += t; mag += fabs(t); }
      const int64_t at = k * N + n;
      if (masked ? !(mask[at >> 5] >> (at & 31) & 1) : sw[n] == 0.0f) s = 0;
      const double e = wild ? beyond_rounding(dw[at], s, fabs(s), mag, 6.1e-8) : fabs(dw[at] - s) / (mag + 1e-30);
      at_least(worst, e);
    }
  }
  expect(wild ? "dW, error / (rounding of the result)" : "dW, error / sum |terms|", worst, wild ? 1 : F64 ? 6.1e-8 : 3e-6);
  expect("bias gradient", worst_b, wild ? 1 : 6.1e-8);
}
}  // namespace aqt
int main() {
  using namespace aqt;
  constexpr int kNone = AQT_EPI_NONE, kSwish = AQT_EPI_SWISH, kGlu = AQT_EPI_GLU;
  forward<1, 2, 4, 2, 1, 128, false, kGlu>(70, 150, 70); forward<1, 2, 4, 2, 1, 128, true, kSwish>(129, 131, 129);
  forward<1, 1, 2, 4, 1, 128, true, kNone>(67, 257, 130); forward<1, 2, 2, 2, 1, 128, true, kGlu>(65, 33, 30);
  forward<1, 2, 4, 1, 1, 128, false, kSwish>(131, 17, 65); forward<1, 1, 1, 1, 8, 64, false, kNone>(33, 517, 31);
  forward<1, 1, 1, 1, 8, 64, true, kSwish>(1, 31, 1); forward<1, 2, 1, 1, 8, 64, true, kGlu>(40, 129, 34);
  forward<1, 2, 1, 1, 8, 64, false, kGlu>(9, 15, 18); forward<1, 1, 1, 1, 8, 64, true, kNone>(9, 3, 5);
  from_rows<false>(33, 64, 36, 8); from_rows<true>(1, 68, 4, 8); from_rows<true>(40, 512, 33, 4); from_rows<false>(31, 508, 31, 8); from_rows<false>(65, 132, 70, 8);
  from_dense<kNone>(33, 64, 36, 8, true); from_dense<kSwish>(31, 68, 60, 4, true); from_dense<kNone>(1, 256, 4, 3, false); from_dense<kSwish>(70, 252, 100, 8, false);
  from_dense<kNone>(40, 132, 32, 4, true);
  rows_f64<1, 1, 8, false, 0>(33, 17, 300); rows_f64<1, 1, 8, false, 0>(5, 15, 3); rows_f64<2, 1, 8, true, 1 + kSwish>(34, 33, 77);
  rows_f64<1, 4, 1, false, 0>(65, 66, 37); rows_f64<1, 4, 1, true, 1 + kNone>(31, 65, 17); rows_f64<1, 4, 1, true, 1 + kNone>(3, 3, 15);
  rows_f64<2, 2, 1, false, 1 + kGlu>(33, 70, 33); rows_f64<2, 1, 8, true, 1 + kGlu>(33, 34, 129); rows_f64<2, 2, 1, false, 1 + kGlu>(2, 2, 1);
  rows_exact<4, false, 0>(65, 66, 64, kTame); rows_exact<5, false, 0>(33, 170, 200, kInfinite, 2); rows_exact<5, false, 0>(64, 33, 133, kFar);
  rows_exact<5, true, 1 + kNone>(17, 97, 131, kFar, 2); rows_exact<4, true, 1 + kGlu>(70, 70, 65, kInfinite); rows_exact<4, false, 1 + kGlu>(5, 98, 190, kFar);
  rows_exact<5, false, 1 + kSwish>(9, 19, 127, kTame); rows_exact<4, true, 1 + kNone>(64, 64, 128, kInfinite);
  rows_any<1, false, 0, false>(33, 128, 96); rows_any<2, false, 0, false>(33, 128, 32); rows_any<2, true, 1 + kGlu, false>(33, 128, 320);
  rows_any<1, false, 0, true>(7, 32, 4640); rows_any<1, true, 1 + kSwish, true>(3, 32, 4128);
  weights<double>(70, 66, 65, 64, false); weights<double>(130, 3, 2, 64, true); weights<double>(33, 64, 70, 64, true); weights<double>(1, 1, 1, 64, false);
  weights<double>(200, 130, 5, 128, true);
  weights<double, 4>(70, 66, 65, 64, false); weights<double, 5>(200, 81, 33, 128, true, kInfinite); weights<double, 5>(64, 97, 5, 64, true, kFar);
  weights<double, 4>(329, 4, 66, 192, false, kFar); weights<double, 5>(130, 193, 17, 192, true, kInfinite);
  weights<float>(70, 64, 96, 0, true); weights<float>(33, 32, 64, 0, false); weights<float>(1, 32, 32, 0, true); weights<float>(600, 32, 32, 0, false);
  weights<float>(70, 128, 128, 64, true); weights<float>(33, 256, 128, 64, false); weights<float>(1, 128, 128, 32, true);
  printf(bad ? "MISMATCH\n" : "ok\n"); return bad;
}
