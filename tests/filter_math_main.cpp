// Largest errors, in units of the last place, of the filter's logarithm,
// cosine and exponential against 80-bit long double, over evenly spread and
// random arguments and the ends of the ranges.
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "pfr_filter_math.h"

static double ulps(double got, long double want) {
  int e;
  frexpl(want, &e);
  const long double ulp = ldexpl(1.0L, e - 53);  // want in [2^(e-1), 2^e)
  return (double)(fabsl((long double)got - want) / ulp);
}

int main() {
  static pfr::MathTables T;
  const long double pi = acosl(-1.0L);
  for (int i = 0; i < pfr::kLogBins; ++i) {
    const pfr::LogEntry t = pfr::kLogTable[i];
    T.lg[i] = {t.rc, t.hi};
    T.lo[i] = t.lo;
    // the table itself: rc a binary32 number near 1 / m, log rc to 2^-42 and the rest
    const long double rc = t.rc * (i >= pfr::kHalfBin ? 2.0L : 1.0L), lg = logl(rc);
    if ((double)(float)t.rc != t.rc || ldexp(t.hi, 42) != rint(ldexp(t.hi, 42)) ||
        fabsl(t.hi - lg) > ldexpl(1.0L, -43) || fabsl((lg - t.hi) - t.lo) > ldexpl(1.0L, -63) ||
        fabsl((1.0L + (i + 0.5L) / pfr::kLogBins) * t.rc - 1.0L) > ldexpl(1.0L, -8)) {
      printf("table entry %d\n", i);
      return 1;
    }
  }
  for (int i = 0; i < pfr::kCosBins; ++i)
    T.cs[i] = {(double)cosl(2 * pi * i / pfr::kCosBins), (double)sinl(2 * pi * i / pfr::kCosBins)};
  double log_max = 0, cos_max = 0, exp_max = 0;
  auto word = [&](uint32_t x) {
    const long double want = -logl(((long double)x + 1.0L) * 0x1p-32L);
    const double got = pfr::neg_log_u1(x, &T);
    if (want > 0) log_max = fmax(log_max, ulps(got, want));
    else if (got != 0.0) log_max = HUGE_VAL;
    // a unit of the last place of 1 and below: near its zeros the cosine's
    // error is that of the sine and angle, absolute
    const double c = pfr::cos_turns(x, &T);
    cos_max = fmax(cos_max, (double)(fabsl(c - cosl(2 * pi * x * 0x1p-32L)) / 0x1p-53L));
  };
  uint64_t state = 1;
  auto random = [&]() {
    state = state * 6364136223846793005ull + 1442695040888963407ull;
    return state >> 11;
  };
  for (uint32_t k = 0; k < 4096; ++k) {
    word(k);
    word(0xFFFFFFFFu - k);
    for (int b = 12; b < 32; ++b) word((1u << b) - 2048 + k);
  }
  for (int k = 0; k < 1000000; ++k) word((uint32_t)(random() >> 21));
  auto at = [&](double x) {
    const long double want = expl((long double)x);
    if (want >= 0x1p-1000L) exp_max = fmax(exp_max, ulps(pfr::exp_neg(x), want));
  };
  for (int k = 0; k < 1000000; ++k) {
    const double u = (double)random() * 0x1p-53;
    at(-u);
    at(-40.0 * u);
    at(-690.0 * u);
    at(-ldexp(u, -(k % 60)));
  }
  if (pfr::exp_neg(0.0) != 1.0 || pfr::exp_neg(-INFINITY) != 0.0 || pfr::exp_neg(-1e300) != 0.0 ||
      !std::isnan(pfr::exp_neg(NAN)))
    exp_max = HUGE_VAL;
  printf("%.4f %.4f %.4f\n", log_max, cos_max, exp_max);
  return 0;
}
