// pfr_filter_math.h -- the elementary functions of the filter's move and
// initialisation, in binary64.
//
// The general library functions (argument reduction for any argument, special
// cases) were most of the move's time.  Here the arguments are known: u1 =
// y 2^-32 with y a whole number in [1, 2^32], an angle that is a whole number
// of 2^-32 turns, and a log-weight at most 0.
//   -log u1   y = m 2^e; a table of 128 intervals of m gives rc ~ 1 / m and
//             log rc, and log(m rc) is a short series in r = m rc - 1 (m from
//             sqrt 2 up counts as m / 2, so that u1 near 1 keeps its relative
//             precision: kk = 0, log rc = 0).  r is exact, and so is the sum
//             of kk ln 2 and log rc to 2^-42; what is left of both and the
//             series beyond r are added to that sum's rounding error before
//             they are added to the sum, so only the last addition rounds.
//   cos       a table of 256 angles and the addition theorem
//   exp       2^k e^r, |r| <= ln 2 / 2, the exponential series to r^13 / 13!
//             (below 2^-57 beyond), 1 + r + r^2 / 2 with their rounding errors
// Largest errors over some million arguments, in units of the last place, beside
// the device library's functions: logarithm 0.501 (0.63), exponential 0.542
// (0.86); the cosine, absolute, 1.5 units of 2^-53, where cos(2 pi u) in binary64
// loses every digit near its zeros.
//
// Compiles for the host too, where the errors are tested.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define PFR_MATH __device__ __forceinline__
#else
#define PFR_MATH static inline
#endif

namespace pfr {

constexpr int kLogBins = 128, kCosBins = 256;
constexpr int kHalfBin = 53;  // m from 1 + 53/128 = 1.4140625 on
constexpr double kLn2Hi = 0x1.62e42fefa3800p-1;   // ln 2 to 42 bits: times 0..1154 exact
constexpr double kLn2Lo = 0x1.ef35793c76730p-45;  // ln 2 - kLn2Hi

struct alignas(16) MathPair {
  double x, y;
};
struct MathTables {
  MathPair lg[kLogBins];  // rc (times 1/2 where m counts as m / 2), log rc to 2^-42
  MathPair cs[kCosBins];  // cosine and sine of 2 pi i / 256
  double lo[kLogBins];    // the rest of log rc
};

// Interval i of m: rc, the binary32 number next to the inverse of its centre (1
// in the two intervals at m = 1 and 2, so that log u1 = log(1 + r) there), and
// log rc as a multiple of 2^-42 and a remainder.
struct LogEntry {
  double rc, hi, lo;
};
constexpr LogEntry kLogTable[kLogBins] = {
    {0x1p0, 0.0, 0.0},
    {0x1.fa11cap-1, -0x1.7dc49e782p-7, 0x1.ea453db5aedfap-44},
    {0x1.f6310ap-1, -0x1.3cea5df47p-6, 0x1.68e0bb2d11538p-44},
    {0x1.f25f64p-1, -0x1.b9fc0afbp-6, 0x1.b97bf0ae65efdp-44},
    {0x1.ee9c8p-1, -0x1.1b0d90924p-5, 0x1.3381e9ae9df1p-44},
    {0x1.eae808p-1, -0x1.58a5b57c9p-5, 0x1.b23e395718b0ep-45},
    {0x1.e741aap-1, -0x1.95c836cc9p-5, 0x1.c0be197c4f058p-45},
    {0x1.e3a918p-1, -0x1.d276b22dbp-5, -0x1.6b943c787885bp-46},
    {0x1.e01e02p-1, -0x1.075982499p-4, 0x1.b8e3f64b59fedp-44},
    {0x1.dca01ep-1, -0x1.253f6120ap-4, -0x1.4189d7b69873fp-44},
    {0x1.d92f22p-1, -0x1.42edcd9a64p-4, -0x1.bc6a0ea7d0151p-46},
    {0x1.d5cac8p-1, -0x1.60658ad374p-4, -0x1.0c3b9dee9c50dp-44},
    {0x1.d272cap-1, -0x1.7da76907bp-4, -0x1.2cee8c481006fp-44},
    {0x1.cf26e6p-1, -0x1.9ab4225204p-4, 0x1.8a2072678cdf7p-45},
    {0x1.cbe6dap-1, -0x1.b78c7d2b1p-4, 0x1.24f7f3c3d1dd4p-44},
    {0x1.c8b266p-1, -0x1.d4313a96ccp-4, 0x1.93d5a79144461p-45},
    {0x1.c5894ep-1, -0x1.f0a3039118p-4, 0x1.d36060343122ep-44},
    {0x1.c26b54p-1, -0x1.06714f3ca6p-3, 0x1.a38539cde76e2p-45},
    {0x1.bf583ep-1, -0x1.14785c6e74p-3, -0x1.5ed771057a4a1p-46},
    {0x1.bc4fd6p-1, -0x1.2266f328a6p-3, 0x1.4c7e1b83f8e84p-45},
    {0x1.b951e2p-1, -0x1.303d74c648p-3, 0x1.15295ccdb166fp-50},
    {0x1.b65e2ep-1, -0x1.3dfc2c26ccp-3, -0x1.8abf362b930e7p-45},
    {0x1.b37484p-1, -0x1.4ba37269a6p-3, 0x1.420f9b3ecb41dp-44},
    {0x1.b094b4p-1, -0x1.5933896982p-3, -0x1.2eb88b6918e2p-48},
    {0x1.adbe88p-1, -0x1.66acd4072ap-3, -0x1.aa1c5bfc6c77p-44},
    {0x1.aaf1d2p-1, -0x1.740f93fc04p-3, 0x1.08b1018f0b768p-44},
    {0x1.a82e66p-1, -0x1.815c059c36p-3, 0x1.00262792efc78p-44},
    {0x1.a5741p-1, -0x1.8e92902886p-3, -0x1.a8b74b13f58d5p-44},
    {0x1.a2c2a8p-1, -0x1.9bb36547ep-3, 0x1.1dc18a1c998d1p-45},
    {0x1.a01a02p-1, -0x1.a8becdf082p-3, -0x1.e38524f20ae63p-44},
    {0x1.9d79f2p-1, -0x1.b5b51740fcp-3, 0x1.4a9066c043ed5p-44},
    {0x1.9ae24ep-1, -0x1.c2968890c2p-3, 0x1.cd402ded86c9bp-45},
    {0x1.9852fp-1, -0x1.cf6359209cp-3, -0x1.7b9639a216c06p-45},
    {0x1.95cbbp-1, -0x1.dc1bcdcabep-3, -0x1.916e1a63196c6p-44},
    {0x1.934c68p-1, -0x1.e8c0250aa6p-3, 0x1.6804b80e8e72ap-45},
    {0x1.90d4f2p-1, -0x1.f550a0ecb8p-3, 0x1.2d402a0afc21ep-45},
    {0x1.8e6528p-1, -0x1.00e6c38ad5p-2, -0x1.e188d52b24cadp-50},
    {0x1.8bfce8p-1, -0x1.071b860cd6p-2, 0x1.bcb83a3e019fbp-44},
    {0x1.899c1p-1, -0x1.0d46b3d9abp-2, -0x1.d41a1f63b293bp-44},
    {0x1.87427cp-1, -0x1.13686fa13bp-2, 0x1.d3c4299d6a45p-44},
    {0x1.84f00cp-1, -0x1.1980d34542p-2, -0x1.b7dde7a364a5fp-45},
    {0x1.82a4ap-1, -0x1.1f8ffa248ap-2, -0x1.7956c040cc921p-45},
    {0x1.806018p-1, -0x1.2596011df7p-2, -0x1.8e7c4224ea3f8p-44},
    {0x1.7e2256p-1, -0x1.2b9301378ap-2, 0x1.67ac9d6e70e7ep-45},
    {0x1.7beb3ap-1, -0x1.31871a4144p-2, -0x1.8fd1d948b82f3p-46},
    {0x1.79baa6p-1, -0x1.37726827fep-2, 0x1.e74b62c4944f9p-44},
    {0x1.779082p-1, -0x1.3d54f7e81fp-2, -0x1.c6e41598fe6f7p-44},
    {0x1.756cacp-1, -0x1.432ef2f84fp-2, 0x1.fb037931707cfp-44},
    {0x1.734f0cp-1, -0x1.490068ec01p-2, 0x1.8b63dfe19117ep-44},
    {0x1.713786p-1, -0x1.4ec97582p-2, -0x1.3a68baf27d709p-45},
    {0x1.6f2602p-1, -0x1.548a2aa6ddp-2, -0x1.33e5762fda1e4p-45},
    {0x1.6d1a62p-1, -0x1.5a42ac334dp-2, 0x1.bc98f2d791854p-50},
    {0x1.6b149p-1, -0x1.5ff308ea79p-2, -0x1.ed6839f21e439p-45},
    {0x1.691474p-1, 0x1.602d09a709p-2, 0x1.ea08976e418afp-46},
    {0x1.6719f4p-1, 0x1.5a8caf83eep-2, -0x1.95dbb0a7f5b78p-48},
    {0x1.6524f8p-1, 0x1.54f430c7bep-2, 0x1.a6d34c08ca452p-46},
    {0x1.63356cp-1, 0x1.4f638013aap-2, -0x1.fcfcacb2de886p-44},
    {0x1.614b36p-1, 0x1.49da7dbfccp-2, 0x1.06992cdaaef3ap-44},
    {0x1.5f6644p-1, 0x1.4459202d3ap-2, -0x1.812e892274dc8p-47},
    {0x1.5d867cp-1, 0x1.3edf458417p-2, -0x1.f0a9e297faafcp-44},
    {0x1.5babccp-1, 0x1.396ce231bcp-2, -0x1.5d92c5673e352p-47},
    {0x1.59d62p-1, 0x1.3401e3eaedp-2, -0x1.1b8f355526e72p-44},
    {0x1.58056p-1, 0x1.2e9e2b8e12p-2, 0x1.42f0c128d1317p-45},
    {0x1.56397cp-1, 0x1.2941b0b987p-2, -0x1.21944b72f6c33p-44},
    {0x1.54725ep-1, 0x1.23ec584decp-2, -0x1.6e8b4c8a5991dp-44},
    {0x1.52aff6p-1, 0x1.1e9e183c8ap-2, -0x1.8479f53c15f98p-44},
    {0x1.50f22ep-1, 0x1.1956d385bcp-2, 0x1.7d24e3ad1a45cp-45},
    {0x1.4f38f6p-1, 0x1.14167e6767p-2, 0x1.e09a3024d7322p-44},
    {0x1.4d843cp-1, 0x1.0edd064378p-2, 0x1.016a52d84528bp-47},
    {0x1.4bd3eep-1, 0x1.09aa57a26cp-2, 0x1.b4efd61736304p-44},
    {0x1.4a27fap-1, 0x1.047e5e31e8p-2, 0x1.d51000d0a1e6dp-45},
    {0x1.488052p-1, 0x1.feb22276ap-3, 0x1.f31a7de006adbp-45},
    {0x1.46dce4p-1, 0x1.f474b5c4ep-3, -0x1.bd7ebf1cfa71bp-44},
    {0x1.453d9ep-1, 0x1.ea4448d84ap-3, 0x1.5e6b1e372f262p-44},
    {0x1.43a274p-1, 0x1.e020d27236p-3, -0x1.5be04ad6ece1fp-45},
    {0x1.420b52p-1, 0x1.d60a157104p-3, -0x1.5e3b0efc4c134p-44},
    {0x1.40782ep-1, 0x1.cc001295b4p-3, -0x1.e8a5a5cc9ecfap-46},
    {0x1.3ee8f4p-1, 0x1.c20289a18p-3, -0x1.93292e55ce12p-45},
    {0x1.3d5d9ap-1, 0x1.b81178d382p-3, 0x1.d85063c1da89ep-46},
    {0x1.3bd60ep-1, 0x1.ae2ca9be72p-3, 0x1.7995d2e588b3ep-44},
    {0x1.3a5244p-1, 0x1.a4540b3e6ap-3, 0x1.5f7b5c8243af3p-44},
    {0x1.38d22ep-1, 0x1.9a877e06bap-3, 0x1.43bcdbf159cafp-44},
    {0x1.3755bep-1, 0x1.90c6e177ccp-3, -0x1.a47277693cd71p-46},
    {0x1.35dce6p-1, 0x1.8712139d0ep-3, 0x1.328dec2f9af9fp-44},
    {0x1.34679ap-1, 0x1.7d68fe72f6p-3, -0x1.532a417f5df39p-45},
    {0x1.32f5cep-1, 0x1.73cb8adcfep-3, -0x1.da53d8d1d318ap-44},
    {0x1.318776p-1, 0x1.6a39a0a3bep-3, -0x1.90ad56665b947p-44},
    {0x1.301c82p-1, 0x1.60b30b830ap-3, -0x1.73d67499879a4p-44},
    {0x1.2eb4eap-1, 0x1.5737cbb818p-3, 0x1.9b93b26b86e55p-44},
    {0x1.2d50ap-1, 0x1.4dc7b817bcp-3, 0x1.c75b60ae1d464p-47},
    {0x1.2bef98p-1, 0x1.4462b3bc9cp-3, -0x1.89360a737fc77p-44},
    {0x1.2a91cap-1, 0x1.3b08bc0d8p-3, -0x1.aec7d7275f517p-44},
    {0x1.293726p-1, 0x1.31b996aba4p-3, 0x1.f02c263a6137bp-44},
    {0x1.27dfa4p-1, 0x1.28753ef11ap-3, 0x1.734fc359868aep-44},
    {0x1.268b38p-1, 0x1.1f3b93bf26p-3, -0x1.6066e9b067a88p-46},
    {0x1.2539d8p-1, 0x1.160c80c4b2p-3, 0x1.ec142a900b313p-45},
    {0x1.23eb7ap-1, 0x1.0ce7f0c4ccp-3, 0x1.3eb1bac2710cdp-46},
    {0x1.22a012p-1, 0x1.03cdbf7d1ep-3, 0x1.817f07169ba68p-44},
    {0x1.215798p-1, 0x1.f57bc799p-4, 0x1.76a4c9ea8aff8p-46},
    {0x1.201202p-1, 0x1.e3708b5304p-4, 0x1.05bd3e6c69521p-45},
    {0x1.1ecf44p-1, 0x1.d1797ba218p-4, 0x1.35f51b5f061bp-44},
    {0x1.1d8f56p-1, 0x1.bf9680f9fcp-4, 0x1.3f81b8d7724dep-45},
    {0x1.1c523p-1, 0x1.adc78265bp-4, -0x1.579d209c2345ap-44},
    {0x1.1b17c6p-1, 0x1.9c0c2ba4d4p-4, -0x1.ad1951e8b42b6p-44},
    {0x1.19e012p-1, 0x1.8a647d391cp-4, 0x1.c19482f9f6ccdp-44},
    {0x1.18ab08p-1, 0x1.78d01f23d8p-4, 0x1.6711794b0e70cp-47},
    {0x1.1778a2p-1, 0x1.674f0ee364p-4, 0x1.a65accca2708bp-44},
    {0x1.1648d6p-1, 0x1.55e10e20ep-4, 0x1.922500e0afb3bp-47},
    {0x1.151b9ap-1, 0x1.4485dc8dbcp-4, 0x1.fa67a68d15f4bp-44},
    {0x1.13f0e8p-1, 0x1.333d734184p-4, -0x1.ff3b6ace50af5p-49},
    {0x1.12c8b8p-1, 0x1.2207ac8784p-4, 0x1.472c4fc004aa9p-44},
    {0x1.11a302p-1, 0x1.10e4612cbp-4, -0x1.7e109a845d805p-44},
    {0x1.107fbcp-1, 0x1.ffa694dab8p-5, 0x1.2fd08983860dfp-45},
    {0x1.0f5eep-1, 0x1.dda8b7c68p-5, -0x1.1caac64d4aed9p-45},
    {0x1.0e4066p-1, 0x1.bbced3a69p-5, -0x1.885088bdfb456p-46},
    {0x1.0d2446p-1, 0x1.9a188df74p-5, -0x1.0ed8aceb405d4p-44},
    {0x1.0c0a78p-1, 0x1.7885892358p-5, -0x1.0d92d084f92a2p-46},
    {0x1.0af2f8p-1, 0x1.5715df404p-5, -0x1.8e055df93ffbep-44},
    {0x1.09ddbap-1, 0x1.35c8b2ca1p-5, 0x1.820c4def45c63p-44},
    {0x1.08cabcp-1, 0x1.149e568008p-5, -0x1.3030c9a1c45fap-44},
    {0x1.07b9f2p-1, 0x1.e72bccc14p-6, -0x1.93062499a534bp-45},
    {0x1.06ab5ap-1, 0x1.a55f624c6p-6, -0x1.dec419f2b5285p-45},
    {0x1.059eeap-1, 0x1.63d615c69p-6, 0x1.7ab2f895961afp-47},
    {0x1.04949cp-1, 0x1.228f827eap-6, 0x1.686df2803cc03p-45},
    {0x1.038c6cp-1, 0x1.c3177b4c8p-7, -0x1.44245fce37d0bp-44},
    {0x1.02865p-1, 0x1.4192bb968p-7, 0x1.95f4755d3a613p-46},
    {0x1.018244p-1, 0x1.8121bb458p-8, 0x1.a1bbb82e18d5cp-46},
    {0x1p-1, 0.0, 0.0},
};

PFR_MATH uint64_t math_bits(double v) {
  uint64_t b;
  __builtin_memcpy(&b, &v, sizeof b);
  return b;
}
PFR_MATH double math_double(uint64_t b) {
  double v;
  __builtin_memcpy(&v, &b, sizeof v);
  return v;
}

// -log((x + 1) 2^-32)
PFR_MATH double neg_log_u1(uint32_t x, const MathTables* T) {
  const uint64_t yb = math_bits((double)x + 1.0);
  const uint32_t hi = (uint32_t)(yb >> 32);
  const uint32_t i = (hi >> 13) & (kLogBins - 1);
  const double m = math_double((yb & 0xFFFFFFFFFFFFFull) | 0x3FF0000000000000ull);
  const int kk = 1023 + 32 - (int)(hi >> 20) - (i >= (uint32_t)kHalfBin ? 1 : 0);
  const MathPair t = T->lg[i];
  const double r = __builtin_fma(m, t.x, -1.0);  // exact, |r| below 2^-7
  double p = __builtin_fma(r, 1.0 / 8.0, -1.0 / 7.0);
  p = __builtin_fma(p, r, 1.0 / 6.0);
  p = __builtin_fma(p, r, -1.0 / 5.0);
  p = __builtin_fma(p, r, 1.0 / 4.0);
  p = __builtin_fma(p, r, -1.0 / 3.0);
  p = __builtin_fma(p, r, 1.0 / 2.0);  // r - log(1 + r) = r^2 p
  const double kd = (double)kk;
  const double a = __builtin_fma(kd, kLn2Hi, t.y);  // exact; 0, or larger than r
  const double s = a - r, e = (a - s) - r;
  return s + (e + __builtin_fma(p * r, r, __builtin_fma(kd, kLn2Lo, T->lo[i])));
}

// cos(2 pi x 2^-32)
PFR_MATH double cos_turns(uint32_t x, const MathTables* T) {
  const uint32_t v = x + 0x800000u;
  const MathPair t = T->cs[v >> 24];
  const double d = (double)((int32_t)(v & 0xFFFFFFu) - 0x800000) * (6.283185307179586 * 0x1p-32);
  const double z = d * d;
  const double cm =
      z * __builtin_fma(z, __builtin_fma(z, -1.0 / 720.0, 1.0 / 24.0), -0.5);  // cos d - 1
  const double s3 =
      __builtin_fma(z, __builtin_fma(z, -1.0 / 5040.0, 1.0 / 120.0), -1.0 / 6.0);
  const double sn = __builtin_fma(d * z, s3, d);
  return __builtin_fma(t.x, cm, __builtin_fma(-t.y, sn, t.x));
}

// exp(x) for x <= 0 (NaN stays NaN)
PFR_MATH double exp_neg(double x) {
  x = x < -800.0 ? -800.0 : x;  // below -746 the result is 0
  const double k = __builtin_rint(x * 1.4426950408889634);
  const double rh = __builtin_fma(k, -kLn2Hi, x), rl = k * kLn2Lo;  // rh exact
  const double r = rh - rl, rest = (rh - r) - rl;
  double p = __builtin_fma(r, 1.0 / 6227020800.0, 1.0 / 479001600.0);
  p = __builtin_fma(p, r, 1.0 / 39916800.0);
  p = __builtin_fma(p, r, 1.0 / 3628800.0);
  p = __builtin_fma(p, r, 1.0 / 362880.0);
  p = __builtin_fma(p, r, 1.0 / 40320.0);
  p = __builtin_fma(p, r, 1.0 / 5040.0);
  p = __builtin_fma(p, r, 1.0 / 720.0);
  p = __builtin_fma(p, r, 1.0 / 120.0);
  p = __builtin_fma(p, r, 1.0 / 24.0);
  p = __builtin_fma(p, r, 1.0 / 6.0);
  const double g = 0.5 * r, h = g * r, he = __builtin_fma(g, r, -h);  // h + he = r^2 / 2
  const double q = r + h, qe = h - (q - r);                            // q + qe = r + h
  const double s = 1.0 + q, se = q - (s - 1.0);                        // s + se = 1 + q
  p = __builtin_fma(p * h, 2.0 * r, __builtin_fma(rest, q, rest) + he);
  return __builtin_ldexp(s + (se + (qe + p)), (int)k);
}

}  // namespace pfr
