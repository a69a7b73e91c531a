// pfr_alt.hip -- the collective-free resamplers: Metropolis (Code 2 of the
// paper) and rejection (Code 3), one lane per particle on a counter-based
// Philox stream.
//
// Lane results depend only on (particle, step/trial, filter, offset) through
// the Philox counter, never on which lane or wave did the work, so every
// launch shape gives the same bits.
#include "pfr_kernels.h"
#include <algorithm>
#include <cstring>

namespace pfr {

// ------------------------------------------------------------------ Metropolis
// Lane i runs B steps of an independent Metropolis chain started at k = i.
// Step s takes (j, u) from words 3s, 3s+1, 3s+2 of the lane's Philox stream
// (word m = word m&3 of counter (i, TRIAL<<28 | m>>2, filter, offset)) and
// moves to j when u * w_k <= w_j.  The proposals and their weight loads do not
// depend on the chain state: a group of 4 steps takes 3 Philox calls and
// issues its 4 gathers at once, and the gathers of group m+1 are in flight
// while the accept decisions of group m run in order (two register sets, used
// alternately, so that no load has to complete before it is consumed).
struct MGroup {
  uint32_t j[4];
  uint32_t u[4];
  double wj[4];
  int nq;
};

// pl: the lane's Philox parts for particle i (philox_lane); the step number,
// filter and offset are the same on every lane of the wave.
template <typename T>
__device__ __forceinline__ void metropolis_fetch(const T* __restrict__ ws, Key key, uint32_t i,
                                                 const PhiloxLane& pl, uint32_t filt,
                                                 uint32_t offset, uint32_t n, int32_t steps,
                                                 int32_t m, MGroup& g) {
  uint32_t x[12];
  const int32_t left = steps - 4 * m;
  const int ncall = left >= 4 ? 3 : (3 * left + 3) / 4;
#pragma unroll
  for (int c3 = 0; c3 < 3; ++c3) {
    if (c3 < ncall) {
      const uint4 v = philox_lane_call(pl, key, DOM_TRIAL, (uint32_t)(3 * m + c3), filt, offset);
      x[4 * c3 + 0] = v.x;
      x[4 * c3 + 1] = v.y;
      x[4 * c3 + 2] = v.z;
      x[4 * c3 + 3] = v.w;
    }
  }
  g.nq = left >= 4 ? 4 : left;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    g.j[q] = q < g.nq ? index_draw(x[3 * q], x[3 * q + 1], n) : i;
    g.u[q] = x[3 * q + 2];
    g.wj[q] = (double)ws[g.j[q]];
  }
}

template <typename T>
__device__ __forceinline__ void metropolis_accept(const MGroup& g, uint32_t& k, double& wk) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (q < g.nq && accept_exact<T>(u_accept(g.u[q]), wk, g.wj[q])) {
      k = g.j[q];
      wk = g.wj[q];
    }
  }
}

// A workgroup takes the particles [p0, p1) of the global array (chunk per
// workgroup) and walks the segments that overlap them; a segment of at most
// CAP weights is first copied into LDS, so that every random weight load of
// its chains is an LDS read.  The chains do not depend on the launch shape.
// Four consecutive weights; a segment starts anywhere, so the wide access is
// aligned to one weight only.
template <typename T>
struct alignas(sizeof(T)) Weights4 {
  T v[4];
};
template <typename T>
__device__ __forceinline__ Weights4<T> load_weights4(const T* __restrict__ w) {
  typedef T V __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  const V t = *reinterpret_cast<const V*>(w);
  return Weights4<T>{{t.x, t.y, t.z, t.w}};
}

// A segment of n weights into LDS (16-byte aligned), 16 bytes a lane, or a
// weight each where the threads suffice (the last of n, when they are not a
// multiple of four, are a second wait: 65536 segments of 128 .. 256 without
// max_len, one step, 368 -> 347 us).
template <typename T>
__device__ __forceinline__ void stage_weights(const T* __restrict__ w, uint32_t n, T* sw) {
  if (n <= blockDim.x) {
    if (threadIdx.x < n) sw[threadIdx.x] = w[threadIdx.x];
    return;
  }
#pragma unroll 4
  for (uint32_t q = threadIdx.x; q < n / 4; q += blockDim.x) {
    const Weights4<T> t = load_weights4(w + 4 * q);
#pragma unroll
    for (int k = 0; k < 4; ++k) sw[4 * q + k] = t.v[k];
  }
  if (threadIdx.x < (n & 3u)) sw[(n & ~3u) + threadIdx.x] = w[(n & ~3u) + threadIdx.x];
}

template <typename T>
__device__ __forceinline__ uint32_t metropolis_chain(const T* ws, Key key, uint32_t i,
                                                     uint32_t filt, uint32_t offset, uint32_t n,
                                                     int32_t steps) {
  uint32_t k = i;
  double wk = (double)ws[i];
  const PhiloxLane pl = philox_lane(key, i, filt, offset);
  const int32_t groups = (steps + 3) / 4;
  for (int32_t m = 0; m < groups; ++m) {
    MGroup g;
    metropolis_fetch(ws, key, i, pl, filt, offset, n, steps, m, g);
    metropolis_accept<T>(g, k, wk);
  }
  return k;
}

// ------------------------------------------------------------------ bound table
// For a vector too long for LDS, an upper bound of the weights, one per bucket
// of S = 2^shift consecutive particles, lets most proposals be rejected
// without loading w_j: if u * w_k > ub >= w_j the step (or trial) rejects.
// The bound is a power of two, 2^(cM - 127 - c4): cM is the largest bucket
// code of the vector and c4 = min(15, cM - c) the 4-bit distance of the
// bucket's code c, where 2^(c - 127) >= the bucket maximum.  Two buckets per
// LDS byte: 128 KB cover 2^18 buckets.  The skip test compares the rounded
// product u * (a lower bound of w_k) with ub with a margin of 2^-20 relative,
// far above the product's rounding, so a skipped step is one that the exact
// test rejects; the output is the same.
constexpr int kTableBuckets = 1 << 18;  // nibbles in LDS (128 KB)
constexpr int kTableThreads = 1024;
constexpr int kCodeThreads = 256;

__device__ __forceinline__ uint32_t bound_code(float v) {
  const uint32_t b = __float_as_uint(v);
  return (b >> 23) + ((b & 0x7FFFFFu) != 0u);  // 0 .. 255 for finite v >= 0
}
__device__ __forceinline__ uint32_t bound_code(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const int e = (int)((b >> 52) & 0x7FF);
  if (e == 0) return 0u;  // zero or below 2^-1022
  const int c = e - 1023 + 127 + (((b & 0xFFFFFFFFFFFFFull) != 0ull) ? 1 : 0);
  return c < 0 ? 0u : (c > 255 ? 255u : (uint32_t)c);
}

// One thread per bucket: its 8-bit code; per workgroup the largest code.
// Invalid weights (negative, non-finite) give code 255, which disables the
// skips of the vector (the kernels then load every weight).
template <typename T>
__global__ __launch_bounds__(kCodeThreads) void k_bound_codes(const T* __restrict__ w, int64_t n,
                                                              int shift,
                                                              uint8_t* __restrict__ codes,
                                                              uint32_t* __restrict__ wg_max) {
  __shared__ uint32_t slot[kCodeThreads / kWave];
  const int64_t b = (int64_t)blockIdx.x * kCodeThreads + threadIdx.x;
  const int64_t S = (int64_t)1 << shift;
  uint32_t c = 0;
  if ((b << shift) < n) {
    const int64_t e = ((b + 1) << shift) < n ? ((b + 1) << shift) : n;
    for (int64_t k = b << shift; k < e; ++k) {
      const T v = w[k];
      const uint32_t ck = weight_ok(v) ? bound_code(v) : 255u;
      c = ck > c ? ck : c;
    }
    codes[b] = (uint8_t)c;
  }
  (void)S;
  c = wave_reduce(c, OpMax());
  if (lane_id() == 0) slot[threadIdx.x / kWave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t m = slot[0];
    for (int k = 1; k < kCodeThreads / kWave; ++k) m = slot[k] > m ? slot[k] : m;
    wg_max[blockIdx.x] = m;
  }
}

struct BoundTable {
  static constexpr bool kUsed = true;
  const uint8_t* nib;  // LDS, two 4-bit codes per byte
  int shift;
  // high word of the binary64 bound 2^(cM - 127) of the largest bucket, or
  // 0xFFFFFFFF when the table is unusable (no product exceeds it)
  uint32_t hi_top;
  // bucket b = j >> shift sits in byte b >> 1, low nibble for even b; the
  // nibble's bit offset 4 (b & 1) is bit `shift` of j moved to bit 2
  // (shift >= 2)
  __device__ __forceinline__ uint32_t c4(uint32_t j) const {
    return __builtin_amdgcn_ubfe((uint32_t)nib[j >> (shift + 1)], (j >> (shift - 2)) & 4u, 4u);
  }
  // true when u * lb > ub(j) = 2^(cM - 127 - c4), i.e. u * w_k > w_j for every
  // w_k >= lb.  The test reads only the high word of p = fl(u * lb) (the same
  // product the exact accept test forms): high(p) > high(ub) means
  // p >= ub (1 + 2^-20), and since p exceeds u * lb by at most a factor
  // 1 + 2^-53, u * lb > ub follows.  Adding c4 << 20 to high(p) instead of
  // subtracting it from the exponent of ub keeps the test to two integer
  // instructions; neither side wraps (high(p) < 2^31).
  __device__ __forceinline__ bool rejects(double u, double lb, uint32_t j) const {
    const uint32_t hp = (uint32_t)((uint64_t)__double_as_longlong(u * lb) >> 32);
    return hp + (c4(j) << 20) > hi_top;
  }
};

// The 4-bit table, packed once per call: every workgroup takes the largest
// code from the per-workgroup maxima of k_bound_codes, each thread packs 8
// codes into one word (the code array is padded to a multiple of 8; the
// padding is never looked up), and workgroup 0 stores the largest code.
constexpr int kPackThreads = 256;

__global__ __launch_bounds__(kPackThreads) void k_pack_table(const uint8_t* __restrict__ codes,
                                                             const uint32_t* __restrict__ wg_max,
                                                             uint32_t n_wg, uint32_t nb,
                                                             uint32_t* __restrict__ nib,
                                                             uint32_t* __restrict__ cm_out) {
  __shared__ uint32_t slot[kPackThreads / kWave];
  uint32_t m = 0;
  for (uint32_t k = threadIdx.x; k < n_wg; k += kPackThreads) m = wg_max[k] > m ? wg_max[k] : m;
  m = wave_reduce(m, OpMax());
  if (lane_id() == 0) slot[threadIdx.x / kWave] = m;
  __syncthreads();
  uint32_t cM = slot[0];
  for (int k = 1; k < kPackThreads / kWave; ++k) cM = slot[k] > cM ? slot[k] : cM;
  const uint32_t p = blockIdx.x * kPackThreads + threadIdx.x;
  if (8 * p < nb) {
    const uint2 v = reinterpret_cast<const uint2*>(codes)[p];
    uint32_t packed = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t c = ((q < 4 ? v.x : v.y) >> (8 * (q & 3))) & 0xFFu;
      const uint32_t d = c > cM ? 15u : (cM - c > 15u ? 15u : cM - c);
      packed |= d << (4 * q);
    }
    nib[p] = packed;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *cm_out = cM;
}

// The rejection table in one pass, without the vector's largest code: the
// distances are taken from c_ref, the code of the caller's w_max, which
// bounds every valid weight.  A bucket whose code reaches c_ref (or whose
// weights are invalid, code 255) gets distance 0, i.e. the bound
// 2^(c_ref - 127) >= w_max, which no trial's u * w_max exceeds: it is never
// skipped, and the exact test decides as without the table.  One thread per
// bucket; eight lanes OR their nibbles into one word, stored by the first.
template <typename T>
__global__ __launch_bounds__(kCodeThreads) void k_bound_nibbles(const T* __restrict__ w,
                                                                int64_t n, int shift, uint32_t nb,
                                                                uint32_t c_ref,
                                                                uint32_t* __restrict__ nib,
                                                                uint32_t* __restrict__ cm_out) {
  const int64_t b = (int64_t)blockIdx.x * kCodeThreads + threadIdx.x;
  uint32_t d = 0;
  if (b < (int64_t)nb) {
    const int64_t e = ((b + 1) << shift) < n ? ((b + 1) << shift) : n;
    uint32_t c = 0;
    for (int64_t k = b << shift; k < e; ++k) {
      const T v = w[k];
      const uint32_t ck = weight_ok(v) ? bound_code(v) : 255u;
      c = ck > c ? ck : c;
    }
    d = c >= c_ref ? 0u : (c_ref - c > 15u ? 15u : c_ref - c);
  }
  uint32_t word = d << (4 * (threadIdx.x & 7u));
  word |= __shfl_xor(word, 1);
  word |= __shfl_xor(word, 2);
  word |= __shfl_xor(word, 4);
  if ((threadIdx.x & 7u) == 0 && b < (int64_t)nb) nib[b >> 3] = word;
  if (blockIdx.x == 0 && threadIdx.x == 0) *cm_out = c_ref;
}

// Workgroup prologue: the packed table copied into LDS with 16-byte loads (the
// packed array is padded to a multiple of 16 bytes).
__device__ BoundTable load_bound_table(const uint32_t* __restrict__ nib_g,
                                       const uint32_t* __restrict__ cm, uint32_t nb, int shift,
                                       uint8_t* nib) {
  const uint32_t n4 = (nb + 31) / 32;  // 16-byte pieces (32 nibbles each)
  const uint4* __restrict__ src = reinterpret_cast<const uint4*>(nib_g);
  uint4* dst = reinterpret_cast<uint4*>(nib);
  for (uint32_t p = threadIdx.x; p < n4; p += blockDim.x) dst[p] = src[p];
  const uint32_t cM = *cm;
  __syncthreads();
  BoundTable t;
  t.nib = nib;
  t.shift = shift;
  // 2^(cM - 127) has binary64 exponent field cM - 127 + 1023 = cM + 896
  t.hi_top = cM < 255u ? (cM + 896u) << 20 : 0xFFFFFFFFu;
  return t;
}

// A bound per particle (or per 2 or 4 of them) in LDS, for a segment too long
// for its weights to be staged: 16 bits, twice what the 32-bit weights would
// leave room for.  The bound is the weight rounded up to 16 leading bits of
// its format (binary32: 7 fraction bits, binary64: 4), so nearly every
// proposal that it cannot reject is accepted, and the loads of w_j that are
// left are about the accepted moves.  Invalid weights never cause a skip that
// the exact test would not take (their code is the largest, or the comparison
// fails), so the result is the plain chain's for any input.  Measured on 256
// segments of 60000 binary32 weights against plain chains, whose gathers miss
// the L2: B = 354 294 -> 624 G steps/s, B = 16 281 -> 534.
constexpr uint32_t kCodes = 65536;  // 128 KB
constexpr uint32_t kCodesMaxShift = 2;
// Whether a workgroup's part of a segment pays for the segment's codes: its
// particles times the steps (or trials) of each must be a share of the n weights
// to be read.  That share is smaller where the chip is full (chunks of 5120 up:
// the plain gathers wait for one another, and the codes are staged many times
// over one another's chains) than where a workgroup runs alone; in batches small
// enough for one chain per thread the codes never paid.  Binary32 weights, plain /
// codes: 256 segments of 60000, 2 / 4 steps 144 / 131, 247 / 178 us; 64 of 262143,
// 4 / 12 / 16 steps 311 / 514, 807 / 882, 1010 / 1082; 6 of 100000, 16 / 30 / 60
// steps 43 / 49, 77 / 77, 147 / 135; 4 of 60000, 120 steps 109 / 139.
__device__ __forceinline__ bool codes_pay(int64_t chunk, int64_t part, uint32_t n, double each) {
  const double work = (double)part * each;
  return chunk > 1024 && work >= (chunk >= 5120 ? 0.4 : 1.0) * (double)n;
}
__device__ __forceinline__ uint32_t bound16(float v) {
  return (uint32_t)(((uint64_t)__float_as_uint(v) + 0xFFFFu) >> 16);  // -NaN: 0x10000, cut to 0xFFFF
}
__device__ __forceinline__ uint32_t bound16(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  return weight_ok(v) ? (uint32_t)((b + 0xFFFFFFFFFFFFull) >> 48) & 0x7FFFu : 0x7FF0u;
}

template <typename T>
struct CodeTable {
  static constexpr bool kUsed = true;
  const uint16_t* code;  // LDS
  uint32_t shift;        // particle j's bound is code[j >> shift]
  // True when p = fl(u w_k) shows u w_k > w_j: the high word of p (as a signed
  // number: a negative or zero p never rejects) exceeds that of the bound in
  // binary64, so p >= bound (1 + 2^-20), far above the rounding of p.
  __device__ __forceinline__ bool rejects(double u, double wk, uint32_t j) const {
    const uint32_t c = code[j >> shift];
    const int32_t hi = sizeof(T) == 4 ? (int32_t)((c << 13) + 0x38000000u) : (int32_t)(c << 16);
    return (int32_t)((uint64_t)__double_as_longlong(u * wk) >> 32) > hi;
  }
};

template <typename T>
__device__ __forceinline__ CodeTable<T> stage_codes(const T* __restrict__ w, uint32_t n,
                                                    uint16_t* code) {
  CodeTable<T> t{code, 0};
  while (((n - 1) >> t.shift) >= kCodes) ++t.shift;
  auto enc = [](T v) -> uint32_t {
    const uint32_t c = bound16(v);
    return c > 0xFFFFu ? 0xFFFFu : c;
  };
  if (t.shift == 0) {
#pragma unroll 4
    for (uint32_t q = threadIdx.x; q < n / 4; q += blockDim.x) {
      const Weights4<T> x = load_weights4(w + 4 * q);
      reinterpret_cast<uint2*>(code)[q] =
          make_uint2(enc(x.v[0]) | (enc(x.v[1]) << 16), enc(x.v[2]) | (enc(x.v[3]) << 16));
    }
    if (threadIdx.x < (n & 3u)) {
      const uint32_t j = (n & ~3u) + threadIdx.x;
      code[j] = (uint16_t)enc(w[j]);
    }
  } else {  // two or four weights a code
    const bool four = t.shift == 2;
    auto put = [&](uint32_t q, uint32_t a, uint32_t b) {
      if (four) code[q] = (uint16_t)max(a, b);
      else reinterpret_cast<uint32_t*>(code)[q] = a | (b << 16);
    };
#pragma unroll 4
    for (uint32_t q = threadIdx.x; q < n / 4; q += blockDim.x) {
      const Weights4<T> x = load_weights4(w + 4 * q);
      put(q, max(enc(x.v[0]), enc(x.v[1])), max(enc(x.v[2]), enc(x.v[3])));
    }
    if (threadIdx.x == 0 && (n & 3u)) {
      uint32_t c[4] = {0, 0, 0, 0};
      for (uint32_t k = 0; k < (n & 3u); ++k) c[k] = enc(w[(n & ~3u) + k]);
      put(n / 4, max(c[0], c[1]), max(c[2], c[3]));
    }
  }
  return t;
}

// The waves of a SIMD issue oldest first, so that of equal chains the oldest
// wave's ends long before the others', which are then too few to fill the
// SIMD (one wave in four ended at 58 % of the workgroup's time).  A wave
// therefore lowers its priority with each quarter of its chain: those behind
// go first, and all stay within a quarter.  2^20 weights, B = 354: 610 -> 586
// us.  (Later steps, at 3/4, 15/16 and 63/64 of the chain: 605.)
struct ChainPriority {
  int32_t q;
  __device__ __forceinline__ explicit ChainPriority(int32_t B) : q((B + 15) / 16) {
    __builtin_amdgcn_s_setprio(3);
  }
  __device__ __forceinline__ void step(int32_t m) const {  // m: groups of four steps done
    if (m == q) __builtin_amdgcn_s_setprio(2);
    else if (m == 2 * q) __builtin_amdgcn_s_setprio(1);
    else if (m == 3 * q) __builtin_amdgcn_s_setprio(0);
  }
};

// Metropolis with a bound table.  A skip needs the exact current w_k, so
// the gathers cannot be issued ahead of the decisions of earlier steps;
// instead each lane runs K independent chains in lockstep: at every step the
// chains whose proposal the table cannot reject issue their loads together
// and the K decisions follow.  Lane l runs the particles ib + c STRIDE,
// c < K, below i1, of the segment of n weights ws (wv: its buffer view).
template <typename T, int K, int STRIDE, typename Table>
__device__ __forceinline__ void metropolis_lockstep(const T* __restrict__ ws,
                                                    __amdgpu_buffer_rsrc_t wv, uint32_t n,
                                                    int32_t B, Key key, uint32_t filter,
                                                    uint32_t offset, const Table& tab,
                                                    uint32_t ib, uint32_t i1,
                                                    int32_t* __restrict__ as) {
  if (ib >= i1) return;
  uint32_t k[K];
  double wk[K];
  PhiloxLane pl[K];
#pragma unroll
  for (int c = 0; c < K; ++c) {
    // a dead chain (past the end) runs a copy of the lane's first and is not stored
    const uint32_t i = ib + c * STRIDE;
    k[c] = i < i1 ? i : ib;
    wk[c] = (double)ws[k[c]];
    pl[c] = philox_lane(key, k[c], filter, offset);
  }
  ChainPriority prio(B);
  for (int32_t m = 0; 4 * m < B; ++m) {
    prio.step(m);
    const int32_t left = B - 4 * m;
    const int ncall = left >= 4 ? 3 : (3 * left + 3) / 4;
    const int nq = left >= 4 ? 4 : left;
    uint32_t x[K][12];
#pragma unroll
    for (int c = 0; c < K; ++c) {
#pragma unroll
      for (int c3 = 0; c3 < 3; ++c3) {
        if (c3 < ncall) {
          // step, filter and offset are the same on every lane (one segment)
          const uint4 v =
              philox_lane_call(pl[c], key, DOM_TRIAL, (uint32_t)(3 * m + c3), filter, offset);
          x[c][4 * c3 + 0] = v.x;
          x[c][4 * c3 + 1] = v.y;
          x[c][4 * c3 + 2] = v.z;
          x[c][4 * c3 + 3] = v.w;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q < nq) {
        uint32_t j[K];
        double u[K], v[K];
        bool need[K];
        T raw[K];
#pragma unroll
        for (int c = 0; c < K; ++c) {
          j[c] = index_draw(x[c][3 * q], x[c][3 * q + 1], n);
          u[c] = u_accept(x[c][3 * q + 2]);
          need[c] = !tab.rejects(u[c], wk[c], j[c]);
        }
        // the K gathers go out together (the scheduler, left to itself, may wait
        // for the first before the second: 256 segments of 60000, 100 steps, 1870
        // -> 2045 us); lanes with nothing to load read zero
#pragma unroll
        for (int c = 0; c < K; ++c)
          raw[c] = buffer_gather<T>(wv, need[c] ? j[c] * (uint32_t)sizeof(T) : kNoLoad);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < K; ++c) v[c] = (double)raw[c];
#pragma unroll
        for (int c = 0; c < K; ++c) {
          // selects, not a branch: the gathered value is used on every lane,
          // so the gathers cannot be sunk into per-chain branches
          const bool acc = need[c] & accept_exact<T>(u[c], wk[c], v[c]);
          k[c] = acc ? j[c] : k[c];
          wk[c] = acc ? v[c] : wk[c];
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < K; ++c)
    if (ib + c * STRIDE < i1) as[ib + c * STRIDE] = (int32_t)k[c];
}

template <typename T, int K>
__global__ __launch_bounds__(kTableThreads) void k_metropolis_table(
    const T* __restrict__ w, int64_t n, int32_t B, Key key, uint32_t offset, uint32_t filter,
    int32_t* __restrict__ a, int64_t chunk, const uint32_t* __restrict__ nib_g,
    const uint32_t* __restrict__ cm, uint32_t nb, int shift) {
  __shared__ __align__(16) uint8_t nib[kTableBuckets / 2];
  offset = counter_offset(key, offset);
  const BoundTable tab = load_bound_table(nib_g, cm, nb, shift, nib);
  // n * sizeof(T) < 2^31 (checked by the launcher)
  const __amdgpu_buffer_rsrc_t wv = buffer_view(w, (uint32_t)(n * (int64_t)sizeof(T)));
  const int64_t p0 = (int64_t)blockIdx.x * chunk;
  const int64_t p1 = p0 + chunk < n ? p0 + chunk : n;
  for (int64_t g = p0; g < p1; g += (int64_t)K * kTableThreads) {
    const uint32_t i = (uint32_t)g + threadIdx.x;
    // a remainder of one or two chains a lane runs those alone (B = 354, us:
    // 2^20 + 1 particles 1543 -> 1429, 2^20 + 2^17 2126 -> 1883, 1.5 M
    // 3417 -> 2834)
    if (K > 1 && p1 - g <= kTableThreads)
      metropolis_lockstep<T, 1, kTableThreads>(w, wv, (uint32_t)n, B, key, filter, offset, tab, i,
                                               (uint32_t)p1, a);
    else if (K > 2 && p1 - g <= 2 * kTableThreads)
      metropolis_lockstep<T, 2, kTableThreads>(w, wv, (uint32_t)n, B, key, filter, offset, tab, i,
                                               (uint32_t)p1, a);
    else
      metropolis_lockstep<T, K, kTableThreads>(w, wv, (uint32_t)n, B, key, filter, offset, tab, i,
                                               (uint32_t)p1, a);
  }
}

// ------------------------------------------------------------------ staged Metropolis
// Workgroups go to the eight XCDs in turn, each with its own L2.  Chunk index
// of a workgroup such that runs of about 65536 particles (whole segments, in a
// batch) stay on one XCD: their weights are then read from its L2, where
// chunks dealt out one by one would keep a copy of every segment in flight in
// all eight.
__device__ __forceinline__ int64_t xcd_chunk(int64_t chunk, uint32_t b, uint32_t chunks) {
  const uint32_t G = (uint32_t)max((int64_t)1, 65536 / chunk);
  const uint32_t s0 = b - b % (8 * G);
  if (s0 + 8 * G > chunks) return b;  // the last, partial group of runs
  const uint32_t r = b - s0;
  return s0 + (r & 7u) * G + (r >> 3);
}

// A queue of chunks for workgroups that stay on their CU and take the next
// chunk when they are done with one: a launch of a workgroup per chunk hands
// them out in order, and with one or two workgroups to a CU a free CU may wait.
// Eight heads, one per XCD, in lines of their own; a workgroup serves the
// chunks of its XCD's head (t % 8, so that xcd_chunk keeps its runs together)
// and then those of the others.  Every workgroup ends when all eight are used
// up.  Up to kQueueFilters segments: with more of them the shares even out by
// themselves, and the cost prefix is longer (16384 segments of 64 .. 512, fewer
// than 8 / 60 / 200 steps: without 106 / 356 / 985 us, with 121 / 363 / 939;
// 8192 of 512 .. 2048 106 / 418 / 1220 and 124 / 461 / 1397; 4096 of 128 .. 4096
// 72 / 268 / 806 and 72 / 248 / 660).  4096 ragged vectors of 256 .. 65536, B = 4 .. 354, with the
// permutation: 4.25 -> 3.94 ms; with the waves of a workgroup taking 64 chains
// at a time instead of a fixed share, 3.70; with chunks twice as long, 3.47.
constexpr uint32_t kHeadStride = 32;
constexpr size_t kQueueBytes = 8 * kHeadStride * sizeof(uint32_t);
constexpr uint32_t kQueueFilters = 4096;
struct ChunkQueue {
  uint32_t* heads;
  uint32_t chunks;
};
// The next chunk, the same on every thread, or at least q.chunks at the end.
// The first is the workgroup's own number (gridDim.x is at most q.chunks, and a
// multiple of 8 when it is less); the heads count those beyond.  Eight lanes look
// at all heads at once, so that the end, when nothing is left, costs one load
// and not an atomic per head (64 segments of 4096, which have a workgroup per
// chunk and no queue to look at: 21 -> 16 us).
__device__ __forceinline__ uint32_t next_chunk(const ChunkQueue& q, bool first, uint32_t* slot) {
  if (first) return blockIdx.x;
  if (gridDim.x >= q.chunks) return q.chunks;
  __syncthreads();  // the last chunk's number has been read, and its LDS
  if (threadIdx.x < kWave) {
    const uint32_t lane = lane_id(), x = (blockIdx.x + lane) & 7u;  // its own XCD's first
    uint32_t t = q.chunks;
    while (true) {
      uint32_t c = 0;
      if (lane < 8)
        c = __hip_atomic_load(q.heads + x * kHeadStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint64_t some = ballot(lane < 8 && gridDim.x + c * 8u + x < q.chunks);
      if (some == 0) break;  // (heads only grow: nothing will come)
      const uint32_t pick = (blockIdx.x + (uint32_t)__ffsll((long long)some) - 1u) & 7u;
      if (lane == 0) c = atomicAdd(q.heads + pick * kHeadStride, 1u);
      t = gridDim.x + uniform_u32(c) * 8u + pick;
      if (t < q.chunks) break;
      t = q.chunks;
    }
    if (lane == 0) *slot = t;
  }
  __syncthreads();
  return uniform_u32(*slot);
}

// A batch whose segments have their own step counts is cut by cost instead of
// by particles: chunk t starts where the cost prefix, a segment's particles
// times its steps (and two for the rest), reaches t / gridDim of the total,
// rounded to whole passes of the workgroup.  Equal chunks leave the chip
// waiting for the last ones of B = 354 (4096 ragged vectors
// of 256 .. 65536 particles, B = 4 .. 354: 4.94 against 3.87 ms).
// One workgroup, four segments per thread and round; bound by the latency of
// its rounds (4096 segments: one per thread and round 10 us, four 4).
__global__ __launch_bounds__(1024) void k_cost_prefix(const int64_t* __restrict__ offsets,
                                                      uint32_t n_filters,
                                                      const int32_t* __restrict__ B,
                                                      uint64_t* __restrict__ cost,
                                                      uint32_t* __restrict__ heads) {
  constexpr int kF = 4;
  if (threadIdx.x < 8) heads[threadIdx.x * kHeadStride] = 0;
  __shared__ uint64_t s_w[1024 / kWave];
  const uint32_t wave = threadIdx.x / kWave, lane = lane_id();
  uint64_t carry = 0;
  for (uint32_t f0 = kF * threadIdx.x; f0 - kF * threadIdx.x < n_filters; f0 += kF * 1024) {
    int64_t o[kF + 1];
    int32_t b[kF];
#pragma unroll
    for (int k = 0; k <= kF; ++k) o[k] = offsets[min(f0 + k, n_filters)];
#pragma unroll
    for (int k = 0; k < kF; ++k) b[k] = B[min(f0 + k, n_filters - 1)];
    uint64_t x[kF], sum = 0;
#pragma unroll
    for (int k = 0; k < kF; ++k) {  // (no particles past the end)
      x[k] = sum;
      sum += (uint64_t)(o[k + 1] - o[k]) * ((uint64_t)max(b[k], 0) + 2);
    }
    const uint64_t incl = wave_incl_add_u64(sum);
    if (lane == kWave - 1) s_w[wave] = incl;
    __syncthreads();
    uint64_t before = carry + incl - sum;
#pragma unroll
    for (uint32_t w2 = 0; w2 < 1024 / kWave; ++w2) {
      const uint64_t t = s_w[w2];
      before += w2 < wave ? t : 0ull;
      carry += t;
    }
#pragma unroll
    for (int k = 0; k < kF; ++k)
      if (f0 + k < n_filters) cost[f0 + k] = before + x[k];
    __syncthreads();
  }
  if (threadIdx.x == 0) cost[n_filters] = carry;
}

// First particle of chunk t of `chunks` (whole waves call it).
__device__ __forceinline__ int64_t cost_start(const uint64_t* __restrict__ cost,
                                              const int64_t* __restrict__ offsets,
                                              uint32_t n_filters, int64_t n_total, uint32_t t,
                                              uint32_t chunks, uint32_t cap) {
  if (t == 0) return 0;
  if (t >= chunks) return n_total;
  const uint64_t total = cost[n_filters], q = total / chunks, r = total % chunks;
  const uint64_t target = q * t + r * t / chunks;
  const uint32_t f = wave_find_segment(cost, n_filters, target);
  const uint64_t n = (uint64_t)(offsets[f + 1] - offsets[f]);
  const uint64_t span = cost[f + 1] - cost[f];
  // (of equal prefixes the last is found: f's cost is positive unless no cost follows)
  uint64_t i = span ? (target - cost[f]) / (span / n) : 0ull;
  const uint64_t unit = n > cap ? 2048 : 1024;
  i = (i + unit / 2) / unit * unit;
  return offsets[f] + (int64_t)(i < n ? i : n);
}

// Chains of one vector that gather from global memory (chunk particles per
// workgroup), the gathers of the next group of steps in flight while the
// current group is decided.  Bound by the gathers' latency in short vectors and
// their rate in long ones; without the batches' segments, queue and cost cuts
// it keeps eight waves per SIMD (2^18 binary32 weights, 1 / 8 steps: 7.4 / 17.4
// us, as a case of the batch kernel 9.1 / 18.7).
template <typename T>
__global__ __launch_bounds__(256) void k_metropolis_global(const T* __restrict__ w, int64_t n_total,
                                                           int32_t B,
                                                           const int32_t* __restrict__ B_dev,
                                                           Key key, uint32_t offset, uint32_t filt,
                                                           int32_t* __restrict__ a,
                                                           int64_t chunk) {
  offset = counter_offset(key, offset);
  const int64_t p0 = (int64_t)blockIdx.x * chunk;
  const int64_t p1 = p0 + chunk < n_total ? p0 + chunk : n_total;
  const uint32_t n = (uint32_t)n_total;
  const int32_t steps = B_dev ? B_dev[0] : B;
  const int32_t groups = (steps + 3) / 4;
  for (int64_t g = p0 + threadIdx.x; g < p1; g += 256) {
    const uint32_t i = (uint32_t)g;
    uint32_t k = i;
    double wk = (double)w[i];
    const PhiloxLane pl = philox_lane(key, i, filt, offset);
    MGroup ga, gb;
    if (groups > 0) metropolis_fetch(w, key, i, pl, filt, offset, n, steps, 0, ga);
    for (int32_t m = 0; m < groups; m += 2) {
      if (m + 1 < groups) metropolis_fetch(w, key, i, pl, filt, offset, n, steps, m + 1, gb);
      metropolis_accept<T>(ga, k, wk);
      if (m + 2 < groups) metropolis_fetch(w, key, i, pl, filt, offset, n, steps, m + 2, ga);
      if (m + 1 < groups) metropolis_accept<T>(gb, k, wk);
    }
    a[g] = (int32_t)k;
  }
}

// QUEUED: a batch cut by cost, chunks from the queue; else chunk blockIdx.x.
// Where the LDS holds two workgroups of 1024 threads, the registers have to as
// well: eight waves per SIMD.  With the queue's scalars in every form it was
// seven, and one workgroup (4096 segments of 256, 16 / 100 steps: 109 / 513 us,
// with two 73 / 329).  The workgroups of 256 threads, a wave per SIMD, keep the
// registers that the chain alone would have, and in binary32 a plain loop (one
// vector of 16384, 354 steps: in shares 62.7 us, so 58.4; of 4097 in binary64
// 64.7 and 66.2).
template <typename T, int CAP, int THREADS, bool QUEUED>
__global__ __launch_bounds__(THREADS, THREADS > 256 && CAP * sizeof(T) <= 65536 ? 8 : 1)
void k_metropolis_staged(
    const T* __restrict__ w, int64_t n_total, const int64_t* __restrict__ offsets,
    uint32_t n_filters, int32_t B, const int32_t* __restrict__ B_dev, Key key, uint32_t offset,
    uint32_t filter_base, int32_t* __restrict__ a, int64_t chunk,
    const uint64_t* __restrict__ cost, ChunkQueue queue) {
  // 128 KB of weights, or 65536 codes of a segment longer than that
  constexpr bool kCoded = THREADS == 1024 && CAP * sizeof(T) == 2 * kCodes;
  __shared__ __align__(16) T sw[CAP];
  offset = counter_offset(key, offset);
  __shared__ uint32_t s_chunk, s_next;
  // particles of the segment part that are left go to the waves as they get
  // free, 64 chains (or 128) at a time: the first index of the wave's share, at
  // least the part's length at the end.  (Workgroups of 256 threads, and parts of
  // at most a chain per thread, have nothing to hand out: the shares in order
  // keep short segments' waves even over the SIMDs.)
  constexpr bool kTakes = THREADS > 256;
  auto take = [&](uint32_t chains) -> uint32_t {
    uint32_t old = 0;
    if (lane_id() == 0) old = atomicAdd(&s_next, chains);
    return uniform_u32(old);
  };
  for (bool first = true;; first = false) {
    const uint32_t b = QUEUED ? next_chunk(queue, first, &s_chunk) : blockIdx.x;
    if (b >= queue.chunks) break;
    const int64_t t = offsets ? xcd_chunk(chunk, b, queue.chunks) : (int64_t)b;
    int64_t p0 = t * chunk, p1 = p0 + chunk < n_total ? p0 + chunk : n_total;
    if (QUEUED) {
      p0 = cost_start(cost, offsets, n_filters, n_total, (uint32_t)t, queue.chunks, CAP);
      p1 = cost_start(cost, offsets, n_filters, n_total, (uint32_t)t + 1, queue.chunks, CAP);
    }
    uint32_t f = offsets && p0 < p1 ? wave_find_segment(offsets, n_filters, p0) : 0u;
    for (int64_t g0 = p0; g0 < p1; ++f) {
      const int64_t base = offsets ? offsets[f] : 0;
      const int64_t end = offsets ? offsets[f + 1] : n_total;
      const int64_t q1 = end < p1 ? end : p1;
      if (q1 <= g0) continue;  // empty segment
      const uint32_t n = (uint32_t)(end - base);
      const int32_t steps = B_dev ? B_dev[f] : B;
      const uint32_t filt = filter_base + f;
      if (n <= (uint32_t)CAP) {
        __syncthreads();  // the previous segment's chains are done with sw
        const uint32_t len = (uint32_t)(q1 - g0), i0 = (uint32_t)(g0 - base);
        const bool shares = kTakes && len > (uint32_t)THREADS;
        if (shares && threadIdx.x == 0) s_next = 0;
        stage_weights(w + base, n, sw);
        __syncthreads();
        if constexpr (!kTakes && sizeof(T) == 4) {
          for (uint32_t k = threadIdx.x; k < len; k += THREADS)
            a[g0 + k] = (int32_t)metropolis_chain(sw, key, i0 + k, filt, offset, n, steps);
        } else {
          uint32_t k0 = shares ? take(kWave) : uniform_u32(threadIdx.x & ~(uint32_t)(kWave - 1));
          while (k0 < len) {
            const uint32_t k = k0 + lane_id();
            if (k < len)
              a[g0 + k] = (int32_t)metropolis_chain(sw, key, i0 + k, filt, offset, n, steps);
            k0 = shares ? take(kWave) : k0 + THREADS;
          }
        }
      } else if (kCoded && n <= kCodes << kCodesMaxShift &&
                 codes_pay(chunk, q1 - g0, n, (double)steps)) {
        uint16_t* const code = reinterpret_cast<uint16_t*>(sw);
        __syncthreads();
        if (threadIdx.x == 0) s_next = 0;
        const CodeTable<T> tab = stage_codes(w + base, n, code);
        __syncthreads();
        const __amdgpu_buffer_rsrc_t wv = buffer_view(w + base, n * (uint32_t)sizeof(T));
        const uint32_t i0 = (uint32_t)(g0 - base), i1 = (uint32_t)(q1 - base);
        // two chains a lane, or one for the last
        for (uint32_t k, taken = 0; taken < i1 - i0;) {
          const bool two = i1 - i0 - taken > 2 * kWave;
          k = take(two ? 2 * kWave : kWave);
          taken = k + (two ? 2 * kWave : kWave);
          if (two)
            metropolis_lockstep<T, 2, kWave>(w + base, wv, n, steps, key, filt, offset, tab,
                                             i0 + k + lane_id(), i1, a + base);
          else
            metropolis_lockstep<T, 1, kWave>(w + base, wv, n, steps, key, filt, offset, tab,
                                             i0 + k + lane_id(), i1, a + base);
        }
      } else {  // a longer segment in a staged launch: plain chains
        for (int64_t g = g0 + threadIdx.x; g < q1; g += THREADS)
          a[g] = (int32_t)metropolis_chain(w + base, key, (uint32_t)(g - base), filt, offset, n,
                                           steps);
      }
      g0 = q1;
    }
    if (!QUEUED) break;
  }
}

// ------------------------------------------------------------------ rejection
// Particle i: trial 0 proposes j = i; trial t >= 1 proposes j from Philox
// counter (i, TRIAL<<28 | t, filter, offset); every trial takes its u from the
// same block.  The first trial with u * w_max <= w_j wins.  After max_trials
// rejections the particle keeps a_i = i and FLAG_TRIAL_CAP is raised.
//
// Scheduling (the variable task-length problem of the paper's section 2.2):
// the waves of a workgroup hand out its particles among themselves through an
// LDS counter, a wave taking as many as it has free lanes, so that none runs
// out of work while another still holds a long range.  When the particles are
// used up, those still running in a wave share all its lanes: compacted to the
// first m lanes, each gets 64 / m lanes (shares that differ by at most one) that
// try consecutive trials of it at once, and the lowest accepting trial wins.
// That is the same answer as trying the trials one by one, so the output does
// not depend on the schedule, and the slowest particle of a wave does not run
// alone on one lane.
constexpr int kRejBatch = 4;  // trials per lane and pass while acceptance is rare
constexpr uint32_t kNoParticle = 0xFFFFFFFFu;

// No bound table: every weight is read (from LDS, or from global memory).
struct NoTable {
  static constexpr bool kUsed = false;
};

// Trials t .. t + NQ - 1 of particle i: true when one accepts, j the lowest
// accepting one's proposal.  The draws, then the table checks, then the weight
// loads together, then the decisions: one wait per pass.  With a table, a
// trial that needs no load reads nothing (an out-of-range buffer offset).
// TINY: the bound may lie below 2^-900, where a difference can round to zero
// (accept_exact); elsewhere one fused multiply-add decides.
template <int NQ, bool TINY, typename T, typename Table>
__device__ __forceinline__ bool rejection_try(const T* ws, __amdgpu_buffer_rsrc_t wv, uint32_t i,
                                              uint32_t t, uint32_t n, uint32_t filt, double wmax,
                                              uint32_t max_trials, Key key, uint32_t offset,
                                              const Table& tab, uint32_t& j) {
  const uint32_t left = t < max_trials ? max_trials - t : 0u;
  uint32_t jq[NQ];
  double uq[NQ], vq[NQ];
  bool live[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const uint4 x = draw(key, i, DOM_TRIAL, t + (uint32_t)q, filt, offset);
    jq[q] = index_draw(x.x, x.y, n);
    if (q == 0) jq[q] = t == 0 ? i : jq[q];
    uq[q] = u_accept(x.z);
    live[q] = (uint32_t)q < left;
    if constexpr (Table::kUsed) live[q] = live[q] & !tab.rejects(uq[q], wmax, jq[q]);
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    if constexpr (Table::kUsed)
      vq[q] = (double)buffer_gather<T>(wv, live[q] ? jq[q] * (uint32_t)sizeof(T) : kNoLoad);
    else
      vq[q] = (double)ws[jq[q]];
  }
  bool any = false;
#pragma unroll
  for (int q = NQ - 1; q >= 0; --q) {
    const bool acc =
        live[q] & (TINY ? accept_exact<double>(uq[q], wmax, vq[q])
                        : __fma_rn(uq[q], wmax, -vq[q]) <= 0.0);
    j = acc ? jq[q] : j;
    any |= acc;
  }
  return any;
}

// floor(x / m) = x kShareMagic[m] >> 18 for x <= 4095, m <= 64 (x m < 2^18)
struct ShareMagic {
  uint32_t v[kWave + 1];
};
constexpr ShareMagic share_magic() {
  ShareMagic s{};
  for (uint32_t m = 1; m <= kWave; ++m) s.v[m] = (1u << 18) / m + 1u;
  return s;
}
static __constant__ const ShareMagic kShare = share_magic();

// One wave works through the particles [i0, i1) (local indices) of one segment
// (weights ws, length n, filter id filt, output as) together with the other
// waves of its workgroup (queue: the LDS counter, 0 at the start).  VALU bound,
// mostly by Philox, where acceptance is rare: 1024 vectors of 16000 binary32
// weights at 1.8 % acceptance 621 G trials/s (2.04 ms), 467 with per-trial
// conditions on the pass's length, the exact test's underflow branch and
// 64-bit particle indices; at 70 %, where a pass is one trial and the queue,
// 94 us against 176.  Even lane shares in the tail (64 / m, not its floor, and
// no search for the m-th running lane) took 4096 vectors of 4000 from 3.16 to
// 2.26 ms.
template <bool TINY, typename T, typename Table>
__device__ void rejection_wave_range(const T* ws, __amdgpu_buffer_rsrc_t wv, uint32_t n,
                                     uint32_t filt, double wmax, uint32_t i0, uint32_t i1,
                                     uint32_t max_trials, Key key, uint32_t offset,
                                     int32_t* __restrict__ as, uint32_t& my_flags,
                                     const Table& tab, uint32_t* queue) {
  const uint32_t lane = lane_id();
  const uint32_t len = i1 - i0;
  uint32_t cur = kNoParticle;  // the particle this lane works on
  uint32_t t = 0;              // its next trial
  uint64_t tried = 0, accepted = 0;  // wave-uniform counts
  auto rank_in = [](uint64_t mask) -> uint32_t {  // set bits below this lane
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
  };
  auto give_up = [&]() {  // the trial cap: the particle keeps its own index
    as[cur] = (int32_t)cur;
    my_flags |= FLAG_TRIAL_CAP;
    cur = kNoParticle;
  };

  // main phase.  Each pass tries NQ trials of every lane's particle: 4 while
  // the wave's acceptance rate so far is below 1/2 (long runs of rejections,
  // where four trials share one pass's overhead), else 1 (further trials would
  // be wasted draws and loads).  The results do not depend on it.
  while (true) {
    const uint64_t freem = ballot(cur == kNoParticle);
    if (freem != 0) {
      uint32_t old = 0;
      if (lane == 0) old = atomicAdd(queue, (uint32_t)__popcll(freem));
      const uint32_t next = uniform_u32(old);
      const uint32_t mine = next + rank_in(freem);
      if (cur == kNoParticle && mine < len) {
        cur = i0 + mine;
        t = 0;
      }
      if (next + (uint32_t)__popcll(freem) >= len) break;  // used up for every wave
    }
    bool won = false;
    if (accepted * 2u < tried) {
      uint32_t j = 0;
      won = rejection_try<kRejBatch, TINY>(ws, wv, cur, t, n, filt, wmax, max_trials, key, offset,
                                           tab, j);
      if (won) as[cur] = (int32_t)j;
      t += kRejBatch;
      tried += (uint64_t)kRejBatch * kWave;
    } else {
      uint32_t j = 0;
      won = rejection_try<1, TINY>(ws, wv, cur, t, n, filt, wmax, max_trials, key, offset, tab, j);
      if (won) as[cur] = (int32_t)j;
      t += 1;
      tried += kWave;
    }
    accepted += (uint64_t)__popcll(ballot(won));
    if (won) cur = kNoParticle;
    else if (t >= max_trials) give_up();
  }

  // tail phase (the counts go on: the tail is all there is when the range is
  // shorter than a wave)
  while (true) {
    const uint64_t act = ballot(cur != kNoParticle);
    if (act == 0) break;
    const uint32_t m = (uint32_t)__popcll(act);
    // the particles left move to lanes 0 .. m - 1
    const uint32_t rank = rank_in(act);
    const uint32_t to = cur != kNoParticle ? rank : m + (lane - rank);
    cur = (uint32_t)__builtin_amdgcn_ds_permute((int)(to << 2), (int)cur);
    t = (uint32_t)__builtin_amdgcn_ds_permute((int)(to << 2), (int)t);
    // lane l helps particle g = floor(l m / 64); particle g's helpers start at
    // ceil(64 g / m)
    const uint32_t magic = kShare.v[m];
    auto start = [&](uint32_t g) -> uint32_t {
      return g >= m ? (uint32_t)kWave : ((64u * g + m - 1u) * magic) >> 18;
    };
    const uint32_t g = (lane * m) >> 6;
    const uint32_t oi = shfl_u32(cur, (int)g), ot = shfl_u32(t, (int)g);
    const uint32_t s_own = start(lane), e_own = start(lane + 1u);
    const uint32_t r = lane - start(g);
    uint32_t j = 0, batch;
    bool acc;
    if (accepted * 2u < tried) {
      batch = kRejBatch;
      acc = rejection_try<kRejBatch, TINY>(ws, wv, oi, ot + batch * r, n, filt, wmax, max_trials,
                                           key, offset, tab, j);
    } else {
      batch = 1;
      acc = rejection_try<1, TINY>(ws, wv, oi, ot + r, n, filt, wmax, max_trials, key, offset,
                                   tab, j);
    }
    const uint64_t accm = ballot(acc);
    const uint32_t size = e_own - s_own;  // helpers of this lane's own particle
    uint64_t mine = 0;
    if (cur != kNoParticle)
      mine = accm & ((size >= kWave ? ~0ull : ((1ull << size) - 1ull)) << s_own);
    const int src = mine ? __ffsll((long long)mine) - 1 : (int)lane;
    const uint32_t jw = shfl_u32(j, src);
    const bool won = mine != 0;
    if (won) {
      as[cur] = (int32_t)jw;
      cur = kNoParticle;
    } else if (cur != kNoParticle) {
      t += batch * size;
      if (t >= max_trials) give_up();
    }
    tried += (uint64_t)batch * kWave;
    accepted += (uint64_t)__popcll(ballot(won));
  }
}

// Trials per particle to expect of the particles [i0, i1) of a segment, from
// the first trials of as many as the workgroup has threads.
template <typename T>
__device__ __forceinline__ double mean_trials(const T* __restrict__ w, uint32_t i0, uint32_t i1,
                                              uint32_t filt, double wmax, Key key,
                                              uint32_t offset) {
  const uint32_t i = i0 + threadIdx.x;
  const bool in = i < i1;
  const uint4 x = draw(key, i, DOM_TRIAL, 0, filt, offset);
  const int won = __syncthreads_count(in && u_accept(x.z) * wmax <= (double)w[in ? i : i0]);
  return (double)min(i1 - i0, blockDim.x) / (double)max(won, 1);
}

// A workgroup takes the particles [p0, p1) and walks the segments that overlap
// them; the waves hand out each segment part among themselves (an LDS
// counter reset between the part's barriers).  A segment of at most CAP
// weights is first copied into LDS, of a longer one its bound codes where they
// pay for it (256 vectors of 60000 binary32 weights at 1.3 % acceptance: 4.3 ms
// with gathers from global memory, 2.1 ms with codes; at 71 %: 91 and 112 us).
// The chunks go to the XCDs in runs
// that share a segment (xcd_chunk).
template <typename T, int CAP, int THREADS>
__global__ __launch_bounds__(THREADS) void k_rejection(
    const T* __restrict__ w, int64_t n_total, const int64_t* __restrict__ offsets,
    uint32_t n_filters, double w_max, const double* __restrict__ w_max_dev, uint32_t max_trials,
    Key key, uint32_t offset, uint32_t filter_base, int32_t* __restrict__ a,
    uint32_t* __restrict__ flags, int64_t chunk) {
  constexpr bool kCoded = THREADS == 1024 && CAP * sizeof(T) == 2 * kCodes;
  __shared__ __align__(16) T sw[CAP > 0 ? CAP : 1];
  __shared__ uint32_t queue;  // particles of the segment part handed out so far
  offset = counter_offset(key, offset);
  const int64_t p0 =
      (offsets ? xcd_chunk(chunk, blockIdx.x, gridDim.x) : (int64_t)blockIdx.x) * chunk;
  const int64_t p1 = p0 + chunk < n_total ? p0 + chunk : n_total;
  uint32_t my_flags = 0;
  uint32_t f = offsets ? wave_find_segment(offsets, n_filters, p0) : 0u;
  for (int64_t g0 = p0; g0 < p1; ++f) {
    const int64_t base = offsets ? offsets[f] : 0;
    const int64_t end = offsets ? offsets[f + 1] : n_total;
    const int64_t q1 = end < p1 ? end : p1;
    if (q1 <= g0) continue;  // empty segment
    const uint32_t n = (uint32_t)(end - base);
    const double wmax = w_max_dev ? w_max_dev[f] : w_max;
    const bool tiny = !(wmax >= 0x1p-900);
    const uint32_t i0 = (uint32_t)(g0 - base), i1 = (uint32_t)(q1 - base);
    const T* __restrict__ wf = w + base;
    int32_t* __restrict__ af = a + base;
    const uint32_t filt = filter_base + f;
    const __amdgpu_buffer_rsrc_t none = buffer_view(wf, 0u);
    __syncthreads();  // the previous part's trials are done with sw and the queue
    if (threadIdx.x == 0) queue = 0;
    if (CAP > 0 && !tiny && n <= (uint32_t)CAP) {
      stage_weights(wf, n, sw);
      __syncthreads();
      rejection_wave_range<false>((const T*)sw, none, n, filt, wmax, i0, i1, max_trials, key,
                                  offset, af, my_flags, NoTable{}, &queue);
    } else if (kCoded && !tiny && wmax <= 0x1p127 && n <= kCodes << kCodesMaxShift &&
               codes_pay(chunk, i1 - i0, n, mean_trials(wf, i0, i1, filt, wmax, key, offset))) {
      // (a product beyond binary32's range could exceed the code of an infinity)
      const CodeTable<T> tab = stage_codes(wf, n, reinterpret_cast<uint16_t*>(sw));
      __syncthreads();
      rejection_wave_range<false>(wf, buffer_view(wf, n * (uint32_t)sizeof(T)), n, filt, wmax, i0,
                                  i1, max_trials, key, offset, af, my_flags, tab, &queue);
    } else if (CAP == 0 && !tiny) {
      __syncthreads();
      rejection_wave_range<false>(wf, none, n, filt, wmax, i0, i1, max_trials, key, offset, af,
                                  my_flags, NoTable{}, &queue);
    } else {
      __syncthreads();
      rejection_wave_range<true>(wf, none, n, filt, wmax, i0, i1, max_trials, key, offset, af,
                                 my_flags, NoTable{}, &queue);
    }
    g0 = q1;
  }
  if (flags) {
    const uint32_t wf = wave_reduce(my_flags, OpOr());
    if (lane_id() == 0 && wf) atomicOr(flags, wf);
  }
}

// One vector with the LDS bound table; the workgroup's waves hand out its
// chunk among themselves.  (w_max at least 2^-900: checked by the launcher.)
template <typename T>
__global__ __launch_bounds__(kTableThreads) void k_rejection_table(
    const T* __restrict__ w, int64_t n, double w_max, uint32_t max_trials, Key key,
    uint32_t offset, uint32_t filter, int32_t* __restrict__ a, uint32_t* __restrict__ flags,
    int64_t chunk, const uint32_t* __restrict__ nib_g, const uint32_t* __restrict__ cm,
    uint32_t nb, int shift) {
  __shared__ __align__(16) uint8_t nib[kTableBuckets / 2];
  __shared__ uint32_t queue;  // particles of the chunk handed out so far
  offset = counter_offset(key, offset);
  if (threadIdx.x == 0) queue = 0;  // before the barrier of the table's load
  const BoundTable tab = load_bound_table(nib_g, cm, nb, shift, nib);
  const int64_t p0 = (int64_t)blockIdx.x * chunk;
  const int64_t p1 = p0 + chunk < n ? p0 + chunk : n;
  uint32_t my_flags = 0;
  // n * sizeof(T) < 2^31 (checked by the launcher)
  if (p0 < p1)
    rejection_wave_range<false>(w, buffer_view(w, (uint32_t)(n * (int64_t)sizeof(T))),
                                (uint32_t)n, filter, w_max, (uint32_t)p0, (uint32_t)p1,
                                max_trials, key, offset, a, my_flags, tab, &queue);
  if (flags) {
    const uint32_t wf = wave_reduce(my_flags, OpOr());
    if (lane_id() == 0 && wf) atomicOr(flags, wf);
  }
}

// ------------------------------------------------------------------ launchers
// LDS capacity (weights) for the longest segment: 16, 64 or 128 KB, or none
// when some segment is longer (or the lengths are unknown and the vector is
// long) -- then every weight load goes to global memory.
template <typename T>
int staged_capacity(int64_t max_len, int64_t n_total, uint32_t n_filters) {
  constexpr int64_t per_kb = 1024 / (int64_t)sizeof(T);
  if (n_filters == 1) {
    if (n_total <= 16 * per_kb) return (int)(16 * per_kb);
    if (n_total <= 64 * per_kb) return (int)(64 * per_kb);
    return 0;
  }
  // batches: up to the tuned largest tier; longer segments run in the same
  // launch from global memory
  if (max_len <= 0) max_len = (int64_t)128 * per_kb;
  const int64_t top = (int64_t)tuning().batch_stage_max_kb;
  if (max_len <= 16 * per_kb || top == 16) return (int)(16 * per_kb);
  if (max_len <= 64 * per_kb || top == 64) return (int)(64 * per_kb);
  return (int)(128 * per_kb);
}

// Particles per workgroup of 1024 threads of a batch: as many as `most`, less
// where that would leave CUs idle (two workgroups each).
int64_t chunk_for(int64_t n_total, int64_t most) {
  return std::min(most, std::max<int64_t>(1024, (n_total / 512 + 1023) / 1024 * 1024));
}
// The same where most segments are too long for the 128 KB tier, so that nearly
// every chunk is one part of one segment: equal chunks in whole rounds of the
// workgroups that the chip holds at once, one to a CU (16 of 40000 binary32
// weights, 4 steps: 313 chunks, a second round for the last 57, 23 us, 209 chunks
// 17; 64 of 2^15 .. 2^16, rejection at 4 %: 492 chunks 121 us, 246 103).  Chunks
// of several short segments differ in cost, and small ones even that out (500 of
// 2^8 .. 2^14 binary64 weights, 100 steps: 464 chunks 340 us, 232 375).
int64_t batch_chunk(int cap, size_t weight, int64_t n_total, uint32_t n_filters, int64_t most) {
  if (cap * weight <= 65536 || n_total / n_filters <= cap) return chunk_for(n_total, most);
  const int64_t rounds = (n_total + 256 * most - 1) / (256 * most);
  const int64_t even = (n_total + 256 * rounds - 1) / (256 * rounds);
  return std::min(most, (even + 1023) / 1024 * 1024);
}

template <typename T>
hipError_t launch_metropolis_t(const void* wv, int64_t n_total, const int64_t* offsets,
                               uint32_t n_filters, int64_t max_len, int32_t B,
                               const int32_t* B_dev, Key key, uint32_t offset,
                               uint32_t filter_base, int32_t* a, void* ws, hipStream_t stream) {
  const T* w = (const T*)wv;
  constexpr int per_kb = 1024 / (int)sizeof(T);
  const int cap = staged_capacity<T>(max_len, n_total, n_filters);
  const uint64_t* const uniform = nullptr;
  auto once = [](unsigned grid) { return ChunkQueue{nullptr, grid}; };
  if (cap == 0) {
    // one vector of up to 128 KB of weights: staged as below (one workgroup per
    // CU for the LDS); a longer one gathers from global memory, with at most the
    // tuned number of chains per workgroup, and few enough to use every CU (60000
    // binary32 weights, 16 / 354 steps: 2048 30 / 541 us, 256 9 / 90; as bound codes
    // in LDS 14 / 105)
    if (n_total <= 128 * per_kb) {
      const int64_t chunk1 = 256;
      const unsigned grid = (unsigned)((n_total + chunk1 - 1) / chunk1);
      hipLaunchKernelGGL((k_metropolis_staged<T, 128 * per_kb, 256, false>), dim3(grid), dim3(256),
                         0, stream, w, n_total, offsets, n_filters, B, B_dev, key, offset,
                         filter_base, a, chunk1, uniform, once(grid));
      return hipGetLastError();
    }
    const int64_t chunk =
        std::min<int64_t>(tuning().metropolis_chunk, (n_total / 256 + 255) / 256 * 256);
    const unsigned grid = (unsigned)((n_total + chunk - 1) / chunk);
    hipLaunchKernelGGL(k_metropolis_global<T>, dim3(grid), dim3(256), 0, stream, w, n_total, B,
                       B_dev, key, offset, filter_base, a, chunk);
    return hipGetLastError();
  }
  // segments longer than the LDS tier run in the same launch
  if (!offsets || n_filters <= 1) {
    // one short vector: every workgroup stages all of it and runs 256 of its
    // chains, one per lane, so that long chains (large B) spread over many CUs
    // instead of running four to a lane on one to four of them
    const int64_t chunk1 = 256;
    const dim3 grid1((unsigned)((n_total + chunk1 - 1) / chunk1));
    if (cap == 16 * per_kb)
      hipLaunchKernelGGL((k_metropolis_staged<T, 16 * per_kb, 256, false>), grid1, dim3(256), 0, stream,
                         w, n_total, offsets, n_filters, B, B_dev, key, offset, filter_base, a,
                         chunk1, uniform, once(grid1.x));
    else
      hipLaunchKernelGGL((k_metropolis_staged<T, 64 * per_kb, 256, false>), grid1, dim3(256), 0, stream,
                         w, n_total, offsets, n_filters, B, B_dev, key, offset, filter_base, a,
                         chunk1, uniform, once(grid1.x));
    return hipGetLastError();
  }
  if (n_total <= 256 * 256) {
    // a small batch: one chain per lane and 256 chains per workgroup, as for
    // one short vector, so that its long chains spread over the chip
    const dim3 grid1((unsigned)((n_total + 255) / 256));
    if (cap == 16 * per_kb)
      hipLaunchKernelGGL((k_metropolis_staged<T, 16 * per_kb, 256, false>), grid1, dim3(256), 0, stream,
                         w, n_total, offsets, n_filters, B, B_dev, key, offset, filter_base, a,
                         (int64_t)256, uniform, once(grid1.x));
    else if (cap == 64 * per_kb)
      hipLaunchKernelGGL((k_metropolis_staged<T, 64 * per_kb, 256, false>), grid1, dim3(256), 0, stream,
                         w, n_total, offsets, n_filters, B, B_dev, key, offset, filter_base, a,
                         (int64_t)256, uniform, once(grid1.x));
    else
      hipLaunchKernelGGL((k_metropolis_staged<T, 128 * per_kb, 256, false>), grid1, dim3(256), 0, stream,
                         w, n_total, offsets, n_filters, B, B_dev, key, offset, filter_base, a,
                         (int64_t)256, uniform, once(grid1.x));
    return hipGetLastError();
  }
  // the tuned chunk, twice that from the queue, less where it would leave CUs
  // idle
  const bool queued = ws && B_dev && n_filters <= kQueueFilters;
  // (from the queue twice the tuned chunk, but several to a workgroup)
  const int64_t tuned = tuning().batch_metropolis_chunk;
  const int64_t chunk =
      queued ? chunk_for(n_total, 2 * tuned)
             : batch_chunk(cap, sizeof(T), n_total, n_filters, tuned);
  // with a workspace and step counts of its own per segment: cut by cost, and
  // the chunks handed out as workgroups get free
  const unsigned chunks = (unsigned)((n_total + chunk - 1) / chunk);
  const uint64_t* cost = nullptr;
  ChunkQueue queue = once(chunks);
  if (queued) {
    queue.heads = (uint32_t*)ws;
    uint64_t* prefix = (uint64_t*)((char*)ws + kQueueBytes);
    hipLaunchKernelGGL(k_cost_prefix, dim3(1), dim3(1024), 0, stream, offsets, n_filters, B_dev,
                       prefix, queue.heads);
    cost = prefix;
  }
  const unsigned stay = cap * sizeof(T) > 65536 ? 256 : 512;  // what the chip holds at once
  const dim3 grid(queued && chunks > stay ? stay : chunks);
  auto launch = [&](auto plain, auto from_queue) {
    hipLaunchKernelGGL(queued ? from_queue : plain, grid, dim3(1024), 0, stream, w, n_total, offsets,
                       n_filters, B, B_dev, key, offset, filter_base, a, chunk, cost, queue);
  };
  if (cap == 16 * per_kb)
    launch(k_metropolis_staged<T, 16 * per_kb, 1024, false>,
           k_metropolis_staged<T, 16 * per_kb, 1024, true>);
  else if (cap == 64 * per_kb)
    launch(k_metropolis_staged<T, 64 * per_kb, 1024, false>,
           k_metropolis_staged<T, 64 * per_kb, 1024, true>);
  else
    launch(k_metropolis_staged<T, 128 * per_kb, 1024, false>,
           k_metropolis_staged<T, 128 * per_kb, 1024, true>);
  return hipGetLastError();
}

// Bound-table geometry for one vector of n weights: buckets of 2^shift
// particles, at most kTableBuckets of them.
struct TableGeom {
  int shift;
  uint32_t nb, n_wg;
  size_t wg_off, codes_off, nib_off, cm_off, bytes;
};

TableGeom table_geom(int64_t n) {
  TableGeom g;
  g.shift = 2;  // at least 4 particles per bucket (BoundTable::c4 needs shift >= 2)
  while ((((n - 1) >> g.shift) + 1) > kTableBuckets) ++g.shift;
  g.nb = (uint32_t)(((n - 1) >> g.shift) + 1);
  g.n_wg = (g.nb + kCodeThreads - 1) / kCodeThreads;
  g.wg_off = 0;
  g.codes_off = ((size_t)g.n_wg * 4 + 255) & ~(size_t)255;
  g.nib_off = g.codes_off + (((size_t)g.nb + 7) / 8 * 8 + 255) / 256 * 256;
  // packed nibbles, padded to 16-byte pieces; then the largest code
  g.cm_off = g.nib_off + (((size_t)g.nb + 31) / 32 * 16 + 255) / 256 * 256;
  g.bytes = g.cm_off + 256;
  return g;
}

// A vector long enough for the table path: not staged in LDS, and long enough
// that the table prologue pays off.
template <typename T>
bool use_table(int64_t n_total, uint32_t n_filters, int64_t max_len) {
  // the table kernels gather through a buffer resource, whose byte range
  // must stay below 2^31
  return n_filters == 1 && n_total >= (1 << 16) &&
         n_total * (int64_t)sizeof(T) < ((int64_t)1 << 31) &&
         staged_capacity<T>(max_len, n_total, n_filters) == 0;
}

size_t alt_workspace_bytes(bool f64, int64_t n_total, uint32_t n_filters, int64_t max_len) {
  const bool t = f64 ? use_table<double>(n_total, n_filters, max_len)
                     : use_table<float>(n_total, n_filters, max_len);
  return t ? table_geom(n_total).bytes : 0;
}

// Metropolis: the same, and for a batch the cost prefix of its segments.
size_t metropolis_workspace_bytes(bool f64, int64_t n_total, uint32_t n_filters,
                                  int64_t max_len) {
  if (n_filters > kQueueFilters) return 0;
  if (n_filters > 1)  // the chunk queue, the cost prefix
    return kQueueBytes + ((((size_t)n_filters + 1) * sizeof(uint64_t) + 255) & ~(size_t)255);
  return alt_workspace_bytes(f64, n_total, n_filters, max_len);
}

template <typename T>
hipError_t launch_bound_codes(const T* w, int64_t n, const TableGeom& g, void* ws,
                              hipStream_t stream) {
  char* base = (char*)ws;
  hipLaunchKernelGGL(k_bound_codes<T>, dim3(g.n_wg), dim3(kCodeThreads), 0, stream, w, n, g.shift,
                     (uint8_t*)(base + g.codes_off), (uint32_t*)(base + g.wg_off));
  const uint32_t words = (g.nb + 7) / 8;
  hipLaunchKernelGGL(k_pack_table, dim3((words + kPackThreads - 1) / kPackThreads),
                     dim3(kPackThreads), 0, stream, (const uint8_t*)(base + g.codes_off),
                     (const uint32_t*)(base + g.wg_off), g.n_wg, g.nb,
                     (uint32_t*)(base + g.nib_off), (uint32_t*)(base + g.cm_off));
  return hipGetLastError();
}

// bound_code of a finite positive binary64 on the host: 2^(c - 127) >= v
uint32_t ref_code(double v) {
  uint64_t bits;
  memcpy(&bits, &v, sizeof bits);
  const int e = (int)((bits >> 52) & 0x7FF);
  if (e == 0) return 0u;  // below 2^-1022: every code reaches it
  const int c = e - 1023 + 127 + ((bits & 0xFFFFFFFFFFFFFull) != 0ull ? 1 : 0);
  return c < 0 ? 0u : (c > 255 ? 255u : (uint32_t)c);
}

// Workgroups of the table kernels: one per CU, each with a chunk of particles.
constexpr int64_t kTableGrid = 256;

template <typename T>
hipError_t launch_metropolis_table(const T* w, int64_t n, int32_t B, Key key, uint32_t offset,
                                   uint32_t filter, int32_t* a, void* ws, hipStream_t stream) {
  const TableGeom g = table_geom(n);
  hipError_t e = launch_bound_codes(w, n, g, ws, stream);
  if (e != hipSuccess) return e;
  const int64_t chunk = (n + kTableGrid - 1) / kTableGrid;
  char* base = (char*)ws;
  const dim3 grid((unsigned)((n + chunk - 1) / chunk));
  const uint32_t* nib = (const uint32_t*)(base + g.nib_off);
  const uint32_t* cm = (const uint32_t*)(base + g.cm_off);
  // chains per lane: as many as the chunk fills (four from 2^20 particles up);
  // more than that would run copies of dead chains on every lane
  if (chunk <= kTableThreads)
    hipLaunchKernelGGL((k_metropolis_table<T, 1>), grid, dim3(kTableThreads), 0, stream, w, n, B,
                       key, offset, filter, a, chunk, nib, cm, g.nb, g.shift);
  else if (chunk <= 2 * kTableThreads || sizeof(T) == 8)
    // (binary64 stays at two chains: four spill, 1.25 against 1.05 ms at 2^20)
    hipLaunchKernelGGL((k_metropolis_table<T, 2>), grid, dim3(kTableThreads), 0, stream, w, n, B,
                       key, offset, filter, a, chunk, nib, cm, g.nb, g.shift);
  else if constexpr (sizeof(T) == 4)
    hipLaunchKernelGGL((k_metropolis_table<T, 4>), grid, dim3(kTableThreads), 0, stream, w, n, B,
                       key, offset, filter, a, chunk, nib, cm, g.nb, g.shift);
  return hipGetLastError();
}

hipError_t launch_metropolis(bool f64, const void* w, int64_t n_total, const int64_t* offsets,
                             uint32_t n_filters, int64_t max_len, int32_t B, const int32_t* B_dev,
                             Key key, uint32_t offset, uint32_t filter_base, int32_t* a, void* ws,
                             size_t ws_bytes, hipStream_t stream) {
  // the table pays off once chains are long (small beta, most proposals rejected),
  // and where the vector has more of them than plain chains of one per lane fill
  // the chip with (binary32, 60 / 354 steps, table against plain: 65536 particles
  // 28.2 / 114 and 19.6 / 86 us, 72000 29.6 / 123 and 29.2 / 140)
  const int32_t min_B = tuning().metropolis_table_min_B;
  if (ws && !B_dev && min_B > 0 && B >= min_B && n_total > (1 << 16) &&
      ws_bytes >= alt_workspace_bytes(f64, n_total, n_filters, max_len) &&
      (f64 ? use_table<double>(n_total, n_filters, max_len)
           : use_table<float>(n_total, n_filters, max_len)))
    return f64 ? launch_metropolis_table((const double*)w, n_total, B, key, offset, filter_base,
                                         a, ws, stream)
               : launch_metropolis_table((const float*)w, n_total, B, key, offset, filter_base, a,
                                         ws, stream);
  if (n_filters <= 1 || ws_bytes < metropolis_workspace_bytes(f64, n_total, n_filters, max_len))
    ws = nullptr;  // a batch's workspace: the chunk queue and the cost prefix
  return f64 ? launch_metropolis_t<double>(w, n_total, offsets, n_filters, max_len, B, B_dev, key,
                                           offset, filter_base, a, ws, stream)
             : launch_metropolis_t<float>(w, n_total, offsets, n_filters, max_len, B, B_dev, key,
                                          offset, filter_base, a, ws, stream);
}


template <typename T>
hipError_t launch_rejection_t(const void* wv, int64_t n_total, const int64_t* offsets,
                              uint32_t n_filters, int64_t max_len, double w_max,
                              const double* w_max_dev, uint32_t max_trials, Key key,
                              uint32_t offset, uint32_t filter_base, int32_t* a, uint32_t* flags,
                              hipStream_t stream) {
  const T* w = (const T*)wv;
  constexpr int per_kb = 1024 / (int)sizeof(T);
  const int cap = staged_capacity<T>(max_len, n_total, n_filters);
  const bool single = !offsets || n_filters <= 1;
  if (cap == 0) {
    // a short single vector: 256 particles per workgroup, so that its long
    // trial sequences spread over more CUs
    const int64_t chunk = single && n_total < (1 << 19) ? 256
                                                          : (int64_t)tuning().rejection_per_wave * 4;
    hipLaunchKernelGGL((k_rejection<T, 0, 256>), dim3((unsigned)((n_total + chunk - 1) / chunk)),
                       dim3(256), 0, stream, w, n_total, offsets, n_filters, w_max, w_max_dev,
                       max_trials, key, offset, filter_base, a, flags, chunk);
    return hipGetLastError();
  }
  if (single) {
    // one vector in LDS: every 256-thread workgroup stages all of it and takes
    // 256 of its particles (one per lane on average)
    const int64_t chunk1 = 256;
    const dim3 grid1((unsigned)((n_total + chunk1 - 1) / chunk1));
    if (cap == 16 * per_kb)
      hipLaunchKernelGGL((k_rejection<T, 16 * per_kb, 256>), grid1, dim3(256), 0, stream, w,
                         n_total, offsets, n_filters, w_max, w_max_dev, max_trials, key, offset,
                         filter_base, a, flags, chunk1);
    else
      hipLaunchKernelGGL((k_rejection<T, 64 * per_kb, 256>), grid1, dim3(256), 0, stream, w,
                         n_total, offsets, n_filters, w_max, w_max_dev, max_trials, key, offset,
                         filter_base, a, flags, chunk1);
    return hipGetLastError();
  }
  if (n_total <= 256 * 256) {
    // a small batch: 256 particles per 256-thread workgroup, as for one short
    // vector, so that long trial sequences spread over the chip: 16 vectors of
    // 4000 at 1.8 % acceptance 45 us, in chunks of 16384 it was 798.  Up to 256
    // workgroups; with more of them the staging repeated in each costs more
    // (every workgroup copies all of its segment).
    const dim3 grid1((unsigned)((n_total + 255) / 256));
    if (cap == 16 * per_kb)
      hipLaunchKernelGGL((k_rejection<T, 16 * per_kb, 256>), grid1, dim3(256), 0, stream, w,
                         n_total, offsets, n_filters, w_max, w_max_dev, max_trials, key, offset,
                         filter_base, a, flags, (int64_t)256);
    else if (cap == 64 * per_kb)
      hipLaunchKernelGGL((k_rejection<T, 64 * per_kb, 256>), grid1, dim3(256), 0, stream, w,
                         n_total, offsets, n_filters, w_max, w_max_dev, max_trials, key, offset,
                         filter_base, a, flags, (int64_t)256);
    else
      hipLaunchKernelGGL((k_rejection<T, 128 * per_kb, 256>), grid1, dim3(256), 0, stream, w,
                         n_total, offsets, n_filters, w_max, w_max_dev, max_trials, key, offset,
                         filter_base, a, flags, (int64_t)256);
    return hipGetLastError();
  }
  // the tuned chunk, less where it would leave CUs idle (64 vectors of 4000 at
  // 1.8 % acceptance: 85 us against 818; 64 of 30000: 312 against 716)
  const int64_t chunk = batch_chunk(cap, sizeof(T), n_total, n_filters,
                                    (int64_t)tuning().batch_rejection_per_wave * 16);
  const dim3 grid((unsigned)((n_total + chunk - 1) / chunk));
  if (cap == 16 * per_kb)
    hipLaunchKernelGGL((k_rejection<T, 16 * per_kb, 1024>), grid, dim3(1024), 0, stream, w,
                       n_total, offsets, n_filters, w_max, w_max_dev, max_trials, key, offset,
                       filter_base, a, flags, chunk);
  else if (cap == 64 * per_kb)
    hipLaunchKernelGGL((k_rejection<T, 64 * per_kb, 1024>), grid, dim3(1024), 0, stream, w,
                       n_total, offsets, n_filters, w_max, w_max_dev, max_trials, key, offset,
                       filter_base, a, flags, chunk);
  else
    hipLaunchKernelGGL((k_rejection<T, 128 * per_kb, 1024>), grid, dim3(1024), 0, stream, w,
                       n_total, offsets, n_filters, w_max, w_max_dev, max_trials, key, offset,
                       filter_base, a, flags, chunk);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_rejection_table(const T* w, int64_t n, double w_max, uint32_t max_trials,
                                  Key key, uint32_t offset, uint32_t filter, int32_t* a,
                                  uint32_t* flags, void* ws, hipStream_t stream) {
  const TableGeom g = table_geom(n);
  char* base = (char*)ws;
  hipLaunchKernelGGL(k_bound_nibbles<T>, dim3((g.nb + kCodeThreads - 1) / kCodeThreads),
                     dim3(kCodeThreads), 0, stream, w, n, g.shift, g.nb, ref_code(w_max),
                     (uint32_t*)(base + g.nib_off), (uint32_t*)(base + g.cm_off));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // chunks of 16 waves x rejection_per_wave particles, several per CU
  const int64_t chunk = (int64_t)tuning().rejection_per_wave * (kTableThreads / kWave);
  hipLaunchKernelGGL(k_rejection_table<T>, dim3((unsigned)((n + chunk - 1) / chunk)),
                     dim3(kTableThreads), 0, stream, w, n, w_max, max_trials, key, offset, filter,
                     a, flags, chunk, (const uint32_t*)(base + g.nib_off),
                     (const uint32_t*)(base + g.cm_off), g.nb, g.shift);
  return hipGetLastError();
}

hipError_t launch_rejection(bool f64, const void* w, int64_t n_total, const int64_t* offsets,
                            uint32_t n_filters, int64_t max_len, double w_max,
                            const double* w_max_dev, uint32_t max_trials, Key key,
                            uint32_t offset, uint32_t filter_base, int32_t* a, uint32_t* flags,
                            void* ws, size_t ws_bytes, hipStream_t stream) {
  // below 2^20 particles the plain kernel was faster at every y measured (0..4)
  if (ws && !w_max_dev && w_max >= 0x1p-900 && tuning().rejection_table &&
      n_total >= (1 << 20) &&
      ws_bytes >= alt_workspace_bytes(f64, n_total, n_filters, max_len) &&
      (f64 ? use_table<double>(n_total, n_filters, max_len)
           : use_table<float>(n_total, n_filters, max_len)))
    return f64 ? launch_rejection_table((const double*)w, n_total, w_max, max_trials, key, offset,
                                        filter_base, a, flags, ws, stream)
               : launch_rejection_table((const float*)w, n_total, w_max, max_trials, key, offset,
                                        filter_base, a, flags, ws, stream);
  return f64 ? launch_rejection_t<double>(w, n_total, offsets, n_filters, max_len, w_max,
                                          w_max_dev, max_trials, key, offset, filter_base, a,
                                          flags, stream)
             : launch_rejection_t<float>(w, n_total, offsets, n_filters, max_len, w_max,
                                         w_max_dev, max_trials, key, offset, filter_base, a,
                                         flags, stream);
}

}  // namespace pfr
