// pfr_filter.hip -- the bootstrap particle filter of Code 1 for a 1-D
// linear-Gaussian state-space model, batched over F filters of n particles:
//   x_0 ~ N(0, s0^2),   x_t = phi x_{t-1} + q e_t,   y_t = x_t + r v_t.
// The bootstrap choice (section 1) takes the transition density as K_t and
// the observation density as G_t.  Step t of Code 1 runs, for every filter:
// ancestors from the previous weights, the permutation that makes in-place
// propagation safe (section 2.3, eq. predicate), the in-place copy
// x_i <- x_{c_i} for c_i != i, propagation and weighting.  The log-weights are
// shifted by their maximum in binary64 before exponentiation (the
// renormalisation identity of appendix E), the weights handed to the next
// resampling are binary32 values in (0, 1] with maximum exactly 1, and
// log Z accumulates max + log(mean exp(lw - max)) in binary64.
//
// The step index t lives in device memory; the last kernel of a step advances
// it, so one captured graph of a step can be replayed for t = 1..T.
//
// Random numbers: the initial state of particle i of filter f takes Philox
// counter (i, INIT<<28, f, offset), its propagation noise at step t the counter
// (i, NOISE<<28 | t, f, offset); a standard normal is formed from words 0 and
// 1 by the Box-Muller transform with u1 = (x0 + 1) 2^-32 and u2 = x1 2^-32.
#include "pfr_filter_math.h"
#include "pfr_kernels.h"

namespace pfr {

namespace {

// ---------------------------------------------------------------- functions
// lgssm_init forms the tables of pfr_filter_math.h in the workspace; a
// workgroup copies them to LDS.
__device__ __forceinline__ void fill_tables(MathTables* T, int tid, int threads) {
  for (int i = tid; i < kCosBins; i += threads)
    T->cs[i] = MathPair{cospi(i * (2.0 / kCosBins)), sinpi(i * (2.0 / kCosBins))};
  for (int i = tid; i < kLogBins; i += threads) {
    const LogEntry t = kLogTable[i];
    T->lg[i] = MathPair{t.rc, t.hi};
    T->lo[i] = t.lo;
  }
}
static_assert(sizeof(MathTables) == kFilterTableBytes, "table bytes of the filter state");
__device__ __forceinline__ void load_tables(MathTables* T, const void* __restrict__ src, int tid,
                                            int threads) {
  for (int i = tid; i < (int)(sizeof(MathTables) / 16); i += threads)
    reinterpret_cast<uint4*>(T)[i] = reinterpret_cast<const uint4*>(src)[i];
}

// Square root of t = 0 or 2^-40 < t < 2^10: the reciprocal square root
// estimate, a coupled Newton step (Goldschmidt), then one on the root.  The
// correctly rounded root of 2 neg_log_u1(x) for each of the 2^32 words x.
__device__ __forceinline__ double sqrt_pos(double t) {
  const double y = __builtin_amdgcn_rsq(t);
  double g = t * y, h = 0.5 * y;
  double d = __fma_rn(-h, g, 0.5);
  g = __fma_rn(g, d, g);
  h = __fma_rn(h, d, h);
  d = __fma_rn(-g, g, t);
  g = __fma_rn(d, h, g);
  return t == 0.0 ? 0.0 : g;
}

__device__ __forceinline__ double normal_bm(uint32_t x0, uint32_t x1, const MathTables* T) {
  return sqrt_pos(2.0 * neg_log_u1(x0, T)) * cos_turns(x1, T);
}

template <int THREADS, typename Op>
__device__ double block_reduce(double v, double* slot, Op op) {
  const int wave = (int)threadIdx.x / kWave, lane = (int)threadIdx.x % kWave;
  v = wave_reduce(v, op);
  __syncthreads();
  if (lane == 0) slot[wave] = v;
  __syncthreads();
  double t = slot[0];
  for (int w2 = 1; w2 < THREADS / kWave; ++w2) t = op(t, slot[w2]);
  __syncthreads();
  return t;
}

constexpr int kFT = 512;  // threads per workgroup of the initialisation

__global__ __launch_bounds__(kFT) void k_lg_init(int32_t n_filters, int32_t n, double s0, Key key,
                                                 uint32_t offset, uint32_t filter_base,
                                                 float* __restrict__ x, float* __restrict__ w,
                                                 double* __restrict__ logz,
                                                 int32_t* __restrict__ B_dev,
                                                 uint32_t* __restrict__ t_dev,
                                                 int64_t* __restrict__ offsets,
                                                 uint32_t* __restrict__ done,
                                                 uint32_t* __restrict__ bstart,
                                                 uint32_t* __restrict__ estart,
                                                 MathTables* __restrict__ tables) {
  __shared__ MathTables T;
  fill_tables(&T, (int)threadIdx.x, kFT);
  __syncthreads();
  if (blockIdx.x == 0)
    for (int i = (int)threadIdx.x; i < (int)(sizeof(MathTables) / 16); i += kFT)
      reinterpret_cast<uint4*>(tables)[i] = reinterpret_cast<const uint4*>(&T)[i];
  const int64_t total = (int64_t)n_filters * n;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += stride) {
    const int32_t f = (int32_t)(g / n), i = (int32_t)(g - (int64_t)f * n);
    const uint4 u = draw(key, (uint32_t)i, DOM_INIT, 0, filter_base + (uint32_t)f, offset);
    x[g] = (float)(s0 * normal_bm(u.x, u.y, &T));
    w[g] = 1.0f;
  }
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g <= n_filters; g += stride) {
    offsets[g] = g * n;
    bstart[g] = (uint32_t)(g * ((n + kBlock - 1) / kBlock));
    estart[g] = (uint32_t)(g * ((n + 1 + kBlock - 1) / kBlock));
    if (g < n_filters) {
      logz[g] = 0.0;
      B_dev[g] = 1;
    }
    if (g == 0) {
      *t_dev = 1u;
      *done = 0u;
    }
  }
}

// One workgroup per filter: copy, propagate, weight, log Z and the Metropolis
// step count for the next resampling, B = ceil(log eps / log(1 - beta)) with
// beta = mean(w) (the shifted weights have maximum 1).
// inv_r = 1 / r in binary64: the scaled residual is (y - x) * inv_r, one
// multiply where a division would cost a dozen VALU instructions (it may
// differ from (y - x) / r in the last bit).
// Filters of up to CAP particles keep their new states in LDS until the
// largest log-weight is known: the states are gathered from x, all of them
// before any is written, so the copy needs no pass of its own, and x is read
// and written once.  Longer filters (CAP = 0) copy first and go through x
// twice.  A thread takes quads of consecutive particles.  Every workgroup
// counts itself once it has read t; the last one advances it.  VALU bound
// (172 VALU instructions a particle, a Philox call among them): 1024 filters of
// 16384 188 -> 105 us (library functions, three passes over x).
typedef float QuadF __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t QuadI __attribute__((ext_vector_type(4), aligned(4)));

template <int CAP, int THREADS>
__global__ __launch_bounds__(THREADS) void k_lg_move(int32_t n, double phi, double q,
                                                     double inv_r, double log_norm,
                                                     double log_eps,
                                                     const double* __restrict__ y, int32_t T,
                                                     uint32_t* __restrict__ t_dev,
                                                     uint32_t* __restrict__ done,
                                                     const void* __restrict__ tables, Key key,
                                                     uint32_t offset, uint32_t filter_base,
                                                     const int32_t* __restrict__ c,
                                                     float* __restrict__ x,
                                                     float* __restrict__ w,
                                                     double* __restrict__ logz,
                                                     int32_t* __restrict__ B_dev,
                                                     uint32_t* __restrict__ flags) {
  __shared__ MathTables tab;
  __shared__ double slot[THREADS / kWave];
  __shared__ __align__(16) float xs[CAP > 0 ? CAP : 4];
  const uint32_t f = blockIdx.x;
  const int64_t base = (int64_t)f * n;
  const uint32_t t = *t_dev;
  const int tid = (int)threadIdx.x;
  __syncthreads();  // every thread has read t
  if (tid == 0 && atomicAdd(done, 1u) == gridDim.x - 1u) {
    *done = 0u;
    *t_dev = t + 1u;
  }
  if (t < 1u || t > (uint32_t)T) {  // no observation for this step
    if (flags && f == 0 && tid == 0) atomicOr(flags, FLAG_BAD_STEP);
    return;
  }
  const double yt = y[t - 1];
  const int32_t* __restrict__ cf = c + base;
  float* __restrict__ xf = x + base;
  float* __restrict__ wf = w + base;
  const int32_t nq = (n + 3) / 4;
  load_tables(&tab, tables, tid, THREADS);
  if (CAP == 0) {
    // in-place copy: slots that are read satisfy c_j = j and are never written
    for (int32_t i = tid; i < n; i += THREADS) {
      const int32_t ci = cf[i];
      if (ci != i) xf[i] = xf[ci];
    }
  }
  __syncthreads();
  // the squared scaled residual d^2; the log-weight is -d^2 / 2 + log_norm, so
  // the smallest d^2 gives the largest one, and lw - max lw = (min d^2 - d^2) / 2
  auto residual2 = [&](float xn) -> double {
    const double d = (yt - (double)xn) * inv_r;
    return d * d;
  };
  double least = __builtin_huge_val();
  for (int32_t qd = tid; qd < nq; qd += THREADS) {
    const int32_t i0 = 4 * qd;
    const bool whole = i0 + 4 <= n;
    float xo[4];
    if (CAP > 0) {
      int32_t ci[4];
      if (whole) {
        const QuadI v = *reinterpret_cast<const QuadI*>(cf + i0);
        ci[0] = v.x; ci[1] = v.y; ci[2] = v.z; ci[3] = v.w;
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) ci[k] = i0 + k < n ? cf[i0 + k] : 0;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) xo[k] = xf[ci[k]];
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) xo[k] = i0 + k < n ? xf[i0 + k] : 0.0f;
    }
    float xn[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint4 u = draw(key, (uint32_t)(i0 + k), DOM_NOISE, t, filter_base + f, offset);
      xn[k] = (float)(phi * (double)xo[k] + q * normal_bm(u.x, u.y, &tab));
    }
    if (!whole) {  // past the end: an infinite residual, weight 0
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (i0 + k >= n) xn[k] = __builtin_huge_valf();
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) least = fmin(least, residual2(xn[k]));
    if (CAP > 0) {
      *reinterpret_cast<float4*>(xs + i0) = make_float4(xn[0], xn[1], xn[2], xn[3]);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (i0 + k < n) xf[i0 + k] = xn[k];
    }
  }
  least = block_reduce<THREADS>(least, slot, OpMin());  // (its barriers: all states were read)
  const double mx = -0.5 * least + log_norm;
  double sum = 0.0;
  for (int32_t qd = tid; qd < nq; qd += THREADS) {
    const int32_t i0 = 4 * qd;
    float xn[4], wn[4];
    if (CAP > 0) {
      const float4 v = *reinterpret_cast<const float4*>(xs + i0);
      xn[0] = v.x; xn[1] = v.y; xn[2] = v.z; xn[3] = v.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) xn[k] = i0 + k < n ? xf[i0 + k] : __builtin_huge_valf();
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double e = exp_neg(__fma_rn(-0.5, residual2(xn[k]), 0.5 * least));
      wn[k] = (float)e;
      sum += e;
    }
    if (i0 + 4 <= n) {
      QuadF v;
      v.x = wn[0]; v.y = wn[1]; v.z = wn[2]; v.w = wn[3];
      *reinterpret_cast<QuadF*>(wf + i0) = v;
      if (CAP > 0) {
        v.x = xn[0]; v.y = xn[1]; v.z = xn[2]; v.w = xn[3];
        *reinterpret_cast<QuadF*>(xf + i0) = v;
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (i0 + k < n) {
          wf[i0 + k] = wn[k];
          if (CAP > 0) xf[i0 + k] = xn[k];
        }
      }
    }
  }
  sum = block_reduce<THREADS>(sum, slot, OpAdd());
  if (tid == 0) {
    const double beta = sum / (double)n;
    logz[f] += mx + log(beta);
    double B = beta >= 1.0 ? 1.0 : ceil(log_eps / log1p(-beta));
    B = B < 1.0 ? 1.0 : (B > 65536.0 ? 65536.0 : B);
    B_dev[f] = (int32_t)B;
  }
}

}  // namespace

hipError_t launch_lgssm_init(int32_t n_filters, int32_t n, double s0, Key key, uint32_t offset,
                             uint32_t filter_base, float* x, float* w, double* logz,
                             int32_t* B_dev, uint32_t* t_dev, const FilterState& st,
                             hipStream_t stream) {
  const int64_t total = (int64_t)n_filters * n;
  int64_t grid = (total + kFT - 1) / kFT;
  if (grid < 1) grid = 1;
  if (grid > 2048) grid = 2048;  // each workgroup forms the tables first
  hipLaunchKernelGGL(k_lg_init, dim3((uint32_t)grid), dim3(kFT), 0, stream, n_filters, n, s0, key,
                     offset, filter_base, x, w, logz, B_dev, t_dev, st.offsets, st.done,
                     st.bstart, st.estart, (MathTables*)st.tables);
  return hipGetLastError();
}

hipError_t launch_lgssm_move(int32_t n_filters, int32_t n, double phi, double q, double r,
                             double log_eps, const double* y, int32_t T, uint32_t* t_dev,
                             const FilterState& st, Key key, uint32_t offset,
                             uint32_t filter_base, const int32_t* c, float* x, float* w,
                             double* logz, int32_t* B_dev, uint32_t* flags, hipStream_t stream) {
  const double log_norm = -log(r) - 0.5 * log(6.283185307179586);
  auto launch = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3((uint32_t)n_filters), dim3(threads), 0, stream, n, phi, q,
                       1.0 / r, log_norm, log_eps, y, T, t_dev, st.done, st.tables, key, offset,
                       filter_base,
                       c, x, w, logz, B_dev, flags);
  };
  // workgroups to a CU: eight (by waves), two and one (by LDS); filters too
  // long for LDS below
  if (n <= 2048) launch(k_lg_move<2048, 256>, 256);
  else if (n <= 16384) launch(k_lg_move<16384, 1024>, 1024);
  else if (n <= 32768) launch(k_lg_move<32768, 1024>, 1024);
  else launch(k_lg_move<0, 1024>, 1024);
  return hipGetLastError();
}

}  // namespace pfr
