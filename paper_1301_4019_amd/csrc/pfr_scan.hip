// pfr_scan.hip -- the collective resamplers: multinomial (Code 5 of the
// paper), stratified (Code 7) and systematic (Code 8).
//
// All three compute the scaled prefix r_i = n W_i / W_n of the weights and map
// sorted points onto it:
//   stratified   point q_s = s + 1 - u_s in (s, s+1], ancestor = min{i : r_i >= q_s}
//   systematic   the same with one offset u for all strata
//   multinomial  p_k = n S_k / S_n from exponential spacings (sorted uniforms),
//                ancestor = #{i < n-1 : r_i <= p_k}
// i.e. Code 7/8 followed by Code 11, and Code 5 with an upper-bound search.
//
// Exact prefix sums.  The paper shows that a float32 prefix sum biases these
// schemes for large n.  Here each block of 1024 weights is quantised to
// integers q = floor(w * 2^s_b) < 2^53 relative to the block maximum (every
// float32 weight within 2^29 of the block maximum is represented exactly),
// block sums are exact 64-bit integers, and the carries between blocks are
// exact 128-bit integers at one global scale.  Integer sums do not depend on
// the order of addition, so the prefix is deterministic, monotone, exactly
// flat across zero weights and consistent at every block boundary; the only
// rounding is the final map r = n * I / I_total to binary64, itself monotone
// with r = n at the end.
//
// Short vectors and short segments of a batch (up to 4096 and 16384 weights,
// stratified and systematic): one workgroup each, one launch (k_scan_one).
// One vector beyond that:
//   records one record per block (validity, block scale, quantised sum), one
//           wave per block, and one sum per exponential-spacing block of the
//           multinomial scheme (whose points are kept for the emission).
//   carries turn the records into the global scale, the exact carries C_b and
//           the total, and scan the exponential-block sums.  With at most
//           direct_max_blocks blocks this step is folded into the emission:
//           every emit workgroup reduces all records (and block sums) itself,
//           which costs less than one more launch.
//   emit    each block rebuilds its exact prefix, I = C_b + local prefix, and
//           r = n I / Q: one block per workgroup of four waves with its own
//           carries, one block per wave (16 consecutive weights per lane)
//           after the carries pass.  Stratified / systematic: every particle
//           computes its cumulative offspring O_i = #{s : q_s <= r_i} in O(1),
//           and the block's output range [O(C_b), O(C_b+1)) is filled through
//           LDS markers and a max-scan, then written coalesced.  Multinomial:
//           each block reads the exponential blocks whose points fall in its
//           r-range and settles its particles with interleaved binary searches
//           in LDS.
// Ragged batches of longer segments run the same steps over all blocks of all
// segments, or inside one workgroup per segment.
#include "pfr_kernels.h"

#include <algorithm>

namespace pfr {

namespace {
#include "pfr_scan_common.h"


// ---------------------------------------------------------------- records
// Record of the block at base: validity, reference exponent (block maximum),
// quantised sum.  Same value in every thread.
template <typename T>
__device__ BlockRec block_record(const T* __restrict__ w, int64_t n, int64_t base, WgScratch* s) {
  T x[kPer];
  load4(w, n, base, x);
  uint32_t bad = 0;
  uint32_t emax = 1;
#pragma unroll
  for (int v = 0; v < kPer; ++v) {
    if (!weight_ok(x[v])) bad = FLAG_BAD_WEIGHTS;
    else emax = max(emax, (uint32_t)exp_field(x[v]));
  }
  // pack (bad, emax) into one max-reduction: bad dominates
  const uint32_t key = (bad << 16) | emax;
  const uint32_t red = wg_reduce(key, OpMax(), (uint32_t*)s->i);
  BlockRec r;
  r.bad = red >> 16;
  const int e_ref = (int)(red & 0xFFFFu);
  uint64_t sum = 0;
  if (!r.bad) {
#pragma unroll
    for (int v = 0; v < kPer; ++v) sum += quantize(x[v], e_ref);
  }
  r.sum = wg_reduce(sum, OpAdd(), s->u);
  r.scale = scale_of<T>(e_ref);
  return r;
}


__device__ __forceinline__ u128 conv_rec(const BlockRec& r, int32_t gscale) {
  return shift_u128((u128)r.sum, gscale - r.scale);
}

// ---------------------------------------------------------------- carries
// From nb records: global scale, exact exclusive carries C[0..nb] (C[nb] is
// the total) and status.  Whole workgroup; records are read in chunks of
// kBlock, 4 consecutive per thread, all loads of a chunk issued together.
struct Totals {
  u128 Q;
  int32_t gscale;
  uint32_t status;
};

template <typename RecPtr, typename CPtr>
__device__ Totals carries_from_records(uint32_t nb, RecPtr recs, CPtr C, WgScratch* s) {
  const int tid = (int)threadIdx.x;
  uint32_t bad = 0;
  uint32_t smin_key = 0xFFFFFFFFu;  // scale + 2^31, min over non-empty blocks
  for (uint32_t base = 0; base < nb; base += kBlock) {
    BlockRec r[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const uint32_t b = base + (uint32_t)tid * kPer + k;
      if (b < nb) r[k] = recs[b];
      else r[k].sum = 0, r[k].scale = 0, r[k].bad = 0;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      bad |= r[k].bad;
      if (r[k].sum) smin_key = min(smin_key, (uint32_t)r[k].scale ^ 0x80000000u);
    }
  }
  bad = wg_reduce(bad, OpOr(), (uint32_t*)s->i);
  smin_key = wg_reduce(smin_key, OpMin(), (uint32_t*)s->i);
  Totals t;
  // every converted block sum is below 2^(63 + gscale - smin); nb of them stay
  // below 2^kCarryBits
  t.gscale = (smin_key == 0xFFFFFFFFu)
                 ? 0
                 : (int32_t)(smin_key ^ 0x80000000u) + (kCarryBits - 63) - ceil_log2(nb);
  u128 carry = 0;
  for (uint32_t base = 0; base < nb; base += kBlock) {
    u128 v[kPer];
    u128 mine = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const uint32_t b = base + (uint32_t)tid * kPer + k;
      v[k] = (b < nb) ? conv_rec(recs[b], t.gscale) : (u128)0;
      mine += v[k];
    }
    u128 tot;
    u128 run = carry + wg_exclusive(mine, s->v, &tot);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const uint32_t b = base + (uint32_t)tid * kPer + k;
      if (b < nb) C[b] = run;
      run += v[k];
    }
    carry += tot;
  }
  if (tid == 0) C[nb] = carry;
  __syncthreads();
  t.Q = carry;
  t.status = bad;
  if (!bad && carry == 0) t.status |= FLAG_ZERO_TOTAL;
  return t;
}

// ---------------------------------------------------------------- kernels
// ---------------------------------------------------------------- carries
// Two levels.  The records fall into groups of kGrp = 1024 consecutive
// blocks.  k_carry_groups (one 256-thread workgroup per group, all in
// parallel) fixes the group's own scale gs_g from its largest block, exactly
// as the global scale is fixed from the largest block overall (with the
// group's 2^10 blocks in place of nb, so group sums stay below 2^100), and
// writes every block's exclusive prefix P_b inside the group at that scale
// and the group total T_g.  The group workgroup that finishes last (a count
// in the header, zeroed by the records pass) takes the global scale from the
// group keys, converts each T_g to it (a shift: truncation when gs_g is
// finer) and scans them into Tx_g; the total Q is Tx_G.  The
// carry of block b in group g is then
//   C_b = Tx_g + floor(P_b 2^(gscale - gs_g)),  C_nb = Q,
// an integer function of the records alone, monotone in b and continuous at
// group ends (P at a group's end is T_g).  It differs from converting every
// block to the global scale by truncation only (one unit of the global scale
// per group), within the bound of the per-block quantisation.  The
// exponential-block sums of the multinomial scheme are plain integers and
// take the same two levels without scales.
constexpr int kGrpLog = 10;
constexpr uint32_t kGrp = 1u << kGrpLog;
constexpr int kGPer = (int)kGrp / kT;  // blocks per thread of a group workgroup (4)

struct CarryGroup {
  u128 T;        // group total at the group's scale (exponential groups: plain sum)
  int32_t gs;    // the group's scale
  uint32_t key;  // min over non-empty blocks of scale ^ 2^31, ~0u if none
  uint32_t bad;
  uint32_t pad;
};

// conv_rec with 64-bit shifts only.  A non-empty block's shift is at most
// kCarryBits - 63 (a group's or the global scale exceeds no non-empty block's
// scale by more), and an empty block converts to zero under any shift, so
// clamping the left shift to 63 changes nothing.
static_assert(kCarryBits - 63 < 64, "left shifts of block sums stay below 64");
__device__ __forceinline__ u128 conv_rec_fast(const BlockRec& r, int32_t scale) {
  const int sh = scale - r.scale;
  const uint64_t s = r.sum;
  const uint32_t l = (uint32_t)min(max(sh, 0), 63), d = (uint32_t)min(-sh, 64);
  const uint64_t lo = sh >= 0 ? s << l : (d >= 64 ? 0ull : s >> d);
  const uint64_t hi = l > 0 ? s >> (64 - l) : 0ull;
  return ((u128)hi << 64) | lo;
}

// Exclusive scan of the kGrp values x (kGPer consecutive per thread) of one
// workgroup; returns the thread's exclusive base and the workgroup total.
__device__ __forceinline__ u128 group_scan(u128 (&x)[kGPer], u128* s_w, u128* total) {
  const int wave = (int)threadIdx.x / kWave, lane = (int)threadIdx.x % kWave;
  u128 run = 0;
#pragma unroll
  for (int k = 0; k < kGPer; ++k) {
    const u128 v = x[k];
    x[k] = run;
    run += v;
  }
  const u128 inc = wave_incl_add_u128(run);
  if (lane == kWave - 1) s_w[wave] = inc;
  __syncthreads();
  u128 before = inc - run, tot = 0;
#pragma unroll
  for (int w2 = 0; w2 < kNW; ++w2) {
    const u128 t = s_w[w2];
    before += w2 < wave ? t : (u128)0;
    tot += t;
  }
  *total = tot;
  return before;
}

// Exclusive scan, in index order, of val(j) for j < m by a workgroup of NT
// threads (CK consecutive values per thread per chunk); put(j, prefix) gets
// each result.  Returns the total; s_w holds NT / 64 values.
template <int NT, int CK, typename Val, typename Put>
__device__ u128 wg_scan_blocked(uint32_t m, Val val, Put put, u128* s_w) {
  constexpr int NW = NT / kWave;
  constexpr uint32_t chunk = (uint32_t)NT * CK;
  const int tid = (int)threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  u128 carry = 0;
  for (uint32_t c0 = 0; c0 < m; c0 += chunk) {
    const uint32_t j0 = c0 + (uint32_t)tid * CK;
    u128 x[CK];
#pragma unroll
    for (int k = 0; k < CK; ++k) x[k] = j0 + (uint32_t)k < m ? val(j0 + (uint32_t)k) : (u128)0;
    u128 run = 0;
#pragma unroll
    for (int k = 0; k < CK; ++k) {
      const u128 v = x[k];
      x[k] = run;
      run += v;
    }
    const u128 inc = wave_incl_add_u128(run);
    if (lane == kWave - 1) s_w[wave] = inc;
    __syncthreads();
    u128 before = carry + (inc - run), tot = 0;
#pragma unroll 2
    for (int w2 = 0; w2 < NW; ++w2) {
      const u128 t = s_w[w2];
      before += w2 < wave ? t : (u128)0;
      tot += t;
    }
#pragma unroll
    for (int k = 0; k < CK; ++k)
      if (j0 + (uint32_t)k < m) put(j0 + (uint32_t)k, before + x[k]);
    carry += tot;
    __syncthreads();
  }
  return carry;
}

// The top level over the G group records (and the Ge exponential ones): global
// scale, status, Tx[0..G] and TEx[0..Ge].  Run by the group workgroup that
// finishes last (kT threads; G <= 2048 for n < 2^31, one chunk).
template <bool MULTI>
__device__ void carry_top(uint32_t nb, uint32_t G, uint32_t Ge,
                          const CarryGroup* __restrict__ groups,
                          const CarryGroup* __restrict__ egroups, u128* __restrict__ Tx,
                          u128* __restrict__ TEx, ScanHeader* __restrict__ hdr, uint32_t* s_u,
                          u128* s_w) {
  const int tid = (int)threadIdx.x;
  uint32_t bad = 0, key = 0xFFFFFFFFu;
  for (uint32_t g = (uint32_t)tid; g < G; g += kT) {
    bad |= groups[g].bad;
    key = min(key, groups[g].key);
  }
  key = wg_reduce(key, OpMin(), s_u);
  bad = wg_reduce(bad, OpOr(), s_u + kNW);
  const int32_t gscale =
      key == 0xFFFFFFFFu ? 0 : (int32_t)(key ^ 0x80000000u) + (kCarryBits - 63) - ceil_log2(nb);
  const u128 Q = wg_scan_blocked<kT, 8>(
      G, [&](uint32_t g) { return shift_u128(groups[g].T, gscale - groups[g].gs); },
      [&](uint32_t g, u128 c) { Tx[g] = c; }, s_w);
  if (MULTI) {
    const u128 S = wg_scan_blocked<kT, 8>(
        Ge, [&](uint32_t g) { return egroups[g].T; }, [&](uint32_t g, u128 c) { TEx[g] = c; },
        s_w);
    if (tid == 0) TEx[Ge] = S;
  }
  if (tid == 0) {
    Tx[G] = Q;
    uint32_t status = bad;
    if (!bad && Q == 0) status |= FLAG_ZERO_TOTAL;
    hdr->status = status;
    hdr->gscale = gscale;
    hdr->Q = Q;
  }
}

// The group step: group g of the weight blocks (weights) or of the
// exponential blocks; its scale, every block's prefix inside it and its
// record.  All kT threads call it.
__device__ void carry_group(bool weights, uint32_t g, uint32_t m,
                            const BlockRec* __restrict__ recs,
                            const uint64_t* __restrict__ esums, u128* __restrict__ out,
                            CarryGroup* __restrict__ rec_out, u128* s_w, uint32_t* s_u) {
  const int tid = (int)threadIdx.x;
  const uint32_t j0 = g * kGrp + (uint32_t)tid * kGPer;
  u128 x[kGPer];
  uint32_t key = 0xFFFFFFFFu, bad = 0;
  int32_t gs = 0;
  if (weights) {
    BlockRec r[kGPer];
#pragma unroll
    for (int k = 0; k < kGPer; ++k) {
      if (j0 + k < m) r[k] = recs[j0 + k];
      else r[k].sum = 0, r[k].scale = 0, r[k].bad = 0;
    }
#pragma unroll
    for (int k = 0; k < kGPer; ++k) {
      bad |= r[k].bad;
      if (r[k].sum) key = min(key, (uint32_t)r[k].scale ^ 0x80000000u);
    }
    key = wg_reduce(key, OpMin(), s_u);
    bad = wg_reduce(bad, OpOr(), s_u + kNW);
    gs = key == 0xFFFFFFFFu ? 0 : (int32_t)(key ^ 0x80000000u) + (kCarryBits - 63) - kGrpLog;
#pragma unroll
    for (int k = 0; k < kGPer; ++k) x[k] = conv_rec_fast(r[k], gs);
  } else {
#pragma unroll
    for (int k = 0; k < kGPer; ++k) x[k] = j0 + k < m ? (u128)esums[j0 + k] : (u128)0;
  }
  u128 total;
  const u128 before = group_scan(x, s_w, &total);
#pragma unroll
  for (int k = 0; k < kGPer; ++k)
    if (j0 + k < m) out[j0 + k] = before + x[k];
  if (tid == 0) {
    CarryGroup c;
    c.T = total;
    c.gs = gs;
    c.key = key;
    c.bad = bad;
    c.pad = 0;
    rec_out[g] = c;
  }
}

// With a single group in all (strata schemes up to 2^20 particles) its
// workgroup goes on to the top level: no count and no fences.  Otherwise one
// workgroup per group, and the last to finish runs the top level (measured:
// one workgroup taking the three groups of a 2^20 multinomial call in turn,
// 9.7 us, is slower than three in parallel with the count, 8.8 us).
constexpr uint32_t kFewGroups = 1;

template <bool MULTI>
__global__ __launch_bounds__(kT) void k_carry_groups(uint32_t nb, uint32_t nbe, uint32_t G,
                                                     const BlockRec* __restrict__ recs,
                                                     const uint64_t* __restrict__ esums,
                                                     u128* __restrict__ P, u128* __restrict__ PE,
                                                     CarryGroup* __restrict__ groups,
                                                     CarryGroup* __restrict__ egroups,
                                                     uint32_t Ge, u128* __restrict__ Tx,
                                                     u128* __restrict__ TEx,
                                                     ScanHeader* __restrict__ hdr) {
  __shared__ u128 s_w[kNW];
  __shared__ uint32_t s_u[2 * kNW];
  __shared__ uint32_t s_last;
  if (G + (MULTI ? Ge : 0u) <= kFewGroups) {
    for (uint32_t g = 0; g < G; ++g) {
      carry_group(true, g, nb, recs, esums, P, groups, s_w, s_u);
      __syncthreads();  // the scratch is reused; the group records are read by all
    }
    if (MULTI) {
      for (uint32_t g = 0; g < Ge; ++g) {
        carry_group(false, g, nbe, recs, esums, PE, egroups, s_w, s_u);
        __syncthreads();
      }
    }
    carry_top<MULTI>(nb, G, Ge, groups, egroups, Tx, TEx, hdr, s_u, s_w);
    return;
  }
  const bool weights = blockIdx.x < G;
  if (!MULTI && !weights) return;  // (never: the grid has G workgroups then)
  const uint32_t g = weights ? blockIdx.x : blockIdx.x - G;
  carry_group(weights, g, weights ? nb : nbe, recs, esums, weights ? P : PE,
              weights ? groups : egroups, s_w, s_u);
  if (threadIdx.x == 0) {
    // the last group to finish (the records pass zeroed the count) runs the
    // top level: release this group's record, count it, acquire the others
    __threadfence();
    s_last = atomicAdd(&hdr->groups_done, 1u) == G + (MULTI ? Ge : 0u) - 1u ? 1u : 0u;
  }
  __syncthreads();
  if (!s_last) return;
  __threadfence();
  carry_top<MULTI>(nb, G, Ge, groups, egroups, Tx, TEx, hdr, s_u, s_w);
}

// The exact carry C_b of block b (0 <= b <= nb) from the two levels.
struct Carries {
  const u128* __restrict__ P;
  const u128* __restrict__ Tx;
  const CarryGroup* __restrict__ grp;
  uint32_t nb, G;
  int32_t gscale;
  __device__ __forceinline__ u128 operator[](uint32_t b) const {
    if (b >= nb) return Tx[G];
    const uint32_t g = b >> kGrpLog;
    return Tx[g] + shift_u128(P[b], gscale - grp[g].gs);
  }
};

// The exponential-block carries CE[e] (0 <= e <= nbe) from the two levels.
struct ECarries {
  const u128* __restrict__ PE;
  const u128* __restrict__ TEx;
  uint32_t nbe, Ge;
  __device__ __forceinline__ u128 operator[](uint32_t e) const {
    if (e >= nbe) return TEx[Ge];
    return TEx[e >> kGrpLog] + PE[e];
  }
};

__host__ __device__ constexpr uint32_t carry_groups(uint32_t nblocks) {
  return (nblocks + kGrp - 1) / kGrp;
}

// Direct carries: with at most kDirectMax blocks every emit workgroup derives
// the global scale, its own exact carry and the total from all records itself,
// which saves the carry kernel.
constexpr uint32_t kDirectMax = kT * 8;

// ---------------------------------------------------------------- one block per wave
// The stratified and systematic emission and the records pass run one
// 1024-weight block per wave, lane l holding particles 16 l .. 16 l + 15 of
// the block, four waves (four consecutive blocks) per workgroup.  A block's
// prefix then needs no workgroup barrier: the lane sums its 16 quantised
// weights and one DPP scan over the wave gives the lane's offset.  r is formed
// from the exact block carry by an affine map in binary64,
//   r_i = min(fl(L_i c + r(C_b)), r(C_{b+1})),  c = n 2^(gscale - scale_b) / Q,
// with L_i the block's exact integer prefix (below 2^63) rounded once: the map
// is monotone in L_i, flat over zero weights and clamped to the block's range,
// so O_i is monotone across blocks as well; it adds at most five roundings of
// n 2^-53 to the error of r against the exact value.
constexpr int kWPer = kBlock / kWave;  // particles per lane (16)
constexpr int kWavesPerWG = kT / kWave;
constexpr int kUTabW = 2048;           // stratum offset words cached per wave

template <typename T>
__device__ __forceinline__ void wave_load(const T* __restrict__ w, int64_t n, int64_t base,
                                          T (&x)[kWPer]) {
  const int64_t idx = base + (int64_t)lane_id() * kWPer;
  const bool aligned = ((reinterpret_cast<uintptr_t>(w + idx) & 15u) == 0);
  if (aligned && idx + kWPer <= n) {
    if constexpr (sizeof(T) == 4) {
      const float4* p = reinterpret_cast<const float4*>(w + idx);
#pragma unroll
      for (int k = 0; k < kWPer / 4; ++k) {
        const float4 t = p[k];
        x[4 * k] = t.x; x[4 * k + 1] = t.y; x[4 * k + 2] = t.z; x[4 * k + 3] = t.w;
      }
    } else {
      const double2* p = reinterpret_cast<const double2*>(w + idx);
#pragma unroll
      for (int k = 0; k < kWPer / 2; ++k) {
        const double2 t = p[k];
        x[2 * k] = t.x; x[2 * k + 1] = t.y;
      }
    }
  } else {
#pragma unroll
    for (int v = 0; v < kWPer; ++v) x[v] = (idx + v < n) ? w[idx + v] : (T)0;
  }
}

// The block's weights in an order in which every load instruction is
// coalesced (lane l takes the 16-byte pieces l, l + 64, ... of the block), for
// the record, whose maximum and sum do not depend on the order.  Values past
// the vector's end are zero.
template <typename T>
__device__ __forceinline__ void wave_load_unordered(const T* __restrict__ w, int64_t n,
                                                    int64_t base, T (&x)[kWPer]) {
  constexpr int kV = 16 / (int)sizeof(T);  // values per 16-byte piece
  const int lane = (int)lane_id();
  const bool aligned = ((reinterpret_cast<uintptr_t>(w + base) & 15u) == 0);
  if (aligned && base + kBlock <= n) {
#pragma unroll
    for (int k = 0; k < kWPer / kV; ++k) {
      const int64_t idx = base + (int64_t)(k * kWave + lane) * kV;
      if constexpr (sizeof(T) == 4) {
        const float4 t = *reinterpret_cast<const float4*>(w + idx);
        x[4 * k] = t.x; x[4 * k + 1] = t.y; x[4 * k + 2] = t.z; x[4 * k + 3] = t.w;
      } else {
        const double2 t = *reinterpret_cast<const double2*>(w + idx);
        x[2 * k] = t.x; x[2 * k + 1] = t.y;
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < kWPer / kV; ++k)
#pragma unroll
      for (int v = 0; v < kV; ++v) {
        const int64_t idx = base + (int64_t)(k * kWave + lane) * kV + v;
        x[kV * k + v] = idx < n ? w[idx] : (T)0;
      }
  }
}

// wave_load of a whole, 16-byte aligned float32 block through 4 KB of the
// wave's LDS: the global loads are coalesced (lane l takes the 16-byte pieces
// l, l + 64, ...) and the lanes read their 16 consecutive weights back.  Piece
// u sits at u ^ ((u >> 4) & 3), so that 16 lanes reading pieces 4l + k touch
// 16 different bank groups.  Other blocks and binary64 load directly.
template <typename T>
__device__ __forceinline__ void wave_load_staged(const T* __restrict__ w, int64_t n, int64_t base,
                                                 T (&x)[kWPer], int32_t* stage) {
  if constexpr (sizeof(T) == 4) {
    const bool aligned = ((reinterpret_cast<uintptr_t>(w + base) & 15u) == 0);
    if (stage && aligned && base + kBlock <= n) {
      const int lane = (int)lane_id();
      const float4* g = reinterpret_cast<const float4*>(w + base);
      float4* S = reinterpret_cast<float4*>(stage);
      float4 t[kWPer / 4];
#pragma unroll
      for (int k = 0; k < kWPer / 4; ++k) t[k] = g[k * kWave + lane];
#pragma unroll
      for (int k = 0; k < kWPer / 4; ++k) {
        const int u = k * kWave + lane;
        S[u ^ ((u >> 4) & 3)] = t[k];
      }
      wave_lds_sync();
#pragma unroll
      for (int k = 0; k < kWPer / 4; ++k) {
        const int u = lane * (kWPer / 4) + k;
        const float4 v = S[u ^ ((u >> 4) & 3)];
        x[4 * k] = v.x; x[4 * k + 1] = v.y; x[4 * k + 2] = v.z; x[4 * k + 3] = v.w;
      }
      wave_lds_sync();
      return;
    }
  }
  wave_load(w, n, base, x);
}

// quantize() without branches: q = floor(v 2^scale) for every finite v >= 0
// of a block whose scale keeps q below 2^53.  binary32: scaling by a power of
// two is exact (a result below 2^-126 may round, but it floors to zero
// anyway), the floor is exact, and q splits exactly into two 32-bit halves
// (t - hi 2^32 keeps at most t's 24 significant bits).  binary64: the
// significand shifted by scale + exponent - 1075, truncated.
template <typename T>
__device__ __forceinline__ uint64_t quantize_nb(T v, int scale) {
  if constexpr (sizeof(T) == 4) {
    const float t = floorf(ldexpf(v, scale));
    const float hi = floorf(t * 0x1p-32f);
    const float lo = __builtin_fmaf(hi, -0x1p32f, t);
    // the pair as one value, or sums of it become two additions
    uint64_t q = ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
    asm("" : "+v"(q));
    return q;
  } else {
    typedef WTraits<T> Tr;
    const uint64_t b = Tr::bits(v);
    const uint32_t ef = (uint32_t)((b >> 52) & 0x7FFu);
    const uint64_t m = (b & 0xFFFFFFFFFFFFFull) | (ef ? (1ull << 52) : 0ull);
    const int sh = (int)(ef < 1u ? 1u : ef) - 1075 + scale;
    const uint64_t up = m << (sh & 63);
    const uint64_t dn = m >> (uint32_t)min(-sh, 63);
    return sh >= 0 ? up : dn;
  }
}

// u64 -> binary64, rounded once (the high half converts exactly).
__device__ __forceinline__ double u64_to_f64(uint64_t x) {
  uint32_t hi = (uint32_t)(x >> 32);
  asm("" : "+v"(hi));  // a 32-bit conversion
  return __fma_rn((double)hi, 0x1p32, (double)(uint32_t)x);
}

// r (or a point p) of the local prefix L by a block's affine map, clamped to
// the block's upper end; the whole block sum is that end exactly.  No branch:
// the two selects cost less than the exec masks of one.
__device__ __forceinline__ double affine_r(uint64_t L, uint64_t total, double c, double lo,
                                           double hi) {
  const double rv = fmin(__fma_rn(u64_to_f64(L), c, lo), hi);
  return L == total ? hi : rv;
}

// O(r) = #{s : s + 1 - u_s <= r}, exactly, for 0 <= r <= n < 2^31 and
// t = 1 - u_m in (0, 1], m = floor(r): m + [frac(r) >= t].  At r = n the
// fraction is 0, so any t gives n.
__device__ __forceinline__ uint32_t cum_at(double r, double t) {
  return (uint32_t)(int32_t)r + (__builtin_amdgcn_fract(r) >= t ? 1u : 0u);
}

// Record of the block at base (one wave): validity, reference exponent, sum.
template <typename T>
__device__ __forceinline__ BlockRec wave_block_record(const T* __restrict__ w, int64_t n, int64_t base) {
  T x[kWPer];
  wave_load_unordered(w, n, base, x);
  uint32_t bad = 0, emax = 1;
#pragma unroll
  for (int v = 0; v < kWPer; ++v) {
    if (!weight_ok(x[v])) bad = FLAG_BAD_WEIGHTS;
    else emax = max(emax, (uint32_t)exp_field(x[v]));
  }
  const uint32_t key = wave_reduce((bad << 16) | emax, OpMax());
  BlockRec r;
  r.bad = key >> 16;
  const int e_ref = (int)(key & 0xFFFFu);
  r.scale = scale_of<T>(e_ref);
  uint64_t sum = 0;
  if (!r.bad) {
#pragma unroll
    for (int v = 0; v < kWPer; ++v) sum += quantize_nb(x[v], r.scale);
  }
  r.sum = readlane(wave_incl_add_u64(sum), kWave - 1);
  return r;
}

// r of the wave's block: lane l gets r_i of particles P0 + 16 l + v (values
// past the vector's end repeat the last one), and the block's range
// [r(C_b), r(C_{b+1})].
struct BlockR {
  double r[kWPer];
  double lo, hi;
};

template <typename T>
__device__ __forceinline__ void block_r_wave(const T* __restrict__ w, int64_t n, int64_t P0,
                                             const BlockRec rec, u128 Cb, u128 Cb1,
                                             int32_t gscale, u128 Q, BlockR& R,
                                             int32_t* stage = nullptr) {
  const RMap rm = make_rmap(Q, n);
  R.lo = rm(Cb);
  R.hi = rm(Cb1);
  const int32_t scale = (int32_t)__builtin_amdgcn_readfirstlane(rec.scale);
  const int sh = (int32_t)__builtin_amdgcn_readfirstlane(gscale) - scale;
  const double c = ldexp(rm.Nd * rm.invQ, sh);
  T x[kWPer];
  wave_load_staged(w, n, P0, x, stage);
  uint64_t q[kWPer];
  uint64_t acc = 0;
#pragma unroll
  for (int v = 0; v < kWPer; ++v) {
    acc += quantize_nb(x[v], scale);
    q[v] = acc;
  }
  const uint64_t incl = wave_incl_add_u64(acc);
  const uint64_t off = incl - acc;
  const uint64_t total = readlane(incl, kWave - 1);
  // every particle from the block's last positive weight on has the whole
  // block sum, i.e. r = r(C_{b+1}) exactly: that particle then ends the
  // block's range, as in exact arithmetic
#pragma unroll
  for (int v = 0; v < kWPer; ++v) {
    R.r[v] = affine_r(off + q[v], total, c, R.lo, R.hi);
  }
}

// Expansion of cumulative offspring into ancestors, 1024 outputs at a time:
// the block's outputs are [O_lo, O_hi) and particle P0 + 16 lane + v takes
// [Op[v], O[v]).  A marker at the first output of every run, a max-scan (16
// values per lane in registers, then over the wave), the result written back
// to LDS and stored row by row (coalesced).
__device__ __forceinline__ void expand_wave(const uint32_t (&O)[kWPer], const uint32_t (&Op)[kWPer],
                                            uint32_t O_lo, uint32_t O_hi, int64_t P0, int64_t n,
                                            int32_t* __restrict__ a_out, int32_t* M) {
  const int lane = (int)lane_id();
  O_hi = min(O_hi, (uint32_t)n);  // (never binds: every O is at most n)
  int32_t carry = -1;  // particle covering the first output of the chunk
  int4* M4 = reinterpret_cast<int4*>(M) + lane * (kWPer / 4);
  const int32_t P0_32 = (int32_t)P0;
  for (uint32_t cs = O_lo; cs < O_hi; cs += kBlock) {
    const uint32_t len = min((uint32_t)kBlock, O_hi - cs);
#pragma unroll
    for (int k = 0; k < kWPer / 4; ++k) M4[k] = make_int4(-1, -1, -1, -1);
    wave_lds_sync();
    // (a particle that starts no run in this chunk writes the spare slot)
#pragma unroll
    for (int v = 0; v < kWPer; ++v) {
      const uint32_t pos = Op[v] - cs;
      M[(O[v] > Op[v] && pos < len) ? pos : (uint32_t)kBlock] = lane * kWPer + v;
    }
    wave_lds_sync();
    int32_t m[kWPer];
#pragma unroll
    for (int k = 0; k < kWPer / 4; ++k) {
      const int4 t = M4[k];
      m[4 * k] = t.x; m[4 * k + 1] = t.y; m[4 * k + 2] = t.z; m[4 * k + 3] = t.w;
    }
#pragma unroll
    for (int k = 1; k < kWPer; ++k) m[k] = max(m[k], m[k - 1]);
    const int32_t incl = wave_incl_max_i32(m[kWPer - 1]);
    const int32_t before = max(carry, (int32_t)wave_shift_up_u32((uint32_t)incl, 0xFFFFFFFFu));
#pragma unroll
    for (int k = 0; k < kWPer; ++k) m[k] = max(m[k], before);
    carry = (int32_t)__builtin_amdgcn_readlane(m[kWPer - 1], kWave - 1);
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < kWPer / 4; ++k) {
      M4[k] = make_int4(m[4 * k], m[4 * k + 1], m[4 * k + 2], m[4 * k + 3]);
    }
    wave_lds_sync();
    int32_t* __restrict__ a_chunk = a_out + cs;  // the same on every lane
#pragma unroll
    for (int j = 0; j < kWPer; ++j) {
      const uint32_t p = (uint32_t)lane + (uint32_t)j * kWave;
      if (p < len) a_chunk[p] = P0_32 + M[p];
    }
    wave_lds_sync();
  }
}

// The claimed slots of the wave's block, 16 bits a lane.
__device__ __forceinline__ void wave_claim_bits(const uint32_t (&O)[kWPer],
                                                const uint32_t (&Op)[kWPer], int64_t P0,
                                                uint32_t* __restrict__ claim) {
  uint32_t bits = 0;
#pragma unroll
  for (int v = 0; v < kWPer; ++v) bits |= (O[v] > Op[v] ? 1u : 0u) << v;
  reinterpret_cast<uint16_t*>(claim)[(P0 >> 4) + lane_id()] = (uint16_t)bits;
}
// The identity of a zero or invalid total over a block: every position claims
// its own slot.  Called by `threads` consecutive threads, the first one t = 0.
__device__ __forceinline__ void block_identity(int64_t P0, int64_t n, int t, int threads,
                                               int32_t* __restrict__ a,
                                               uint32_t* __restrict__ claim) {
  for (int64_t i = P0 + t; i < min(P0 + kBlock, n); i += threads) a[i] = (int32_t)i;
  if (claim && t < kBlock / 32) claim[(P0 >> 5) + t] = 0xFFFFFFFFu;
}

template <bool SYSTEMATIC>
struct StrataWaveLds {
  alignas(16) int32_t M[kBlock + 4];                   // expansion markers, then the expanded chunk; M[kBlock] spare
  uint32_t u[SYSTEMATIC ? 1 : kUTabW];     // raw offset words of strata [m_lo, m_lo + kUTabW)
};

// Stratified / systematic emission of one block by one wave: the block's
// particles are P0 .. P0 + cnt - 1 of a vector of n, with exclusive exact
// carry Cb and inclusive Cb1 at global scale gscale, total Q.  Writes a_out[s]
// = P0 + i for every s in [O_{i-1}, O_i); with claim also the claimed slots of
// Code 10's Prepermute, one bit per particle (the output is sorted, so a slot
// is claimed when its particle has offspring; the winners, the first positions
// of the runs, show in the ancestry itself).
template <typename T, bool SYSTEMATIC>
__device__ __forceinline__ void emit_block_wave(const T* __restrict__ w, int64_t n, int64_t P0,
                                                const BlockRec rec, u128 Cb, u128 Cb1,
                                                int32_t gscale, u128 Q, Key key, uint32_t filter,
                                                uint32_t offset, int32_t* __restrict__ a_out,
                                                StrataWaveLds<SYSTEMATIC>* L,
                                                uint32_t* __restrict__ claim) {
  const int lane = (int)lane_id();
  const int cnt = (int)min((int64_t)kBlock, n - P0);
  BlockR R;
  block_r_wave(w, n, P0, rec, Cb, Cb1, gscale, Q, R, L->M);
  if (!(R.hi > R.lo) && !claim) return;  // an empty range has no outputs

  // stratum offsets of the strata the block's range touches
  const int64_t m_lo = (int64_t)floor(R.lo);
  const int64_t m_hi = min(n - 1, (int64_t)floor(R.hi));
  const bool table = !SYSTEMATIC && (m_hi - m_lo + 1 <= kUTabW);
  const double t_sys =
      SYSTEMATIC ? 1.0 - u_offset(draw_uniform(key, 0, DOM_STRATA, 0, filter, offset).x) : 0.0;
  if (table && m_hi >= m_lo) {
    for (int64_t cc = (m_lo >> 2) + lane; cc <= (m_hi >> 2); cc += kWave) {
      const uint4 xw = draw(key, (uint32_t)cc, DOM_STRATA, 0, filter, offset);
      const uint32_t xs[4] = {xw.x, xw.y, xw.z, xw.w};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t m = cc * 4 + v;
        if (m >= m_lo && m <= m_hi) L->u[m - m_lo] = xs[v];
      }
    }
    wave_lds_sync();
  }
  const int32_t n32 = (int32_t)n, mlo32 = (int32_t)m_lo;
  auto cum_sys = [&](double rv) -> uint32_t { return cum_at(rv, t_sys); };
  auto cum_tab = [&](double rv) -> uint32_t {
    const int32_t m = (int32_t)rv;
    return cum_at(rv, 1.0 - u_offset(L->u[m >= n32 ? 0 : m - mlo32]));
  };
  auto cum_draw = [&](double rv) -> uint32_t {
    return cum_at(rv, 1.0 - u_offset(stratum_word(key, filter, offset, (int32_t)rv)));
  };
  uint32_t O[kWPer];
  uint32_t O_lo, O_hi;
  if (SYSTEMATIC) {
#pragma unroll
    for (int v = 0; v < kWPer; ++v) O[v] = cum_sys(R.r[v]);
    O_lo = cum_sys(R.lo);
    O_hi = cum_sys(R.hi);
  } else if (table) {
#pragma unroll
    for (int v = 0; v < kWPer; ++v) O[v] = cum_tab(R.r[v]);
    O_lo = cum_tab(R.lo);
    O_hi = cum_tab(R.hi);
  } else {
#pragma unroll
    for (int v = 0; v < kWPer; ++v) O[v] = cum_draw(R.r[v]);
    O_lo = cum_draw(R.lo);
    O_hi = cum_draw(R.hi);
  }
  O_lo = (uint32_t)__builtin_amdgcn_readfirstlane(O_lo);
  O_hi = (uint32_t)__builtin_amdgcn_readfirstlane(O_hi);
  uint32_t Op[kWPer];
  Op[0] = wave_shift_up_u32(O[kWPer - 1], O_lo);
#pragma unroll
  for (int v = 1; v < kWPer; ++v) Op[v] = O[v - 1];

  if (claim) wave_claim_bits(O, Op, P0, claim);
  expand_wave(O, Op, O_lo, O_hi, P0, n, a_out, L->M);
}

// ---------------------------------------------------------------- multinomial, one block per wave
// The points p_k = n S_k / S_n of the exponential spacings are formed per
// exponential block as r is per weight block: the block's exact carry CE[e]
// plus the lane's quantised spacings, by the affine map (p of the block's
// last spacing pinned to r(CE[e+1]), so blocks meet exactly).  A weight
// block's particles need O_i = #{k : p_k < r_i}, the cumulative offspring:
// particle i is then the ancestor of outputs [O_{i-1}, O_i), which is
// a_k = #{i : r_i <= p_k}, the upper-bound search of Code 5 (below n - 1, as
// i < cnt).  O_i comes from a binary search over the 1024 points of the one
// exponential block whose range holds r_i, in LDS; the wave walks the
// exponential blocks from the one holding the first point at or above
// r(C_b) to the one holding the first at or above r(C_{b+1}) (usually one or
// two), and the expansion is the one of the stratified scheme.
struct MultiWaveLds {
  double P[kBlock];                   // the points of one exponential block
  alignas(16) int32_t M[kBlock + 4];  // expansion markers; M[kBlock] spare
};

// The lane's 16 quantised spacings of exponential block e (indices
// 1024 e + 16 lane + v): as the records pass stored them (STORED), or drawn
// again (the one-workgroup batch path, which keeps no spacings).
template <bool STORED>
__device__ __forceinline__ void exp_values_wave(Key key, uint32_t filter, uint32_t offset,
                                                int64_t n, uint32_t e,
                                                const uint64_t* __restrict__ evals,
                                                uint64_t (&q)[kWPer]) {
  const int lane = (int)lane_id();
  if constexpr (STORED) {
    const ulonglong2* p =
        reinterpret_cast<const ulonglong2*>(evals + (size_t)e * kBlock + lane * kWPer);
#pragma unroll
    for (int k = 0; k < kWPer / 2; ++k) {
      const ulonglong2 t = p[k];
      q[2 * k] = t.x;
      q[2 * k + 1] = t.y;
    }
  } else {
#pragma unroll
    for (int c = 0; c < kWPer / 4; ++c) {
      const uint32_t call = e * (uint32_t)(kBlock / 4) + (uint32_t)lane * (kWPer / 4) + c;
      const uint4 x = draw(key, call, DOM_EXP, 0, filter, offset);
      const uint32_t xs[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t k = (int64_t)call * 4 + v;
        const double ev = neg_log_spacing(xs[v]);
        q[4 * c + v] = (k <= n) ? (uint64_t)(ev * 0x1p48) : 0ull;
      }
    }
  }
}

// Exponential block holding the first point at or above x: the number of
// blocks whose last point P(b + 1) = em(CE[b + 1]) lies below x.  The last
// points sit within a few blocks of (b + 1) 1024 n / (n + 1), so one probe of
// 256 consecutive boundaries (four per lane) around the guess settles it; a
// bisection is the fallback.
template <typename CEPtr>
__device__ __forceinline__ uint32_t exp_block_of(double x, int64_t n, CEPtr CE, uint32_t nbe,
                                                 const RMap& em) {
  const double per_block = (double)kBlock * (double)n / (double)(n + 1);
  int64_t w0 = (int64_t)(x / per_block) - 128;  // first probed boundary index b + 1
  if (w0 < 1) w0 = 1;
  const int64_t last = (int64_t)nbe - 1;  // boundaries 1 .. nbe - 1
  const int lane = (int)lane_id();
  uint32_t below = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t b = w0 + lane * 4 + k;
    below += (b <= last && em(CE[b]) < x) ? 1u : 0u;
  }
  below = wave_reduce(below, OpAdd());
  const int64_t w1 = min(w0 + 255, last);
  const int64_t span = w1 - w0 + 1;
  const bool ok = w0 > last || ((w0 == 1 || below > 0) && (w1 == last || (int64_t)below < span));
  if (ok) return (uint32_t)(w0 > last ? last : w0 - 1 + below);
  uint32_t lo = 1, hi = nbe;  // #{b in [1, nbe - 1] : P(b) < x}
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (em(CE[mid]) < x) lo = mid + 1;
    else hi = mid;
  }
  return lo - 1;
}

template <typename T, bool STORED, typename CEPtr>
__device__ __forceinline__ void emit_multi_wave(const T* __restrict__ w, int64_t n, int64_t P0,
                                                const BlockRec rec, u128 Cb, u128 Cb1,
                                                int32_t gscale, u128 Q, Key key, uint32_t filter,
                                                uint32_t offset, CEPtr CE, uint32_t nbe,
                                                const uint64_t* __restrict__ evals,
                                                int32_t* __restrict__ a_out, MultiWaveLds* L,
                                                uint32_t* __restrict__ claim = nullptr) {
  const int lane = (int)lane_id();
  const int cnt = (int)min((int64_t)kBlock, n - P0);
  BlockR R;
  block_r_wave(w, n, P0, rec, Cb, Cb1, gscale, Q, R, L->M);
  if (!(R.hi > R.lo) && !claim) return;  // an empty range has no outputs
  const RMap em = make_rmap(CE[nbe], n);
  const double ce = em.Nd * em.invQ;
  const uint32_t e_first = (uint32_t)__builtin_amdgcn_readfirstlane(exp_block_of(R.lo, n, CE, nbe, em));
  const uint32_t e_last = (uint32_t)__builtin_amdgcn_readfirstlane(exp_block_of(R.hi, n, CE, nbe, em));
  uint32_t O[kWPer];
#pragma unroll
  for (int v = 0; v < kWPer; ++v) O[v] = 0;
  uint32_t det = 0;  // bit v: O[v] is known
  uint32_t O_lo = 0, O_hi = 0;
  bool lo_det = false, hi_det = false;
  double2* P2 = reinterpret_cast<double2*>(L->P) + lane * (kWPer / 2);
  // lower bound in the block's points (x at most its last point)
  auto lb = [&](double x) -> uint32_t {
    uint32_t pos = (L->P[kBlock / 2 - 1] < x) ? (uint32_t)(kBlock / 2) : 0u;
#pragma unroll
    for (uint32_t st = kBlock / 4; st > 0; st >>= 1) pos += (L->P[pos + st - 1] < x) ? st : 0u;
    return pos;
  };
  for (uint32_t e = e_first; e <= e_last; ++e) {
    uint64_t q[kWPer];
    exp_values_wave<STORED>(key, filter, offset, n, e, evals, q);
    uint64_t acc = 0;
#pragma unroll
    for (int v = 0; v < kWPer; ++v) {
      acc += q[v];
      q[v] = acc;
    }
    const uint64_t incl = wave_incl_add_u64(acc);
    const uint64_t off = incl - acc;
    const uint64_t total = readlane(incl, kWave - 1);
    const double p_base = em(CE[e]), p_top = em(CE[e + 1]);
#pragma unroll
    for (int k = 0; k < kWPer / 2; ++k) {
      double pv[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        pv[h] = affine_r(off + q[2 * k + h], total, ce, p_base, p_top);
      }
      P2[k] = make_double2(pv[0], pv[1]);
    }
    wave_lds_sync();
    const uint32_t base = e * (uint32_t)kBlock;
    // the particles this block settles: not settled yet and r <= its last
    // point; eight of the lane's searches run step by step together, so that
    // their LDS reads are in flight at the same time (eight, not sixteen,
    // bounds the registers the reads hold: three waves per SIMD instead of one)
    uint32_t need = 0;
#pragma unroll
    for (int v = 0; v < kWPer; ++v)
      need |= (!((det >> v) & 1u) && R.r[v] <= p_top) ? (1u << v) : 0u;
#pragma unroll
    for (int h = 0; h < kWPer; h += kWPer / 2) {
      const uint32_t need_h = need & (((1u << (kWPer / 2)) - 1u) << h);
      if (ballot(need_h != 0)) {
        uint32_t pos[kWPer / 2];
#pragma unroll
        for (int v = 0; v < kWPer / 2; ++v)
          pos[v] = (L->P[kBlock / 2 - 1] < R.r[h + v]) ? (uint32_t)(kBlock / 2) : 0u;
#pragma unroll
        for (uint32_t st = kBlock / 4; st > 0; st >>= 1) {
#pragma unroll
          for (int v = 0; v < kWPer / 2; ++v)
            pos[v] += (L->P[pos[v] + st - 1] < R.r[h + v]) ? st : 0u;
        }
#pragma unroll
        for (int v = 0; v < kWPer / 2; ++v)
          if ((need_h >> (h + v)) & 1u) O[h + v] = base + pos[v];
      }
    }
    det |= need;
    if (!lo_det && R.lo <= p_top) {
      O_lo = base + lb(R.lo);
      lo_det = true;
    }
    if (!hi_det && R.hi <= p_top) {
      O_hi = base + lb(R.hi);
      hi_det = true;
    }
    wave_lds_sync();
  }
  O_lo = (uint32_t)__builtin_amdgcn_readfirstlane(O_lo);
  O_hi = (uint32_t)__builtin_amdgcn_readfirstlane(O_hi);
  uint32_t Op[kWPer];
  Op[0] = wave_shift_up_u32(O[kWPer - 1], O_lo);
#pragma unroll
  for (int v = 1; v < kWPer; ++v) Op[v] = O[v - 1];
  if (claim) wave_claim_bits(O, Op, P0, claim);
  expand_wave(O, Op, O_lo, O_hi, P0, n, a_out, L->M);
}

// Weight records, one block per wave (blockIdx.x < wgs_b), and for the
// multinomial scheme the exponential blocks (one per workgroup beyond them).
template <typename T, bool MULTI>
__global__ __launch_bounds__(kT) void k_scan_records_w(const T* __restrict__ w, int64_t n,
                                                       uint32_t nb, uint32_t wgs_b, Key key,
                                                       uint32_t offset, uint32_t filter,
                                                       BlockRec* __restrict__ recs,
                                                       uint64_t* __restrict__ esums,
                                                       uint64_t* __restrict__ evals,
                                                       ScanHeader* __restrict__ hdr) {
  offset = counter_offset(key, offset);
  if (blockIdx.x == 0 && threadIdx.x == 0) hdr->groups_done = 0;  // for the carries pass
  if (blockIdx.x < wgs_b) {
    const uint32_t b = blockIdx.x * kWavesPerWG +
                       (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (b >= nb) return;
    const BlockRec r = wave_block_record(w, n, (int64_t)b * kBlock);
    if (lane_id() == 0) recs[b] = r;
  } else if (MULTI) {
    __shared__ WgScratch s;
    const uint32_t b = blockIdx.x - wgs_b;
    uint64_t q[kPer];
    exp_values(key, filter, offset, n, b, q);
    store_exp_values(evals, b, q);
    const uint64_t sum = wg_reduce(q[0] + q[1] + q[2] + q[3], OpAdd(), s.u);
    if (threadIdx.x == 0) esums[b] = sum;
  }
}

// ---------------------------------------------------------------- one block per workgroup
// The emission of a single vector with one 1024-weight block per workgroup of
// four waves, four weights per thread.  At up to about a thousand blocks the
// wave form above leaves one wave per SIMD, whose serial latency (16 weights a
// lane, and some 20 KB of straight-line code fetched once) is the call; here
// the chain is a quarter as long, and its code is fetched for four times the
// waves.  Kernel time, systematic, 2^16 / 2^18 / 2^20 weights: 8.7 / 10.9 / 13.1
// (with the carries pass) -> 5.8 / 6.4 / 9.9 us; from 2^21 on the wave form is
// faster (2^21 10.6 against 13.6 us, 2^24 38 against 70 us: fewer barriers).
//
// Carries.  Each workgroup reduces all records itself, up to kGrp blocks four
// per thread; the values are those of the carries pass.
struct WgCarry {
  u128 Cb, Cb1, Q;
  int32_t gscale;
  uint32_t status;
};

struct CarryScratch {
  uint32_t key[kNW], bad[kNW];
  u128 before[kNW], all[kNW];
};

// min over the workgroup of the scale keys and or of the bad flags, in
// registers of every thread after the barrier inside.
__device__ __forceinline__ void wg_key_bad(uint32_t& key, uint32_t& bad, CarryScratch* s) {
  const int wave = (int)threadIdx.x / kWave;
  key = ~wave_max_u32(~key);
  bad = ballot(bad != 0) ? FLAG_BAD_WEIGHTS : 0u;
  if (lane_id() == 0) {
    s->key[wave] = key;
    s->bad[wave] = bad;
  }
  __syncthreads();
#pragma unroll
  for (int w2 = 0; w2 < kNW; ++w2) {
    key = min(key, s->key[w2]);
    bad |= s->bad[w2];
  }
}
// Workgroup sums of two 128-bit values.
__device__ __forceinline__ void wg_sum2(u128& x, u128& y, CarryScratch* s) {
  const int wave = (int)threadIdx.x / kWave;
  x = wave_incl_add_u128(x);
  y = wave_incl_add_u128(y);
  if (lane_id() == kWave - 1) {
    s->before[wave] = x;
    s->all[wave] = y;
  }
  __syncthreads();
  x = y = 0;
#pragma unroll
  for (int w2 = 0; w2 < kNW; ++w2) {
    x += s->before[w2];
    y += s->all[w2];
  }
}

// Blocks up to which the records are converted straight to the global scale;
// beyond, up to one group, they go through the group's scale, as in the
// carries pass (the two differ, by truncation, only for blocks 2^27 times
// lighter than the heaviest).
constexpr uint32_t kStraight = 256;

__device__ __forceinline__ WgCarry direct_carries(uint32_t nb, uint32_t b,
                                                  const BlockRec* __restrict__ recs,
                                                  const BlockRec& own, CarryScratch* s,
                                                  uint32_t straight = kStraight) {
  // record j = r kT + thread, so that a load covers consecutive records
  constexpr int kR = (int)(kDirectMax / kT);
  uint32_t key = 0xFFFFFFFFu, bad = 0;
  u128 before = 0, all = 0;
  if (nb <= kGrp) {
    BlockRec r[kGPer];
#pragma unroll
    for (int k = 0; k < kGPer; ++k) {
      const uint32_t j = (uint32_t)k * kT + threadIdx.x;
      if (j < nb) r[k] = recs[j];
      else r[k].sum = 0, r[k].scale = 0, r[k].bad = 0;
    }
#pragma unroll
    for (int k = 0; k < kGPer; ++k) {
      bad |= r[k].bad;
      if (r[k].sum) key = min(key, (uint32_t)r[k].scale ^ 0x80000000u);
    }
    wg_key_bad(key, bad, s);
    const bool none = key == 0xFFFFFFFFu;
    const int32_t top = (int32_t)(key ^ 0x80000000u) + (kCarryBits - 63);
    const int32_t gscale = none ? 0 : top - ceil_log2(nb);
    const int32_t via = none ? 0 : nb <= straight ? gscale : top - kGrpLog;
#pragma unroll
    for (int k = 0; k < kGPer; ++k) {
      const uint32_t j = (uint32_t)k * kT + threadIdx.x;
      const u128 v = conv_rec_fast(r[k], via);
      all += v;
      before += j < b ? v : (u128)0;
    }
    wg_sum2(before, all, s);
    WgCarry c;
    c.gscale = gscale;
    c.Cb = shift_u128(before, gscale - via);
    c.Cb1 = shift_u128(before + conv_rec_fast(own, via), gscale - via);
    c.Q = shift_u128(all, gscale - via);
    c.status = bad | (!bad && c.Q == 0 ? FLAG_ZERO_TOTAL : 0u);
    return c;
  }
  for (int k = 0; k < kR; ++k) {
    const uint32_t j = (uint32_t)k * kT + threadIdx.x;
    if (j < nb) {
      const BlockRec r = recs[j];
      bad |= r.bad;
      if (r.sum) key = min(key, (uint32_t)r.scale ^ 0x80000000u);
    }
  }
  wg_key_bad(key, bad, s);
  const int32_t gscale = key == 0xFFFFFFFFu ? 0
                                            : (int32_t)(key ^ 0x80000000u) + (kCarryBits - 63) -
                                                  ceil_log2(nb);
  for (int k = 0; k < kR; ++k) {
    const uint32_t j = (uint32_t)k * kT + threadIdx.x;
    if (j < nb) {
      const u128 v = conv_rec_fast(recs[j], gscale);
      all += v;
      before += j < b ? v : (u128)0;
    }
  }
  wg_sum2(before, all, s);
  WgCarry c;
  c.gscale = gscale;
  c.Cb = before;
  c.Cb1 = before + conv_rec_fast(own, gscale);
  c.Q = all;
  c.status = bad | (!bad && c.Q == 0 ? FLAG_ZERO_TOTAL : 0u);
  return c;
}

// Four consecutive weights of the block (zeros past the end); the vector
// starts anywhere, so the wide load is aligned to one weight only.
template <typename T>
__device__ __forceinline__ void load4_any(const T* __restrict__ w, int64_t n, int64_t base,
                                          T (&x)[kPer]) {
  const int64_t idx = base + (int64_t)threadIdx.x * kPer;
  if (idx + kPer <= n) {
    typedef T V __attribute__((ext_vector_type(4), aligned(sizeof(T))));
    const V t = *reinterpret_cast<const V*>(w + idx);
    x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w;
  } else {
#pragma unroll
    for (int v = 0; v < kPer; ++v) x[v] = (idx + v < n) ? w[idx + v] : (T)0;
  }
}

// r of the thread's four particles and of the particle before them (the
// formula of block_r_wave; the block's lower end before its first particle).
struct WgR {
  double r[kPer], prev, lo, hi;
};
struct PrefixScratch {
  uint64_t sum[kNW];
};
// The thread's quantised weights as inclusive prefixes inside the thread, and
// their sum, which goes to the scratch per wave (a barrier must follow).
template <typename T>
__device__ __forceinline__ uint64_t wg_quantize(const T (&x)[kPer], int32_t scale,
                                                uint64_t (&q)[kPer], PrefixScratch* s) {
  uint64_t acc = 0;
#pragma unroll
  for (int v = 0; v < kPer; ++v) {
    acc += quantize_nb(x[v], scale);
    q[v] = acc;
  }
  const uint64_t incl = wave_incl_add_u64(acc);
  if (lane_id() == kWave - 1) s->sum[threadIdx.x / kWave] = incl;
  return incl - acc;  // exclusive inside the wave
}
__device__ __forceinline__ void wg_block_r(const uint64_t (&q)[kPer], uint64_t off,
                                           const PrefixScratch* s, int32_t scale,
                                           const WgCarry& C, int64_t n, WgR& R) {
  const int wave = (int)threadIdx.x / kWave;
  uint64_t total = 0;
#pragma unroll
  for (int w2 = 0; w2 < kNW; ++w2) {
    off += w2 < wave ? s->sum[w2] : 0ull;
    total += s->sum[w2];
  }
  const RMap rm = make_rmap(C.Q, n);
  R.lo = rm(C.Cb);
  R.hi = rm(C.Cb1);
  const double c = ldexp(rm.Nd * rm.invQ, C.gscale - scale);
  auto r_of = [&](uint64_t L) -> double { return affine_r(L, total, c, R.lo, R.hi); };
  R.prev = off ? r_of(off) : R.lo;  // (no weight before: the block's lower end)
#pragma unroll
  for (int v = 0; v < kPer; ++v) R.r[v] = r_of(off + q[v]);
}

// Expansion of cumulative offspring into ancestors, as expand_wave: 2048
// outputs a round, eight consecutive ones per thread, 16-byte stores.
constexpr int kOut = 8;  // outputs per thread and round
struct ExpandLds {
  alignas(16) int32_t M[kT * kOut + 4];
  int32_t top[kNW];
};
__device__ __forceinline__ void wg_markers_clear(ExpandLds* L) {
  int4* M4 = reinterpret_cast<int4*>(L->M) + threadIdx.x * (kOut / 4);
#pragma unroll
  for (int k = 0; k < kOut / 4; ++k) M4[k] = make_int4(-1, -1, -1, -1);
}
typedef int32_t OutQuad __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void store_quad(int32_t* __restrict__ p, uint32_t i, uint32_t len,
                                           int32_t v0, int32_t v1, int32_t v2, int32_t v3) {
  if (i + 4 <= len) {
    OutQuad q;
    q.x = v0; q.y = v1; q.z = v2; q.w = v3;
    *reinterpret_cast<OutQuad*>(p + i) = q;
  } else {
    if (i < len) p[i] = v0;
    if (i + 1 < len) p[i + 1] = v1;
    if (i + 2 < len) p[i + 2] = v2;
  }
}
// The markers are cleared (with a barrier behind it) before the first call.
__device__ __forceinline__ void wg_expand(const uint32_t (&O)[kPer], uint32_t Oprev,
                                          uint32_t O_lo, uint32_t O_hi, int32_t P0, int64_t n,
                                          int32_t* __restrict__ a_out, ExpandLds* L) {
  constexpr uint32_t kRound = kT * kOut;
  const int tid = (int)threadIdx.x, wave = tid / kWave;
  O_hi = min(O_hi, (uint32_t)n);  // (never binds: every O is at most n)
  int32_t carry = -1;             // particle covering the first output of the round
  for (uint32_t cs = O_lo; cs < O_hi; cs += kRound) {
    const uint32_t len = min(kRound, O_hi - cs);
    if (cs != O_lo) {
      __syncthreads();  // the last round's markers and tops have been read
      wg_markers_clear(L);
      __syncthreads();
    }
    uint32_t p = Oprev;
#pragma unroll
    for (int v = 0; v < kPer; ++v) {
      const uint32_t pos = p - cs;
      if (O[v] > p && pos < len) L->M[pos] = tid * kPer + v;
      p = O[v];
    }
    __syncthreads();
    const int4* M4 = reinterpret_cast<const int4*>(L->M) + tid * (kOut / 4);
    int32_t m[kOut];
#pragma unroll
    for (int k = 0; k < kOut / 4; ++k) {
      const int4 t = M4[k];
      m[4 * k] = t.x; m[4 * k + 1] = t.y; m[4 * k + 2] = t.z; m[4 * k + 3] = t.w;
    }
#pragma unroll
    for (int k = 1; k < kOut; ++k) m[k] = max(m[k], m[k - 1]);
    const int32_t incl = wave_incl_max_i32(m[kOut - 1]);
    if (lane_id() == kWave - 1) L->top[wave] = incl;
    __syncthreads();
    int32_t before = (int32_t)wave_shift_up_u32((uint32_t)incl, 0xFFFFFFFFu);
    before = max(before, carry);
#pragma unroll
    for (int w2 = 0; w2 < kNW; ++w2) {
      const int32_t t = L->top[w2];
      before = w2 < wave ? max(before, t) : before;
      carry = max(carry, t);
    }
#pragma unroll
    for (int k = 0; k < kOut; ++k) m[k] = P0 + max(m[k], before);
    const uint32_t i = (uint32_t)tid * kOut;
    int32_t* __restrict__ ap = a_out + cs;
#pragma unroll
    for (int k = 0; k < kOut; k += 4)
      store_quad(ap, i + k, len, m[k], m[k + 1], m[k + 2], m[k + 3]);
  }
}

// The claim bits of the thread's particles (1: it has outputs); the nibbles of
// eight lanes make a word.
__device__ __forceinline__ void wg_claim_bits(const uint32_t (&O)[kPer], uint32_t Oprev,
                                              int64_t P0, uint32_t* __restrict__ claim) {
  const int tid = (int)threadIdx.x;
  uint32_t p = Oprev, bits = 0;
#pragma unroll
  for (int v = 0; v < kPer; ++v) {
    bits |= (O[v] > p ? 1u : 0u) << v;
    p = O[v];
  }
  bits <<= 4 * (tid & 7);
  bits |= dpp_u32<kDppXor1>(0u, bits);
  bits |= dpp_u32<kDppXor2>(0u, bits);
  bits |= dpp_u32<kDppHalfMirror>(0u, bits);
  if ((tid & 7) == 0) claim[(P0 >> 5) + (tid >> 3)] = bits;
}

template <bool SYSTEMATIC>
struct StrataWgLds {
  ExpandLds ex;
  CarryScratch cs;
  PrefixScratch ps;
  uint32_t u[SYSTEMATIC ? 1 : kUTabW];  // offset words of strata [m_lo, m_lo + kUTabW)
};

template <typename T, int SCHEME>
__global__ __launch_bounds__(kT) void k_scan_emit_b(const T* __restrict__ w, int64_t n,
                                                    uint32_t nb, Key key, uint32_t offset,
                                                    uint32_t filter,
                                                    const BlockRec* __restrict__ recs,
                                                    int32_t* __restrict__ a,
                                                    uint32_t* __restrict__ flags,
                                                    uint32_t* __restrict__ claim) {
  static_assert(SCHEME != SCHEME_MULTINOMIAL, "strata schemes only");
  constexpr bool SYSTEMATIC = SCHEME == SCHEME_SYSTEMATIC;
  __shared__ StrataWgLds<SYSTEMATIC> L;
  const uint32_t b = blockIdx.x;
  const int tid = (int)threadIdx.x;
  const int64_t P0 = (int64_t)b * kBlock;
  T x[kPer];
  load4_any(w, n, P0, x);
  const BlockRec rec = recs[b];
  offset = counter_offset(key, offset);
  wg_markers_clear(&L.ex);
  const WgCarry c = direct_carries(nb, b, recs, rec, &L.cs);
  if (flags && b == 0 && tid == 0 && c.status) atomicOr(flags, c.status);
  if (c.status & (FLAG_BAD_WEIGHTS | FLAG_ZERO_TOTAL)) {
    block_identity(P0, n, tid, kT, a, claim);
    return;
  }
  uint64_t q[kPer];
  const uint64_t off = wg_quantize(x, rec.scale, q, &L.ps);
  __syncthreads();
  WgR R;
  wg_block_r(q, off, &L.ps, rec.scale, c, n, R);
  if (!(R.hi > R.lo) && !claim) return;  // an empty range has no outputs

  const int32_t n32 = (int32_t)n;
  const int32_t m_lo = (int32_t)floor(R.lo);
  const int32_t m_hi = min(n32 - 1, (int32_t)floor(R.hi));
  const bool table = !SYSTEMATIC && m_hi - m_lo + 1 <= kUTabW;
  const double t_sys =
      SYSTEMATIC ? 1.0 - u_offset(draw_uniform(key, 0, DOM_STRATA, 0, filter, offset).x) : 0.0;
  if (!SYSTEMATIC) {
    if (table) {
      for (int32_t cc = (m_lo >> 2) + tid; cc <= (m_hi >> 2); cc += kT) {
        const uint4 xw = draw(key, (uint32_t)cc, DOM_STRATA, 0, filter, offset);
        const uint32_t xs[4] = {xw.x, xw.y, xw.z, xw.w};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int32_t m = cc * 4 + v;
          if (m >= m_lo && m <= m_hi) L.u[m - m_lo] = xs[v];
        }
      }
    }
    __syncthreads();
  }
  auto cum = [&](double rv) -> uint32_t {
    if (SYSTEMATIC) return cum_at(rv, t_sys);
    const int32_t m = (int32_t)rv;
    return cum_at(rv, 1.0 - u_offset(table ? L.u[m >= n32 ? 0 : m - m_lo]
                                           : stratum_word(key, filter, offset, m)));
  };
  uint32_t O[kPer];
  const uint32_t Oprev = cum(R.prev);
#pragma unroll
  for (int v = 0; v < kPer; ++v) O[v] = cum(R.r[v]);
  const uint32_t O_lo = uniform_u32(cum(R.lo)), O_hi = uniform_u32(cum(R.hi));
  if (claim) wg_claim_bits(O, Oprev, P0, claim);
  wg_expand(O, Oprev, O_lo, O_hi, (int32_t)P0, n, a, &L.ex);
}

template <typename T, int SCHEME>
__global__ __launch_bounds__(kT) void k_scan_emit_w(const T* __restrict__ w, int64_t n,
                                                    uint32_t nb, Key key, uint32_t offset,
                                                    uint32_t filter,
                                                    const ScanHeader* __restrict__ hdr,
                                                    const BlockRec* __restrict__ recs,
                                                    Carries C, int32_t* __restrict__ a,
                                                    uint32_t* __restrict__ flags,
                                                    uint32_t* __restrict__ claim) {
  static_assert(SCHEME != SCHEME_MULTINOMIAL, "strata schemes only");
  offset = counter_offset(key, offset);
  __shared__ StrataWaveLds<SCHEME == SCHEME_SYSTEMATIC> L[kWavesPerWG];
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t b = blockIdx.x * kWavesPerWG + wave;
  if (b >= nb) return;
  const uint32_t status = hdr->status;
  const int32_t gscale = hdr->gscale;
  C.gscale = gscale;
  const u128 Cb = C[b], Cb1 = C[b + 1], Q = hdr->Q;
  if (flags && b == 0 && threadIdx.x == 0 && status) atomicOr(flags, status);
  const int64_t P0 = (int64_t)b * kBlock;
  if (status & (FLAG_BAD_WEIGHTS | FLAG_ZERO_TOTAL)) {
    block_identity(P0, n, (int)lane_id(), kWave, a, claim);
    return;
  }
  emit_block_wave<T, SCHEME == SCHEME_SYSTEMATIC>(w, n, P0, recs[b], Cb, Cb1, gscale, Q, key,
                                                   filter, offset, a, &L[wave], claim);
}

// Multinomial emission, one weight block per wave (after the carries); with
// claim also the claimed slots (the multinomial ancestry is sorted, as the
// strata schemes' is).
template <typename T>
__global__ __launch_bounds__(kT) void k_scan_emit_mw(const T* __restrict__ w, int64_t n,
                                                     uint32_t nb, uint32_t nbe, Key key,
                                                     uint32_t offset, uint32_t filter,
                                                     const ScanHeader* __restrict__ hdr,
                                                     const BlockRec* __restrict__ recs,
                                                     Carries C, ECarries CE,
                                                     const uint64_t* __restrict__ evals,
                                                     int32_t* __restrict__ a,
                                                     uint32_t* __restrict__ flags,
                                                     uint32_t* __restrict__ claim) {
  offset = counter_offset(key, offset);
  __shared__ MultiWaveLds L[kWavesPerWG];
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t b = blockIdx.x * kWavesPerWG + wave;
  if (b >= nb) return;
  const uint32_t status = hdr->status;
  if (flags && b == 0 && threadIdx.x == 0 && status) atomicOr(flags, status);
  const int64_t P0 = (int64_t)b * kBlock;
  if (status & (FLAG_BAD_WEIGHTS | FLAG_ZERO_TOTAL)) {
    block_identity(P0, n, (int)lane_id(), kWave, a, claim);
    return;
  }
  C.gscale = hdr->gscale;
  emit_multi_wave<T, true>(w, n, P0, recs[b], C[b], C[b + 1], C.gscale, hdr->Q, key, filter,
                           offset, CE, nbe, evals, a, &L[wave], claim);
}

// The multinomial emission with one block per workgroup (at most kGrp blocks,
// whose carries go through the group's scale as in the carries pass, and
// kDirectMulti exponential blocks).  The workgroup forms its own weight carries from the
// records and, in the same two barriers, the prefix of the exponential block
// sums, kept in LDS as the last point of every block.  Each particle finds the
// exponential block of its r there (a few steps between the first and the last
// block that the workgroup's range touches), and only blocks that hold the r
// of some particle are rebuilt from their stored spacings and searched, which
// matters where one weight covers many of them.  r, points and comparisons
// are those of emit_multi_wave.  Bound by the serial chain (carries, prefix,
// ten LDS steps per searched block, expansion); four workgroups per CU at 2^20
// weights: 23 us, where carries and one block per wave took 9 and 29 (a wave
// per SIMD).  About half of it is instruction issue, a quarter the carries.
constexpr uint32_t kDirectMulti = 5 * kT;
struct MultiWgLds {
  double top[kDirectMulti + 1];  // top[e]: point of the exponential prefix up to block e
  double P[kBlock];              // the points of one exponential block
  ExpandLds ex;
  CarryScratch cs;
  PrefixScratch ps;
  u128 esum[kNW];
  uint64_t wsum[kNW];
  uint32_t used[kDirectMulti / 32];  // exponential blocks that hold some r
  uint32_t O_lo, O_hi;
};

template <typename T>
__global__ __launch_bounds__(kT) void k_scan_emit_mb(const T* __restrict__ w, int64_t n,
                                                     uint32_t nb, uint32_t nbe,
                                                     const BlockRec* __restrict__ recs,
                                                     const uint64_t* __restrict__ esums,
                                                     const uint64_t* __restrict__ evals,
                                                     uint32_t straight, int32_t* __restrict__ a,
                                                     uint32_t* __restrict__ flags,
                                                     uint32_t* __restrict__ claim) {
  constexpr int kE = (int)(kDirectMulti / kT);  // exponential blocks per thread
  __shared__ MultiWgLds L;
  const uint32_t b = blockIdx.x;
  const int tid = (int)threadIdx.x, wave = (int)uniform_u32((uint32_t)tid / kWave);
  const int64_t P0 = (int64_t)b * kBlock;
  T x[kPer];
  load4_any(w, n, P0, x);
  const BlockRec rec = recs[b];
  u128 ee[kE];  // inclusive prefixes of the thread's exponential block sums
  {
    u128 run = 0;
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      const uint32_t e = (uint32_t)tid * kE + (uint32_t)k;
      run += e < nbe ? (u128)esums[e] : (u128)0;
      ee[k] = run;
    }
    const u128 inc = wave_incl_add_u128(run);
    if (lane_id() == kWave - 1) L.esum[wave] = inc;
#pragma unroll
    for (int k = 0; k < kE; ++k) ee[k] += inc - run;
  }
  wg_markers_clear(&L.ex);
  if (tid < (int)(kDirectMulti / 32)) L.used[tid] = 0;
  const WgCarry c = direct_carries(nb, b, recs, rec, &L.cs, straight);
  if (flags && b == 0 && tid == 0 && c.status) atomicOr(flags, c.status);
  if (c.status & (FLAG_BAD_WEIGHTS | FLAG_ZERO_TOTAL)) {
    block_identity(P0, n, tid, kT, a, claim);
    return;
  }
  u128 ebefore = 0, S = 0;
#pragma unroll
  for (int w2 = 0; w2 < kNW; ++w2) {
    const u128 t = L.esum[w2];
    ebefore += w2 < wave ? t : (u128)0;
    S += t;
  }
  const RMap em = make_rmap(S, n);
  if (tid == 0) L.top[0] = em((u128)0);
#pragma unroll
  for (int k = 0; k < kE; ++k) L.top[tid * kE + k + 1] = em(ebefore + ee[k]);
  uint64_t q[kPer];
  const uint64_t off = wg_quantize(x, rec.scale, q, &L.ps);
  __syncthreads();
  WgR R;
  wg_block_r(q, off, &L.ps, rec.scale, c, n, R);
  if (!(R.hi > R.lo)) {  // an empty range has no outputs
    if (claim && (tid & 7) == 0) claim[(P0 >> 5) + (tid >> 3)] = 0;
    return;
  }

  // exponential block of a value: the blocks whose last point lies below it
  auto block_between = [&](double rv, uint32_t lo, uint32_t hi) -> uint32_t {
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (L.top[mid + 1] < rv) lo = mid + 1;
      else hi = mid;
    }
    return lo;
  };
  // the ends of the range: one probe of 64 blocks around the expected one
  // (the boundaries scatter by half a block at 2^20 points), else a bisection
  auto block_of = [&](double rv) -> uint32_t {
    const double per_block = (double)kBlock * (double)n / (double)(n + 1);
    const uint32_t last = nbe - 1;
    uint32_t e0 = (uint32_t)(rv / per_block);
    e0 = e0 > 32u ? e0 - 32u : 0u;
    e0 = min(e0, last);
    const uint32_t e = e0 + lane_id();
    const uint32_t below =
        (uint32_t)__popcll(ballot(e < last && L.top[e < last ? e + 1 : 0] < rv));
    const bool ok = (e0 == 0 || below > 0) && (e0 + kWave >= last || below < kWave);
    return uniform_u32(ok ? e0 + below : block_between(rv, 0u, last));
  };
  const uint32_t e_first = block_of(R.lo), e_last = block_of(R.hi);
  double rr[kPer + 1];
  uint32_t re[kPer + 1], O[kPer + 1];
  rr[0] = R.prev;
#pragma unroll
  for (int v = 0; v < kPer; ++v) rr[v + 1] = R.r[v];
#pragma unroll
  for (int v = 0; v <= kPer; ++v) {
    O[v] = 0;
    re[v] = block_between(rr[v], e_first, e_last);
    if (v == 0 || re[v] != re[v - 1]) atomicOr(&L.used[re[v] >> 5], 1u << (re[v] & 31u));
  }
  __syncthreads();
  const double ce = em.Nd * em.invQ;
  for (uint32_t word = e_first >> 5; word <= e_last >> 5; ++word) {
    uint32_t bits = uniform_u32(L.used[word]);
    while (bits) {
      const uint32_t e = word * 32u + (uint32_t)__ffs((int)bits) - 1u;
      bits &= bits - 1u;
      uint64_t p[kPer];
      load_exp_values(evals, e, p);
#pragma unroll
      for (int v = 1; v < kPer; ++v) p[v] += p[v - 1];
      const uint64_t incl = wave_incl_add_u64(p[kPer - 1]);
      if (lane_id() == kWave - 1) L.wsum[wave] = incl;
      __syncthreads();
      uint64_t before = incl - p[kPer - 1], total = 0;
#pragma unroll
      for (int w2 = 0; w2 < kNW; ++w2) {
        before += w2 < wave ? L.wsum[w2] : 0ull;
        total += L.wsum[w2];
      }
      const double p_base = L.top[e], p_top = L.top[e + 1];
      double pv[kPer];
#pragma unroll
      for (int v = 0; v < kPer; ++v) pv[v] = affine_r(before + p[v], total, ce, p_base, p_top);
      double2* P2 = reinterpret_cast<double2*>(L.P) + tid * (kPer / 2);
      P2[0] = make_double2(pv[0], pv[1]);
      P2[1] = make_double2(pv[2], pv[3]);
      __syncthreads();
      bool any = false;
#pragma unroll
      for (int v = 0; v <= kPer; ++v) any |= re[v] == e;
      if (any) {
        // points below r: at most 1023, as r is at most the last one
        uint32_t pos[kPer + 1];
#pragma unroll
        for (int v = 0; v <= kPer; ++v) pos[v] = 0;
#pragma unroll
        for (uint32_t st = kBlock / 2; st > 0; st >>= 1) {
#pragma unroll
          for (int v = 0; v <= kPer; ++v) pos[v] += (L.P[pos[v] + st - 1] < rr[v]) ? st : 0u;
        }
#pragma unroll
        for (int v = 0; v <= kPer; ++v) O[v] = re[v] == e ? e * (uint32_t)kBlock + pos[v] : O[v];
      }
    }
  }
  if (tid == 0) L.O_lo = O[0];
  if (tid == kT - 1) L.O_hi = O[kPer];  // its r is the range's upper end
  __syncthreads();
  const uint32_t Ov[kPer] = {O[1], O[2], O[3], O[4]};
  if (claim) wg_claim_bits(Ov, O[0], P0, claim);
  wg_expand(Ov, O[0], uniform_u32(L.O_lo), uniform_u32(L.O_hi), (int32_t)P0, n, a, &L.ex);
}

// ---------------------------------------------------------------- whole vector in one workgroup
// Stratified / systematic resampling of a vector (or of every short segment of
// a batch) of at most NB blocks by one workgroup in one launch: the weights
// are read once and stay quantised in registers from the records to the
// emission.  Thread t takes the quads of four weights t, t + THREADS, ...; a
// block is four waves of one round.  All outputs fit one marker pass, since
// there are as many as particles.  Records, scale, carries and r are those of
// the block-parallel kernels.  Bound by the latency of its phases.  Per call (captured), systematic:
// n = 1000 8.3 -> 3.9 us, 4096 9.4 -> 5.8 us (from 256 threads with 16 weights
// a lane); 65536 segments of 256 535 -> 185 us and 1024 of 16384 61 -> 46 us
// (from records, carries and emission).
//
// PERM: the permutation of Code 10 too.  The claimed slots are the particles
// with outputs, which a thread knows for its own quads; the winners, the first
// outputs of their runs, are the marked positions.  The ancestry is in LDS
// already, so the chains are walked there: the first kOneSteps steps of a quad
// together, the rest from a list.  With the permutation as a second launch
// (k_permute_lds) -> in this one, systematic: one vector of 1000 9.7 -> 7.2 us,
// 4096 of 300 28.5 -> 21.1, 65536 of 256 298 -> 209, 4096 of 4096 127 -> 91,
// 1024 of 16384 97 -> 84 (a step of as many filters: 88 -> 64).
constexpr uint32_t kMarked = 0x80000000u;
constexpr int kOneSteps = 3;
template <int NB>
struct OneWg {
  static constexpr int kThreads = NB >= 4 ? 1024 : 256 * NB;
  static constexpr int kW = kThreads / kWave;               // waves
  static constexpr int kR = NB * kBlock / (4 * kThreads);   // quads per thread
  static constexpr int kParts = NB * 4;                     // waves' shares of blocks
  static constexpr uint32_t kList = NB >= 4 ? 1024 : 256;   // entries of the chains' list
  static_assert(kParts <= kWave, "a wave holds one entry per share");
};

template <typename T, int SCHEME, int NB, bool PERM>
__global__ __launch_bounds__(OneWg<NB>::kThreads,
                             NB == 16 && sizeof(T) == 4 ? 8 : 1) void k_scan_one(
    const T* __restrict__ w_all, int64_t n_total, const int64_t* __restrict__ offsets,
    int64_t above, bool last, Key key, uint32_t offset, uint32_t filter_base,
    int32_t* __restrict__ a_all, int32_t* __restrict__ c_all, uint32_t* __restrict__ flags) {
  typedef OneWg<NB> G;
  constexpr bool SYSTEMATIC = SCHEME == SCHEME_SYSTEMATIC;
  static_assert(SCHEME != SCHEME_MULTINOMIAL, "strata schemes only");
  __shared__ __align__(16) int32_t M[NB * kBlock];
  __shared__ __align__(16) uint32_t u[SYSTEMATIC ? 4 : NB * kBlock];
  __shared__ uint32_t s_key[G::kParts];
  __shared__ uint64_t s_sum[G::kParts];
  __shared__ int32_t s_top[G::kParts];
  __shared__ uint32_t s_list[PERM ? G::kList : 1], s_count;
  const uint32_t f = blockIdx.x;
  const int64_t base = offsets ? offsets[f] : 0;
  const int64_t n = offsets ? offsets[f + 1] - base : n_total;
  if (n <= above) return;  // another launch's segment
  if (n > (int64_t)NB * kBlock) {
    // another launch's, or longer than the batch's max_len: identity + flag
    if (!last) return;
    for (int64_t i = threadIdx.x; i < n; i += G::kThreads) {
      a_all[base + i] = (int32_t)i;
      if (PERM) c_all[base + i] = (int32_t)i;
    }
    if (threadIdx.x == 0 && flags) atomicOr(flags, FLAG_BAD_COUNTS);
    return;
  }
  const T* __restrict__ w = w_all + base;
  int32_t* __restrict__ a = a_all + base;
  const uint32_t filter = filter_base + f;
  offset = counter_offset(key, offset);
  const int tid = (int)threadIdx.x, wave = (int)uniform_u32((uint32_t)tid / kWave);
  const int lane = (int)lane_id();
  const int32_t n32 = (int32_t)n;
  const uint32_t nb = ((uint32_t)n + kBlock - 1) / kBlock;

  // records: reference exponents
  T x[G::kR][4];
#pragma unroll
  for (int r = 0; r < G::kR; ++r) {
    const int32_t i = r * 4 * G::kThreads + 4 * tid;
    if (i + 4 <= n32) {
      typedef T V __attribute__((ext_vector_type(4), aligned(sizeof(T))));
      const V t = *reinterpret_cast<const V*>(w + i);
      x[r][0] = t.x; x[r][1] = t.y; x[r][2] = t.z; x[r][3] = t.w;
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) x[r][v] = i + v < n32 ? w[i + v] : (T)0;
    }
    reinterpret_cast<int4*>(M)[r * G::kThreads + tid] = make_int4(-1, -1, -1, -1);
  }
  if (!SYSTEMATIC) {
    for (int32_t cc = tid; cc < (n32 + 3) / 4; cc += G::kThreads)
      reinterpret_cast<uint4*>(u)[cc] = draw(key, (uint32_t)cc, DOM_STRATA, 0, filter, offset);
  }
#pragma unroll
  for (int r = 0; r < G::kR; ++r) {
    uint32_t k = 1;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      k = max(k, weight_ok(x[r][v]) ? (uint32_t)exp_field(x[r][v]) : FLAG_BAD_WEIGHTS << 16);
    k = wave_max_u32(k);
    if (lane == 0) s_key[r * G::kW + wave] = k;
  }
  __syncthreads();
  // quantised prefixes inside the waves.  With sixteen weights a thread they
  // are formed again from the weights in the emission: 64 registers instead of
  // 86, and two workgroups to a CU (systematic, 1024 segments of 16384: 64 ->
  // 46 us)
  constexpr bool kAgain = G::kR > 1 && sizeof(T) == 4;
  uint64_t q[kAgain ? 1 : G::kR][4], off[G::kR];
  int32_t scale[G::kR];
#pragma unroll
  for (int r = 0; r < G::kR; ++r) {
    const uint32_t* k4 = s_key + ((r * G::kW + wave) & ~3);
    scale[r] = scale_of<T>((int)(max(max(k4[0], k4[1]), max(k4[2], k4[3])) & 0xFFFFu));
    uint64_t acc = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      acc += quantize_nb(x[r][v], scale[r]);
      if (!kAgain) q[kAgain ? 0 : r][v] = acc;
    }
    const uint64_t incl = wave_incl_add_u64(acc);
    if (lane == kWave - 1) s_sum[r * G::kW + wave] = incl;
    off[r] = incl - acc;
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  // carries, by every wave: lane l holds block l
  uint64_t sum = 0;
  uint32_t bkey = 0;
  if ((uint32_t)lane < nb) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      sum += s_sum[4 * lane + k];
      bkey = max(bkey, s_key[4 * lane + k]);
    }
  }
  BlockRec rec;
  rec.sum = sum;
  rec.scale = scale_of<T>((int)(bkey & 0xFFFFu));
  rec.bad = bkey >> 16;
  const uint32_t bad = ballot(rec.bad != 0) ? FLAG_BAD_WEIGHTS : 0u;
  const uint32_t skey = ~wave_max_u32(sum ? ~((uint32_t)rec.scale ^ 0x80000000u) : 0u);
  const int32_t gscale = skey == 0xFFFFFFFFu ? 0
                                             : (int32_t)(skey ^ 0x80000000u) + (kCarryBits - 63) -
                                                   ceil_log2(nb);
  const u128 val = sum ? conv_rec(rec, gscale) : (u128)0;
  const u128 inc = wave_incl_add_u128(val);
  const u128 Q = readlane(inc, kWave - 1);
  const uint32_t status = bad | (!bad && Q == 0 ? FLAG_ZERO_TOTAL : 0u);
  if (flags && tid == 0 && status) atomicOr(flags, status);
  if (status) {
    for (int32_t i = tid; i < n32; i += G::kThreads) {
      a[i] = i;
      if (PERM) c_all[base + i] = i;
    }
    return;
  }
  if (PERM && tid == 0) s_count = 0;
  uint32_t claimed = 0;  // bit 4 r + v: particle v of the thread's quad r has outputs
  const RMap rm = make_rmap(Q, n);
  const double lo_l = rm(inc - val), hi_l = rm(inc), slope = rm.Nd * rm.invQ;
  const double t_sys =
      SYSTEMATIC ? 1.0 - u_offset(draw_uniform(key, 0, DOM_STRATA, 0, filter, offset).x) : 0.0;
  auto cum = [&](double rv) -> int32_t {
    const int32_t m = (int32_t)rv;
    return (int32_t)cum_at(rv, SYSTEMATIC ? t_sys : 1.0 - u_offset(u[m >= n32 ? 0 : m]));
  };
#pragma unroll
  for (int r = 0; r < G::kR; ++r) {
    const int part = r * G::kW + wave, blk = part >> 2;
    if ((uint32_t)blk >= nb) break;  // the same on every lane of the wave
    const double lo = readlane(lo_l, blk), hi = readlane(hi_l, blk);
    const double c = ldexp(slope, gscale - scale[r]);
    uint64_t total = 0, o = off[r];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t sk = s_sum[4 * blk + k];
      o += k < (part & 3) ? sk : 0ull;
      total += sk;
    }
    auto r_of = [&](uint64_t L) -> double { return affine_r(L, total, c, lo, hi); };
    int32_t p = cum(o ? r_of(o) : lo);
    const int32_t i = r * 4 * G::kThreads + 4 * tid;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (kAgain) {
        asm("" : "+v"(x[r][v]));  // or the compiler keeps the earlier values instead
        o += quantize_nb(x[r][v], scale[r]);
      }
      const int32_t O = cum(r_of(kAgain ? o : o + q[kAgain ? 0 : r][v]));
      // (past the end O stays at the block's upper end: no marker)
      if (O > p) {
        M[p] = i + v;
        if (PERM) claimed |= 1u << (4 * r + v);
      }
      p = O;
    }
    __builtin_amdgcn_sched_barrier(0);  // one round's values in registers at a time
  }
  __syncthreads();
  // expansion: the running maximum of the markers
  int32_t m[G::kR][4], in[G::kR];
  uint32_t won = 0;  // bit 4 r + v: position v of the thread's quad r is marked
#pragma unroll
  for (int r = 0; r < G::kR; ++r) {
    const int4 t = reinterpret_cast<const int4*>(M)[r * G::kThreads + tid];
    if (PERM)
      won |= ((t.x >= 0 ? 1u : 0u) | (t.y >= 0 ? 2u : 0u) | (t.z >= 0 ? 4u : 0u) |
              (t.w >= 0 ? 8u : 0u)) << (4 * r);
    m[r][0] = t.x;
    m[r][1] = max(t.y, m[r][0]);
    m[r][2] = max(t.z, m[r][1]);
    m[r][3] = max(t.w, m[r][2]);
    in[r] = wave_incl_max_i32(m[r][3]);
    if (lane == kWave - 1) s_top[r * G::kW + wave] = in[r];
  }
  __syncthreads();
  const int32_t tops = wave_incl_max_i32(lane < G::kParts ? s_top[lane] : -1);
#pragma unroll
  for (int r = 0; r < G::kR; ++r) {
    const int part = r * G::kW + wave;
    const int32_t upto =
        part > 0 ? (int32_t)__builtin_amdgcn_readlane(tops, part - 1) : -1;
    const int32_t before = max(upto, (int32_t)wave_shift_up_u32((uint32_t)in[r], 0xFFFFFFFFu));
    const uint32_t i = (uint32_t)(r * 4 * G::kThreads + 4 * tid);
#pragma unroll
    for (int v = 0; v < 4; ++v) m[r][v] = max(m[r][v], before);
    if (i < (uint32_t)n32) store_quad(a, i, (uint32_t)n32, m[r][0], m[r][1], m[r][2], m[r][3]);
    if constexpr (PERM) {
      uint32_t y[4];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        y[v] = (uint32_t)m[r][v] | ((won >> (4 * r + v)) & 1u ? kMarked : 0u);
      reinterpret_cast<uint4*>(M)[r * G::kThreads + tid] = make_uint4(y[0], y[1], y[2], y[3]);
    }
  }
  if constexpr (PERM) {
    const uint32_t* MM = reinterpret_cast<const uint32_t*>(M);
    int32_t* __restrict__ c = c_all + base;
    auto walk = [&](uint32_t y) -> uint32_t {  // the end of the chain from the marked value y
      while (y & kMarked) y = MM[y & ~kMarked];
      return y;
    };
    __syncthreads();
#pragma unroll
    for (int r = 0; r < G::kR; ++r) {
      const uint32_t i = (uint32_t)(r * 4 * G::kThreads + 4 * tid);
      if (i >= (uint32_t)n32) break;
      const uint4 t = reinterpret_cast<const uint4*>(MM)[r * G::kThreads + tid];
      uint32_t y[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if ((claimed >> (4 * r + v)) & 1u || i + v >= (uint32_t)n32) y[v] = i + v;
      for (int k = 0; k < kOneSteps && ((y[0] | y[1] | y[2] | y[3]) & kMarked); ++k) {
        uint32_t z[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) z[v] = MM[y[v] & kMarked ? y[v] & ~kMarked : 0u];
#pragma unroll
        for (int v = 0; v < 4; ++v) y[v] = y[v] & kMarked ? z[v] : y[v];
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (y[v] & kMarked) {
          const uint32_t at = atomicAdd(&s_count, 1u);
          if (at < G::kList) s_list[at] = (i + v) << 16 | (y[v] & ~kMarked);
          else y[v] = walk(y[v]);
        }
      }
      store_quad(c, i, (uint32_t)n32, (int32_t)y[0], (int32_t)y[1], (int32_t)y[2], (int32_t)y[3]);
    }
    __syncthreads();  // also orders the chains' slots after the quads stored above
    const uint32_t listed = min(s_count, G::kList);
    for (uint32_t k = (uint32_t)tid; k < listed; k += G::kThreads)
      c[s_list[k] >> 16] = (int32_t)walk((s_list[k] & 0xFFFFu) | kMarked);
  }
}


// ---------------------------------------------------------------- Code 5
// Multinomial resampling with one independent uniform per particle, as Code 5
// prints it: the scaled prefix r_k = n W_k / W_n of the exact sums is written
// out (binary64, the same values the other schemes compare against), then
// particle i draws u_i = m 2^-53 (m: 21 bits of word 0 and 32 of word 1 of its
// uniform-domain Philox call), p_i = n u_i, and takes #{k < n-1 : r_k <= p_i}.
// The search is two-level: every workgroup holds up to kSplit splitters
// r_{(j+1) S - 1} (S a power of two) in LDS, which narrow each point to S
// candidates, and a bisection over those in global memory finishes it.
template <typename T>
__global__ __launch_bounds__(kT) void k_scan_r(const T* __restrict__ w, int64_t n, uint32_t nb,
                                               const ScanHeader* __restrict__ hdr,
                                               const BlockRec* __restrict__ recs, Carries C,
                                               double* __restrict__ r_out) {
  if (hdr->status & (FLAG_BAD_WEIGHTS | FLAG_ZERO_TOTAL)) return;
  const uint32_t b = blockIdx.x * kWavesPerWG +
                     (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (b >= nb) return;
  const int64_t P0 = (int64_t)b * kBlock;
  BlockR R;
  C.gscale = hdr->gscale;
  block_r_wave(w, n, P0, recs[b], C[b], C[b + 1], C.gscale, hdr->Q, R);
  const int64_t i0 = P0 + (int64_t)lane_id() * kWPer;
#pragma unroll
  for (int v = 0; v < kWPer; ++v)
    if (i0 + v < n) r_out[i0 + v] = R.r[v];
}

__global__ void k_scan_status(const ScanHeader* __restrict__ hdr, uint32_t* __restrict__ flags) {
  if (hdr->status) atomicOr(flags, hdr->status);
}

constexpr int kSplit = 4096;

__global__ __launch_bounds__(kT) void k_multinomial_iid(int64_t n,
                                                        const ScanHeader* __restrict__ hdr,
                                                        const double* __restrict__ r,
                                                        int stride_log2, Key key,
                                                        uint32_t offset, uint32_t filter,
                                                        int32_t* __restrict__ a,
                                                        uint32_t* __restrict__ flags) {
  __shared__ double sp[kSplit];
  offset = counter_offset(key, offset);
  const uint32_t status = hdr->status;
  if (flags && blockIdx.x == 0 && threadIdx.x == 0 && status) atomicOr(flags, status);
  const bool identity = (status & (FLAG_BAD_WEIGHTS | FLAG_ZERO_TOTAL)) != 0;
  const int64_t m = n - 1;                  // candidates r_0 .. r_{m-1}
  const int64_t S = (int64_t)1 << stride_log2;
  const int J = (int)(m >> stride_log2);  // splitters inside [0, m), J <= kSplit
  if (!identity)
    for (int j = (int)threadIdx.x; j < J; j += kT) sp[j] = r[((int64_t)(j + 1) << stride_log2) - 1];
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * kT;
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += stride) {
    if (identity) {
      a[i] = (int32_t)i;
      continue;
    }
    const uint4 x = draw(key, (uint32_t)i, DOM_UNIFORM, 0, filter, offset);
    const uint64_t mb = ((uint64_t)(x.x >> 11) << 32) | (uint64_t)x.y;
    const double p = (double)n * ((double)mb * 0x1p-53);
    // splitters: every r_k with k < lo S is <= p; r_{(lo+1) S - 1} > p if lo < J
    int lo = 0, hi = J;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (sp[mid] <= p) lo = mid + 1;
      else hi = mid;
    }
    int64_t L = (int64_t)lo << stride_log2;
    int64_t H = lo < J ? L + S - 1 : m;  // the answer lies in [L, H]
    while (L < H) {
      const int64_t mid = (L + H) >> 1;
      if (r[mid] <= p) L = mid + 1;
      else H = mid;
    }
    a[i] = (int32_t)L;
  }
}

// Ragged batch: one workgroup per filter runs the reduce, the carries and the
// emission of its own segment, with the records and carries in LDS.
constexpr int kBatchMaxBlocks = 256;  // segments up to 2^18 particles

struct BatchLds {
  BlockRec recs[kBatchMaxBlocks];
  u128 C[kBatchMaxBlocks + 1];
  uint64_t esums[kBatchMaxBlocks];
  u128 CE[kBatchMaxBlocks + 1];
};

template <typename T, int SCHEME>
__global__ __launch_bounds__(kT) void k_scan_batched(const T* __restrict__ w, int64_t n_total,
                                                     const int64_t* __restrict__ offsets,
                                                     uint32_t n_filters, int64_t above, Key key,
                                                     uint32_t offset, uint32_t filter_base,
                                                     int32_t* __restrict__ a,
                                                     uint32_t* __restrict__ flags) {
  offset = counter_offset(key, offset);
  __shared__ BatchLds B;
  __shared__ WgScratch s;
  const uint32_t f = blockIdx.x;
  if (f >= n_filters) return;
  const int tid = (int)threadIdx.x;
  const int64_t base = offsets ? offsets[f] : 0;
  const int64_t n = offsets ? offsets[f + 1] - base : n_total;
  if (n <= above) return;  // empty, or another launch's segment
  const T* __restrict__ ws = w + base;
  int32_t* __restrict__ as = a + base;
  const uint32_t filt = filter_base + f;
  const uint32_t nb = (uint32_t)((n + kBlock - 1) / kBlock);
  const uint32_t nbe = (uint32_t)((n + 1 + kBlock - 1) / kBlock);
  if (nbe > kBatchMaxBlocks) {  // segment too long for this path: identity + flag
    for (int64_t i = tid; i < n; i += kT) as[i] = (int32_t)i;
    if (tid == 0 && flags) atomicOr(flags, FLAG_BAD_COUNTS);
    return;
  }
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  for (uint32_t b = wave; b < nb; b += kWavesPerWG) {
    const BlockRec r = wave_block_record(ws, n, (int64_t)b * kBlock);
    if (lane_id() == 0) B.recs[b] = r;
  }
  if (SCHEME == SCHEME_MULTINOMIAL) {
    for (uint32_t b = 0; b < nbe; ++b) {
      uint64_t q[kPer];
      exp_values(key, filt, offset, n, b, q);
      const uint64_t sum = wg_reduce(q[0] + q[1] + q[2] + q[3], OpAdd(), s.u);
      if (tid == 0) B.esums[b] = sum;
    }
  }
  __syncthreads();
  const Totals t = carries_from_records(nb, (const BlockRec*)B.recs, (u128*)B.C, &s);
  if (SCHEME == SCHEME_MULTINOMIAL) exp_carries(nbe, (const uint64_t*)B.esums, (u128*)B.CE, &s);
  if (flags && tid == 0 && t.status) atomicOr(flags, t.status);
  if (t.status & (FLAG_BAD_WEIGHTS | FLAG_ZERO_TOTAL)) {
    for (int64_t i = tid; i < n; i += kT) as[i] = (int32_t)i;
    return;
  }
  if constexpr (SCHEME == SCHEME_MULTINOMIAL) {
    __shared__ MultiWaveLds L[kWavesPerWG];
    for (uint32_t b = wave; b < nb; b += kWavesPerWG)
      emit_multi_wave<T, false>(ws, n, (int64_t)b * kBlock, B.recs[b], B.C[b], B.C[b + 1],
                                t.gscale, t.Q, key, filt, offset, (const u128*)B.CE, nbe,
                                (const uint64_t*)nullptr, as, &L[wave]);
  } else {
    __shared__ StrataWaveLds<SCHEME == SCHEME_SYSTEMATIC> L[kWavesPerWG];
    for (uint32_t b = wave; b < nb; b += kWavesPerWG)
      emit_block_wave<T, SCHEME == SCHEME_SYSTEMATIC>(ws, n, (int64_t)b * kBlock, B.recs[b],
                                                       B.C[b], B.C[b + 1], t.gscale, t.Q, key,
                                                       filt, offset, as, &L[wave], nullptr);
  }
}

// ---------------------------------------------------------------- segmented batches
// A batch with a workspace runs block-parallel: every 1024-weight block of
// every segment is one workgroup of the records and of the emit kernel, so a
// long segment no longer runs through one workgroup.  Blocks start at each
// segment's first weight (the same blocks as a single call on the segment),
// and one workgroup per segment forms the segment's exact carries, so the
// result is that of one call per segment.

// Exclusive prefixes over the segments: bstart[f] (weight blocks) and, when
// given, estart[f] (exponential blocks) and tstart[f] (tiles of kSegTile slots
// of the fused permutation).  One workgroup, four segments per thread and
// round; bound by the latency of its rounds (4096 segments 5.7 us; one segment
// per thread of 256, 19.6) and, with few segments, by its size (four: 1024
// threads 3.8 us, 64 threads 1.8).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_seg_prefix(const int64_t* __restrict__ offsets,
                                                        uint32_t n_filters,
                                                        uint32_t* __restrict__ bstart,
                                                        uint32_t* __restrict__ estart,
                                                        uint32_t* __restrict__ tstart) {
  constexpr int kF = 4, kW = THREADS / kWave;
  __shared__ uint32_t s_b[kW], s_e[kW], s_t[kW];
  const uint32_t tid = threadIdx.x, wave = tid / kWave;
  uint32_t cb = 0, ce = 0, ct = 0;  // totals of the rounds before (below 2^32, as the layouts' are)
  for (uint32_t base = 0; base < n_filters; base += kF * THREADS) {
    const uint32_t f0 = base + kF * tid;
    int64_t o[kF + 1];
#pragma unroll
    for (int k = 0; k <= kF; ++k) o[k] = offsets[min(f0 + k, n_filters)];
    uint32_t nb[kF], ne[kF], nt[kF], tb = 0, te = 0, tt = 0;
#pragma unroll
    for (int k = 0; k < kF; ++k) {
      const int64_t n = o[k + 1] - o[k];
      nb[k] = n > 0 ? (uint32_t)((n + kBlock - 1) / kBlock) : 0u;
      ne[k] = n > 0 ? (uint32_t)((n + 1 + kBlock - 1) / kBlock) : 0u;
      nt[k] = n > 0 ? (uint32_t)((n + kSegTile - 1) / kSegTile) : 0u;
      tb += nb[k];
      te += ne[k];
      tt += nt[k];
    }
    const uint32_t ib = wave_inclusive_scan(tb, OpAdd()), ie = wave_inclusive_scan(te, OpAdd()),
                   it = wave_inclusive_scan(tt, OpAdd());
    __syncthreads();  // the round before has read the totals
    if (lane_id() == kWave - 1) {
      s_b[wave] = ib;
      s_e[wave] = ie;
      s_t[wave] = it;
    }
    __syncthreads();
    uint32_t b = cb + ib - tb, e = ce + ie - te, t = ct + it - tt;
#pragma unroll
    for (uint32_t w2 = 0; w2 < (uint32_t)kW; ++w2) {
      const uint32_t vb = s_b[w2], ve = s_e[w2], vt = s_t[w2];
      b += w2 < wave ? vb : 0u;
      e += w2 < wave ? ve : 0u;
      t += w2 < wave ? vt : 0u;
      cb += vb;
      ce += ve;
      ct += vt;
    }
#pragma unroll
    for (int k = 0; k < kF; ++k) {
      const uint32_t f = f0 + (uint32_t)k;
      if (f < n_filters) {
        bstart[f] = b;
        if (estart) estart[f] = e;
        if (tstart) tstart[f] = t;
      }
      b += nb[k];
      e += ne[k];
      t += nt[k];
    }
  }
  if (tid == 0) {
    bstart[n_filters] = cb;
    if (estart) estart[n_filters] = ce;
    if (tstart) tstart[n_filters] = ct;
  }
}

// The claim words of segment f, when the emission writes them: whole tiles.
__device__ __forceinline__ uint32_t* seg_claim(const SegClaim& c, uint32_t f) {
  return c.claim ? c.claim + (size_t)c.tstart[f] * (kSegTile / 32) : nullptr;
}

// Records of the segmented multinomial batch: a workgroup per weight block,
// then one per exponential block.
template <typename T>
__global__ __launch_bounds__(kT) void k_seg_records(
    const T* __restrict__ w, const int64_t* __restrict__ offsets, uint32_t n_filters,
    uint32_t grid_b, Key key, uint32_t offset, uint32_t filter_base,
    const uint32_t* __restrict__ bstart, const uint32_t* __restrict__ estart,
    BlockRec* __restrict__ recs, uint64_t* __restrict__ esums, uint64_t* __restrict__ evals) {
  __shared__ WgScratch s;
  offset = counter_offset(key, offset);
  if (blockIdx.x < grid_b) {
    const uint32_t g = blockIdx.x;
    if (g >= bstart[n_filters]) return;
    const uint32_t f = wave_find_segment<uint32_t>(bstart, n_filters, g);
    const int64_t base = offsets[f];
    const int64_t n = offsets[f + 1] - base;
    const BlockRec r = block_record(w + base, n, (int64_t)(g - bstart[f]) * kBlock, &s);
    if (threadIdx.x == 0) recs[g] = r;
  } else {
    const uint32_t g = blockIdx.x - grid_b;
    if (g >= estart[n_filters]) return;
    const uint32_t f = wave_find_segment<uint32_t>(estart, n_filters, g);
    const int64_t n = offsets[f + 1] - offsets[f];
    uint64_t q[kPer];
    exp_values(key, filter_base + f, offset, n, g - estart[f], q);
    store_exp_values(evals, g, q);  // global block g = segment block g - estart[f]
    const uint64_t sum = wg_reduce(q[0] + q[1] + q[2] + q[3], OpAdd(), s.u);
    if (threadIdx.x == 0) esums[g] = sum;
  }
}

// Weight records of the segmented batch, one block per wave (strata schemes).
template <typename T>
__global__ __launch_bounds__(kT) void k_seg_records_w(const T* __restrict__ w,
                                                      const int64_t* __restrict__ offsets,
                                                      uint32_t n_filters,
                                                      const uint32_t* __restrict__ bstart,
                                                      BlockRec* __restrict__ recs) {
  const uint32_t g = blockIdx.x * kWavesPerWG +
                     (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (g >= bstart[n_filters]) return;
  const uint32_t f = wave_find_segment<uint32_t>(bstart, n_filters, g);
  const int64_t base = offsets[f];
  const int64_t n = offsets[f + 1] - base;
  const BlockRec r = wave_block_record(w + base, n, (int64_t)(g - bstart[f]) * kBlock);
  if (lane_id() == 0) recs[g] = r;
}

// Per segment (one workgroup each): global scale, exact carries C (nb + 1 per
// segment, at cstart = bstart[f] + f), total and status, and the
// exponential-block carries of the multinomial scheme (at estart[f] + f).
struct SegHdr {
  u128 Q;
  int32_t gscale;
  uint32_t status;
  uint64_t pad;
};

template <bool MULTI>
__global__ __launch_bounds__(kT) void k_seg_carries(uint32_t n_filters,
                                                    const uint32_t* __restrict__ bstart,
                                                    const uint32_t* __restrict__ estart,
                                                    const BlockRec* __restrict__ recs,
                                                    const uint64_t* __restrict__ esums,
                                                    u128* __restrict__ C, u128* __restrict__ CE,
                                                    SegHdr* __restrict__ hdr) {
  __shared__ WgScratch s;
  const uint32_t f = blockIdx.x;
  if (f >= n_filters) return;
  const uint32_t b0 = bstart[f], nb = bstart[f + 1] - b0;
  if (nb == 0) return;
  const Totals t = carries_from_records(nb, recs + b0, C + b0 + f, &s);
  if (MULTI) {
    const uint32_t e0 = estart[f];
    exp_carries(estart[f + 1] - e0, esums + e0, CE + e0 + f, &s);
  }
  if (threadIdx.x == 0) {
    hdr[f].Q = t.Q;
    hdr[f].gscale = t.gscale;
    hdr[f].status = t.status;
  }
}

// Emission of the segmented batch, one block per wave (strata schemes).
template <typename T, int SCHEME>
__global__ __launch_bounds__(kT) void k_seg_emit_w(
    const T* __restrict__ w, const int64_t* __restrict__ offsets, uint32_t n_filters, Key key,
    uint32_t offset, uint32_t filter_base, const uint32_t* __restrict__ bstart,
    const BlockRec* __restrict__ recs, const u128* __restrict__ C,
    const SegHdr* __restrict__ hdr, int32_t* __restrict__ a, uint32_t* __restrict__ flags,
    SegClaim sc) {
  static_assert(SCHEME != SCHEME_MULTINOMIAL, "strata schemes only");
  __shared__ StrataWaveLds<SCHEME == SCHEME_SYSTEMATIC> L[kWavesPerWG];
  offset = counter_offset(key, offset);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t g = blockIdx.x * kWavesPerWG + wave;
  if (g >= bstart[n_filters]) return;
  const uint32_t f = wave_find_segment<uint32_t>(bstart, n_filters, g);
  const int64_t base = offsets[f];
  const int64_t n = offsets[f + 1] - base;
  const uint32_t b = g - bstart[f];
  int32_t* __restrict__ as = a + base;
  const uint32_t status = hdr[f].status;
  if (flags && b == 0 && lane_id() == 0 && status) atomicOr(flags, status);
  const int64_t P0 = (int64_t)b * kBlock;
  if (status & (FLAG_BAD_WEIGHTS | FLAG_ZERO_TOTAL)) {
    block_identity(P0, n, (int)lane_id(), kWave, as, seg_claim(sc, f));
    return;
  }
  const u128* Cs = C + bstart[f] + f;
  emit_block_wave<T, SCHEME == SCHEME_SYSTEMATIC>(w + base, n, P0, recs[g], Cs[b], Cs[b + 1],
                                                   hdr[f].gscale, hdr[f].Q, key, filter_base + f,
                                                   offset, as, &L[wave], seg_claim(sc, f));
}

// Multinomial emission of the segmented batch, one block per wave; three waves
// per SIMD (168 registers; binary64 took 169 and ran two: 1024 segments of 16384
// 313 us, with three 272).
template <typename T>
__global__ __launch_bounds__(kT, 3) void k_seg_emit_mw(
    const T* __restrict__ w, const int64_t* __restrict__ offsets, uint32_t n_filters, Key key,
    uint32_t offset, uint32_t filter_base, const uint32_t* __restrict__ bstart,
    const uint32_t* __restrict__ estart, const BlockRec* __restrict__ recs,
    const u128* __restrict__ C, const u128* __restrict__ CE, const SegHdr* __restrict__ hdr,
    int32_t* __restrict__ a, uint32_t* __restrict__ flags, const uint64_t* __restrict__ evals,
    SegClaim sc) {
  __shared__ MultiWaveLds L[kWavesPerWG];
  offset = counter_offset(key, offset);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t g = blockIdx.x * kWavesPerWG + wave;
  if (g >= bstart[n_filters]) return;
  const uint32_t f = wave_find_segment<uint32_t>(bstart, n_filters, g);
  const int64_t base = offsets[f];
  const int64_t n = offsets[f + 1] - base;
  const uint32_t b = g - bstart[f];
  int32_t* __restrict__ as = a + base;
  const uint32_t status = hdr[f].status;
  if (flags && b == 0 && lane_id() == 0 && status) atomicOr(flags, status);
  const int64_t P0 = (int64_t)b * kBlock;
  if (status & (FLAG_BAD_WEIGHTS | FLAG_ZERO_TOTAL)) {
    block_identity(P0, n, (int)lane_id(), kWave, as, seg_claim(sc, f));
    return;
  }
  const u128* Cs = C + bstart[f] + f;
  const uint32_t nbe = estart[f + 1] - estart[f];
  emit_multi_wave<T, true>(w + base, n, P0, recs[g], Cs[b], Cs[b + 1], hdr[f].gscale, hdr[f].Q,
                           key, filter_base + f, offset, CE + estart[f] + f, nbe,
                           evals + (size_t)estart[f] * kBlock, as, &L[wave], seg_claim(sc, f));
}

// The two-level carries of a single vector in its workspace.
struct CarrySet {
  Carries C;
  ECarries CE;
  CarryGroup* groups;
  CarryGroup* egroups;
};

CarrySet carry_set(const ScanLayout& L, char* base, uint32_t nb, uint32_t nbe) {
  CarrySet c;
  const uint32_t G = carry_groups(nb), Ge = carry_groups(nbe);
  c.groups = (CarryGroup*)(base + L.groups);
  c.egroups = (CarryGroup*)(base + L.egroups);
  c.C = Carries{(const u128*)(base + L.carries), (const u128*)(c.groups + G), c.groups, nb, G, 0};
  c.CE = ECarries{(const u128*)(base + L.ecarries), (const u128*)(c.egroups + Ge), nbe, Ge};
  return c;
}

template <bool MULTI>
hipError_t launch_carries(const CarrySet& c, ScanHeader* hdr, const BlockRec* recs,
                          const uint64_t* esums, hipStream_t stream) {
  const uint32_t G = c.C.G, Ge = MULTI ? c.CE.Ge : 0u;
  // one workgroup for all groups when there are few
  const uint32_t grid = G + Ge <= kFewGroups ? 1u : G + Ge;
  hipLaunchKernelGGL((k_carry_groups<MULTI>), dim3(grid), dim3(kT), 0, stream, c.C.nb,
                     c.CE.nbe, G, recs, esums, (u128*)c.C.P, (u128*)c.CE.PE, c.groups,
                     c.egroups, Ge, (u128*)c.C.Tx, (u128*)c.CE.TEx, hdr);
  return hipGetLastError();
}

template <typename T, int SCHEME>
hipError_t launch_scan_t(const void* wv, int64_t n, Key key, uint32_t offset, uint32_t filter,
                         int32_t* a, void* ws, uint32_t* flags, hipStream_t stream,
                         uint32_t* claim = nullptr) {
  const T* w = (const T*)wv;
  constexpr bool multi = SCHEME == SCHEME_MULTINOMIAL;
  const ScanLayout L = scan_layout(n, multi);
  char* base = (char*)ws;
  ScanHeader* hdr = (ScanHeader*)base;
  BlockRec* recs = (BlockRec*)(base + L.recs);
  uint64_t* esums = (uint64_t*)(base + L.erecs);
  uint64_t* evals = multi ? (uint64_t*)(base + L.evals) : nullptr;
  const uint32_t nb = (uint32_t)((n + kBlock - 1) / kBlock);
  const uint32_t nbe = multi ? (uint32_t)((n + 1 + kBlock - 1) / kBlock) : 0u;
  const uint32_t wgs_b = (nb + kWavesPerWG - 1) / kWavesPerWG;
  const CarrySet cs = carry_set(L, base, nb, nbe);
  hipLaunchKernelGGL((k_scan_records_w<T, multi>), dim3(wgs_b + nbe), dim3(kT), 0, stream, w, n,
                     nb, wgs_b, key, offset, filter, recs, esums, evals, hdr);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if constexpr (!multi) {
    if (nb <= (uint32_t)tuning().direct_max_blocks && nb <= kDirectMax) {
      hipLaunchKernelGGL((k_scan_emit_b<T, SCHEME>), dim3(nb), dim3(kT), 0, stream, w, n, nb,
                         key, offset, filter, recs, a, flags, claim);
      return hipGetLastError();
    }
  }
  if constexpr (multi) {
    // up to kGrp blocks, one group, the workgroup's own carries win at every
    // length (against the carry kernel and one block per wave: 2^18 20.6 / 41.7
    // us, 2^19 23.6 / 43.8, 2^20 32.4 / 47.3); more would take a second level of
    // carries in every workgroup.  straight: a vector that
    // k_scan_batched resamples without a workspace, whose carries that forms at
    // the global scale at once
    const bool one_wg = n <= (int64_t)tuning().single_wg_max;
    if ((nb <= (uint32_t)tuning().direct_max_blocks || one_wg) && nb <= kGrp &&
        nbe <= kDirectMulti) {
      hipLaunchKernelGGL((k_scan_emit_mb<T>), dim3(nb), dim3(kT), 0, stream, w, n, nb, nbe,
                         recs, esums, (const uint64_t*)evals, one_wg ? kStraight : 0u, a, flags,
                         claim);
      return hipGetLastError();
    }
  }
  e = launch_carries<multi>(cs, hdr, recs, esums, stream);
  if (e != hipSuccess) return e;
  if constexpr (multi) {
    hipLaunchKernelGGL((k_scan_emit_mw<T>), dim3(wgs_b), dim3(kT), 0, stream, w, n, nb, nbe, key,
                       offset, filter, hdr, recs, cs.C, cs.CE, (const uint64_t*)evals, a, flags,
                       claim);
  } else {
    hipLaunchKernelGGL((k_scan_emit_w<T, SCHEME>), dim3(wgs_b), dim3(kT), 0, stream, w,
                       n, nb, key, offset, filter, hdr, recs, cs.C, a, flags, claim);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_scan_scheme(int scheme, const void* w, int64_t n, Key key, uint32_t offset,
                              uint32_t filter, int32_t* a, void* ws, uint32_t* flags,
                              hipStream_t stream) {
  switch (scheme) {
    case SCHEME_MULTINOMIAL:
      return launch_scan_t<T, SCHEME_MULTINOMIAL>(w, n, key, offset, filter, a, ws, flags, stream);
    case SCHEME_STRATIFIED:
      return launch_scan_t<T, SCHEME_STRATIFIED>(w, n, key, offset, filter, a, ws, flags, stream);
    default:
      return launch_scan_t<T, SCHEME_SYSTEMATIC>(w, n, key, offset, filter, a, ws, flags, stream);
  }
}

// One workgroup per segment (or for one vector): the strata schemes in tiers
// of segment length, the multinomial scheme and longer segments through
// k_scan_batched.  max_len: longest segment (0 = unknown); the tier that ends
// the call for it gives longer ones the identity.  c: the permuted ancestry
// too (strata schemes, max_len known and at most kOneWgMax).
template <typename T, int SCHEME>
hipError_t launch_batched_t(const T* w, int64_t n_total, const int64_t* offsets,
                            uint32_t n_filters, int64_t max_len, Key key, uint32_t offset,
                            uint32_t filter_base, int32_t* a, int32_t* c, uint32_t* flags,
                            hipStream_t stream) {
  int64_t above = 0;
  if constexpr (SCHEME != SCHEME_MULTINOMIAL) {
    if (!offsets) max_len = n_total;
    const bool equal = max_len > 0 && max_len * (int64_t)n_filters == n_total;
    auto tier = [&](auto plain, auto perm, int threads, int64_t upto) {
      // a tier is left to the next one where every segment is longer, or where
      // few segments would only add launches
      if (max_len > 0 && above >= max_len) return;
      if ((max_len <= 0 || max_len > upto) && (equal || (upto < kOneWgMax && n_filters <= 256)))
        return;
      const bool last = max_len > 0 && max_len <= upto;
      // (a launch holds fewer than 2^32 threads: 4 M segments of 1024)
      const uint32_t most = (uint32_t)((((uint64_t)1 << 32) - 1) / (uint64_t)threads);
      for (uint32_t f0 = 0; f0 < n_filters; f0 += most)
        hipLaunchKernelGGL(c ? perm : plain, dim3(std::min(most, n_filters - f0)), dim3(threads), 0,
                           stream, w, n_total, offsets ? offsets + f0 : nullptr, above, last, key,
                           offset, filter_base + f0, a, c, flags);
      above = upto;
    };
    tier(k_scan_one<T, SCHEME, 1, false>, k_scan_one<T, SCHEME, 1, true>, OneWg<1>::kThreads,
         1024);
    tier(k_scan_one<T, SCHEME, 4, false>, k_scan_one<T, SCHEME, 4, true>, OneWg<4>::kThreads,
         4096);
    tier(k_scan_one<T, SCHEME, 16, false>, k_scan_one<T, SCHEME, 16, true>, OneWg<16>::kThreads,
         kOneWgMax);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || (max_len > 0 && max_len <= kOneWgMax)) return e;
  }
  hipLaunchKernelGGL((k_scan_batched<T, SCHEME>), dim3(n_filters), dim3(kT), 0, stream, w, n_total,
                     offsets, n_filters, above, key, offset, filter_base, a, flags);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_batched_scheme(int scheme, const void* w, int64_t n_total,
                                 const int64_t* offsets, uint32_t n_filters, int64_t max_len,
                                 Key key, uint32_t offset, uint32_t filter_base, int32_t* a,
                                 int32_t* c, uint32_t* flags, hipStream_t stream) {
  const T* wt = (const T*)w;
  switch (scheme) {
    case SCHEME_MULTINOMIAL:
      return launch_batched_t<T, SCHEME_MULTINOMIAL>(wt, n_total, offsets, n_filters, max_len, key,
                                                     offset, filter_base, a, c, flags, stream);
    case SCHEME_STRATIFIED:
      return launch_batched_t<T, SCHEME_STRATIFIED>(wt, n_total, offsets, n_filters, max_len, key,
                                                    offset, filter_base, a, c, flags, stream);
    default:
      return launch_batched_t<T, SCHEME_SYSTEMATIC>(wt, n_total, offsets, n_filters, max_len, key,
                                                    offset, filter_base, a, c, flags, stream);
  }
}

template <typename T, int SCHEME>
hipError_t launch_segmented_t(const T* w, int64_t n_total, const int64_t* offsets,
                              uint32_t n_filters, Key key, uint32_t offset, uint32_t filter_base,
                              int32_t* a, void* ws, uint32_t* flags, uint32_t* bstart,
                              uint32_t* estart, const SegClaim& sc, hipStream_t stream) {
  constexpr bool multi = SCHEME == SCHEME_MULTINOMIAL;
  const SegLayout L = seg_layout(n_total, n_filters, multi);
  char* base = (char*)ws;
  BlockRec* recs = (BlockRec*)(base + L.recs);
  uint64_t* esums = (uint64_t*)(base + L.esums);
  uint64_t* evals = multi ? (uint64_t*)(base + L.evals) : nullptr;
  hipError_t e = hipSuccess;
  if (!bstart) {  // (else the caller keeps the block prefixes)
    bstart = (uint32_t*)(base + L.bstart);
    estart = multi ? (uint32_t*)(base + L.estart) : nullptr;
    auto prefix = [&](auto kernel, int threads) {
      hipLaunchKernelGGL(kernel, dim3(1), dim3(threads), 0, stream, offsets, n_filters, bstart,
                         estart, sc.tstart);
    };
    if (n_filters <= 256) prefix(k_seg_prefix<64>, 64);
    else if (n_filters <= 1024) prefix(k_seg_prefix<256>, 256);
    else prefix(k_seg_prefix<1024>, 1024);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const uint32_t wgs_b = (L.grid_b + kWavesPerWG - 1) / kWavesPerWG;
  if constexpr (multi)
    hipLaunchKernelGGL((k_seg_records<T>), dim3(L.grid_b + L.grid_e), dim3(kT), 0, stream,
                       w, offsets, n_filters, L.grid_b, key, offset, filter_base, bstart, estart,
                       recs, esums, evals);
  else
    hipLaunchKernelGGL((k_seg_records_w<T>), dim3(wgs_b), dim3(kT), 0, stream, w, offsets,
                       n_filters, bstart, recs);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  u128* C = (u128*)(base + L.carries);
  u128* CE = (u128*)(base + L.ecarries);
  SegHdr* hdr = (SegHdr*)(base + L.hdr);
  hipLaunchKernelGGL((k_seg_carries<multi>), dim3(n_filters), dim3(kT), 0, stream, n_filters,
                     bstart, estart, recs, esums, C, CE, hdr);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if constexpr (multi)
    hipLaunchKernelGGL((k_seg_emit_mw<T>), dim3(wgs_b), dim3(kT), 0, stream, w, offsets,
                       n_filters, key, offset, filter_base, bstart, estart, recs, C, CE, hdr, a,
                       flags, (const uint64_t*)evals, sc);
  else
    hipLaunchKernelGGL((k_seg_emit_w<T, SCHEME>), dim3(wgs_b), dim3(kT), 0, stream, w, offsets,
                       n_filters, key, offset, filter_base, bstart, recs, C, hdr, a, flags, sc);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_segmented_scheme(int scheme, const void* w, int64_t n_total,
                                   const int64_t* offsets, uint32_t n_filters, Key key,
                                   uint32_t offset, uint32_t filter_base, int32_t* a, void* ws,
                                   uint32_t* flags, uint32_t* bstart, uint32_t* estart,
                                   const SegClaim& sc, hipStream_t stream) {
  const T* wt = (const T*)w;
  switch (scheme) {
    case SCHEME_MULTINOMIAL:
      return launch_segmented_t<T, SCHEME_MULTINOMIAL>(wt, n_total, offsets, n_filters, key,
                                                       offset, filter_base, a, ws, flags, bstart,
                                                       estart, sc, stream);
    case SCHEME_STRATIFIED:
      return launch_segmented_t<T, SCHEME_STRATIFIED>(wt, n_total, offsets, n_filters, key,
                                                      offset, filter_base, a, ws, flags, bstart,
                                                       estart, sc, stream);
    default:
      return launch_segmented_t<T, SCHEME_SYSTEMATIC>(wt, n_total, offsets, n_filters, key,
                                                      offset, filter_base, a, ws, flags, bstart,
                                                       estart, sc, stream);
  }
}

}  // namespace

SegLayout seg_layout(int64_t n_total, uint32_t n_filters, bool multinomial) {
  SegLayout L;
  // upper bounds of the block counts: each segment adds at most one partial block
  L.grid_b = (uint32_t)(n_total / kBlock + n_filters);
  L.grid_e = multinomial ? (uint32_t)((n_total + n_filters) / kBlock + n_filters) : 0u;
  L.bstart = 0;
  L.estart = align256(((size_t)n_filters + 1) * sizeof(uint32_t));
  L.recs = L.estart + (multinomial ? align256(((size_t)n_filters + 1) * sizeof(uint32_t)) : 0);
  L.esums = L.recs + align256((size_t)L.grid_b * sizeof(BlockRec));
  L.carries = L.esums + align256((size_t)L.grid_e * sizeof(uint64_t));
  L.ecarries = L.carries + align256(((size_t)L.grid_b + n_filters) * sizeof(u128));
  L.hdr = L.ecarries +
          (multinomial ? align256(((size_t)L.grid_e + n_filters) * sizeof(u128)) : 0);
  L.evals = L.hdr + align256((size_t)n_filters * sizeof(SegHdr));
  L.total = L.evals + (multinomial ? align256((size_t)L.grid_e * kBlock * sizeof(uint64_t)) : 0);
  return L;
}

hipError_t launch_scan_segmented(int scheme, bool f64, const void* w, int64_t n_total,
                                 const int64_t* offsets, uint32_t n_filters, Key key,
                                 uint32_t offset, uint32_t filter_base, int32_t* a, void* ws,
                                 uint32_t* flags, hipStream_t stream, uint32_t* bstart,
                                 uint32_t* estart, const SegClaim& sc) {
  return f64 ? launch_segmented_scheme<double>(scheme, w, n_total, offsets, n_filters, key,
                                               offset, filter_base, a, ws, flags, bstart, estart,
                                               sc, stream)
             : launch_segmented_scheme<float>(scheme, w, n_total, offsets, n_filters, key,
                                              offset, filter_base, a, ws, flags, bstart, estart,
                                               sc, stream);
}

ScanLayout scan_layout(int64_t n, bool multinomial) {
  const size_t nb = (size_t)((n + kBlock - 1) / kBlock);
  const size_t nbe = multinomial ? (size_t)((n + 1 + kBlock - 1) / kBlock) : 0;
  ScanLayout L;
  L.recs = 256;
  L.carries = L.recs + align256(nb * sizeof(BlockRec));
  L.erecs = L.carries + align256((nb + 1) * sizeof(u128));
  L.ecarries = L.erecs + align256(nbe * sizeof(uint64_t));
  L.groups = L.ecarries + align256((nbe + 1) * sizeof(u128));
  const size_t G = carry_groups((uint32_t)nb), Ge = carry_groups((uint32_t)nbe);
  L.egroups = L.groups + align256(G * sizeof(CarryGroup) + (G + 1) * sizeof(u128));
  L.evals = L.egroups + align256(Ge * sizeof(CarryGroup) + (Ge + 1) * sizeof(u128));
  L.total = L.evals + align256(nbe * kBlock * sizeof(uint64_t));
  return L;
}

size_t batch_scan_lds_bytes() { return sizeof(BatchLds) + sizeof(EmitLds); }

hipError_t launch_scan(int scheme, bool f64, const void* w, int64_t n, Key key, uint32_t offset,
                       uint32_t filter, int32_t* a, void* ws, uint32_t* flags,
                       hipStream_t stream) {
  return f64 ? launch_scan_scheme<double>(scheme, w, n, key, offset, filter, a, ws, flags, stream)
             : launch_scan_scheme<float>(scheme, w, n, key, offset, filter, a, ws, flags, stream);
}

size_t multinomial_iid_workspace_bytes(int64_t n) {
  return scan_layout(n, false).total + align256((size_t)n * sizeof(double));
}

template <typename T>
hipError_t launch_multinomial_iid_t(const T* w, int64_t n, Key key, uint32_t offset,
                                    uint32_t filter, int32_t* a, void* ws, uint32_t* flags,
                                    hipStream_t stream) {
  const ScanLayout L = scan_layout(n, false);
  char* base = (char*)ws;
  ScanHeader* hdr = (ScanHeader*)base;
  BlockRec* recs = (BlockRec*)(base + L.recs);
  double* r = (double*)(base + L.total);
  const uint32_t nb = (uint32_t)((n + kBlock - 1) / kBlock);
  const uint32_t wgs_b = (nb + kWavesPerWG - 1) / kWavesPerWG;
  const CarrySet cs = carry_set(L, base, nb, 0u);
  hipLaunchKernelGGL((k_scan_records_w<T, false>), dim3(wgs_b), dim3(kT), 0, stream, w, n, nb,
                     wgs_b, key, offset, filter, recs, (uint64_t*)nullptr, (uint64_t*)nullptr, hdr);
  launch_carries<false>(cs, hdr, recs, nullptr, stream);
  hipLaunchKernelGGL((k_scan_r<T>), dim3(wgs_b), dim3(kT), 0, stream, w, n, nb, hdr, recs, cs.C,
                     r);
  // splitter stride: the smallest power of two leaving at most kSplit splitters
  int sl = 0;
  while (((n - 1) >> sl) > kSplit) ++sl;
  int64_t grid = (n + kT - 1) / kT;
  if (grid > 1024) grid = 1024;
  hipLaunchKernelGGL(k_multinomial_iid, dim3((unsigned)grid), dim3(kT), 0, stream, n, hdr, r, sl,
                     key, offset, filter, a, flags);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_scan_r_t(const T* w, int64_t n, double* r, void* ws, uint32_t* flags,
                           hipStream_t stream) {
  const ScanLayout L = scan_layout(n, false);
  char* base = (char*)ws;
  ScanHeader* hdr = (ScanHeader*)base;
  BlockRec* recs = (BlockRec*)(base + L.recs);
  const uint32_t nb = (uint32_t)((n + kBlock - 1) / kBlock);
  const uint32_t wgs_b = (nb + kWavesPerWG - 1) / kWavesPerWG;
  const CarrySet cs = carry_set(L, base, nb, 0u);
  hipLaunchKernelGGL((k_scan_records_w<T, false>), dim3(wgs_b), dim3(kT), 0, stream, w, n, nb,
                     wgs_b, Key{0, 0, nullptr}, 0u, 0u, recs, (uint64_t*)nullptr,
                     (uint64_t*)nullptr, hdr);
  launch_carries<false>(cs, hdr, recs, nullptr, stream);
  hipLaunchKernelGGL((k_scan_r<T>), dim3(wgs_b), dim3(kT), 0, stream, w, n, nb, hdr, recs, cs.C,
                     r);
  if (flags) hipLaunchKernelGGL(k_scan_status, dim3(1), dim3(1), 0, stream, hdr, flags);
  return hipGetLastError();
}

hipError_t launch_scan_r(bool f64, const void* w, int64_t n, double* r, void* ws, uint32_t* flags,
                         hipStream_t stream) {
  return f64 ? launch_scan_r_t((const double*)w, n, r, ws, flags, stream)
             : launch_scan_r_t((const float*)w, n, r, ws, flags, stream);
}

hipError_t launch_multinomial_iid(bool f64, const void* w, int64_t n, Key key, uint32_t offset,
                                  uint32_t filter, int32_t* a, void* ws, uint32_t* flags,
                                  hipStream_t stream) {
  return f64 ? launch_multinomial_iid_t((const double*)w, n, key, offset, filter, a, ws, flags,
                                        stream)
             : launch_multinomial_iid_t((const float*)w, n, key, offset, filter, a, ws, flags,
                                        stream);
}

hipError_t launch_scan_claimed(int scheme, bool f64, const void* w, int64_t n, Key key,
                               uint32_t offset, uint32_t filter, int32_t* a, void* ws,
                               uint32_t* flags, uint32_t* claim, hipStream_t stream) {
  if (scheme == SCHEME_MULTINOMIAL)
    return f64 ? launch_scan_t<double, SCHEME_MULTINOMIAL>(w, n, key, offset, filter, a, ws,
                                                           flags, stream, claim)
               : launch_scan_t<float, SCHEME_MULTINOMIAL>(w, n, key, offset, filter, a, ws, flags,
                                                          stream, claim);
  if (scheme == SCHEME_STRATIFIED)
    return f64 ? launch_scan_t<double, SCHEME_STRATIFIED>(w, n, key, offset, filter, a, ws, flags,
                                                          stream, claim)
               : launch_scan_t<float, SCHEME_STRATIFIED>(w, n, key, offset, filter, a, ws, flags,
                                                         stream, claim);
  if (scheme == SCHEME_SYSTEMATIC)
    return f64 ? launch_scan_t<double, SCHEME_SYSTEMATIC>(w, n, key, offset, filter, a, ws, flags,
                                                          stream, claim)
               : launch_scan_t<float, SCHEME_SYSTEMATIC>(w, n, key, offset, filter, a, ws, flags,
                                                         stream, claim);
  return hipErrorInvalidValue;
}

hipError_t launch_scan_batched(int scheme, bool f64, const void* w, int64_t n_total,
                               const int64_t* offsets, uint32_t n_filters, int64_t max_len,
                               Key key, uint32_t offset, uint32_t filter_base, int32_t* a,
                               uint32_t* flags, hipStream_t stream, int32_t* c) {
  return f64 ? launch_batched_scheme<double>(scheme, w, n_total, offsets, n_filters, max_len, key,
                                             offset, filter_base, a, c, flags, stream)
             : launch_batched_scheme<float>(scheme, w, n_total, offsets, n_filters, max_len, key,
                                            offset, filter_base, a, c, flags, stream);
}

}  // namespace pfr
