// pfr_aux.hip -- auxiliaries of the resampling step:
//   offspring_to_ancestors  (Code 11 of the paper after an exclusive scan of
//                            the offspring counts)
//   permute_ancestors       (Code 10: Prepermute, chain walk, gather)
#include "pfr_kernels.h"

namespace pfr {

namespace {

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ================================================================ o2a
// Single pass with a decoupled look-back (Merrill & Garland, 2016) over tiles
// of 4096 counts.  Counts are exact integers, so the carry a tile obtains does
// not depend on how far it had to look back.  Tile ids come from a ticket so
// that every tile's predecessors are already running.
//
// Status word of a tile (64 bits):  [63:35] epoch  [34:33] kind  [32:0] value
// kind 1 = aggregate of the tile, 2 = inclusive prefix; a word whose epoch is
// not the current call's is treated as not yet written.  The epoch advances
// when the last tile of a call finishes, so the status array never needs to
// be cleared between calls (a zeroed workspace is a valid initial state).
constexpr int kO2aTile = 4096;
constexpr uint64_t kKindAgg = 1, kKindInc = 2;
constexpr uint64_t kValMask = (1ull << 33) - 1;

struct O2aHeader {
  uint32_t epoch;
  uint32_t tile_ticket;
  uint32_t done;
  uint32_t pad[61];
};

__device__ __forceinline__ uint64_t pack_status(uint32_t epoch, uint64_t kind, uint64_t value) {
  return ((uint64_t)(epoch & 0x1FFFFFFFu) << 35) | (kind << 33) | (value & kValMask);
}
__device__ __forceinline__ uint64_t status_load(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void status_store(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Offspring values of a tile in (g, lane, v) order per wave; negative counts
// count as 0 and counts above n as n + 1 (both raise FLAG_BAD_COUNTS), so sums
// stay far below 2^33 per tile.
__device__ __forceinline__ void load_counts(const int32_t* __restrict__ o, int64_t n, int64_t base,
                                            uint64_t (&q)[16], uint32_t& bad) {
  const int lane = (int)lane_id();
  const bool aligned = ((reinterpret_cast<uintptr_t>(o + base) & 15u) == 0);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int64_t idx = base + (int64_t)g * 256 + lane * 4;
    int32_t v4[4];
    if (aligned && idx + 4 <= n) {
      const int4 t = *reinterpret_cast<const int4*>(o + idx);
      v4[0] = t.x; v4[1] = t.y; v4[2] = t.z; v4[3] = t.w;
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) v4[v] = (idx + v < n) ? o[idx + v] : 0;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      int64_t x = v4[v];
      if (x < 0) { bad = FLAG_BAD_COUNTS; x = 0; }
      if (x > n) { bad = FLAG_BAD_COUNTS; x = n + 1; }
      q[g * 4 + v] = (uint64_t)x;
    }
  }
}

template <int G, int V>
__device__ __forceinline__ uint64_t inclusive_scan16(uint64_t (&q)[16]) {
  uint64_t run = 0;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    uint64_t s = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      s += q[g * V + v];
      q[g * V + v] = s;
    }
    const uint64_t incl = wave_inclusive_scan(s, OpAdd());
    const uint64_t add = run + (incl - s);
#pragma unroll
    for (int v = 0; v < V; ++v) q[g * V + v] += add;
    run += readlane(incl, kWave - 1);
  }
  return run;
}

// Expansion of one tile: positions s in [lo, hi) get P0 + #{i : O_i <= s},
// where O (inclusive cumulative counts, saturated at n + 1) sits in LDS.
__device__ __forceinline__ void expand_tile(const uint32_t* __restrict__ O_lds, int cnt,
                                            int64_t lo, int64_t hi, int64_t P0,
                                            int32_t* __restrict__ a, int tid, int nthreads) {
  for (int64_t s = lo + tid; s < hi; s += nthreads) {
    int l = 0, h = cnt;
    while (l < h) {
      const int m = (l + h) >> 1;
      if ((int64_t)O_lds[m] <= s) l = m + 1;
      else h = m;
    }
    a[s] = (int32_t)(P0 + l);
  }
}

// Builds the tile's cumulative counts in LDS (4 waves x 1024) given its carry
// and returns through the arguments the tile total.
__device__ __forceinline__ void tile_counts_to_lds(uint64_t (&q)[16], uint64_t carry, int64_t n,
                                                   uint32_t* __restrict__ O_lds, int wave,
                                                   const uint64_t* wave_prefix) {
  const int lane = (int)lane_id();
#pragma unroll
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      uint64_t O = carry + wave_prefix[wave] + q[g * 4 + v];
      if (O > (uint64_t)n + 1) O = (uint64_t)n + 1;
      O_lds[wave * 1024 + g * 256 + lane * 4 + v] = (uint32_t)O;
    }
  }
}

__global__ __launch_bounds__(256) void k_o2a(const int32_t* __restrict__ o, int64_t n,
                                             int32_t* __restrict__ a, O2aHeader* __restrict__ hdr,
                                             uint64_t* __restrict__ status,
                                             uint32_t* __restrict__ flags, uint32_t ntiles) {
  __shared__ uint32_t O_lds[kO2aTile];
  __shared__ uint64_t wave_tot[4], wave_prefix[4];
  __shared__ uint32_t s_tile, s_epoch, s_bad;
  __shared__ uint64_t s_carry;
  const int tid = (int)threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  if (tid == 0) {
    s_tile = atomicAdd(&hdr->tile_ticket, 1u);
    s_epoch = __hip_atomic_load(&hdr->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_bad = 0;
  }
  __syncthreads();
  const uint32_t t = s_tile, epoch = s_epoch;
  const int64_t P0 = (int64_t)t * kO2aTile;
  uint64_t q[16];
  uint32_t bad = 0;
  load_counts(o, n, P0 + wave * 1024, q, bad);
  const uint64_t wsum = inclusive_scan16<4, 4>(q);
  if (lane == 0) wave_tot[wave] = wsum;
  bad = wave_reduce(bad, OpOr());
  if (lane == 0 && bad) atomicOr(&s_bad, bad);
  __syncthreads();
  if (tid == 0) {
    uint64_t run = 0;
    for (int w2 = 0; w2 < 4; ++w2) {
      wave_prefix[w2] = run;
      run += wave_tot[w2];
    }
    const uint64_t agg = run > (uint64_t)n + 1 ? (uint64_t)n + 1 : run;
    if (t == 0) {
      s_carry = 0;
      status_store(&status[0], pack_status(epoch, kKindInc, agg));
    } else {
      status_store(&status[t], pack_status(epoch, kKindAgg, agg));
    }
  }
  __syncthreads();
  // look-back by wave 0: lane l inspects tile t-1-l
  if (t > 0 && wave == 0) {
    uint64_t carry = 0;
    int64_t pos = (int64_t)t - 1;  // highest tile not yet accounted for
    while (true) {
      const int64_t j = pos - lane;
      uint64_t st = 0, kind = 0;
      bool ready = true;
      if (j >= 0) {
        st = status_load(&status[j]);
        kind = ((uint32_t)(st >> 35) == (epoch & 0x1FFFFFFFu)) ? ((st >> 33) & 3u) : 0u;
        ready = kind != 0;
      }
      // lanes up to (and including) the nearest inclusive tile must be ready
      const uint64_t inc_mask = ballot(j >= 0 && kind == kKindInc);
      const uint64_t end_mask = inc_mask | ballot(j < 0);
      const int stop = end_mask ? (__ffsll((long long)end_mask) - 1) : kWave;  // first lane that ends the walk
      const uint64_t need = (stop >= kWave - 1) ? ~0ull : ((2ull << stop) - 1);
      if ((ballot(!ready) & need) != 0) {
        __builtin_amdgcn_s_sleep(1);
        continue;
      }
      const uint64_t val = (j >= 0 && lane <= stop) ? (st & kValMask) : 0;
      carry += wave_reduce(val, OpAdd());
      if (stop < kWave) break;
      pos -= kWave;
    }
    if (carry > (uint64_t)n + 1) carry = (uint64_t)n + 1;
    if (lane == 0) {
      s_carry = carry;
      uint64_t inc = carry + wave_prefix[3] + wave_tot[3];
      if (inc > (uint64_t)n + 1) inc = (uint64_t)n + 1;
      status_store(&status[t], pack_status(epoch, kKindInc, inc));
    }
  }
  __syncthreads();
  const uint64_t carry = s_carry;
  tile_counts_to_lds(q, carry, n, O_lds, wave, wave_prefix);
  __syncthreads();
  uint64_t total = carry + wave_prefix[3] + wave_tot[3];
  if (total > (uint64_t)n + 1) total = (uint64_t)n + 1;
  const int cnt = (int)min((int64_t)kO2aTile, n - P0);
  const int64_t lo = min((int64_t)carry, n), hi = min((int64_t)total, n);
  expand_tile(O_lds, cnt, lo, hi, P0, a, tid, 256);
  uint32_t fl = s_bad;
  if (t == ntiles - 1) {
    // positions beyond the last offspring keep the identity
    for (int64_t s = hi + tid; s < n; s += 256) a[s] = (int32_t)s;
    if (total != (uint64_t)n) fl |= FLAG_BAD_COUNTS;
  }
  if (tid == 0) {
    if (fl && flags) atomicOr(flags, fl);
    __threadfence();
    const uint32_t prev = atomicAdd(&hdr->done, 1u);
    if (prev == ntiles - 1) {  // last tile out: next call gets a new epoch
      hdr->tile_ticket = 0;
      hdr->done = 0;
      __hip_atomic_store(&hdr->epoch, (epoch + 1) & 0x1FFFFFFFu, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      __threadfence();
    }
  }
}

// Ragged batch: one workgroup per segment walks its tiles in order and keeps
// the carry in a register.
__global__ __launch_bounds__(256) void k_o2a_batched(const int32_t* __restrict__ o,
                                                     int64_t n_total,
                                                     const int64_t* __restrict__ offsets,
                                                     uint32_t n_filters, int32_t* __restrict__ a,
                                                     uint32_t* __restrict__ flags) {
  __shared__ uint32_t O_lds[kO2aTile];
  __shared__ uint64_t wave_tot[4], wave_prefix[4];
  __shared__ uint32_t s_bad;
  const uint32_t f = blockIdx.x;
  if (f >= n_filters) return;
  const int tid = (int)threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int64_t base = offsets ? offsets[f] : 0;
  const int64_t n = offsets ? offsets[f + 1] - base : n_total;
  const int32_t* __restrict__ os = o + base;
  int32_t* __restrict__ as = a + base;
  if (tid == 0) s_bad = 0;
  uint64_t carry = 0;
  for (int64_t P0 = 0; P0 < n; P0 += kO2aTile) {
    uint64_t q[16];
    uint32_t bad = 0;
    load_counts(os, n, P0 + wave * 1024, q, bad);
    const uint64_t wsum = inclusive_scan16<4, 4>(q);
    if (lane == 0) wave_tot[wave] = wsum;
    bad = wave_reduce(bad, OpOr());
    __syncthreads();
    if (lane == 0 && bad) atomicOr(&s_bad, bad);
    if (tid == 0) {
      uint64_t run = 0;
      for (int w2 = 0; w2 < 4; ++w2) {
        wave_prefix[w2] = run;
        run += wave_tot[w2];
      }
    }
    __syncthreads();
    tile_counts_to_lds(q, carry, n, O_lds, wave, wave_prefix);
    __syncthreads();
    uint64_t total = carry + wave_prefix[3] + wave_tot[3];
    if (total > (uint64_t)n + 1) total = (uint64_t)n + 1;
    const int cnt = (int)min((int64_t)kO2aTile, n - P0);
    expand_tile(O_lds, cnt, min((int64_t)carry, n), min((int64_t)total, n), P0, as, tid, 256);
    carry = total;
    __syncthreads();
  }
  const int64_t hi = min((int64_t)carry, n);
  for (int64_t s = hi + tid; s < n; s += 256) as[s] = (int32_t)s;
  __syncthreads();
  if (tid == 0 && flags) {
    uint32_t fl = s_bad;
    if (carry != (uint64_t)n) fl |= FLAG_BAD_COUNTS;
    if (fl) atomicOr(flags, fl);
  }
}

// ================================================================ permute
// Code 10.  d[j] holds the particle index that claims slot j, or n (unclaimed).
// Prepermute keeps the lowest claimer of every slot.  For a sorted ancestry
// (the output of the collective resamplers) the lowest claimer of slot a_i is
// the first i of its run, so the claim vector is written with plain stores in
// one pass: position i writes slot a_i when it starts a run, and n into every
// slot strictly between a_{i-1} and a_i, which no position claims.  For an
// unsorted ancestry the claim vector is filled with n and the lowest claimer
// found with an atomic minimum (a relaxed load first skips the atomic once a
// lower claimer is in place).
//
// Permute then lets every failed claimer i follow x <- d_x from x = i to an
// unclaimed slot and take it; finally c_j = a_{d_j}.  The chains are disjoint
// paths (the paper's termination argument), one per failed claimer, each
// ending in its own unclaimed slot.  The resolve kernel walks them backwards
// instead: a claimed slot j keeps c_j = j; from an unclaimed slot j it steps
// y <- a_y for as long as position y is the winning claimer of slot a_y
// (d[a_y] == y), which retraces the one chain that ends at j back to its
// failed claimer y, and sets c_j = a_y.  This is the same c as Code 10, reads
// only a and d, and needs no second pass over d.
struct SegIdx {
  int64_t base, n, i;
};

__device__ __forceinline__ SegIdx seg_index(const int64_t* __restrict__ offsets, uint32_t n_filters,
                                            int64_t n_total, int64_t g) {
  SegIdx s;
  if (!offsets) {
    s.base = 0;
    s.n = n_total;
  } else {
    const uint32_t f = find_segment(offsets, n_filters, g);
    s.base = offsets[f];
    s.n = offsets[f + 1] - s.base;
  }
  s.i = g - s.base;
  return s;
}

// ancestor of local position i, with out-of-range values replaced by i
__device__ __forceinline__ int64_t anc_at(const int32_t* __restrict__ a, const SegIdx& s, int64_t i,
                                          bool& bad) {
  const int64_t v = a[s.base + i];
  if (v < 0 || v >= s.n) {
    bad = true;
    return i;
  }
  return v;
}

__global__ __launch_bounds__(256) void k_claim_sorted(const int32_t* __restrict__ a,
                                                      int64_t n_total,
                                                      const int64_t* __restrict__ offsets,
                                                      uint32_t n_filters, int64_t min_len,
                                                      int32_t* __restrict__ d,
                                                      int32_t* __restrict__ e,
                                                      uint32_t* __restrict__ flags) {
  bool bad = false;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n_total; g += stride) {
    const SegIdx s = seg_index(offsets, n_filters, n_total, g);
    if (s.n < min_len) continue;  // permuted in LDS by k_permute_lds
    const int64_t ai = anc_at(a, s, s.i, bad);
    const int64_t prev = (s.i == 0) ? -1 : anc_at(a, s, s.i - 1, bad);
    int32_t* ds = d + s.base;
    e[g] = ai > prev ? (int32_t)ai : (int32_t)(-1 - ai);
    if (ai > prev) {
      ds[ai] = (int32_t)s.i;  // first of its run
      for (int64_t j = prev + 1; j < ai; ++j) ds[j] = (int32_t)s.n;
    }
    if (s.i == s.n - 1) {
      const int64_t top = ai > prev ? ai : prev;
      for (int64_t j = top + 1; j < s.n; ++j) ds[j] = (int32_t)s.n;
    }
  }
  if (flags) {
    const uint32_t b = (uint32_t)wave_reduce((uint32_t)bad, OpOr());
    if (b && lane_id() == 0) atomicOr(flags, FLAG_BAD_ANCESTOR);
  }
}

__global__ __launch_bounds__(256) void k_fill_unclaimed(int32_t* __restrict__ d, int64_t n_total,
                                                        const int64_t* __restrict__ offsets,
                                                        uint32_t n_filters, int64_t min_len) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n_total; g += stride) {
    const SegIdx s = seg_index(offsets, n_filters, n_total, g);
    if (s.n < min_len) continue;
    d[g] = (int32_t)s.n;
  }
}

// Claims of one workgroup are first merged in LDS: a 256-entry table keyed
// by the slot's low bits keeps the smallest (slot, position) pair per entry,
// and a position whose entry holds the same slot with a smaller position
// cannot win, so it issues no global atomic.  Equal ancestors inside a
// workgroup (degenerate weights: every particle descends from one) then cost
// one atomic per workgroup instead of one per particle, all on one address.
// Positions whose entry holds another slot still claim, so the result is the
// same minimum as without the table.  Slots are global indices (< 2^31).
__global__ __launch_bounds__(256) void k_claim_min(const int32_t* __restrict__ a, int64_t n_total,
                                                   const int64_t* __restrict__ offsets,
                                                   uint32_t n_filters, int64_t min_len,
                                                   int32_t* __restrict__ d,
                                                   uint32_t* __restrict__ flags) {
  __shared__ unsigned long long tab[256];
  bool bad = false;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t g0 = (int64_t)blockIdx.x * blockDim.x; g0 < n_total; g0 += stride) {
    const int64_t g = g0 + threadIdx.x;
    bool valid = false;
    uint32_t slot = 0, pos = 0;
    if (g < n_total) {
      const SegIdx s = seg_index(offsets, n_filters, n_total, g);
      if (s.n >= min_len) {
        valid = true;
        slot = (uint32_t)(s.base + anc_at(a, s, s.i, bad));
        pos = (uint32_t)s.i;
      }
    }
    const unsigned long long key = ((unsigned long long)slot << 32) | pos;
    tab[threadIdx.x] = ~0ull;
    __syncthreads();
    if (valid) atomicMin(&tab[slot & 255u], key);
    __syncthreads();
    if (valid) {
      const unsigned long long best = tab[slot & 255u];
      const bool beaten = (uint32_t)(best >> 32) == slot && (uint32_t)best < pos;
      int32_t* dst = &d[slot];
      // d only decreases, so a stale (cached) value that is already <= pos
      // proves the claim lost; only a larger one needs the atomic
      if (!beaten &&
          __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > (int32_t)pos)
        atomicMin(dst, (int32_t)pos);
    }
    __syncthreads();  // the table is reset by the next iteration
  }
  if (flags) {
    const uint32_t b = (uint32_t)wave_reduce((uint32_t)bad, OpOr());
    if (b && lane_id() == 0) atomicOr(flags, FLAG_BAD_ANCESTOR);
  }
}

// Backward walk on the ancestry itself (unsorted input, no marked ancestry):
// from an unclaimed slot j, y = j; while position y won its claim
// (d[a_y] == y) step to y = a_y; then c_j = a_y.  The same walk as k_resolve
// on e = marks(a, d), with the mark of each visited position formed on the
// way (two dependent loads per step instead of one), which saves the pass
// that writes e.  d[j] and a[j] are loaded together.
__global__ __launch_bounds__(256) void k_resolve_ad(const int32_t* __restrict__ a,
                                                    int64_t n_total,
                                                    const int64_t* __restrict__ offsets,
                                                    uint32_t n_filters, int64_t min_len,
                                                    const int32_t* __restrict__ d,
                                                    int32_t* __restrict__ c,
                                                    uint32_t* __restrict__ flags) {
  bool broken = false, bad = false;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n_total; g += stride) {
    const SegIdx s = seg_index(offsets, n_filters, n_total, g);
    if (s.n < min_len) continue;
    const int64_t j = s.i;
    const int64_t dj = d[g];
    int64_t ay = anc_at(a, s, j, bad);
    if (dj >= 0 && dj < s.n) {  // claimed: its winner's ancestor is j
      c[g] = (int32_t)j;
      continue;
    }
    // unclaimed: retrace the chain that ends here back to its failed claimer
    const int32_t* ds = d + s.base;
    int64_t y = j;
    int64_t steps = 0;
    bool br = false;
    while (ds[ay] == y) {  // position y won slot a_y: the chain came through it
      y = ay;
      ay = anc_at(a, s, y, bad);
      if (++steps > s.n) {  // a chain visits distinct slots; only bad input gets here
        br = true;
        break;
      }
    }
    broken |= br;
    c[g] = br ? (int32_t)j : (int32_t)ay;
  }
  if (flags) {
    const uint32_t b = (uint32_t)wave_reduce((uint32_t)(broken ? FLAG_BAD_ANCESTOR : 0u), OpOr());
    if (b && lane_id() == 0) atomicOr(flags, b);
  }
}

// Backward walk on e: one dependent load per chain step.
__global__ __launch_bounds__(256) void k_resolve(int64_t n_total,
                                                 const int64_t* __restrict__ offsets,
                                                 uint32_t n_filters, int64_t min_len,
                                                 const int32_t* __restrict__ d,
                                                 const int32_t* __restrict__ e,
                                                 int32_t* __restrict__ c,
                                                 uint32_t* __restrict__ flags) {
  bool broken = false;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n_total; g += stride) {
    const SegIdx s = seg_index(offsets, n_filters, n_total, g);
    if (s.n < min_len) continue;
    const int64_t j = s.i;
    const int64_t dj = d[g];
    const int32_t* es = e + s.base;
    int64_t ey = es[j];  // loaded with d[g]: the two loads are in flight together
    if (dj >= 0 && dj < s.n) {  // claimed: its winner's ancestor is j
      c[g] = (int32_t)j;
      continue;
    }
    // unclaimed: retrace the chain that ends here back to its failed claimer
    int64_t steps = 0;
    while (ey >= 0) {
      ey = es[ey];
      if (++steps > s.n) {  // a chain visits distinct slots; only bad input gets here
        broken = true;
        break;
      }
    }
    c[g] = broken ? (int32_t)j : (int32_t)(-1 - ey);
  }
  if (flags) {
    const uint32_t b = (uint32_t)wave_reduce((uint32_t)(broken ? FLAG_BAD_ANCESTOR : 0u), OpOr());
    if (b && lane_id() == 0) atomicOr(flags, b);
  }
}

// Segments of at most CAP <= 65536 particles, one workgroup each, entirely in
// LDS (local indices fit 16 bits).  A thread takes the same quads of four
// consecutive positions in every pass, so that loads and stores are 16 bytes
// a lane and what it learns about its own quads stays in registers.  Code 10
// needs of the claims only which slots are claimed and which positions won:
//   sorted     a position wins when it starts a run (a_i > a_{i-1}); one pass
//              gives the winners and a byte per claimed slot (plain stores,
//              where one bit per slot would serialise the atomics of a run);
//              the order is verified on the way, and an input that is not
//              sorted takes the other path
//   any order  an LDS atomic minimum per slot, in windows of the buffer
// Then the ancestry sits in LDS as 16-bit entries, with the winner bit in bit
// 15 up to 32768 particles and in a bitmap beyond, and every unclaimed slot
// walks backwards as in k_resolve, an LDS read per step instead of a read
// beyond the L2: kLockstep steps for the four chains of a quad together, and
// the few longer chains from a list at the end, one a lane (in lockstep to
// their end, a wave's longest chain would hold all its lanes in every round).
// Global traffic: the ancestry once (sorted,
// up to 32768 particles; else twice or more), the permutation once.  Bound by
// the latency of those loads and of the walk.  Measured per call against 32-bit
// claims in LDS up to 16384 particles and the global kernels beyond: 1024
// segments of 16384 107 -> 42 us sorted, 79 -> 50 us unsorted; 600 of 30000
// 426 -> 67 and 1064 -> 79 us; 4096 ragged ones of 256 .. 65536 (4.8e7
// particles) 1.48 -> 0.39 and 3.18 -> 0.45 ms.
constexpr int kLockstep = 6;
constexpr int kPermShort = 2048;      // batches: segments of the 256-thread tier
constexpr int kPermMid = 16384;       // two workgroups of 1024 threads to a CU
constexpr int kPermLong = 32768;      // 96 KB: one pass over a sorted ancestry
constexpr int kPermBatchMax = 65536;  // batches: segments permuted in LDS
constexpr int64_t kPermLongTotal = 1 << 21;  // batches: particles from which kPermMid is passed
// Single vectors up to these lengths are permuted in LDS by one workgroup
// (one launch instead of two to five); beyond them the multi-workgroup
// kernels are faster (kernel time at 8192 sorted, y = 0 / 4: 9.0 / 5.8 us,
// 16384: 21 / 8 against 11.4 / 7.2 us of two launches; unsorted 16384: 14 / 13
// against 19 us of five).
constexpr int kPermSingleMax = 16384;
constexpr int kPermSingleMaxSorted = 8192;
constexpr int kPermSmallWorkspace = 4096;  // up to here a workspace has no room for buckets

// LDS bytes of the shared buffer: 16-bit entries and claim bytes side by side
// up to kPermLong, one after the other in the same place beyond.
constexpr int perm_buffer(int cap) {
  return cap <= kPermShort ? 4 * cap : cap <= kPermLong ? 3 * cap : 2 * cap;
}

// Four consecutive positions from 4 q (entries past n: own index).  Segments
// start anywhere, so the 16-byte access is only 4-byte aligned.
typedef int32_t Quad __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void load_quad(const int32_t* __restrict__ as, uint32_t q, uint32_t n,
                                          int32_t (&v)[4]) {
  const uint32_t i = 4 * q;
  if (i + 4 <= n) {
    const Quad t = *reinterpret_cast<const Quad*>(as + i);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = i + k < n ? as[i + k] : (int32_t)(i + k);
  }
}

// A segment that no launch of the call was made for (longer than the batch's
// max_len) by one workgroup in global memory: lowest claimers by atomic minimum
// into d, then the backward walk of k_resolve_ad.  The claims are read past the
// CU's own cache, where the atomics are.  Slow, and never taken by a call whose
// max_len holds.
template <int THREADS>
__device__ void permute_unforeseen(const int32_t* __restrict__ a, int64_t n, int32_t* d,
                                   int32_t* __restrict__ c, bool& bad) {
  auto anc = [&](int64_t i) -> int64_t {
    const int64_t v = a[i];
    const bool out = v < 0 || v >= n;
    bad |= out;
    return out ? i : v;
  };
  auto claim = [&](int64_t j) -> int32_t {
    return __hip_atomic_load(&d[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  for (int64_t j = threadIdx.x; j < n; j += THREADS)
    __hip_atomic_store(&d[j], (int32_t)n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __threadfence();
  __syncthreads();
  for (int64_t i = threadIdx.x; i < n; i += THREADS) atomicMin(&d[anc(i)], (int32_t)i);
  __threadfence();
  __syncthreads();
  for (int64_t j = threadIdx.x; j < n; j += THREADS) {
    if (claim(j) < (int32_t)n) {
      c[j] = (int32_t)j;
      continue;
    }
    int64_t y = j, ay = anc(j);
    while (claim(ay) == (int32_t)y) {  // (the chain's slots are distinct: it ends)
      y = ay;
      ay = anc(y);
    }
    c[j] = (int32_t)ay;
  }
}

template <int CAP, int THREADS>
__global__ __launch_bounds__(THREADS) void k_permute_lds(
    const int32_t* __restrict__ a, int64_t n_total, const int64_t* __restrict__ offsets,
    int64_t above, int64_t upto, bool last, bool sorted, int32_t* __restrict__ d,
    int32_t* __restrict__ c, uint32_t* __restrict__ flags) {
  constexpr int kBytes = perm_buffer(CAP);
  constexpr uint32_t WIN = kBytes / 4;         // slots of a claim window
  constexpr bool kOnePass = kBytes >= 3 * CAP;  // entries and claim bytes fit together
  constexpr uint32_t kStep = 4 * THREADS;
  constexpr uint32_t kSlow = CAP <= kPermShort ? 256 : 3 * THREADS;
  static_assert(CAP <= 65536 && CAP / (4 * THREADS) <= 16 && WIN % kStep == 0,
                "16-bit indices, 16 quads a thread, windows of whole rounds");
  __shared__ __align__(16) uint8_t buf[kBytes];
  __shared__ uint32_t won[CAP / 32];
  __shared__ uint32_t slow[kSlow], n_slow;
  const int64_t base = offsets ? offsets[blockIdx.x] : 0;
  const int64_t n64 = offsets ? offsets[blockIdx.x + 1] - base : n_total;
  if (n64 <= above || (n64 > upto && !last)) return;  // another launch's segment
  if (n64 > CAP) {
    bool out = false;
    permute_unforeseen<THREADS>(a + base, n64, d + base, c + base, out);
    if (flags && ballot(out) != 0 && lane_id() == 0) atomicOr(flags, FLAG_BAD_ANCESTOR);
    return;
  }
  const uint32_t n = (uint32_t)n64, nq = (n + 3) / 4;
  const bool packed = CAP <= 32768 || n <= 32768u;
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const int32_t* __restrict__ as = a + base;
  uint16_t* const e = reinterpret_cast<uint16_t*>(buf);
  bool bad = false;
  // ancestor of local position i; out-of-range values count as i
  auto anc = [&](uint32_t i, int32_t v) -> uint32_t {
    const bool out = (uint32_t)v >= n && i < n;
    bad |= out;
    return out ? i : (uint32_t)v;
  };
  // the end of the chain that stands at winner y (its winner bit read already)
  auto walk = [&](uint32_t y) -> uint32_t {
    if (packed) {
      y = e[y];
      while (y & 0x8000u) y = e[y & 0x7FFFu];
    } else {
      uint32_t more = 1u;
      while (more) {
        more = (won[y >> 5] >> (y & 31u)) & 1u;
        y = e[y];
      }
    }
    return y;
  };
  if (tid == 0) n_slow = 0;  // (ordered by the barriers before the walk)
  auto put_quad = [&](uint32_t q, const uint32_t (&v)[4], uint32_t nib) {
    const uint32_t w0 = (nib & 1u) << 15, w1 = (nib & 2u) << 30, w2 = (nib & 4u) << 13,
                   w3 = (nib & 8u) << 28;
    reinterpret_cast<uint2*>(e)[q] =
        make_uint2(v[0] | (v[1] << 16) | w0 | w1, v[2] | (v[3] << 16) | w2 | w3);
  };
  // bits 4 r .. 4 r + 3: of the thread's quad tid + r THREADS, which positions
  // won their claims / which slots are claimed
  uint64_t mine_won = 0, mine_claimed = 0;
  if (sorted) {
    uint8_t* const cb = kOnePass ? buf + 2 * CAP : buf;
    for (uint32_t k = tid; k < (n + 15) / 16; k += THREADS)
      reinterpret_cast<uint4*>(cb)[k] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    bool down = false;
#pragma unroll 2
    for (uint32_t r = 0; r * THREADS < nq; ++r) {
      const uint32_t q = r * THREADS + tid;
      int32_t x[4];
      uint32_t v[4], nib = 0;
      load_quad(as, q, n, x);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = anc(4 * q + k, x[k]);
      uint32_t first = 0xFFFFFFFFu;  // -1 before position 0
      if (lane == 0 && q > 0 && q < nq) first = anc(4 * q - 1, as[4 * q - 1]);
      int32_t prev = (int32_t)wave_shift_up_u32(v[3], first);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool in = 4 * q + k < n;
        down |= in && (int32_t)v[k] < prev;
        if (in && (int32_t)v[k] > prev) {
          cb[v[k]] = 1;
          nib |= 1u << k;
        }
        prev = (int32_t)v[k];
      }
      mine_won |= (uint64_t)nib << (4 * r);
      if (kOnePass && q < nq) put_quad(q, v, nib);
      if (!packed) {  // the walk reads other threads' winners: the nibbles of eight lanes
        uint32_t w = nib << (4 * (lane & 7u));
        w |= dpp_u32<kDppXor1>(0u, w);
        w |= dpp_u32<kDppXor2>(0u, w);
        w |= dpp_u32<kDppHalfMirror>(0u, w);
        if ((lane & 7u) == 0 && q < nq) won[q >> 3] = w;
      }
    }
    sorted = !__syncthreads_or(down ? 1 : 0);
    if (sorted) {
      for (uint32_t r = 0; r * THREADS < nq; ++r) {
        const uint32_t q = r * THREADS + tid;
        if (q < nq) {
          const uint32_t x = reinterpret_cast<const uint32_t*>(cb)[q];
          const uint32_t nib = (x | (x >> 7) | (x >> 14) | (x >> 21)) & 15u;
          mine_claimed |= (uint64_t)nib << (4 * r);
        }
      }
    }
  }
  if (!sorted) {
    uint32_t* const d = reinterpret_cast<uint32_t*>(buf);
    for (uint32_t k = tid; k < (n + 31) / 32; k += THREADS) won[k] = 0;
    mine_won = 0;
    for (uint32_t w0 = 0; w0 < n; w0 += WIN) {
      const uint32_t ns = min(WIN, n - w0);
      __syncthreads();  // the buffer is free
      for (uint32_t k = tid; k < (ns + 3) / 4; k += THREADS)
        reinterpret_cast<uint4*>(d)[k] =
            make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
      __syncthreads();
#pragma unroll 2
      for (uint32_t q = tid; q < nq; q += THREADS) {
        int32_t x[4];
        load_quad(as, q, n, x);
        // (an ancestor repeated in its quad has claimed already: 16384 particles
        // of one ancestor, whose claims all meet in one word, 23.2 -> 13.4 us)
        uint32_t claimed = 0xFFFFFFFFu;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t i = 4 * q + k, s = anc(i, x[k]) - w0;
          if (s < ns && i < n && s != claimed) atomicMin(&d[s], i);
          claimed = s;
        }
      }
      __syncthreads();
      for (uint32_t k = tid; k < (ns + 3) / 4; k += THREADS) {
        const uint4 t = reinterpret_cast<const uint4*>(d)[k];
        const uint32_t w[4] = {t.x, t.y, t.z, t.w};
        uint32_t nib = 0;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          if (w[m] < n) {
            nib |= 1u << m;
            atomicOr(&won[w[m] >> 5], 1u << (w[m] & 31u));
          }
        }
        mine_claimed |= (uint64_t)nib << (4 * ((w0 / 4 + k - tid) / THREADS));
      }
    }
    __syncthreads();
    for (uint32_t r = 0; r * THREADS < nq; ++r) {
      const uint32_t q = r * THREADS + tid;
      if (q < nq) mine_won |= (uint64_t)((won[q >> 3] >> (4 * (q & 7u))) & 15u) << (4 * r);
    }
  }
  if (!(kOnePass && sorted)) {
    __syncthreads();  // the buffer is free
#pragma unroll 2
    for (uint32_t r = 0; r * THREADS < nq; ++r) {
      const uint32_t q = r * THREADS + tid;
      if (q >= nq) break;
      int32_t x[4];
      uint32_t v[4];
      load_quad(as, q, n, x);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = anc(4 * q + k, x[k]);
      put_quad(q, v, packed ? (uint32_t)(mine_won >> (4 * r)) & 15u : 0u);
    }
  }
  __syncthreads();
  for (uint32_t r = 0; r * THREADS < nq; ++r) {
    const uint32_t q = r * THREADS + tid;
    if (q >= nq) break;
    const uint2 t = reinterpret_cast<const uint2*>(e)[q];
    const uint32_t cl = (uint32_t)(mine_claimed >> (4 * r)) & 15u;
    uint32_t y[4] = {t.x & 0xFFFFu, t.x >> 16, t.y & 0xFFFFu, t.y >> 16};
    const uint32_t j = 4 * q;
    uint32_t left = 0;  // chains that go on after kLockstep steps
    if (packed) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if ((cl >> k) & 1u || j + k >= n) y[k] = (j + k) & 0x7FFFu;
      for (int s = 0; s < kLockstep && ((y[0] | y[1] | y[2] | y[3]) & 0x8000u); ++s) {
        uint32_t z[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) z[k] = e[y[k] & 0x7FFFu];
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = (y[k] & 0x8000u) ? z[k] : y[k];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) left |= ((y[k] >> 15) & 1u) << k;
    } else {
      left = (uint32_t)(mine_won >> (4 * r)) & 15u & ~cl;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if ((cl >> k) & 1u || j + k >= n) {
          y[k] = (j + k) & 0xFFFFu;
          left &= ~(1u << k);
        }
      }
      for (int s = 0; s < kLockstep && left; ++s) {
        uint32_t z[4], m[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          z[k] = e[y[k]];
          m[k] = won[y[k] >> 5];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const bool go = (left >> k) & 1u;
          const uint32_t more = (m[k] >> (y[k] & 31u)) & 1u;
          left = go && !more ? left & ~(1u << k) : left;
          y[k] = go ? z[k] : y[k];
        }
      }
    }
    if (left) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if ((left >> k) & 1u) {
          const uint32_t at = atomicAdd(&n_slow, 1u);
          if (at < kSlow) slow[at] = ((j + k) << 16) | (y[k] & (packed ? 0x7FFFu : 0xFFFFu));
          else y[k] = walk(y[k] & (packed ? 0x7FFFu : 0xFFFFu));
        }
      }
    }
    if (j + 4 <= n) {
      Quad o;
      o.x = (int32_t)y[0]; o.y = (int32_t)y[1]; o.z = (int32_t)y[2]; o.w = (int32_t)y[3];
      *reinterpret_cast<Quad*>(c + base + j) = o;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (j + k < n) c[base + j + k] = (int32_t)y[k];
    }
  }
  __syncthreads();  // also orders the chains' slots after the quads stored above
  const uint32_t ns = min(n_slow, (uint32_t)kSlow);
  for (uint32_t t = tid; t < ns; t += THREADS) {
    const uint32_t s = slow[t];
    c[base + (s >> 16)] = (int32_t)walk(s & 0xFFFFu);
  }
  if (flags && ballot(bad) != 0 && lane == 0) atomicOr(flags, FLAG_BAD_ANCESTOR);
}

// One short vector, 1 <= n <= kPermShort: a particle or two per thread, so the
// time is the latency of the phases, and fewer of them and less code beat
// k_permute_lds (n = 1000: 2.6 - 3.4 against 3.0 - 3.7 us).  Claims by an LDS
// atomic minimum for any order; the marks then overwrite the claims.
constexpr int kSmallThreads = 1024;
__global__ __launch_bounds__(kSmallThreads) void k_permute_small(const int32_t* __restrict__ a,
                                                                 int32_t n,
                                                                 int32_t* __restrict__ c,
                                                                 uint32_t* __restrict__ flags) {
  __shared__ int32_t de[kPermShort];
  __shared__ uint32_t claimed[kPermShort / 32];
  constexpr int kPer = kPermShort / kSmallThreads;  // particles per thread
  const int tid = (int)threadIdx.x;
  bool bad = false;
  // ancestor of local position i; out-of-range values count as i
  auto anc = [&](int32_t i) -> int32_t {
    const int32_t v = a[i];
    return (v < 0 || v >= n) ? i : v;
  };
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t i = tid + q * kSmallThreads;
    de[i] = n;
    if (q * kSmallThreads < kPermShort / 32 && i < kPermShort / 32) claimed[i] = 0u;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t i = tid + q * kSmallThreads;
    if (i < n) {
      const int32_t v = a[i];
      if (v < 0 || v >= n) bad = true;
      atomicMin(&de[(v < 0 || v >= n) ? i : v], i);
    }
  }
  __syncthreads();
  int32_t ev[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t i = tid + q * kSmallThreads;
    ev[q] = 0;
    if (i < n) {
      const int32_t ai = anc(i);
      ev[q] = de[ai] == i ? ai : -1 - ai;
      if (de[i] < n) atomicOr(&claimed[i >> 5], 1u << (i & 31));
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t i = tid + q * kSmallThreads;
    if (i < n) de[i] = ev[q];
  }
  __syncthreads();
  bool broken = false;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int32_t j = tid + q * kSmallThreads;
    if (j >= n) continue;
    if ((claimed[j >> 5] >> (j & 31)) & 1u) {
      c[j] = j;
      continue;
    }
    int32_t ey = de[j];
    int32_t steps = 0;
    bool br = false;
    while (ey >= 0) {
      ey = de[ey];
      if (++steps > n) {
        br = true;
        break;
      }
    }
    broken |= br;
    c[j] = br ? j : -1 - ey;
  }
  if (flags) {
    const uint32_t fl = (bad || broken) ? FLAG_BAD_ANCESTOR : 0u;
    const uint32_t b = wave_reduce(fl, OpOr());
    if (b && lane_id() == 0) atomicOr(flags, b);
  }
}

// ---------------------------------------------------------------- bucketed claim
// The claim vector of one unsorted vector without global atomics.  The slots
// fall into B buckets of S consecutive slots and the positions into W chunks
// of C; (1) every chunk counts its claims per bucket, (2) one workgroup per
// bucket scans its chunks' counts (the bucket totals give the buckets' bases),
// (3) every chunk writes its (position, slot) pairs to those places (the
// order inside a bucket does not matter), and (4) one workgroup per bucket
// takes the minimum claimer of each of its slots in LDS, writes that part of
// d (unclaimed: n) and the mark e_i = a_i of every winner; (3) has marked
// every position as a loser (-1 - a_i) before.  Claims that lose inside their
// own chunk get no pair.  k_resolve then walks e.  The minimum does not depend
// on the order, so d and e are those of the atomic claim.  Traffic: a read
// four times (8 + 8 bytes, half from the L2), 4 + 8 + 8 bytes of marks and
// pairs, 4 of d, and one scattered 4-byte write per claimed slot.
struct BucketGeom {
  int64_t n;
  uint32_t S, C, B, W;  // slots per bucket, positions per chunk, buckets, chunks
  int log2S;
  size_t cnt_off, tot_off, pairs_off, bytes;  // workspace parts after d and e
};

constexpr int kBucketMax = 4096;  // buckets (LDS counters of the chunk kernels)
constexpr int kBucketSlotsMax = 32768;
constexpr int kBucketThreads = 1024;
constexpr int kClaimThreads = 1024;

__host__ __device__ inline uint32_t pow2_at_least(int64_t x) {
  uint32_t p = 1;
  while ((int64_t)p < x && p < (1u << 30)) p <<= 1;
  return p;
}

BucketGeom bucket_geom(int64_t n) {
  BucketGeom g;
  g.n = n;
  // about 256 buckets and 1024 chunks: S and C powers of two, S from 4096 to
  // kBucketSlotsMax (the claim kernel's LDS table), C from 4096
  const uint32_t t = pow2_at_least((n + 255) / 256), tc = pow2_at_least((n + 1023) / 1024);
  g.S = t < 4096 ? 4096 : (t > (uint32_t)kBucketSlotsMax ? (uint32_t)kBucketSlotsMax : t);
  g.C = tc < 4096 ? 4096 : tc;
  g.log2S = 0;
  while ((1u << g.log2S) < g.S) ++g.log2S;
  g.B = (uint32_t)((n + g.S - 1) / g.S);
  g.W = (uint32_t)((n + g.C - 1) / g.C);
  const size_t base = 2 * align256((size_t)n * sizeof(int32_t));  // d, e
  const size_t pairs = (size_t)g.B * g.W;
  g.cnt_off = base;
  g.tot_off = g.cnt_off + align256(pairs * sizeof(uint32_t));
  g.pairs_off = g.tot_off + align256((size_t)g.B * sizeof(uint32_t));
  g.bytes = g.pairs_off + align256((size_t)n * sizeof(uint64_t));
  return g;
}

// the bucketed claim applies to single vectors of up to 2^31 - 1 particles
// whose bucket count fits the chunk kernels' LDS counters
bool bucket_claim_fits(int64_t n) {
  return n > 0 && n < ((int64_t)1 << 31) && bucket_geom(n).B <= (uint32_t)kBucketMax;
}

// slot claimed by position i (out-of-range ancestors claim their own index)
__device__ __forceinline__ uint32_t claim_slot(int32_t v, uint32_t i, uint32_t n, bool& bad) {
  if (v < 0 || (uint32_t)v >= n) {
    bad = true;
    return i;
  }
  return (uint32_t)v;
}

// Positions of chunk w, four per thread and round, their loads issued together
// (clamped to the chunk; f(i, slot) is called for the positions inside it).
template <typename F>
__device__ __forceinline__ void chunk_claims(const int32_t* __restrict__ a, uint32_t n,
                                             uint32_t p0, uint32_t p1, bool& bad, F f) {
  for (uint32_t i0 = p0; i0 < p1; i0 += 4 * kBucketThreads) {
    int32_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      v[k] = a[min(i0 + (uint32_t)(k * kBucketThreads) + threadIdx.x, p1 - 1)];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t i = i0 + (uint32_t)(k * kBucketThreads) + threadIdx.x;
      if (i < p1) f(i, claim_slot(v[k], i, n, bad));
    }
  }
}

// Equal claims inside a chunk are merged first: an LDS table keyed by the
// slot's low bits keeps the smallest (slot, position) per entry, and a
// position whose entry holds its slot with a smaller position has lost (it is
// not the minimum claimer), so it needs no pair.  Distinct slots sharing an
// entry all keep their pairs.  An ancestry with one parent then gives one
// pair per chunk instead of one per particle.
constexpr int kDedup = 4096;
__device__ __forceinline__ void dedup_fill(const int32_t* __restrict__ a, uint32_t n, uint32_t p0,
                                           uint32_t p1, unsigned long long* tab, bool& bad) {
  for (uint32_t k = threadIdx.x; k < kDedup; k += kBucketThreads) tab[k] = ~0ull;
  __syncthreads();
  chunk_claims(a, n, p0, p1, bad, [&](uint32_t i, uint32_t slot) {
    atomicMin(&tab[slot & (kDedup - 1)], ((unsigned long long)slot << 32) | i);
  });
  __syncthreads();
}
__device__ __forceinline__ bool dedup_lost(const unsigned long long* tab, uint32_t slot,
                                           uint32_t i) {
  const unsigned long long best = tab[slot & (kDedup - 1)];
  return (uint32_t)(best >> 32) == slot && (uint32_t)best < i;
}

__global__ __launch_bounds__(kBucketThreads) void k_bucket_count(
    const int32_t* __restrict__ a, uint32_t n, int log2S, uint32_t C, uint32_t B, uint32_t W,
    uint32_t* __restrict__ cnt, uint32_t* __restrict__ flags) {
  __shared__ uint32_t hist[kBucketMax];
  __shared__ unsigned long long tab[kDedup];
  const uint32_t w = blockIdx.x;
  for (uint32_t b = threadIdx.x; b < B; b += kBucketThreads) hist[b] = 0;
  bool bad = false;
  const uint32_t p0 = w * C, p1 = min(n, p0 + C);
  dedup_fill(a, n, p0, p1, tab, bad);
  chunk_claims(a, n, p0, p1, bad, [&](uint32_t i, uint32_t slot) {
    if (!dedup_lost(tab, slot, i)) atomicAdd(&hist[slot >> log2S], 1u);
  });
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < B; b += kBucketThreads) cnt[(size_t)b * W + w] = hist[b];
  if (flags) {
    const uint32_t f = (uint32_t)wave_reduce((uint32_t)bad, OpOr());
    if (f && lane_id() == 0) atomicOr(flags, FLAG_BAD_ANCESTOR);
  }
}

// Exclusive scan in place of each bucket's W chunk counts (row b of the
// bucket-major count matrix), one workgroup per bucket; the row total goes to
// tot[b].  The bucket's first pair, the sum of the totals of the buckets
// before it, is formed by its readers (bucket_bases).
__global__ __launch_bounds__(kBucketThreads) void k_bucket_rows(uint32_t* __restrict__ cnt,
                                                                uint32_t W,
                                                                uint32_t* __restrict__ tot) {
  __shared__ uint32_t s_w[kBucketThreads / kWave];
  const int tid = (int)threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  uint32_t* row = cnt + (size_t)blockIdx.x * W;
  uint32_t carry = 0;
  for (uint32_t c0 = 0; c0 < W; c0 += kBucketThreads) {
    const uint32_t j = c0 + (uint32_t)tid;
    const uint32_t x = j < W ? row[j] : 0u;
    const uint32_t inc = wave_incl_add_u32(x);
    if (lane == kWave - 1) s_w[wave] = inc;
    __syncthreads();
    uint32_t before = carry + inc - x, t = 0;
    for (int w2 = 0; w2 < kBucketThreads / kWave; ++w2) {
      before += w2 < wave ? s_w[w2] : 0u;
      t += s_w[w2];
    }
    if (j < W) row[j] = before;
    carry += t;
    __syncthreads();
  }
  if (tid == 0) tot[blockIdx.x] = carry;
}

// base[b] = sum of tot[b'] for b' < b, for b <= B, by the calling workgroup
// (kBucketThreads threads, B <= kBucketMax; s_w holds kBucketThreads / 64).
__device__ void bucket_bases(const uint32_t* __restrict__ tot, uint32_t B, uint32_t* base,
                             uint32_t* s_w) {
  const int tid = (int)threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  constexpr int kPerT = kBucketMax / kBucketThreads;  // 4 consecutive buckets per thread
  uint32_t x[kPerT], run = 0;
#pragma unroll
  for (int k = 0; k < kPerT; ++k) {
    const uint32_t b = (uint32_t)tid * kPerT + k;
    const uint32_t v = b < B ? tot[b] : 0u;
    x[k] = run;
    run += v;
  }
  const uint32_t inc = wave_incl_add_u32(run);
  if (lane == kWave - 1) s_w[wave] = inc;
  __syncthreads();
  uint32_t before = inc - run;
  for (int w2 = 0; w2 < wave; ++w2) before += s_w[w2];
#pragma unroll
  for (int k = 0; k < kPerT; ++k) {
    const uint32_t b = (uint32_t)tid * kPerT + k;
    if (b <= B) base[b] = before + x[k];
  }
  __syncthreads();
}

__global__ __launch_bounds__(kBucketThreads) void k_bucket_scatter(
    const int32_t* __restrict__ a, uint32_t n, int log2S, uint32_t C, uint32_t B, uint32_t W,
    const uint32_t* __restrict__ off, const uint32_t* __restrict__ tot,
    uint64_t* __restrict__ pairs, int32_t* __restrict__ e) {
  __shared__ uint32_t cur[kBucketMax + 1];
  __shared__ uint32_t s_w[kBucketThreads / kWave];
  __shared__ unsigned long long tab[kDedup];
  const uint32_t w = blockIdx.x;
  bucket_bases(tot, B, cur, s_w);
  for (uint32_t b = threadIdx.x; b < B; b += kBucketThreads) cur[b] += off[(size_t)b * W + w];
  bool bad = false;
  const uint32_t p0 = w * C, p1 = min(n, p0 + C);
  dedup_fill(a, n, p0, p1, tab, bad);
  // every position is marked as a loser here (in order, coalesced); the
  // claim kernel then marks the winners, one per claimed slot
  chunk_claims(a, n, p0, p1, bad, [&](uint32_t i, uint32_t slot) {
    e[i] = -1 - (int32_t)slot;
    if (!dedup_lost(tab, slot, i)) {  // (a loser here: a smaller position of the chunk claims it)
      const uint32_t r = atomicAdd(&cur[slot >> log2S], 1u);
      pairs[r] = ((uint64_t)i << 32) | slot;
    }
  });
}

// The pairs [q0, q1) of a bucket, four per thread and round, loads together.
template <typename F>
__device__ __forceinline__ void bucket_pairs(const uint64_t* __restrict__ pairs, uint32_t q0,
                                             uint32_t q1, F f) {
  for (uint32_t b0 = q0; b0 < q1; b0 += 4 * kClaimThreads) {
    uint64_t p[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      p[k] = pairs[min(b0 + (uint32_t)(k * kClaimThreads) + threadIdx.x, q1 - 1)];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (b0 + (uint32_t)(k * kClaimThreads) + threadIdx.x < q1)
        f((uint32_t)(p[k] >> 32), (uint32_t)p[k]);
  }
}

__global__ __launch_bounds__(kClaimThreads) void k_bucket_claim(
    uint32_t n, uint32_t S, const uint32_t* __restrict__ tot,
    const uint64_t* __restrict__ pairs, int32_t* __restrict__ d, int32_t* __restrict__ e) {
  __shared__ uint32_t tab[kBucketSlotsMax];
  __shared__ uint32_t s_q[kClaimThreads / kWave];
  const uint32_t b = blockIdx.x;
  const uint32_t s0 = b * S, ns = min(S, n - s0);
  for (uint32_t k = threadIdx.x; k < ns; k += kClaimThreads) tab[k] = n;
  // the bucket's first pair: the pairs of the buckets before it
  uint32_t q = 0;
  for (uint32_t k = threadIdx.x; k < b; k += kClaimThreads) q += tot[k];
  q = wave_reduce(q, OpAdd());
  if (lane_id() == 0) s_q[threadIdx.x / kWave] = q;
  __syncthreads();
  uint32_t q0 = 0;
  for (int w2 = 0; w2 < kClaimThreads / kWave; ++w2) q0 += s_q[w2];
  const uint32_t q1 = q0 + tot[b];
  bucket_pairs(pairs, q0, q1, [&](uint32_t i, uint32_t slot) { atomicMin(&tab[slot - s0], i); });
  __syncthreads();
  for (uint32_t k = threadIdx.x; k < ns; k += kClaimThreads) {
    const uint32_t i = tab[k];
    d[s0 + k] = (int32_t)i;
    if (i < n) e[i] = (int32_t)(s0 + k);  // the winner of slot s0 + k
  }
}

// ---------------------------------------------------------------- resolve, sorted ancestry
// The walk of k_resolve on a sorted ancestry itself, with one bit per slot for
// the claims: position y won its claim when it starts its run (a_y != a_{y-1},
// two neighbouring words), so neither the claim vector nor the marked ancestry
// is written and read.  A chain moves by the ancestry's drift, of the order of
// sqrt(n), per step.  Up to kWindowMax particles a workgroup therefore holds
// the ancestry around its tile of slots in LDS, where most chains stay (a step
// costs an LDS read instead of one beyond the L2): a few steps for the four
// chains of a quad together, then the longer ones from a list, one a lane.
// Chains that leave the window go on in global memory, as do all of them in
// longer vectors.
constexpr int kWinThreads = 512;
constexpr int64_t kWindowMax = 1 << 21;
constexpr uint32_t kWon = 0x80000000u;

// a_y with the winner bit, from global memory
__device__ __forceinline__ uint32_t marked_at(const int32_t* __restrict__ a, uint32_t y) {
  const uint32_t v = (uint32_t)a[y];
  const uint32_t p = y > 0 ? (uint32_t)a[y - 1] : 0xFFFFFFFFu;
  return v != p ? v | kWon : v;
}

template <uint32_t TILE, uint32_t HALO, int STEPS>
struct WindowLds {
  static constexpr uint32_t kTile = TILE, kHalo = HALO, kSpan = TILE + 2 * HALO;
  static constexpr int kSteps = STEPS;
  static constexpr uint32_t kSlow = 1024;  // entries of the list
  alignas(16) uint32_t win[kSpan];
  uint2 slow[kSlow];
  uint32_t n_slow;
};

// The slots [t0, t0 + kTile) of a vector (or segment) of n particles.
template <typename Lds>
__device__ __forceinline__ void resolve_window(const int32_t* __restrict__ a, uint32_t n,
                                               uint32_t t0, const uint32_t* __restrict__ claim,
                                               int32_t* __restrict__ c, Lds* L) {
  constexpr uint32_t kQuads = Lds::kTile / (4 * kWinThreads);  // of a thread
  static_assert(Lds::kTile % (4 * kWinThreads) == 0 && Lds::kSpan % (4 * kWinThreads) == 0,
                "whole rounds");
  uint32_t* const win = L->win;
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t lo = t0 > Lds::kHalo ? t0 - Lds::kHalo : 0u;
  const uint32_t hi = min(n, t0 + Lds::kTile + Lds::kHalo), span = hi - lo;
  if (tid == 0) L->n_slow = 0;
  uint32_t cl[kQuads];
#pragma unroll
  for (uint32_t g = 0; g < kQuads; ++g) {
    const uint32_t j = t0 + 4 * (g * kWinThreads + tid);
    cl[g] = j < n ? (claim[j >> 5] >> (j & 31u)) & 15u : 0u;
  }
#pragma unroll
  for (uint32_t r = 0; r < Lds::kSpan / (4 * kWinThreads); ++r) {
    if (r * 4 * kWinThreads >= span) break;
    const uint32_t q = r * kWinThreads + tid;  // whole waves: the shift below reads lane - 1
    int32_t x[4];
    load_quad(a + lo, q, span, x);
    uint32_t first = 0xFFFFFFFFu;
    if (lane == 0 && lo + 4 * q > 0 && 4 * q < span) first = (uint32_t)a[lo + 4 * q - 1];
    uint32_t prev = wave_shift_up_u32((uint32_t)x[3], first);
    uint32_t m[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      m[k] = (uint32_t)x[k] != prev ? (uint32_t)x[k] | kWon : (uint32_t)x[k];
      prev = (uint32_t)x[k];
    }
    reinterpret_cast<uint4*>(win)[q] = make_uint4(m[0], m[1], m[2], m[3]);
  }
  __syncthreads();
  // the end of the chain that goes on at position y
  auto walk = [&](uint32_t y) -> uint32_t {
    while (true) {
      const uint32_t m = y - lo < span ? win[y - lo] : marked_at(a, y);
      if (!(m & kWon)) return m;
      y = m & ~kWon;
    }
  };
#pragma unroll
  for (uint32_t g = 0; g < kQuads; ++g) {
    const uint32_t j = t0 + 4 * (g * kWinThreads + tid);
    if (j >= n) continue;
    const uint4 t = reinterpret_cast<const uint4*>(win)[(j - lo) / 4];
    uint32_t y[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if ((cl[g] >> k) & 1u || j + k >= n) y[k] = j + k;
    for (int s = 0; s < Lds::kSteps && ((y[0] | y[1] | y[2] | y[3]) & kWon); ++s) {
      uint32_t z[4];
      bool in[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t i = (y[k] & ~kWon) - lo;
        in[k] = (y[k] & kWon) && i < span;
        z[k] = win[in[k] ? i : 0u];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) y[k] = in[k] ? z[k] : y[k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (y[k] & kWon) {
        const uint32_t at = atomicAdd(&L->n_slow, 1u);
        if (at < Lds::kSlow) L->slow[at] = make_uint2(j + k, y[k] & ~kWon);
        else y[k] = walk(y[k] & ~kWon);
      }
    }
    if (j + 4 <= n) {
      Quad o;
      o.x = (int32_t)y[0]; o.y = (int32_t)y[1]; o.z = (int32_t)y[2]; o.w = (int32_t)y[3];
      *reinterpret_cast<Quad*>(c + j) = o;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (j + k < n) c[j + k] = (int32_t)y[k];
    }
  }
  __syncthreads();  // also orders the chains' slots after the quads stored above
  const uint32_t ns = min(L->n_slow, Lds::kSlow);
  for (uint32_t t = tid; t < ns; t += kWinThreads) {
    const uint2 e = L->slow[t];
    c[e.x] = (int32_t)walk(e.y);
  }
}

typedef WindowLds<2048, 3072, 8> VectorWindow;
__global__ __launch_bounds__(kWinThreads) void k_resolve_window(const int32_t* __restrict__ a,
                                                                uint32_t n,
                                                                const uint32_t* __restrict__ claim,
                                                                int32_t* __restrict__ c) {
  __shared__ VectorWindow L;
  resolve_window(a, n, blockIdx.x * VectorWindow::kTile, claim, c, &L);
}

// The same over the segments of a batch, a workgroup per tile.  There are
// tiles enough to fill the chip, so they are larger against their margins (a
// chain moves less in a segment of 2^16 than in a vector of 2^20), and four
// workgroups fit a CU.  Bound by the LDS reads of the chains.  Segments in LDS
// whole (k_permute_lds) leave one workgroup per CU on those of 2^16, and a last
// round that is nearly empty: 4096 ragged segments of 2^8 .. 2^16, 48 M
// particles, 386 -> 155 us, the call 571 -> 342 us.  After three steps half
// the lanes have nothing to do: the list takes the rest (8 steps: 349 us; 16:
// 365; margins of 2048: 354).
typedef WindowLds<(uint32_t)kSegTile, 1024, 3> SegWindow;
__global__ __launch_bounds__(kWinThreads) void k_resolve_segments(
    const int32_t* __restrict__ a, const int64_t* __restrict__ offsets, uint32_t n_filters,
    SegClaim sc, int32_t* __restrict__ c) {
  __shared__ SegWindow L;
  const uint32_t t = blockIdx.x;
  if (t >= sc.tstart[n_filters]) return;
  const uint32_t f = wave_find_segment<uint32_t>(sc.tstart, n_filters, t), t0 = sc.tstart[f];
  const int64_t base = offsets[f];
  resolve_window(a + base, (uint32_t)(offsets[f + 1] - base), (t - t0) * SegWindow::kTile,
                 sc.claim + (size_t)t0 * (kSegTile / 32), c + base, &L);
}


__global__ __launch_bounds__(256) void k_resolve_sorted(const int32_t* __restrict__ a, int64_t n,
                                                        const uint32_t* __restrict__ claim,
                                                        int32_t* __restrict__ c) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += stride) {
    uint32_t m = marked_at(a, (uint32_t)j);  // in flight with the claim word
    if ((claim[j >> 5] >> (j & 31)) & 1u) m = (uint32_t)j;
    while (m & kWon) m = marked_at(a, m & ~kWon);
    c[j] = (int32_t)m;
  }
}

int grid_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return (int)b;
}

}  // namespace

size_t o2a_workspace_bytes(int64_t n_total) {
  const size_t tiles = (size_t)((n_total + kO2aTile - 1) / kO2aTile);
  return 256 + align256(tiles * sizeof(uint64_t));
}

hipError_t launch_offspring_to_ancestors(const int32_t* o, int64_t n_total, const int64_t* offsets,
                                         uint32_t n_filters, int32_t* a, void* ws,
                                         uint32_t* flags, hipStream_t stream) {
  if (offsets || n_filters > 1 || n_total <= kO2aTile) {
    hipLaunchKernelGGL(k_o2a_batched, dim3(offsets ? n_filters : 1u), dim3(256), 0, stream, o,
                       n_total, offsets, offsets ? n_filters : 1u, a, flags);
    return hipGetLastError();
  }
  const uint32_t ntiles = (uint32_t)((n_total + kO2aTile - 1) / kO2aTile);
  O2aHeader* hdr = (O2aHeader*)ws;
  uint64_t* status = (uint64_t*)((char*)ws + 256);
  hipLaunchKernelGGL(k_o2a, dim3(ntiles), dim3(256), 0, stream, o, n_total, a, hdr, status, flags,
                     ntiles);
  return hipGetLastError();
}

// Workspace: the claim vector d and the marked ancestry e, n int32 each; a
// single unsorted vector beyond the LDS path also gets the bucketed claim's
// counts and pairs (8 more bytes per particle), without which it takes the
// atomic claim.
size_t permute_workspace_min_bytes(int64_t n_total) {
  return 2 * align256((size_t)n_total * sizeof(int32_t));
}
size_t permute_workspace_bytes(int64_t n_total, uint32_t n_filters) {
  if (n_filters <= 1 && n_total > kPermSmallWorkspace && bucket_claim_fits(n_total))
    return bucket_geom(n_total).bytes;
  return permute_workspace_min_bytes(n_total);
}

// Batches whose segments fit in LDS, and short single vectors, are permuted
// there (k_permute_lds, one workgroup per segment); longer segments go
// through the global kernels.  max_len: longest segment (0 = unknown).
hipError_t launch_permute(const int32_t* a, int64_t n_total, const int64_t* offsets,
                          uint32_t n_filters, int64_t max_len, bool sorted, int32_t* c, void* ws,
                          size_t ws_bytes, uint32_t* flags, hipStream_t stream) {
  int32_t* d = (int32_t*)ws;
  int32_t* e = (int32_t*)((char*)ws + align256((size_t)n_total * sizeof(int32_t)));
  const int grid = grid_for(n_total);
  int64_t min_len = 0;  // shorter segments are done in LDS
  if (!(offsets && n_filters > 1) && n_total <= (sorted ? kPermSingleMaxSorted : kPermSingleMax)) {
    // a short single vector: one workgroup, one launch
    if (n_total <= kPermShort)
      hipLaunchKernelGGL(k_permute_small, dim3(1), dim3(kSmallThreads), 0, stream, a,
                         (int32_t)n_total, c, flags);
    else
      hipLaunchKernelGGL((k_permute_lds<kPermMid, 1024>), dim3(1), dim3(1024), 0, stream, a,
                         n_total, (const int64_t*)nullptr, (int64_t)0, (int64_t)kPermSingleMax,
                         false, sorted, d, c, flags);
    return hipGetLastError();
  }
  if (offsets && n_filters > 1) {
    // four tiers by segment length, each launch taking its own segments:
    // short ones in 256-thread workgroups (eight to a CU), those up to the
    // tuned length in 1024 threads (two to a CU), those up to 32768 and to
    // 65536 in 1024 threads (one to a CU); longer ones below.  A tier takes
    // the shorter segments too, and their launches fall away, when there are
    // none (every segment has the full length) or when all segments together
    // do not fill the chip once.  The one workgroup of a long segment takes
    // 30 to 70 us, so below kPermLongTotal particles the global kernels,
    // spread over the chip, run the long ones (four of 60000: 22 against 67
    // us; 256 of them 313 against 68 us).  So do they where the LDS tiers come
    // on top of the global kernels, for which the batch has longer segments or
    // none that are known of, and too little would be left to them: by the
    // average segment and, for a sorted ancestry, whose global kernels are
    // fast, by the particles (global against LDS and global, us: 30 of 2^16 ..
    // 2^17.9 sorted 120 / 190, unsorted 329 / 394; 60 of 2^15.8 .. 2^16.2 121 /
    // 163 and 312 / 275; 100 of 2^14.5 .. 2^17 sorted 121 / 154; 200 of 2^15 ..
    // 2^16.5 332 / 304; without max_len 100 of 60000 174 / 117, 100 of 2^15 .. 2^16
    // 142 / 113, 64 of them 63 / 78).
    const int64_t mid = tuning().batch_permute_lds_max;
    const bool equal = max_len > 0 && max_len * (int64_t)n_filters == n_total;
    const bool bounded = max_len > 0 && max_len <= kPermBatchMax;
    const int64_t mean = n_total / (int64_t)n_filters;
    const bool beyond = sorted ? mean > kPermBatchMax || n_total < 2 * kPermLongTotal ||
                                     (max_len > 0 && mean > 52000 &&
                                      n_total < 4 * kPermLongTotal)
                               : 4 * mean > 5 * kPermBatchMax;
    const bool spread = n_total < kPermLongTotal || (!bounded && beyond);
    const int64_t top = spread ? mid : kPermBatchMax;
    const int64_t upto[4] = {kPermShort, mid, kPermLong, kPermBatchMax};
    constexpr uint32_t kSlots[4] = {0, 512, 256, 256};  // workgroups the chip holds at once
    const int64_t need = max_len > 0 ? (max_len < top ? max_len : top) : top;
    int64_t above = 0;
    for (int t = 0; t < 4 && above < need; ++t) {
      if (upto[t] < need && (equal || n_filters <= kSlots[upto[1] < need ? (upto[2] < need ? 3 : 2) : 1]))
        continue;
      const dim3 g(n_filters);
      // (the tier that ends the call takes what is longer than max_len too)
      const bool last = max_len > 0 && max_len <= top && upto[t] >= need;
      auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, g, dim3(threads), 0, stream, a, n_total, offsets, above, upto[t],
                           last, sorted, d, c, flags);
      };
      if (t == 0) launch(k_permute_lds<kPermShort, 256>, 256);
      else if (t == 1) launch(k_permute_lds<kPermMid, 1024>, 1024);
      else if (t == 2) launch(k_permute_lds<kPermLong, 1024>, 1024);
      else launch(k_permute_lds<kPermBatchMax, 1024>, 1024);
      above = upto[t];
    }
    hipError_t e0 = hipGetLastError();
    if (e0 != hipSuccess) return e0;
    if (max_len > 0 && max_len <= top) return hipSuccess;
    min_len = top + 1;
  }
  if (sorted) {
    hipLaunchKernelGGL(k_claim_sorted, dim3(grid), dim3(256), 0, stream, a, n_total, offsets,
                       n_filters, min_len, d, e, flags);
    hipLaunchKernelGGL(k_resolve, dim3(grid), dim3(256), 0, stream, n_total, offsets, n_filters,
                       min_len, d, e, c, flags);
    return hipGetLastError();
  }
  if (!(offsets && n_filters > 1) && bucket_claim_fits(n_total) &&
      ws_bytes >= bucket_geom(n_total).bytes) {
    // one vector: the bucketed claim writes d and e, then the walk on e
    const BucketGeom g = bucket_geom(n_total);
    char* base = (char*)ws;
    uint32_t* cnt = (uint32_t*)(base + g.cnt_off);
    uint32_t* tot = (uint32_t*)(base + g.tot_off);
    uint64_t* pairs = (uint64_t*)(base + g.pairs_off);
    const uint32_t n = (uint32_t)n_total;
    hipLaunchKernelGGL(k_bucket_count, dim3(g.W), dim3(kBucketThreads), 0, stream, a, n, g.log2S,
                       g.C, g.B, g.W, cnt, flags);
    hipLaunchKernelGGL(k_bucket_rows, dim3(g.B), dim3(kBucketThreads), 0, stream, cnt, g.W, tot);
    hipLaunchKernelGGL(k_bucket_scatter, dim3(g.W), dim3(kBucketThreads), 0, stream, a, n,
                       g.log2S, g.C, g.B, g.W, (const uint32_t*)cnt, (const uint32_t*)tot, pairs,
                       e);
    hipLaunchKernelGGL(k_bucket_claim, dim3(g.B), dim3(kClaimThreads), 0, stream, n, g.S,
                       (const uint32_t*)tot, (const uint64_t*)pairs, d, e);
    hipLaunchKernelGGL(k_resolve, dim3(grid), dim3(256), 0, stream, n_total, offsets, n_filters,
                       min_len, d, e, c, flags);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_fill_unclaimed, dim3(grid), dim3(256), 0, stream, d, n_total, offsets,
                     n_filters, min_len);
  hipLaunchKernelGGL(k_claim_min, dim3(grid), dim3(256), 0, stream, a, n_total, offsets,
                     n_filters, min_len, d, flags);
  hipLaunchKernelGGL(k_resolve_ad, dim3(grid), dim3(256), 0, stream, a, n_total, offsets,
                     n_filters, min_len, d, c, flags);
  return hipGetLastError();
}

// The permutation workspace is at least 8 bytes per particle: room for the
// bits of whole blocks from 1025 particles on.
hipError_t launch_resolve_sorted(const int32_t* a, int64_t n, const uint32_t* claim, int32_t* c,
                                 hipStream_t stream) {
  if (n <= kWindowMax)
    hipLaunchKernelGGL(k_resolve_window, dim3((unsigned)((n + VectorWindow::kTile - 1) / VectorWindow::kTile)),
                       dim3(kWinThreads), 0, stream, a, (uint32_t)n, claim, c);
  else
    hipLaunchKernelGGL(k_resolve_sorted, dim3(grid_for(n)), dim3(256), 0, stream, a, n, claim, c);
  return hipGetLastError();
}

// whole tiles: each segment adds at most one partial one
static size_t seg_claim_words(int64_t n_total, uint32_t n_filters) {
  return (size_t)(n_total / kSegTile + n_filters) * (kSegTile / 32);
}
size_t seg_claim_bytes(int64_t n_total, uint32_t n_filters) {
  return align256(seg_claim_words(n_total, n_filters) * sizeof(uint32_t)) +
         align256(((size_t)n_filters + 1) * sizeof(uint32_t));
}
SegClaim seg_claim_in(void* ws, int64_t n_total, uint32_t n_filters) {
  SegClaim sc;
  sc.claim = (uint32_t*)ws;
  sc.tstart = (uint32_t*)((char*)ws +
                          align256(seg_claim_words(n_total, n_filters) * sizeof(uint32_t)));
  return sc;
}

hipError_t launch_resolve_segments(const int32_t* a, int64_t n_total, const int64_t* offsets,
                                   uint32_t n_filters, const SegClaim& sc, int32_t* c,
                                   hipStream_t stream) {
  hipLaunchKernelGGL(k_resolve_segments, dim3((unsigned)(n_total / kSegTile + n_filters)),
                     dim3(kWinThreads), 0, stream, a, offsets, n_filters, sc, c);
  return hipGetLastError();
}

__global__ void k_zero_u32(uint32_t* __restrict__ p, size_t count) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = 0;
}

hipError_t launch_zero_u32(uint32_t* p, size_t count, hipStream_t stream) {
  if (count == 0) return hipSuccess;
  size_t blocks = (count + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)blocks), dim3(256), 0, stream, p, count);
  return hipGetLastError();
}

}  // namespace pfr
