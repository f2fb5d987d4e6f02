// kb_assemble.hpp -- assembly of lower-triangular CSR K on gfx950.
//
// Every element contributes nen(nen+1)/2 lower pairs (Alg. 1 mapping): the node of
// rank r in its element (by global id) owns the r+1 pairs (itself, smaller ids) whose
// global row is that node.  Assembly (Eq. 6) sums the pairs with equal (row, col).
//
// Data movement: a partition by row, then a streaming reduction in LDS.
//   begin    status and counters cleared, padded coordinates (32 bytes per node), and a
//            sample of the elements that tells whether they are numbered with locality.
//   count    per tile of elements: pairs per row bucket (row >> s1), tile-major; or, the
//            direct way (few sub-buckets, or locality), pairs per sub-bucket (row >> s2).
//   offsets  column scan of the tile-major counts: each tile's write offset in each
//            bucket; or the scan of the sub-bucket counts.
//   pass 1   per tile (one element per lane): integrate the element (or read given
//            values), stage its pairs in LDS grouped by bucket or sub-bucket, write each
//            group's run as (row, col, value) arrays, or (row_local << colbits | col,
//            value).  Also the largest value exponent, which fixes the exact-sum scale.
//   pass 2   (not the direct way) per fixed-size segment of a bucket: histogram of
//            sub-buckets; per bucket, a prefix over its segments for each sub-bucket;
//            then LDS-staged scatter into contiguous sub-bucket ranges; pairs are
//            repacked as (row_local << colbits | col, value).
//   pass 3   per sub-bucket: stream its pairs into an LDS hash table keyed by the
//            packed (row, col); each value is added as a 128-bit fixed-point integer
//            (scale 2^F from the largest exponent), so every sum is exact and its
//            result does not depend on the order of the additions: the output is
//            bitwise deterministic although the partition orders pairs through
//            atomics.  Entries are then ordered by (row, col) and converted once
//            (correct rounding of the exact sum to the value type).
//   final    scan of per-sub-bucket unique counts; row_ptr and the compacted col/vals.
// Sub-buckets whose distinct entries overflow the table are reduced in parts (k_pass3_parts) or
// by k_heavy.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kb_element.hpp"
#include "kb_kernels.hpp"
#include "kbuild.h"

namespace kb {

constexpr uint32_t kEmptyKey = 0xFFFFFFFFu;  // packed keys never use bit 31

// ----------------------------------------------------------------- block helpers
// exclusive scan of one uint32 per thread across the block; *total = block sum.
// smem must hold (blockDim/64 + 1) words.  Contains barriers: call from all threads.
__device__ __forceinline__ uint32_t block_scan_u32(uint32_t v, uint32_t* smem, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) smem[wave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t s = 0;
    for (int w = 0; w < nw; ++w) {
      uint32_t t = smem[w];
      smem[w] = s;
      s += t;
    }
    smem[nw] = s;
  }
  __syncthreads();
  const uint32_t r = x - v + smem[wave];
  *total = smem[nw];
  __syncthreads();
  return r;
}

// in-place exclusive scan of a[0..n) in LDS (n arbitrary); returns the total.
template <typename T>
__device__ __forceinline__ uint32_t block_scan_array(T* a, int n, uint32_t* smem) {
  const int per = (n + (int)blockDim.x - 1) / (int)blockDim.x;
  const int lo = threadIdx.x * per;
  uint32_t s = 0;
  for (int i = 0; i < per; ++i)
    if (lo + i < n) s += (uint32_t)a[lo + i];
  uint32_t total;
  uint32_t off = block_scan_u32(s, smem, &total);
  for (int i = 0; i < per; ++i)
    if (lo + i < n) {
      const uint32_t v = (uint32_t)a[lo + i];
      a[lo + i] = (T)off;
      off += v;
    }
  __syncthreads();
  return total;
}

// Called by every workgroup (256 threads) of a grid of `blocks` once it has added to
// cnt[0 .. n) (atomics): the last one to arrive turns the counts into exclusive offsets,
// starts[0 .. n] and, in place, cnt.  *done starts at zero.
__device__ __forceinline__ void last_block_starts(uint32_t* cnt, int n, uint32_t* starts, uint32_t* done,
                                                  uint32_t blocks) {
  __shared__ uint32_t s_scan[8], s_last;
  // This thread's additions done before the arrival.  Nothing but atomics passes between the
  // workgroups, so the wait stands for a release fence, which would write back the L2.  That is
  // particular to gfx9, not a release of the HIP memory model: there s_waitcnt vmcnt(0) also
  // waits for atomics that return nothing, which by then are done where every XCD sees them, as
  // the agent-scope loads below do (later families count such atomics apart, in vscnt).
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomicAdd(done, 1u) == blocks - 1 ? 1u : 0u;
  __syncthreads();
  if (!s_last) return;
  uint32_t carry = 0;
  for (int b0 = 0; b0 < n; b0 += blockDim.x) {
    const int b = b0 + threadIdx.x;
    const uint32_t v = b < n ? __hip_atomic_load(&cnt[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    uint32_t total;
    const uint32_t ex = carry + block_scan_u32(v, s_scan, &total);
    if (b < n) {
      starts[b] = ex;
      cnt[b] = ex;
    }
    carry += total;
  }
  if (threadIdx.x == 0) starts[n] = carry;
}

// ------------------------------------------------------- exact fixed-point sums
// A finite double v is m * 2^(E-1075) (m < 2^53).  With the scale F = 1117 - Emax,
// where Emax is the largest biased exponent of all values, q = v * 2^F is below 2^95
// in magnitude, so up to 2^31 of them sum exactly in a 128-bit two's complement
// integer.  Bits below 2^-F are dropped (truncation toward zero, independent of
// order).  Non-finite values contribute 0 (they are flagged elsewhere).
__device__ __forceinline__ int biased_exponent(double v) {
  return (int)((__double_as_longlong(v) >> 52) & 0x7FF);
}

__device__ __forceinline__ void to_fixed(double v, int F, uint64_t& lo, uint64_t& hi) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  int E = (int)((b >> 52) & 0x7FF);
  uint64_t m = b & ((1ull << 52) - 1);
  lo = 0;
  hi = 0;
  if (E == 0x7FF) return;
  if (E == 0)
    E = 1;  // subnormal
  else
    m |= 1ull << 52;
  if (m == 0) return;
  const int sh = E - 1075 + F;
  if (sh >= 64) {
    hi = m << (sh - 64);
  } else if (sh > 0) {
    lo = m << sh;
    hi = m >> (64 - sh);
  } else if (sh == 0) {
    lo = m;
  } else if (sh > -64) {
    lo = m >> (-sh);
  }
  if (b >> 63) {  // negate (two's complement)
    lo = ~lo + 1;
    hi = ~hi + (lo == 0 ? 1ull : 0ull);
  }
}

// A double or float value's q = trunc(v * 2^F) (non-finite: zero; |q| < 2^95) as chunks
// c0 + c1 * 2^48 with c0 in [0, 2^48) and c1 signed: sums of up to 2^16 such terms fit in one
// unsigned / signed 64-bit word each, so they can be accumulated without carries (and in any
// order).  Formed in FP64 arithmetic, where every step is exact: v 2^F only moves the exponent
// (|q| < 2^95; a result below 2^-1022 truncates to 0 either way), trunc and floor give
// integers, and c1 = floor(q / 2^48), c0 = q - c1 2^48 in [0, 2^48) are multiples of
// q's last bit below 2^53 of it.  Each integer then becomes a 64-bit word by an exact
// FP64 addition: c0 + 2^52 and c1 + 1.5 2^52 (|c1| < 2^47) lie in [2^52, 2^53), where
// the spacing is 1, so their bit patterns are those of the constants plus the integer
// (two's complement for a negative c1), and the constants' low 32 bits are zero: one
// 32-bit subtraction from the high word leaves the integer: the same as from to_fixed's
// q, without forming the 128-bit integer and without branches.
__device__ __forceinline__ void to_chunks(double v, int F, uint64_t& c0, int64_t& c1) {
  const double d = isfinite(v) ? v : 0.0;
  const double q = trunc(ldexp(d, F));
  const double h = floor(ldexp(q, -48));
  const double l = fma(h, -0x1p48, q);  // [0, 2^48)
  const uint64_t bl = (uint64_t)__double_as_longlong(l + 0x1p52);
  const uint64_t bh = (uint64_t)__double_as_longlong(h + 0x1.8p52);
  c0 = bl - 0x4330000000000000ull;
  c1 = (int64_t)(bh - 0x4338000000000000ull);
}
__device__ __forceinline__ void to_chunks(float v, int F, uint64_t& c0, int64_t& c1) {
  to_chunks((double)v, F, c0, c1);  // a float is exactly a double
}

// chunk sums back to the exact 128-bit value
__device__ __forceinline__ void join48(uint64_t s0, int64_t s1, uint64_t& lo, uint64_t& hi) {
  const uint64_t a_lo = (uint64_t)s1 << 48;
  const uint64_t a_hi = (uint64_t)(s1 >> 16);  // arithmetic shift keeps the sign
  lo = s0 + a_lo;
  hi = a_hi + (lo < s0 ? 1ull : 0ull);
}

// exact 128-bit value -> V (double or float), rounded once to nearest; then scaled by
// 2^-F (exact unless the result is subnormal).  The 64 leading bits carry a sticky bit
// for the rest, so the one rounding of the 64-bit integer to V is that of the whole.
template <typename V>
__device__ __forceinline__ V from_fixed_as(uint64_t lo, uint64_t hi, int F) {
  const bool neg = (int64_t)hi < 0;
  if (neg) {
    lo = ~lo + 1;
    hi = ~hi + (lo == 0 ? 1ull : 0ull);
  }
  uint64_t top = lo;
  int sh = 0;
  if (hi != 0) {
    const int lz = __clzll((long long)hi);
    top = lz ? ((hi << lz) | (lo >> (64 - lz))) : hi;
    const uint64_t rest = lz ? (lo << lz) : lo;
    top |= rest ? 1ull : 0ull;  // sticky bit: 64 > 53 + 2 bits, so the rounding stays correct
    sh = 64 - lz;
  }
  V d;
  if constexpr (sizeof(V) == 8)
    d = ldexp(ldexp((double)top, sh), -F);
  else
    d = ldexpf(ldexpf((float)top, sh), -F);
  return neg ? -d : d;
}
__device__ __forceinline__ double from_fixed(uint64_t lo, uint64_t hi, int F) {
  return from_fixed_as<double>(lo, hi, F);
}

// What V's rounding h of an exact value left out, rounded to V: h + residual holds the
// value to about twice V's precision.  h * 2^F is an integer (the value rounded), so its
// fixed-point form is exact and the difference is exact before its one rounding.
template <typename V>
__device__ __forceinline__ V fixed_residual(uint64_t lo, uint64_t hi, int F, V h) {
  uint64_t a, b;
  to_fixed((double)h, F, a, b);
  const uint64_t dl = lo - a;
  const uint64_t dh = hi - b - (lo < a ? 1ull : 0ull);
  return from_fixed_as<V>(dl, dh, F);
}

// ---------------------------------------------------------------- where pairs go
// Pass 1 partitions its tile's pairs by bucket (row >> s1, then pass 2 splits each bucket
// into sub-buckets) or sends them straight to their sub-buckets (row >> s2), which skips
// pass 2: its histogram, offsets and scatter, a read and a write of every pair.  A tile's
// run in a sub-bucket takes one global atomic for its places, so the direct way pays when
// a tile's pairs fall in few sub-buckets:
//   - kDirect, few sub-buckets in the whole mesh (host: at most kSlotsArray, and at most
//     kDirectRuns runs in all): one LDS counter per sub-bucket;
//   - kAsk: elements and nodes numbered with locality.  k_begin counts the sub-buckets
//     that kSamples evenly spaced tiles touch, and every kernel after it takes the direct
//     way if the sampled runs average at least kDirectRun pairs.  A sample is the first
//     256 elements of a tile: in grid order their runs have 115 pairs and more, and under
//     a random numbering of the nodes a run is a node, about 30 at most (there the longest
//     rows would overfill the direct way's tables: 95,000 tets in grid order with random
//     nodes, pass 3 15 us on two levels and 117 direct).  An LDS hash of
//     kSlotsHash slots then maps a tile's sub-buckets to counters; a row whose sub-bucket
//     finds no slot takes its places one by one.
// The sums are exact, so both ways give the same matrix bit for bit.
enum { kTwoLevel = 0, kDirect = 1, kAsk = 2 };
constexpr int kSlotsHash = 512, kSlotsArray = 1024, kSlotProbes = 16;
constexpr int kSamples = 8;
constexpr uint32_t kDirectRun = 32;
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;

// head words of a build: [0] largest exponent, [1] heavy sub-buckets, [2] and [3]
// workgroups done (k_heavy, k_count), [4] sub-buckets listed for k_pass3_parts, then the way
// taken (kAsk) and the samples
constexpr int kHeadWay = 15, kHeadVotes = 16, kHeadWords = 64;

// the way sampled: votes[2 i], votes[2 i + 1] are the sub-buckets and the pairs of tile i
__device__ __forceinline__ bool votes_direct(const uint32_t* __restrict__ votes) {
  uint64_t runs = 0, pairs = 0;
#pragma unroll
  for (int i = 0; i < kSamples; ++i) {
    runs += votes[2 * i];
    pairs += votes[2 * i + 1];
  }
  return runs * kDirectRun <= pairs;
}

// elements in random order too: runs of a few pairs (8 nodes of a brick: 4.5; in grid order
// with random nodes 9)
__device__ __forceinline__ bool votes_scattered(const uint32_t* __restrict__ votes) {
  uint64_t runs = 0, pairs = 0;
#pragma unroll
  for (int i = 0; i < kSamples; ++i) {
    runs += votes[2 * i];
    pairs += votes[2 * i + 1];
  }
  return runs * 6 > pairs;
}

// *way: written by k_count (1: direct, 2: two levels, elements in random order)
__device__ __forceinline__ bool goes_direct(int mode, const uint32_t* __restrict__ way) {
  return mode == kAsk ? *way == 1 : mode == kDirect;
}

// The sub-buckets of each way: rows per sub-bucket 2^s2[way] and their number, way 1 being
// the direct one.  Rows of a mesh numbered with locality have much the same length, so the
// direct way's sub-buckets may fill pass 3's table to kDirectLoad where the two-level
// way's may not (under a random numbering the last rows are twice the average): 32 rows of
// bricks instead of 16 (27M bricks FP64, pass 3 5.9 -> 4.9 ms; randomly numbered 1M bricks
// 0.28 -> 0.33 ms).  Where rows are of unlike length all the same, k_pass3_parts takes over.
struct SubBuckets {
  int s2[2], nsub[2];
  int mode;
  const uint32_t* way;
  __device__ __forceinline__ int pick() const { return goes_direct(mode, way) ? 1 : 0; }
};

// The LDS counters of a tile: one per bucket (two levels), per sub-bucket of the mesh
// (direct, array), or per sub-bucket that the tile touches (direct, hash: key[] holds the
// sub-bucket of each slot).  The ways are separate code under one branch at the top of
// each kernel: as run-time cases of the same code they cost the two-level kernels 5%
// (20.25M tets, pass 1 2.03 -> 2.12 ms) in scalar registers.
template <bool DIRECT>
struct TileSlots {
  uint32_t* cnt;  // [n] pairs per slot, then local run starts
  uint32_t* key;  // [n] sub-bucket of the slot (hash)
  int n;          // counters in use
  int shift;      // row -> bucket or sub-bucket
  bool hash;
  __device__ __forceinline__ TileSlots(uint32_t* cnt_, uint32_t* key_, int mode, int s1, int nb, int s2, int nsub) {
    hash = DIRECT && mode == kAsk;
    cnt = cnt_;
    key = key_;
    n = DIRECT ? (hash ? kSlotsHash : nsub) : nb;
    shift = DIRECT ? s2 : s1;
  }
  __device__ __forceinline__ void clear(int nthreads) const {
    for (int b = threadIdx.x; b < n; b += nthreads) {
      cnt[b] = 0;
      if (hash) key[b] = kEmptyKey;
    }
  }
  // the slot of (sub-)bucket x, or kNoSlot (hash: no free slot within kSlotProbes probes)
  __device__ __forceinline__ uint32_t find(uint32_t x) const {
    if (!DIRECT || !hash) return x;
    constexpr int bits = __builtin_ctz(kSlotsHash);
    uint32_t h = (x * 0x9E3779B1u) >> (32 - bits);
#pragma unroll 1
    for (int p = 0; p < kSlotProbes; ++p) {
      uint32_t k = __hip_atomic_load(&key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (k == kEmptyKey) k = atomicCAS(&key[h], kEmptyKey, x);
      if (k == x || k == kEmptyKey) return h;
      h = (h + 1) & (kSlotsHash - 1);
    }
    return kNoSlot;
  }
  // a row's places as reserve_rows returns them: its slot and its first place in the
  // slot's part of the tile
  __device__ __forceinline__ uint32_t slot(uint32_t q, int32_t row) const {
    return DIRECT ? q >> 16 : (uint32_t)(row >> shift);
  }
  __device__ __forceinline__ uint32_t place(uint32_t q) const { return DIRECT ? q & 0xFFFFu : q; }
};

// Reserve the pairs of local rows OFF .. OFF+N-1 of an element in their slots' LDS
// counters: each run of consecutive rows in one slot takes one atomic for its total
// (under a natural numbering an element's neighbouring nodes mostly share a bucket, and
// per-row increments from neighbouring lanes would serialise on one address); a row
// after the first of its run starts where its predecessor's pairs end.  q: first place of
// the row's r+1 pairs within the slot's part of the tile; direct: slot << 16 | that, or
// kNoSlot.
template <int N, int OFF, int NE, bool DIRECT>
__device__ __forceinline__ void reserve_rows(const TileSlots<DIRECT>& sl, const int32_t (&E)[NE], const int (&r)[NE],
                                             uint32_t (&q)[N]) {
  uint32_t tot[N];  // pairs from row a to the end of its run
  tot[N - 1] = (uint32_t)(r[OFF + N - 1] + 1);
#pragma unroll
  for (int a = N - 2; a >= 0; --a)
    tot[a] = (uint32_t)(r[OFF + a] + 1) +
             ((E[OFF + a] >> sl.shift) == (E[OFF + a + 1] >> sl.shift) ? tot[a + 1] : 0u);
#pragma unroll
  for (int a = 0; a < N; ++a) {
    if (a > 0 && (E[OFF + a] >> sl.shift) == (E[OFF + a - 1] >> sl.shift)) {
      q[a] = DIRECT && q[a - 1] == kNoSlot ? kNoSlot : q[a - 1] + (uint32_t)(r[OFF + a - 1] + 1);
    } else if constexpr (DIRECT) {
      const uint32_t s = sl.find((uint32_t)(E[OFF + a] >> sl.shift));
      q[a] = s == kNoSlot ? kNoSlot : (s << 16 | atomicAdd(&sl.cnt[s], tot[a]));
    } else {
      q[a] = atomicAdd(&sl.cnt[E[OFF + a] >> sl.shift], tot[a]);
    }
  }
}

// ---------------------------------------------------------------------- begin, count
__device__ __forceinline__ double4 padded(const double* __restrict__ coords, int64_t i) {
  return make_double4(coords[3 * i], coords[3 * i + 1], coords[3 * i + 2], 0.0);
}

// First kernel of a build.  Workgroups 0 .. kSamples-1: workgroup 0 clears the status (if
// not null), the entry count and the head words; with kAsk, workgroup i samples the tile at
// i / kSamples of the elements.  The others clear n_zero words at every stride-th word of
// zero (n_tab times: the row counts of the heavy sub-buckets' tables), and the sub-bucket counters,
// and pad the coordinates of the first n_pad nodes (k_count).
template <int NEN>
__global__ __launch_bounds__(256) void k_begin(const int32_t* __restrict__ conn, int64_t n_elem, int64_t n_node,
                                               int tile, int64_t ntiles, int s2, int mode,
                                               uint32_t* __restrict__ status, int64_t* __restrict__ nnz,
                                               uint32_t* __restrict__ head, uint32_t* __restrict__ subcnt,
                                               int64_t nsub, const double* __restrict__ coords,
                                               double4* __restrict__ coords4, int64_t n_pad,
                                               uint32_t* __restrict__ zero, int n_tab, int stride, int n_zero) {
  constexpr int kSet = 4096;  // twice the sub-buckets of a random sample of bricks
  __shared__ uint32_t s_set[kSet];
  __shared__ uint32_t s_runs, s_pairs;
  if (blockIdx.x >= kSamples) {
    const int64_t i0 = (int64_t)(blockIdx.x - kSamples) * blockDim.x + threadIdx.x;
    const int64_t step = (int64_t)(gridDim.x - kSamples) * blockDim.x;
    for (int64_t i = i0; i < (int64_t)n_tab * n_zero; i += step) zero[i / n_zero * stride + i % n_zero] = 0u;
    if (mode != kTwoLevel)
      for (int64_t i = i0; i < nsub; i += step) subcnt[i] = 0u;
    for (int64_t i = i0; i < n_pad; i += step) coords4[i] = padded(coords, i);
    return;
  }
  if (blockIdx.x == 0) {
    if (status && threadIdx.x < KB_STATUS_WORDS) status[threadIdx.x] = 0u;
    if (nnz && threadIdx.x == 0) *nnz = 0;
    if (threadIdx.x < kHeadVotes) head[threadIdx.x] = 0u;
  }
  if (mode != kAsk) return;
  for (int h = threadIdx.x; h < kSet; h += blockDim.x) s_set[h] = kEmptyKey;
  if (threadIdx.x == 0) {
    s_runs = 0u;
    s_pairs = 0u;
  }
  __syncthreads();
  const int64_t t = ntiles * blockIdx.x / kSamples;
  const int64_t e0 = t * tile, e1 = e0 + tile < n_elem ? e0 + tile : n_elem;
  uint32_t runs = 0, pairs = 0;
  const int64_t e = e0 + threadIdx.x;
  int32_t E[NEN];
  if (e < e1) load_conn<NEN>(conn, e, E);
  if (e < e1 && check_conn<NEN>(E, n_node) == 0) {
    pairs += NEN * (NEN + 1) / 2;
#pragma unroll
    for (int a = 0; a < NEN; ++a) {
      const uint32_t x = (uint32_t)(E[a] >> s2);
      if (a > 0 && x == (uint32_t)(E[a > 0 ? a - 1 : 0] >> s2)) continue;
      uint32_t h = (x * 0x9E3779B1u) >> (32 - __builtin_ctz(kSet));
      int p = 0;
#pragma unroll 1
      for (; p < 16; ++p) {
        uint32_t k = __hip_atomic_load(&s_set[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (k == kEmptyKey) {
          k = atomicCAS(&s_set[h], kEmptyKey, x);
          if (k == kEmptyKey) ++runs;
        }
        if (k == kEmptyKey || k == x) break;
        h = (h + 1) & (kSet - 1);
      }
      if (p == 16) ++runs;  // a full set: no locality
    }
  }
  if (runs) atomicAdd(&s_runs, runs);
  if (pairs) atomicAdd(&s_pairs, pairs);
  __syncthreads();
  if (threadIdx.x == 0) {
    head[kHeadVotes + 2 * blockIdx.x] = s_runs;
    head[kHeadVotes + 2 * blockIdx.x + 1] = s_pairs;
  }
}

// A tile's counts added to the sub-bucket counters (direct): one atomic per run.
__device__ __forceinline__ void flush_counts(const TileSlots<true>& sl, uint32_t* __restrict__ subcnt) {
  for (int b = threadIdx.x; b < sl.n; b += blockDim.x) {
    const uint32_t c = sl.cnt[b];
    if (c) atomicAdd(&subcnt[sl.hash ? sl.key[b] : (uint32_t)b], c);
  }
}

// Per tile of `te` elements: pairs per bucket (row >> s1), written tile-major
// hist[t * nb + b]; or, direct, pairs per sub-bucket added to subcnt.  Flags index errors;
// invalid elements contribute nothing.  With kDirect the last workgroup to finish turns
// the counts into the sub-bucket starts sbb[0 .. nsub] and, in place, the write cursors.
// With kAsk the samples decide, and the first workgroup tells the kernels after this one.
// A workgroup counts `per` tiles; direct, where no tile has a histogram of its own, as one
// (the slots are cleared and flushed once: 27M bricks 638 -> 516 us).
template <int NEN, bool DIRECT>
__device__ __forceinline__ void count_elements(const TileSlots<DIRECT>& sl, const int32_t* __restrict__ conn,
                                               int64_t e0, int64_t e1, int64_t n_node, uint32_t* __restrict__ subcnt,
                                               uint32_t* flags) {
  int32_t En[NEN];
  int64_t e = e0 + threadIdx.x;
  if (e < e1) load_conn<NEN>(conn, e, En);
  for (; e < e1; e += blockDim.x) {
    int32_t E[NEN];
#pragma unroll
    for (int a = 0; a < NEN; ++a) E[a] = En[a];
    if (e + blockDim.x < e1) load_conn<NEN>(conn, e + blockDim.x, En);
    const uint32_t f = check_conn<NEN>(E, n_node);
    if (f) {
      *flags |= f;
      continue;
    }
    int r[NEN];
    node_ranks<NEN>(E, r);
    uint32_t q[NEN];
    reserve_rows<NEN, 0>(sl, E, r, q);
    if constexpr (DIRECT) {
#pragma unroll
      for (int a = 0; a < NEN; ++a)
        if (q[a] == kNoSlot) atomicAdd(&subcnt[E[a] >> sl.shift], (uint32_t)(r[a] + 1));
    }
  }
}

// Elements of more than 8 rows come in tiles of a few dozen: a lane takes one row of an
// element (1M bricks of 3 components, 31 elements a tile: 501 -> 436 us).  On two levels only
// those of more than 16, whose ids and ranks overflow a lane's registers (bricks of 3 components
// 97 -> 38 us; tetrahedra of 3, 90 elements a tile: 84 with a lane a row, 65 with one an element).
// s_E: LDS for te elements' ids, then a word each (its errors).
template <int NEN, bool DIRECT>
__device__ __forceinline__ void count_rows(const TileSlots<DIRECT>& sl, uint32_t* s_E, const int32_t* __restrict__ conn,
                                           int64_t e0, int64_t e1, int te, int64_t n_node,
                                           uint32_t* __restrict__ subcnt, uint32_t* flags) {
  uint32_t* s_bad = s_E + te * NEN;
  for (; e0 < e1; e0 += te) {
    const int ne = (int)(e1 - e0 < te ? e1 - e0 : te), n = ne * NEN;
    for (int i = threadIdx.x; i < n; i += blockDim.x) s_E[i] = (uint32_t)conn[e0 * NEN + i];
    for (int i = threadIdx.x; i < ne; i += blockDim.x) s_bad[i] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const int el = i / NEN, a = i - el * NEN;
      const int32_t Ea = (int32_t)s_E[i];
      uint32_t f = Ea < 0 || Ea >= n_node ? KB_F_INDEX : 0u;
#pragma unroll
      for (int b = 0; b < NEN; ++b) f |= b != a && (int32_t)s_E[el * NEN + b] == Ea ? KB_F_REPEAT : 0u;
      if (f) atomicOr(&s_bad[el], f);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const int el = i / NEN;
      if (s_bad[el]) {
        *flags |= s_bad[el];
        continue;
      }
      const int32_t Ea = (int32_t)s_E[i];
      uint32_t r = 0;
#pragma unroll
      for (int b = 0; b < NEN; ++b) r += (int32_t)s_E[el * NEN + b] < Ea ? 1u : 0u;
      const uint32_t s = sl.find((uint32_t)(Ea >> sl.shift));
      if (DIRECT && s == kNoSlot)
        atomicAdd(&subcnt[Ea >> sl.shift], r + 1);
      else
        atomicAdd(&sl.cnt[s], r + 1);
    }
    __syncthreads();
  }
}

template <int NEN, bool DIRECT>
__device__ __forceinline__ void count_tiles(uint32_t* s_h, const int32_t* __restrict__ conn, int64_t n_elem,
                                            int64_t n_node, int te, int64_t ntiles, uint32_t n_pad, int per,
                                                int slot_words, int s1, int nb, int s2, int nsub, int mode,
                                            uint32_t* __restrict__ hist, uint32_t* __restrict__ subcnt,
                                            uint32_t* __restrict__ status) {
  const TileSlots<DIRECT> sl(s_h, s_h + kSlotsHash, mode, s1, nb, s2, nsub);
  const int64_t t0 = (int64_t)(blockIdx.x - n_pad) * per, t1 = t0 + per < ntiles ? t0 + per : ntiles;
  uint32_t flags = 0;
  for (int64_t t = t0; t < t1; ++t) {
    sl.clear(blockDim.x);
    __syncthreads();
    const int64_t e0 = t * te, n = DIRECT ? (t1 - t0) * te : te, e1 = e0 + n < n_elem ? e0 + n : n_elem;
    if constexpr (NEN > 8 && (DIRECT || NEN > 16))
      count_rows<NEN>(sl, s_h + slot_words, conn, e0, e1, te, n_node, subcnt, &flags);
    else
      count_elements<NEN>(sl, conn, e0, e1, n_node, subcnt, &flags);
    __syncthreads();
    if constexpr (DIRECT) {
      flush_counts(sl, subcnt);
      break;
    } else {
      for (int b = threadIdx.x; b < nb; b += blockDim.x) hist[t * nb + b] = s_h[b];
      // (a lane clears the counters that it has written out)
    }
  }
  if (flags) raise_flag(status, flags);
}

// Under a random numbering pass 1 gathers its coordinates from 32-byte records, each in one
// cache line: the first n_pad workgroups copy those of the nodes from pad0 on.  The direct
// way gathers the 24-byte records as given, whose lines its tiles share, and saves the copy
// (27M bricks: 0.31 of 13.6 ms); the nodes before pad0 are copied beside the sampling, which
// takes as long, before the way is known.
template <int NEN>
__global__ __launch_bounds__(256) void k_count(const int32_t* __restrict__ conn, int64_t n_elem, int64_t n_node,
                                               int te, int64_t ntiles, int per, int slot_words, int s1, int nb, int s2,
                                               int nsub, int mode, uint32_t* head, uint32_t* __restrict__ hist,
                                               uint32_t* __restrict__ subcnt, uint32_t* __restrict__ sbb,
                                               uint32_t* __restrict__ status, uint32_t n_pad,
                                               const double* __restrict__ coords, double4* __restrict__ coords4,
                                               int64_t pad0) {
  extern __shared__ uint32_t s_h[];  // the slots' counters, then (hash) their keys
  const bool direct = mode == kAsk ? votes_direct(head + kHeadVotes) : mode == kDirect;
  if (mode == kAsk && blockIdx.x == n_pad && threadIdx.x == 0)
    head[kHeadWay] = direct ? 1u : votes_scattered(head + kHeadVotes) ? 2u : 0u;
  if (blockIdx.x < n_pad) {
    if (direct) return;
    const int64_t step = (int64_t)n_pad * blockDim.x;
    for (int64_t i = pad0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_node; i += step)
      coords4[i] = padded(coords, i);
    return;
  }
  if (direct) {
    count_tiles<NEN, true>(s_h, conn, n_elem, n_node, te, ntiles, n_pad, per, slot_words, s1, nb, s2, nsub, mode,
        hist, subcnt, status);
    if (mode == kDirect) last_block_starts(subcnt, nsub, sbb, &head[3], gridDim.x);
  } else {
    count_tiles<NEN, false>(s_h, conn, n_elem, n_node, te, ntiles, n_pad, per, slot_words, s1, nb, s2, nsub, mode,
        hist, subcnt, status);
  }
}

// Offsets of pass 1's writes, in four kernels.
// Two levels: from the tile-major histogram hist[t][b] (tiles x buckets) without
// transposing it: column sums over chunks of kColChunk tiles, a scan of those per bucket,
// the bucket starts, then each chunk's columns walked again, counts turned into offsets in
// place: hist[t][b] = bstart[b] + (pairs of bucket b in tiles before t).
// Direct (kAsk): the exclusive scan of the sub-bucket counts in the first two kernels, to
// sbb and (in place) to the write cursors; the other two return at once.
constexpr int kColChunk = 64;

// csum[c][b] = sum of hist[t][b] over the tiles of chunk c (grid: chunks x ceil(nb / 256),
// flattened, bucket blocks fastest), or the chunk sums of subcnt
static __global__ __launch_bounds__(kScanThreads) void k_offsets_sums(const uint32_t* __restrict__ hist, int64_t ntiles,
                                                               int nb, int64_t nchunk, uint32_t* __restrict__ csum,
                                                               const uint32_t* __restrict__ subcnt, int64_t nsub,
                                                               int32_t* __restrict__ part, int mode,
                                                               const uint32_t* __restrict__ way) {
  if (goes_direct(mode, way)) {
    if ((int64_t)blockIdx.x * kScanChunk < nsub) scan_chunk_sum((const int32_t*)subcnt, nsub, part);
    return;
  }
  const int64_t nbb = (nb + 255) / 256, c = blockIdx.x / nbb;
  const int b = (int)(blockIdx.x % nbb) * blockDim.x + threadIdx.x;
  if (c >= nchunk || b >= nb) return;
  const int64_t t0 = c * kColChunk, t1 = t0 + kColChunk < ntiles ? t0 + kColChunk : ntiles;
  uint32_t sum = 0;
#pragma unroll 8
  for (int64_t t = t0; t < t1; ++t) sum += hist[t * nb + b];
  csum[c * nb + b] = sum;
}

// one workgroup per bucket b: exclusive scan of csum[.][b] over the chunks, in place; the
// bucket's total to tot[b].  Direct: one workgroup per chunk of subcnt.
static __global__ __launch_bounds__(kScanThreads) void k_offsets_scan(uint32_t* __restrict__ csum, int64_t nchunk,
                                                               int nb, uint32_t* __restrict__ tot, uint32_t* subcnt,
                                                               int64_t nsub, const int32_t* __restrict__ part,
                                                               uint32_t* __restrict__ sbb, int mode,
                                                               const uint32_t* __restrict__ way) {
  if (goes_direct(mode, way)) {
    if ((int64_t)blockIdx.x * kScanChunk < nsub)
      scan_chunk_down((const int32_t*)subcnt, nsub, part, (int32_t*)sbb, (int32_t*)subcnt, nullptr);
    return;
  }
  __shared__ uint32_t s_scan[8];
  const int b = blockIdx.x;
  if (b >= nb) return;
  uint32_t carry = 0;
  for (int64_t c0 = 0; c0 < nchunk; c0 += blockDim.x) {
    const int64_t c = c0 + threadIdx.x;
    const uint32_t v = c < nchunk ? csum[c * nb + b] : 0u;
    uint32_t total;
    const uint32_t ex = block_scan_u32(v, s_scan, &total);
    if (c < nchunk) csum[c * nb + b] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) tot[b] = carry;
}

// single block: bucket starts bstart[0 .. nb] from the bucket totals, and segbase[b] =
// number of pass-2 segments in buckets before b (segbase[nb] = total), a bucket of n
// pairs having ceil(n / seg) segments
static __global__ __launch_bounds__(1024) void k_bucket_starts(const uint32_t* __restrict__ tot, int nb, int seg,
                                                        uint32_t* __restrict__ bstart, uint32_t* __restrict__ segbase,
                                                        int mode, const uint32_t* __restrict__ way) {
  if (goes_direct(mode, way)) return;
  __shared__ uint32_t s_scan[1024 / 64 + 1];
  uint32_t carry = 0, scarry = 0;
  for (int b0 = 0; b0 < nb; b0 += blockDim.x) {
    const int b = b0 + threadIdx.x;
    const uint32_t n = b < nb ? tot[b] : 0u;
    uint32_t total;
    const uint32_t ex = block_scan_u32(n, s_scan, &total);
    if (b < nb) bstart[b] = carry + ex;
    carry += total;
    const uint32_t sex = block_scan_u32((n + seg - 1) / seg, s_scan, &total);
    if (b < nb) segbase[b] = scarry + sex;
    scarry += total;
  }
  if (threadIdx.x == 0) {
    bstart[nb] = carry;
    segbase[nb] = scarry;
  }
}

// counts of chunk c turned into offsets in place (grid as k_offsets_sums); the nb
// workgroups after those write seg2b[s] = bucket of segment s
static __global__ __launch_bounds__(256) void k_offsets_down(uint32_t* __restrict__ hist,
                                                      const uint32_t* __restrict__ csum,
                                                      const uint32_t* __restrict__ bstart, int64_t ntiles, int nb,
                                                      int64_t nchunk, const uint32_t* __restrict__ segbase,
                                                      uint32_t* __restrict__ seg2b, int mode,
                                                      const uint32_t* __restrict__ way) {
  if (goes_direct(mode, way)) return;
  const int64_t nbb = (nb + 255) / 256, c = blockIdx.x / nbb;
  if (c >= nchunk) {
    const int64_t b = blockIdx.x - nchunk * nbb;
    if (b < nb)
      for (uint32_t s = segbase[b] + threadIdx.x; s < segbase[b + 1]; s += blockDim.x) seg2b[s] = (uint32_t)b;
    return;
  }
  const int b = (int)(blockIdx.x % nbb) * blockDim.x + threadIdx.x;
  if (b >= nb) return;
  uint32_t run = bstart[b] + csum[c * nb + b];
  const int64_t t0 = c * kColChunk, t1 = t0 + kColChunk < ntiles ? t0 + kColChunk : ntiles;
#pragma unroll 8
  for (int64_t t = t0; t < t1; ++t) {
    const uint32_t v = hist[t * nb + b];
    hist[t * nb + b] = run;
    run += v;
  }
}

// ------------------------------------------------------------------------ pass 1
// A tile is BLOCK elements, one per lane.  Its pairs are grouped by bucket (row >> s1) or
// sub-bucket (row >> s2) in LDS and each group's run is written at the tile's offset there.
template <typename V>
struct PairOut {
  uint16_t* row1;        // two levels: bucket arrays (row within its bucket, column, value)
  uint32_t* col1;
  V* val1;
  const uint32_t* off1;  // [tile][nb] offsets
  uint32_t* key2;        // direct: sub-bucket arrays (row within its sub-bucket << colbits | column, value)
  V* val2;
  uint32_t* cursor;      // [nsub] next free place
  const uint32_t* way;
  int mode, s1, nb, s2, nsub, colbits;
  // LDS words of the counters: counts and bases (and keys) of the slots
  static size_t slot_words(int mode, int nb, int64_t nsub) {
    const size_t two = 2 * (size_t)nb, hash = 3 * (size_t)kSlotsHash;
    return mode == kTwoLevel ? two : mode == kDirect ? 2 * (size_t)nsub : two > hash ? two : hash;
  }
};

template <typename V, int BLOCK, bool DIRECT>
struct Pass1Smem {
  uint64_t* key;  // [cap] staged (row << 32 | col), direct (slot << 32 | key2)
  V* val;         // [cap] staged values
  uint32_t* scan; // [BLOCK/64 + 1]
  uint32_t* emax; // [1]
  uint32_t* base; // [n] global offset of this tile in each slot
  TileSlots<DIRECT> sl;  // counters (base: n words, cnt: n words, hash: n words of keys)
  static constexpr int kPerLane = DIRECT ? (kSlotsArray + BLOCK - 1) / BLOCK : 1;  // counters per lane at most
  __device__ __forceinline__ Pass1Smem(unsigned char* smem, int cap, const PairOut<V>& o)
      : sl(nullptr, nullptr, o.mode, o.s1, o.nb, o.s2, o.nsub) {
    key = (uint64_t*)smem;
    val = (V*)(key + cap);
    scan = (uint32_t*)(val + cap);
    emax = scan + (BLOCK / 64 + 1);
    base = emax + 1;
    sl.cnt = base + sl.n;
    sl.key = sl.cnt + sl.n;
  }
  // counters cleared; two levels: the tile's offsets read
  __device__ __forceinline__ void begin(const PairOut<V>& o, int64_t t) const {
    if constexpr (DIRECT) {
      sl.clear(BLOCK);
    } else {
      for (int b = threadIdx.x; b < o.nb; b += BLOCK) {
        sl.cnt[b] = 0;
        base[b] = o.off1[t * o.nb + b];
      }
    }
  }
  // direct, after the scan: the tile's places in each sub-bucket, one atomic per run.  The
  // results stay in registers (the caller has other work to do) until put_bases.
  __device__ __forceinline__ void take_bases(const PairOut<V>& o, uint32_t total, uint32_t (&g)[kPerLane]) const {
    if constexpr (!DIRECT) return;
#pragma unroll
    for (int u = 0; u < kPerLane; ++u) {
      const int b = u * BLOCK + threadIdx.x;
      if (b < sl.n) {
        const uint32_t c = (b + 1 < sl.n ? sl.cnt[b + 1] : total) - sl.cnt[b];
        if (c) g[u] = atomicAdd(&o.cursor[sl.hash ? sl.key[b] : (uint32_t)b], c);
      }
    }
  }
  __device__ __forceinline__ void put_bases(const uint32_t (&g)[kPerLane]) const {
    if constexpr (!DIRECT) return;
#pragma unroll
    for (int u = 0; u < kPerLane; ++u) {
      const int b = u * BLOCK + threadIdx.x;
      if (b < sl.n) base[b] = g[u];
    }
  }
};

// the packed lower triangle k as the values of pass1_stage
template <typename V, int T>
struct PackedValues {
  const V (&k)[T];
  __device__ __forceinline__ V operator()(int, int row, int b) const {
    return row >= b ? k[lidx(row, b)] : k[lidx(b, row)];
  }
};

// stage the pairs of local rows R0 .. R0+N-1 (values k(a, row, b) for row = R0 + a): the r+1
// pairs of row E[a] go contiguously into its slot's run (a row without a slot takes its
// places at once)
template <int N, int R0, int NEN, typename V, int BLOCK, bool DIRECT, typename Values>
__device__ __forceinline__ void pass1_stage(const Pass1Smem<V, BLOCK, DIRECT>& sm, const PairOut<V>& o,
                                            const int32_t (&E)[NEN], const uint32_t (&q)[N], const Values& k) {
#pragma unroll
  for (int a = 0; a < N; ++a) {
    const int row = R0 + a;
    // (compared again here: kept from the ranks, the results of all rows' comparisons
    // overflow the scalar registers)
    int32_t F[NEN];
#pragma unroll
    for (int b = 0; b < NEN; ++b) {
      F[b] = E[b];
      asm volatile("" : "+v"(F[b]));
    }
    const uint32_t rl = DIRECT ? ((uint32_t)E[row] & ((1u << o.s2) - 1)) << o.colbits : 0u;
    if (DIRECT && q[a] == kNoSlot) {
      uint32_t n = 0;
#pragma unroll
      for (int b = 0; b < NEN; ++b) n += F[b] <= F[row] ? 1u : 0u;
      uint32_t g = atomicAdd(&o.cursor[E[row] >> o.s2], n);
#pragma unroll
      for (int b = 0; b < NEN; ++b) {
        if (F[b] <= F[row]) {
          o.key2[g] = rl | (uint32_t)F[b];
          o.val2[g] = k(a, row, b);
          ++g;
        }
      }
      continue;
    }
    const uint32_t slot = sm.sl.slot(q[a], E[row]);
    uint32_t pos = sm.sl.cnt[slot] + sm.sl.place(q[a]);
    const uint64_t rk = (uint64_t)(DIRECT ? slot : (uint32_t)E[row]) << 32 | rl;
#pragma unroll
    for (int b = 0; b < NEN; ++b) {
      if (F[b] <= F[row]) {
        sm.key[pos] = rk | (uint32_t)F[b];
        sm.val[pos] = k(a, row, b);
        ++pos;
      }
    }
  }
}

// write the staged pairs: index i lies in slot b, local start cnt[b].  kWriteBatch pairs of
// a lane are under way together: each takes two dependent reads of LDS, and few waves share
// a CU here (pass 1 of 27M bricks FP64 6.60 -> 6.50 ms).  Direct only: the short runs of the
// two-level way then lose the order in which they share lines (17.9M bricks FP32, all
// random: 8.8 -> 9.7 ms).
constexpr int kWriteBatch = 4;
template <typename V, int BLOCK, bool DIRECT>
__device__ __forceinline__ void pass1_write(const Pass1Smem<V, BLOCK, DIRECT>& sm, const PairOut<V>& o,
                                            uint32_t n_items) {
  const auto put = [&](uint32_t g, uint64_t key, V v) {
    if constexpr (DIRECT) {
      o.key2[g] = (uint32_t)key;
    } else {
      o.row1[g] = (uint16_t)((uint32_t)(key >> 32) & ((1u << o.s1) - 1));  // row within its bucket
      o.col1[g] = (uint32_t)key;
    }
    (DIRECT ? o.val2 : o.val1)[g] = v;
  };
  const auto slot = [&](uint64_t key) { return (uint32_t)(key >> 32) >> (DIRECT ? 0 : o.s1); };
  uint32_t i = threadIdx.x;
  for (; DIRECT && i + (kWriteBatch - 1) * BLOCK < n_items; i += kWriteBatch * BLOCK) {
    uint64_t key[kWriteBatch];
    V v[kWriteBatch];
    uint32_t g[kWriteBatch];
#pragma unroll
    for (int u = 0; u < kWriteBatch; ++u) {
      key[u] = sm.key[i + u * BLOCK];
      v[u] = sm.val[i + u * BLOCK];
    }
#pragma unroll
    for (int u = 0; u < kWriteBatch; ++u) {
      const uint32_t b = slot(key[u]);
      g[u] = sm.base[b] + (i + u * BLOCK - sm.sl.cnt[b]);
    }
#pragma unroll
    for (int u = 0; u < kWriteBatch; ++u) put(g[u], key[u], v[u]);
  }
  for (; i < n_items; i += BLOCK) {
    const uint64_t key = sm.key[i];
    const uint32_t b = slot(key);
    put(sm.base[b] + (i - sm.sl.cnt[b]), key, sm.val[i]);
  }
}

// largest finite biased exponent (as doubles) of an element's values: that of the largest
// finite magnitude, compared as bits
template <int T, typename V>
__device__ __forceinline__ uint32_t values_emax(const V (&k)[T]) {
  if constexpr (sizeof(V) == 4) {
    uint32_t m = 0;
#pragma unroll
    for (int p = 0; p < T; ++p) {
      const uint32_t b = __float_as_uint(k[p]) & 0x7FFFFFFFu;
      m = (b > m && b < 0x7F800000u) ? b : m;
    }
    return (uint32_t)biased_exponent((double)__uint_as_float(m));
  } else {
    uint32_t m = 0;
#pragma unroll
    for (int p = 0; p < T; ++p) {
      const uint32_t ep = (uint32_t)biased_exponent((double)k[p]);
      m = (ep > m && ep < 0x7FF) ? ep : m;
    }
    return m;
  }
}

// element values from given per-element lower triangles (assembly-only path)
template <int T, typename V>
__device__ __forceinline__ void read_values(const V* __restrict__ klow, int64_t e, V (&k)[T], uint32_t* flags) {
  bool finite = true;
#pragma unroll
  for (int p = 0; p < T; ++p) {
    k[p] = klow[e * T + p];
    finite = finite && isfinite((double)k[p]);
  }
  if (!finite) *flags |= KB_F_NONFINITE;
}

// where pass 1 gathers its coordinates (k_count)
template <bool DIRECT>
using PassNodes = std::conditional_t<DIRECT, NodesXYZ, NodesPadded>;

// Bricks: one tile per workgroup; tiles are assigned XCD-contiguously, so the runs that
// neighbouring tiles write side by side meet in one L2.  OP: the integrand (unless the
// values are given).
template <int NEN, Prec P, bool FROM_VALUES, int BLOCK, Op OP, bool DIRECT>
__device__ __forceinline__ void pass1_tile(unsigned char* smem, const int32_t (&E)[NEN], const PassNodes<DIRECT> nodes,
    const double* __restrict__ coef, const typename PrecTraits<P>::V* __restrict__ klow,
    int64_t n_elem, int64_t n_node, float tau, const PairOut<typename PrecTraits<P>::V>& o,
    uint32_t* __restrict__ emax, uint32_t* __restrict__ status) {
  using V = typename PrecTraits<P>::V;
  using SM = Pass1Smem<V, BLOCK, DIRECT>;
  constexpr int T = ElemTraits<NEN>::T;
  const SM sm(smem, BLOCK * T, o);
  const int64_t t = xcd_item(blockIdx.x, gridDim.x);
  const int64_t e = t * BLOCK + threadIdx.x;
  sm.begin(o, t);
  if (threadIdx.x == 0) *sm.emax = 0;
  const bool valid = e < n_elem && check_conn<NEN>(E, n_node) == 0;
  double Xn[NEN][3];
  double c_e = 0.0;
  if constexpr (!FROM_VALUES) {
    if (valid) {
      gather_nodes<NEN>(nodes, E, Xn);
      c_e = coef[e];
    }
  }
  __syncthreads();
  uint32_t q[NEN];
  if (valid) {
    int r[NEN];
    node_ranks<NEN>(E, r);
    reserve_rows<NEN, 0>(sm.sl, E, r, q);
  }
  __syncthreads();
  const uint32_t n_items = block_scan_array(sm.sl.cnt, sm.sl.n, sm.scan);
  uint32_t gb[SM::kPerLane];
  sm.take_bases(o, n_items, gb);
  uint32_t flags = 0, fb = 0;
  if (valid) {
    V k[T];
    if constexpr (FROM_VALUES)
      read_values<T>(klow, e, k, &flags);
    else
      element_values_at<NEN, P, OP>(Xn, c_e, tau, k, &flags, &fb);
    atomicMax(sm.emax, values_emax<T>(k));
    pass1_stage<NEN, 0>(sm, o, E, q, PackedValues<V, T>{k});
  }
  if (flags) raise_flag(status, flags);
  if (fb) atomicAdd(&status[1], fb);
  sm.put_bases(gb);
  __syncthreads();
  if (threadIdx.x == 0 && *sm.emax) atomicMax(emax, *sm.emax);
  pass1_write(sm, o, n_items);
}

template <int NEN, Prec P, bool FROM_VALUES, int BLOCK, Op OP = Op::Stiffness>
__global__ __launch_bounds__(BLOCK) void k_pass1(const int32_t* __restrict__ conn, const double* __restrict__ coords,
                                               const double4* __restrict__ coords4,
                                               const double* __restrict__ coef,
                                               const typename PrecTraits<P>::V* __restrict__ klow, int64_t n_elem,
                                               int64_t n_node, float tau,
                                               const PairOut<typename PrecTraits<P>::V> o,
                                               uint32_t* __restrict__ emax, uint32_t* __restrict__ status) {
  extern __shared__ __align__(16) unsigned char smem[];
  int32_t E[NEN] = {};
  const int64_t e = xcd_item(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x;
  if (e < n_elem) load_conn<NEN>(conn, e, E);  // under way while the branch waits for its word
  if (goes_direct(o.mode, o.way))
    pass1_tile<NEN, P, FROM_VALUES, BLOCK, OP, true>(smem, E, NodesXYZ{coords}, coef, klow, n_elem, n_node, tau, o,
        emax, status);
  else
    pass1_tile<NEN, P, FROM_VALUES, BLOCK, OP, false>(smem, E, NodesPadded{coords4}, coef, klow, n_elem, n_node, tau,
        o, emax, status);
}

// The tiles of a persistent workgroup: XCD x owns one contiguous range of the tiles and its
// G workgroups walk it interleaved, so neighbouring runs meet in one L2.  They drift apart,
// though, and where runs are a few pairs long (many buckets, elements in random order) the
// lines that neighbouring tiles share are then written in parts: such a mesh takes a
// workgroup per tile, in the order of dispatch (17.9M bricks FP32, all random: pass 1 10.3 ->
// 9.7 ms; with elements in grid order the walk is the faster one, 7.4 -> 6.5 ms).
__device__ __forceinline__ uint32_t walkers(int mode, const uint32_t* __restrict__ way, uint32_t persist) {
  return mode == kAsk && *way == 2 ? gridDim.x : persist;
}
struct TileWalk {
  int64_t t, hi, step;
  __device__ __forceinline__ TileWalk(int64_t ntiles, int64_t G) {
    const int64_t x = blockIdx.x % kXcds, w = blockIdx.x / kXcds;
    step = G / kXcds + (x < G % kXcds ? 1 : 0);
    const int64_t lo = x * (ntiles / kXcds) + min(x, ntiles % kXcds);
    hi = lo + ntiles / kXcds + (x < ntiles % kXcds ? 1 : 0);
    t = lo + w;
  }
};

// coordinates that are not read again: a later conditional gather otherwise keeps them in
// registers as the value of the lanes that do not gather
template <int N>
__device__ __forceinline__ void forget(double (&x)[N][3]) {
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) asm volatile("" : "=v"(x[a][c]));
}

// Bricks in FP64 from coordinates (an element per lane): two tiles per workgroup of 2 BLOCK
// lanes, so that each SIMD holds two waves while the elements are gathered and integrated.
// The two tiles are then counted, staged and written one after the other through the one
// staging area (BLOCK elements' pairs, which fill the CU's LDS).  Persistent: with one
// workgroup on a CU nothing else covers its start and its gathers, so the next two tiles'
// connectivity is loaded while these are integrated and their nodes are gathered while the
// last one is written (27M bricks: 6.5 -> 5.5 ms).
template <int NEN, Prec P, int BLOCK, Op OP, bool DIRECT>
__device__ __forceinline__ void pass1_two(unsigned char* smem, const int32_t* __restrict__ conn,
    const PassNodes<DIRECT> nodes, const double* __restrict__ coef, int64_t n_elem, int64_t n_node, float tau,
    int64_t ntiles, int64_t G, const PairOut<typename PrecTraits<P>::V>& o, uint32_t* __restrict__ emax,
    uint32_t* __restrict__ status) {
  using V = typename PrecTraits<P>::V;
  using SM = Pass1Smem<V, 2 * BLOCK, DIRECT>;
  constexpr int T = ElemTraits<NEN>::T;
  const SM sm(smem, BLOCK * T, o);
  TileWalk walk((ntiles + 1) / 2, G);  // pairs of tiles
  if (walk.t >= walk.hi) return;
  const int half = threadIdx.x >= BLOCK ? 1 : 0;
  if (threadIdx.x == 0) *sm.emax = 0;
  const auto fetch = [&](int64_t w, int32_t (&E)[NEN]) {
    const int64_t e = w * (2 * BLOCK) + threadIdx.x;
    if (w >= walk.hi || e >= n_elem) return false;
    load_conn<NEN>(conn, e, E);
    return check_conn<NEN>(E, n_node) == 0;
  };
  int32_t E[NEN];
  bool valid = fetch(walk.t, E);
  double Xn[NEN][3];
  double c_e = 0.0;
  if (valid) {
    gather_nodes<NEN>(nodes, E, Xn);
    c_e = coef[walk.t * (2 * BLOCK) + threadIdx.x];
  }
  uint32_t em = 0;  // largest value exponent seen by this lane
  while (true) {
    const int64_t w = walk.t;
    uint32_t flags = 0, fb = 0;
    V k[T];
    if (valid) {  // both tiles' elements
      element_values_at<NEN, P, OP>(Xn, c_e, tau, k, &flags, &fb);
      const uint32_t me = values_emax<T>(k);
      em = me > em ? me : em;
    }
    if (flags) raise_flag(status, flags);
    if (fb) atomicAdd(&status[1], fb);
    int32_t En[NEN];
    const bool vn = fetch(w + walk.step, En);
    uint32_t n_items;
    for (int h = 0;; ++h) {
      sm.begin(o, 2 * w + h);
      __syncthreads();
      uint32_t q[NEN];
      const bool mine = valid && half == h;
      if (mine) {
        int r[NEN];
        node_ranks<NEN>(E, r);
        reserve_rows<NEN, 0>(sm.sl, E, r, q);
      }
      __syncthreads();
      n_items = block_scan_array(sm.sl.cnt, sm.sl.n, sm.scan);
      uint32_t gb[SM::kPerLane];
      sm.take_bases(o, n_items, gb);
      if (mine) pass1_stage<NEN, 0>(sm, o, E, q, PackedValues<V, T>{k});
      sm.put_bases(gb);
      if (h == 1 || 2 * w + 1 >= ntiles) break;
      __syncthreads();
      pass1_write(sm, o, n_items);
      __syncthreads();  // the staging area is reused by the next tile
    }
#pragma unroll
    for (int a = 0; a < NEN; ++a) E[a] = En[a];
    valid = vn;
    forget(Xn);
    if (valid) {
      gather_nodes<NEN>(nodes, E, Xn);
      c_e = coef[(w + walk.step) * (2 * BLOCK) + threadIdx.x];
    }
    __syncthreads();
    pass1_write(sm, o, n_items);
    walk.t = w + walk.step;
    if (walk.t >= walk.hi) break;
    __syncthreads();
  }
  if (em) atomicMax(sm.emax, em);
  __syncthreads();
  if (threadIdx.x == 0 && *sm.emax) atomicMax(emax, *sm.emax);
}

template <int NEN, Prec P, int BLOCK, Op OP = Op::Stiffness>
__global__ __launch_bounds__(2 * BLOCK) void k_pass1_two(const int32_t* __restrict__ conn,
                                                       const double* __restrict__ coords,
                                                       const double4* __restrict__ coords4,
                                                       const double* __restrict__ coef, int64_t n_elem, int64_t n_node,
                                                       float tau, int64_t ntiles,
                                                       const PairOut<typename PrecTraits<P>::V> o,
                                                       uint32_t* __restrict__ emax, uint32_t* __restrict__ status,
                                                       uint32_t persist) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t G = walkers(o.mode, o.way, persist);
  if (blockIdx.x >= G) return;
  if (goes_direct(o.mode, o.way))
    pass1_two<NEN, P, BLOCK, OP, true>(smem, conn, NodesXYZ{coords}, coef, n_elem, n_node, tau, ntiles, G, o, emax,
        status);
  else
    pass1_two<NEN, P, BLOCK, OP, false>(smem, conn, NodesPadded{coords4}, coef, n_elem, n_node, tau, ntiles, G, o, emax,
        status);
}

// offsets of the lane's four rows R0 .. R0+3 in their slots (two levels: per-row atomics
// measured 1-2% faster here than one per run of rows)
template <int R0, bool DIRECT>
__device__ __forceinline__ void pair_reserve_half(const TileSlots<DIRECT>& sl, const int32_t (&E)[8], const int (&r)[8],
                                                  uint32_t (&q)[4]) {
  if constexpr (DIRECT) {
    reserve_rows<4, R0>(sl, E, r, q);
  } else {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      q[a] = atomicAdd(&sl.cnt[E[R0 + a] >> sl.shift], (uint32_t)(r[R0 + a] + 1));
    }
  }
}

// Bricks, stiffness matrix: a lane pair per element (element_values_pair), BLOCK lanes
// and BLOCK / 2 elements per tile.  Twice the waves of one lane per element for the same
// staging LDS, and half the quadrature per lane; lane h counts and stages the pairs of
// rows 4h .. 4h+3.  Persistent: the staging LDS leaves two workgroups per CU, so the next
// tile's connectivity is loaded while the current one is integrated and its nodes are
// gathered while the current one is written.
template <Prec P, int BLOCK, bool DIRECT>
__device__ __forceinline__ void pass1_pair(unsigned char* smem, const int32_t* __restrict__ conn,
    const PassNodes<DIRECT> nodes, const double* __restrict__ coef, int64_t n_elem, int64_t n_node, float tau,
    int64_t ntiles, int64_t G, const PairOut<typename PrecTraits<P>::V>& o, uint32_t* __restrict__ emax,
    uint32_t* __restrict__ status) {
  using V = typename PrecTraits<P>::V;
  using SM = Pass1Smem<V, BLOCK, DIRECT>;
  constexpr int NEN = 8, T = ElemTraits<NEN>::T, TE = BLOCK / 2;
  const SM sm(smem, TE * T, o);
  TileWalk walk(ntiles, G);
  if (walk.t >= walk.hi) return;
  const int h = (int)(threadIdx.x & 1);
  if (threadIdx.x == 0) *sm.emax = 0;
  const auto fetch = [&](int64_t t, int32_t (&E)[NEN]) {
    const int64_t e = t * TE + (threadIdx.x >> 1);
    if (t >= walk.hi || e >= n_elem) return false;
    load_conn<NEN>(conn, e, E);
    return check_conn<NEN>(E, n_node) == 0;
  };
  int32_t E[NEN];
  bool valid = fetch(walk.t, E);
  double xo[4][3];
  double c_e = 0.0;
  if (valid) {
    gather_pair(nodes, E, h, xo);
    c_e = coef[walk.t * TE + (threadIdx.x >> 1)];
  }
  uint32_t em = 0;  // largest value exponent seen by this lane
  while (true) {
    sm.begin(o, walk.t);
    __syncthreads();
    // (a branch per half keeps every index into E and r a constant)
    uint32_t q[4];
    if (valid) {
      int r[NEN];
      node_ranks<NEN>(E, r);
      if (h)
        pair_reserve_half<4>(sm.sl, E, r, q);
      else
        pair_reserve_half<0>(sm.sl, E, r, q);
    }
    __syncthreads();
    const uint32_t n_items = block_scan_array(sm.sl.cnt, sm.sl.n, sm.scan);
    uint32_t gb[SM::kPerLane];
    sm.take_bases(o, n_items, gb);
    const int64_t tn = walk.t + walk.step;
    int32_t En[NEN];
    const bool vn = fetch(tn, En);
    uint32_t flags = 0, fb = 0;
    if (valid) {
      V k[4][8];
      element_values_pair<P>(xo, c_e, tau, h, k, &flags, &fb);
      const auto row_values = [&](int a, int, int b) { return k[a][b]; };
      const uint32_t me = values_emax<32>((const V(&)[32])k);
      em = me > em ? me : em;
      if (h)
        pass1_stage<4, 4>(sm, o, E, q, row_values);
      else
        pass1_stage<4, 0>(sm, o, E, q, row_values);
    }
    if (flags) raise_flag(status, flags);
    if (fb) atomicAdd(&status[1], fb);
    sm.put_bases(gb);
#pragma unroll
    for (int a = 0; a < NEN; ++a) E[a] = En[a];
    valid = vn;
    forget(xo);
    if (valid) {
      gather_pair(nodes, E, h, xo);
      c_e = coef[tn * TE + (threadIdx.x >> 1)];
    }
    __syncthreads();
    pass1_write(sm, o, n_items);
    walk.t = tn;
    if (tn >= walk.hi) break;
    __syncthreads();
  }
  if (em) atomicMax(sm.emax, em);
  __syncthreads();
  if (threadIdx.x == 0 && *sm.emax) atomicMax(emax, *sm.emax);
}

template <Prec P, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_pass1_pair(const int32_t* __restrict__ conn,
                                                    const double* __restrict__ coords,
                                                    const double4* __restrict__ coords4,
                                                    const double* __restrict__ coef, int64_t n_elem, int64_t n_node,
                                                    float tau, int64_t ntiles,
                                                    const PairOut<typename PrecTraits<P>::V> o,
                                                    uint32_t* __restrict__ emax, uint32_t* __restrict__ status,
                                                        uint32_t persist) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t G = walkers(o.mode, o.way, persist);
  if (blockIdx.x >= G) return;
  if (goes_direct(o.mode, o.way))
    pass1_pair<P, BLOCK, true>(smem, conn, NodesXYZ{coords}, coef, n_elem, n_node, tau, ntiles, G, o, emax, status);
  else
    pass1_pair<P, BLOCK, false>(smem, conn, NodesPadded{coords4}, coef, n_elem, n_node, tau, ntiles, G, o, emax,
        status);
}

// Tetrahedra: persistent workgroups.  XCD x owns one contiguous range of tiles and its
// workgroups walk it interleaved (neighbouring runs again meet in one L2).  The next
// tile's connectivity is loaded while the current tile is integrated, and its node
// coordinates while the current tile is written.
template <Prec P, bool FROM_VALUES, int BLOCK, Op OP, bool DIRECT>
__device__ __forceinline__ void pass1_tet(unsigned char* smem, const int32_t* __restrict__ conn,
    const PassNodes<DIRECT> nodes,
    const double* __restrict__ coef, const typename PrecTraits<P>::V* __restrict__ klow,
    int64_t n_elem, int64_t n_node, float tau, int64_t ntiles,
    const PairOut<typename PrecTraits<P>::V>& o, uint32_t* __restrict__ emax,
    uint32_t* __restrict__ status) {
  using V = typename PrecTraits<P>::V;
  using SM = Pass1Smem<V, BLOCK, DIRECT>;
  constexpr int NEN = 4, T = ElemTraits<NEN>::T;
  const SM sm(smem, BLOCK * T, o);
  const int64_t G = gridDim.x, x = blockIdx.x % kXcds, w = blockIdx.x / kXcds;
  const int64_t nw = G / kXcds + (x < G % kXcds ? 1 : 0);
  const int64_t lo = x * (ntiles / kXcds) + min(x, ntiles % kXcds);
  const int64_t hi = lo + ntiles / kXcds + (x < ntiles % kXcds ? 1 : 0);
  int64_t t = lo + w;
  if (t >= hi) return;
  if (threadIdx.x == 0) *sm.emax = 0;

  auto fetch = [&](int64_t tt, int32_t (&Ef)[NEN]) {
    const int64_t e = tt * BLOCK + threadIdx.x;
    if (tt < hi && e < n_elem) {
      load_conn<NEN>(conn, e, Ef);
      return check_conn<NEN>(Ef, n_node) == 0;
    }
    return false;
  };
  int32_t E[NEN];
  bool valid = fetch(t, E);
  double Xn[NEN][3];
  double c_e = 0.0;
  if constexpr (!FROM_VALUES) {
    if (valid) {
      gather_nodes<NEN>(nodes, E, Xn);
      c_e = coef[t * BLOCK + threadIdx.x];
    }
  }
  uint32_t em = 0;  // largest value exponent seen by this lane
  while (true) {
    const int64_t e = t * BLOCK + threadIdx.x;
    sm.begin(o, t);
    __syncthreads();
    uint32_t q[NEN];
    if (valid) {
      int r[NEN];
      node_ranks<NEN>(E, r);
      reserve_rows<NEN, 0>(sm.sl, E, r, q);
    }
    __syncthreads();
    const uint32_t n_items = block_scan_array(sm.sl.cnt, sm.sl.n, sm.scan);
    uint32_t gb[SM::kPerLane];
    sm.take_bases(o, n_items, gb);
    const int64_t tn = t + nw;
    int32_t En[NEN];
    const bool vn = fetch(tn, En);
    uint32_t flags = 0, fb = 0;
    if (valid) {
      V k[T];
      if constexpr (FROM_VALUES)
        read_values<T>(klow, e, k, &flags);
      else
        element_values_at<NEN, P, OP>(Xn, c_e, tau, k, &flags, &fb);
      const uint32_t me = values_emax<T>(k);
      em = me > em ? me : em;
      pass1_stage<NEN, 0>(sm, o, E, q, PackedValues<V, T>{k});
    }
    if (flags) raise_flag(status, flags);
    if (fb) atomicAdd(&status[1], fb);
    sm.put_bases(gb);
#pragma unroll
    for (int a = 0; a < NEN; ++a) E[a] = En[a];
    valid = vn;
    if constexpr (!FROM_VALUES) {
      if (valid) {
        gather_nodes<NEN>(nodes, E, Xn);
        c_e = coef[tn * BLOCK + threadIdx.x];
      }
    }
    __syncthreads();
    pass1_write(sm, o, n_items);
    t = tn;
    if (t >= hi) break;
    __syncthreads();
  }
  if (em) atomicMax(sm.emax, em);
  __syncthreads();
  if (threadIdx.x == 0 && *sm.emax) atomicMax(emax, *sm.emax);
}

template <Prec P, bool FROM_VALUES, int BLOCK, Op OP = Op::Stiffness>
__global__ __launch_bounds__(BLOCK) void k_pass1_tet(const int32_t* __restrict__ conn,
                                                   const double* __restrict__ coords,
                                                   const double4* __restrict__ coords4,
                                                   const double* __restrict__ coef,
                                                   const typename PrecTraits<P>::V* __restrict__ klow, int64_t n_elem,
                                                   int64_t n_node, float tau, int64_t ntiles,
                                                   const PairOut<typename PrecTraits<P>::V> o,
                                                   uint32_t* __restrict__ emax, uint32_t* __restrict__ status) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (goes_direct(o.mode, o.way))
    pass1_tet<P, FROM_VALUES, BLOCK, OP, true>(smem, conn, NodesXYZ{coords}, coef, klow, n_elem, n_node, tau, ntiles,
        o, emax, status);
  else
    pass1_tet<P, FROM_VALUES, BLOCK, OP, false>(smem, conn, NodesPadded{coords4}, coef, klow, n_elem, n_node, tau,
        ntiles, o, emax, status);
}

// Elements of more than eight rows (nodes with several degrees of freedom), values
// given (assembly only).  A tile is `te` elements, few enough that their pairs fit in
// LDS; kWideThreads threads work on it:
//   - per (element, row a): the row's rank r_a among the element's ids, and its run of
//     r_a + 1 places in the tile's part of bucket E_a >> s1 (LDS counters);
//   - per pair, one thread each, values read in storage order (coalesced): pair (p, q)
//     belongs to the row of the larger id (a) and takes place rank(b) of that row's
//     run, b being the other corner (the diagonal takes the last place, r_a);
//   - the staged pairs, grouped by bucket, are written as runs (as for 4 and 8 rows).
constexpr int kWideThreads = 1024;  // threads per wide pass-1 workgroup (one per CU: LDS)

template <int NEN, typename V, bool DIRECT>
__device__ __forceinline__ void pass1_wide(unsigned char* smem, const int32_t* __restrict__ conn,
    const V* __restrict__ klow, int64_t n_elem, int64_t n_node,
    int te, const PairOut<V>& o, uint32_t* __restrict__ emax, uint32_t* __restrict__ status) {
  constexpr int T = ElemTraits<NEN>::T, NT = kWideThreads;
  using SM = Pass1Smem<V, NT, DIRECT>;
  const SM sm(smem, te * T, o);
  // [te * NEN] the tile's connectivity, after the slots' words
  int32_t* s_E = (int32_t*)(sm.base + (DIRECT && sm.sl.hash ? 3 : 2) * sm.sl.n);
  uint32_t* s_q = (uint32_t*)(s_E + te * NEN);  // [te * NEN] run offset of each row in its bucket
  uint32_t* s_rank = s_q + te * NEN;            // [te * NEN] slot << 8 (0xFFFF: none) | rank of each corner's id
  uint32_t* s_ok = s_rank + te * NEN;           // [te] element valid
  uint16_t* s_pq = (uint16_t*)(s_ok + te);      // [T] packed index -> (p << 8 | q)
  const int64_t t = xcd_item(blockIdx.x, gridDim.x);
  const int64_t e0 = t * te;
  const int ne = (int)(n_elem - e0 < te ? n_elem - e0 : te);
  sm.begin(o, t);
  if (threadIdx.x == 0) *sm.emax = 0;
  for (int i = threadIdx.x; i < T; i += NT) {
    int p = 0;
    while ((p + 1) * (p + 2) / 2 <= i) ++p;
    s_pq[i] = (uint16_t)(p << 8 | (i - p * (p + 1) / 2));
  }
  for (int i = threadIdx.x; i < ne * NEN; i += NT) s_E[i] = conn[e0 * NEN + i];
  __syncthreads();
  uint32_t flags = 0;
  for (int el = threadIdx.x; el < ne; el += NT) {
    int32_t E[NEN];
#pragma unroll
    for (int a = 0; a < NEN; ++a) E[a] = s_E[el * NEN + a];
    const uint32_t f = check_conn<NEN>(E, n_node);
    flags |= f;
    s_ok[el] = f == 0;
  }
  __syncthreads();
  for (int j = threadIdx.x; j < ne * NEN; j += NT) {
    const int el = j / NEN;
    if (!s_ok[el]) continue;
    const int32_t Ea = s_E[j];
    uint32_t r = 0;
#pragma unroll
    for (int b = 0; b < NEN; ++b) r += (s_E[el * NEN + b] < Ea) ? 1u : 0u;
    const uint32_t s = sm.sl.find((uint32_t)(Ea >> sm.sl.shift));
    // (a row without a slot: its places in its sub-bucket taken at once)
    s_q[j] = s == kNoSlot ? atomicAdd(&o.cursor[Ea >> o.s2], r + 1) : atomicAdd(&sm.sl.cnt[s], r + 1);
    s_rank[j] = (s & 0xFFFFu) << 8 | r;
  }
  __syncthreads();
  const uint32_t n_items = block_scan_array(sm.sl.cnt, sm.sl.n, sm.scan);  // cnt: local run starts
  uint32_t gb[SM::kPerLane];
  sm.take_bases(o, n_items, gb);
  uint32_t em = 0;
  bool finite = true;
  const V* __restrict__ k = klow + e0 * T;
  for (int i = threadIdx.x; i < ne * T; i += NT) {
    const int el = i / T, kk = i - el * T;
    if (!s_ok[el]) continue;
    const uint32_t pq = s_pq[kk];
    const int p = (int)(pq >> 8), q = (int)(pq & 255u);
    const int32_t Ep = s_E[el * NEN + p], Eq = s_E[el * NEN + q];
    const bool up = Ep >= Eq;
    const int a = up ? p : q, b = up ? q : p;
    const int32_t Ea = up ? Ep : Eq, Eb = up ? Eq : Ep;
    const uint32_t slot = s_rank[el * NEN + a] >> 8, at = s_q[el * NEN + a] + (s_rank[el * NEN + b] & 255u);
    const V v = k[i];
    finite = finite && isfinite((double)v);
    const uint32_t ep = (uint32_t)biased_exponent((double)v);
    em = (ep > em && ep < 0x7FF) ? ep : em;
    const uint32_t key2 = ((uint32_t)Ea & ((1u << o.s2) - 1)) << o.colbits | (uint32_t)Eb;
    if (DIRECT && slot == 0xFFFFu) {
      o.key2[at] = key2;
      o.val2[at] = v;
      continue;
    }
    const uint32_t pos = sm.sl.cnt[slot] + at;
    sm.key[pos] = DIRECT ? (uint64_t)slot << 32 | key2 : (uint64_t)(uint32_t)Ea << 32 | (uint32_t)Eb;
    sm.val[pos] = v;
  }
  if (!finite) flags |= KB_F_NONFINITE;
  if (flags) raise_flag(status, flags);
  if (em) atomicMax(sm.emax, em);
  sm.put_bases(gb);
  __syncthreads();
  if (threadIdx.x == 0 && *sm.emax) atomicMax(emax, *sm.emax);
  pass1_write(sm, o, n_items);
}

template <int NEN, typename V>
__global__ __launch_bounds__(kWideThreads) void k_pass1_wide(const int32_t* __restrict__ conn,
                                                  const V* __restrict__ klow,
                                                  int64_t n_elem, int64_t n_node, int te, const PairOut<V> o,
                                                  uint32_t* __restrict__ emax, uint32_t* __restrict__ status) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (goes_direct(o.mode, o.way))
    pass1_wide<NEN, V, true>(smem, conn, klow, n_elem, n_node, te, o, emax, status);
  else
    pass1_wide<NEN, V, false>(smem, conn, klow, n_elem, n_node, te, o, emax, status);
}

// ----------------------------------------------------- running sums as a source
// A grouped build carries the sums of the groups done so far as a lower CSR (entries in
// row order, with rows[], residuals res[] and nnz in device memory).  The next group's
// pass reads them back as pairs (row, col, value) and (row, col, residual) next to its
// elements' pairs.  Tiles of kCsrTile entries follow the element tiles.  The entries
// are read only if they were written (nnz <= cap); rows outside [0, n_node) are skipped
// (both kernels apply the same test, so counts and writes agree).
// three workgroups per CU beside the hash's slots (2048: two; grouped 20M tets 295 us, 1792: 239)
constexpr int kCsrTile = 1792;

__device__ __forceinline__ int64_t csr_entries(const int64_t* nnz_dev, int64_t cap) {
  const int64_t n = *nnz_dev;
  return (n >= 0 && n <= cap) ? n : 0;
}

constexpr int kCsrThreads = 256, kCsrPer = kCsrTile / kCsrThreads;

template <bool DIRECT>
__device__ __forceinline__ void count_csr(uint32_t* s_h, const int32_t* __restrict__ rows,
                                          const int64_t* __restrict__ nnz_dev, int64_t cap, int64_t n_node, int s1,
                                          int nb, int s2, int nsub, int mode, uint32_t* __restrict__ hist,
                                          uint32_t* __restrict__ subcnt) {
  const TileSlots<DIRECT> sl(s_h, s_h + kSlotsHash, mode, s1, nb, s2, nsub);
  const int64_t t = blockIdx.x;
  sl.clear(kCsrThreads);
  __syncthreads();
  const int64_t n = csr_entries(nnz_dev, cap);
  const int64_t e0 = t * kCsrTile, e1 = e0 + kCsrTile < n ? e0 + kCsrTile : n;
  for (int64_t i = e0 + threadIdx.x; i < e1; i += kCsrThreads) {
    const int32_t r = rows[i];
    if (r < 0 || r >= n_node) continue;
    const uint32_t s = sl.find((uint32_t)(r >> sl.shift));
    if (!DIRECT || s != kNoSlot)
      atomicAdd(&sl.cnt[s], 2u);
    else
      atomicAdd(&subcnt[r >> s2], 2u);
  }
  __syncthreads();
  if constexpr (DIRECT) {
    flush_counts(sl, subcnt);
  } else {
    for (int b = threadIdx.x; b < nb; b += kCsrThreads) hist[t * nb + b] = s_h[b];
  }
}

static __global__ __launch_bounds__(kCsrThreads) void k_hist_csr(const int32_t* __restrict__ rows,
                                                                 const int64_t* __restrict__ nnz_dev, int64_t cap,
                                                                 int64_t n_node, int s1, int nb, int s2, int nsub,
                                                                 int mode, const uint32_t* __restrict__ way,
                                                                 uint32_t* __restrict__ hist,
                                                                 uint32_t* __restrict__ subcnt) {
  extern __shared__ uint32_t s_h[];  // as k_count
  if (goes_direct(mode, way))
    count_csr<true>(s_h, rows, nnz_dev, cap, n_node, s1, nb, s2, nsub, mode, hist, subcnt);
  else
    count_csr<false>(s_h, rows, nnz_dev, cap, n_node, s1, nb, s2, nsub, mode, hist, subcnt);
}

template <typename V, bool DIRECT>
__device__ __forceinline__ void pass1_csr(unsigned char* smem, const int32_t* __restrict__ rows,
    const int32_t* __restrict__ cols,
    const V* __restrict__ vals, const V* __restrict__ res, const int64_t* __restrict__ nnz_dev,
    int64_t cap, int64_t n_node, const PairOut<V>& o, uint32_t* __restrict__ emax) {
  constexpr int NT = kCsrThreads, PER = kCsrPer;
  using SM = Pass1Smem<V, NT, DIRECT>;
  const SM sm(smem, 2 * kCsrTile, o);
  const int64_t t = blockIdx.x;
  sm.begin(o, t);
  if (threadIdx.x == 0) *sm.emax = 0;
  __syncthreads();
  const int64_t n = csr_entries(nnz_dev, cap);
  const int64_t e0 = t * kCsrTile;
  int32_t r[PER];
  uint32_t q[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t i = e0 + u * NT + threadIdx.x;
    r[u] = i < n ? rows[i] : -1;
    if (r[u] >= n_node) r[u] = -1;
    if (r[u] < 0) continue;
    const uint32_t s = sm.sl.find((uint32_t)(r[u] >> sm.sl.shift));
    if constexpr (DIRECT)
      q[u] = s == kNoSlot ? kNoSlot : (s << 16 | atomicAdd(&sm.sl.cnt[s], 2u));
    else
      q[u] = atomicAdd(&sm.sl.cnt[s], 2u);
  }
  __syncthreads();
  const uint32_t n_items = block_scan_array(sm.sl.cnt, sm.sl.n, sm.scan);
  uint32_t gb[SM::kPerLane];
  sm.take_bases(o, n_items, gb);
  uint32_t em = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (r[u] < 0) continue;
    const int64_t i = e0 + u * NT + threadIdx.x;
    const uint32_t col = (uint32_t)cols[i];
    const uint32_t key2 = ((uint32_t)r[u] & ((1u << o.s2) - 1)) << o.colbits | col;
    const V h = vals[i], x = res[i];
    const uint32_t ep = (uint32_t)biased_exponent((double)h);  // |res| <= |h|
    em = (ep > em && ep < 0x7FF) ? ep : em;
    if (DIRECT && q[u] == kNoSlot) {
      const uint32_t g = atomicAdd(&o.cursor[r[u] >> o.s2], 2u);
      o.key2[g] = key2;
      o.val2[g] = h;
      o.key2[g + 1] = key2;
      o.val2[g + 1] = x;
      continue;
    }
    const uint32_t slot = sm.sl.slot(q[u], r[u]);
    const uint32_t pos = sm.sl.cnt[slot] + sm.sl.place(q[u]);
    const uint64_t key = DIRECT ? (uint64_t)slot << 32 | key2 : (uint64_t)(uint32_t)r[u] << 32 | col;
    sm.key[pos] = key;
    sm.val[pos] = h;
    sm.key[pos + 1] = key;
    sm.val[pos + 1] = x;
  }
  if (em) atomicMax(sm.emax, em);
  sm.put_bases(gb);
  __syncthreads();
  if (threadIdx.x == 0 && *sm.emax) atomicMax(emax, *sm.emax);
  pass1_write(sm, o, n_items);
}

template <typename V>
__global__ __launch_bounds__(kCsrThreads) void k_pass1_csr(const int32_t* __restrict__ rows,
                                                         const int32_t* __restrict__ cols,
                                                         const V* __restrict__ vals, const V* __restrict__ res,
                                                         const int64_t* __restrict__ nnz_dev, int64_t cap,
                                                         int64_t n_node, const PairOut<V> o,
                                                         uint32_t* __restrict__ emax) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (goes_direct(o.mode, o.way))
    pass1_csr<V, true>(smem, rows, cols, vals, res, nnz_dev, cap, n_node, o, emax);
  else
    pass1_csr<V, false>(smem, rows, cols, vals, res, nnz_dev, cap, n_node, o, emax);
}

// ------------------------------------------------------------------------ pass 2
// A bucket's pairs are cut into segments of SEG; segment ids run over all buckets
// (segbase[b] is the first segment of bucket b, segbase[nb] their number).

// histogram of sub-buckets ((row >> s2) mod p2) per segment: hist2[s * p2 + j]
// s[k] += 1 for each of N keys, one LDS atomic per run of equal consecutive keys (under a
// natural numbering neighbouring pairs mostly share a sub-bucket, and their increments
// would otherwise serialise on one address: 27M bricks, histogram 2.26 -> 1.01 ms)
template <int N>
__device__ __forceinline__ void count_runs(uint32_t* s, const uint32_t (&k)[N]) {
  uint32_t cur = k[0], run = 1;
#pragma unroll
  for (int i = 1; i < N; ++i) {
    if (k[i] == cur) {
      ++run;
    } else {
      atomicAdd(&s[cur], run);
      cur = k[i];
      run = 1;
    }
  }
  atomicAdd(&s[cur], run);
}

template <int SEG>
__global__ __launch_bounds__(256) void k_hist2(const uint16_t* __restrict__ irow, const uint32_t* __restrict__ bstart,
                                               const uint32_t* __restrict__ segbase,
                                               const uint32_t* __restrict__ seg2b, int nb, int s2, int p2,
                                               uint32_t* __restrict__ hist2, int mode,
                                               const uint32_t* __restrict__ way) {
  extern __shared__ uint32_t s_h[];  // [p2]
  const uint32_t sid = blockIdx.x;
  const uint32_t n_seg = segbase[nb], b = seg2b[sid];
  if (goes_direct(mode, way) || sid >= n_seg) return;  // (b is then not a bucket)
  const uint32_t s = sid - segbase[b];
  for (int j = threadIdx.x; j < p2; j += blockDim.x) s_h[j] = 0;
  __syncthreads();
  const uint32_t be = bstart[b + 1];
  const uint32_t i0 = bstart[b] + s * SEG, i1 = (i0 + SEG < be) ? i0 + SEG : be;
  const uint32_t mask = (uint32_t)p2 - 1;
  // eight row indices per 16-byte load over the 8-aligned middle of the range (irow is
  // 256-byte aligned); the ragged ends one by one
  const uint32_t a0 = (i0 + 7u) & ~7u, a1 = i1 & ~7u;
  if (a0 >= a1) {
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) atomicAdd(&s_h[(irow[i] >> s2) & mask], 1u);
  } else {
    for (uint32_t i = i0 + threadIdx.x; i < a0; i += blockDim.x) atomicAdd(&s_h[(irow[i] >> s2) & mask], 1u);
    for (uint32_t i = a1 + threadIdx.x; i < i1; i += blockDim.x) atomicAdd(&s_h[(irow[i] >> s2) & mask], 1u);
    const uint4* __restrict__ w = (const uint4*)(irow + a0);
    for (uint32_t j = threadIdx.x; j < (a1 - a0) / 8; j += blockDim.x) {
      const uint4 v = w[j];
      const uint32_t k[8] = {((v.x & 0xFFFFu) >> s2) & mask, ((v.x >> 16) >> s2) & mask,
                             ((v.y & 0xFFFFu) >> s2) & mask, ((v.y >> 16) >> s2) & mask,
                             ((v.z & 0xFFFFu) >> s2) & mask, ((v.z >> 16) >> s2) & mask,
                             ((v.w & 0xFFFFu) >> s2) & mask, ((v.w >> 16) >> s2) & mask};
      count_runs<8>(s_h, k);
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < p2; j += blockDim.x) hist2[(int64_t)sid * p2 + j] = s_h[j];
}

// One workgroup per bucket b: for each sub-bucket column j, the exclusive prefix of
// hist2 over the bucket's segments (in place), then the sub-bucket starts
// sbb[b * p2 + j] (sbb[nb * p2] = number of pairs).  A segment's run for sub-bucket j
// starts at sbb[b * p2 + j] + hist2[s * p2 + j].
static __global__ __launch_bounds__(256) void k_colscan(uint32_t* __restrict__ hist2,
                                                 const uint32_t* __restrict__ bstart,
                                                 const uint32_t* __restrict__ segbase, int nb, int p2,
                                                 uint32_t* __restrict__ sbb, int mode,
                                                 const uint32_t* __restrict__ way) {
  if (goes_direct(mode, way)) return;
  __shared__ uint32_t s_tot[1024];
  __shared__ uint32_t s_scan[8];
  const int b = blockIdx.x;
  const uint32_t sa = segbase[b], se = segbase[b + 1];
  for (int j = threadIdx.x; j < p2; j += blockDim.x) {
    uint32_t run = 0;
    uint32_t* col = hist2 + (int64_t)sa * p2 + j;
    uint32_t s = sa;
    for (; s + 8 <= se; s += 8, col += 8 * (int64_t)p2) {  // eight loads in flight
      uint32_t h[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) h[q] = col[q * (int64_t)p2];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        col[q * (int64_t)p2] = run;
        run += h[q];
      }
    }
    for (; s < se; ++s, col += p2) {
      const uint32_t h = *col;
      *col = run;
      run += h;
    }
    s_tot[j] = run;
  }
  __syncthreads();
  block_scan_array(s_tot, p2, s_scan);
  const uint32_t bs = bstart[b];
  for (int j = threadIdx.x; j < p2; j += blockDim.x) sbb[(int64_t)b * p2 + j] = bs + s_tot[j];
  if (b == nb - 1 && threadIdx.x == 0) sbb[(int64_t)nb * p2] = bstart[nb];
}

// scatter a segment into its sub-buckets; output key = row_local << colbits | col
template <typename V, int SEG, int NT>
__global__ __launch_bounds__(NT) void k_scatter2(const uint16_t* __restrict__ irow, const uint32_t* __restrict__ icol,
                                                  const V* __restrict__ ival, const uint32_t* __restrict__ bstart,
                                                  const uint32_t* __restrict__ segbase,
                                                  const uint32_t* __restrict__ seg2b,
                                                  const uint32_t* __restrict__ off2, const uint32_t* __restrict__ sbb,
                                                  int nb, int s2, int p2, int colbits, uint32_t* __restrict__ okey,
                                                  V* __restrict__ oval, int mode,
                                                  const uint32_t* __restrict__ way) {
  extern __shared__ __align__(16) unsigned char smem[];
  V* s_val = (V*)smem;                          // [SEG]
  uint32_t* s_key = (uint32_t*)(s_val + SEG);   // [SEG]
  uint16_t* s_sb = (uint16_t*)(s_key + SEG);    // [SEG] sub-bucket of staged pair
  uint32_t* s_cnt = (uint32_t*)(s_sb + SEG);    // [p2] pairs per sub-bucket, then local starts
  uint32_t* s_off = s_cnt + p2;                 // [p2] global offsets
  uint32_t* s_scan = s_off + p2;                // [NT/64 + 1]
  const uint32_t sid = (uint32_t)xcd_item(blockIdx.x, gridDim.x);
  const uint32_t n_seg = segbase[nb], b = seg2b[sid];
  if (goes_direct(mode, way) || sid >= n_seg) return;  // (b is then not a bucket)
  const uint32_t s = sid - segbase[b];
  for (int j = threadIdx.x; j < p2; j += blockDim.x) {
    s_cnt[j] = 0;
    s_off[j] = sbb[(int64_t)b * p2 + j] + off2[(int64_t)sid * p2 + j];
  }
  __syncthreads();
  const uint32_t be = bstart[b + 1];
  const uint32_t i0 = bstart[b] + s * SEG, i1 = (i0 + SEG < be) ? i0 + SEG : be;
  const uint32_t mask = (uint32_t)p2 - 1, rmask = (1u << s2) - 1;
  constexpr int PER = SEG / NT;
  uint32_t rr[PER], cc[PER], rk[PER];
  V vv[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {  // every load issued first (indices clamped into the segment)
    const uint32_t i = i0 + q * NT + threadIdx.x;
    const uint32_t ic = i < i1 ? i : i0;
    rr[q] = irow[ic];
    cc[q] = icol[ic];
    vv[q] = ival[ic];
  }
  // rank of each pair within its sub-bucket, then the local run starts
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const uint32_t i = i0 + q * NT + threadIdx.x;
    if (i < i1) rk[q] = atomicAdd(&s_cnt[(rr[q] >> s2) & mask], 1u);
  }
  __syncthreads();
  block_scan_array(s_cnt, p2, s_scan);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const uint32_t i = i0 + q * NT + threadIdx.x;
    if (i < i1) {
      const uint32_t j = (rr[q] >> s2) & mask;
      const uint32_t pos = s_cnt[j] + rk[q];
      s_key[pos] = ((rr[q] & rmask) << colbits) | cc[q];
      s_val[pos] = vv[q];
      s_sb[pos] = (uint16_t)j;
    }
  }
  __syncthreads();
  const uint32_t n = i1 - i0;
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
    const uint32_t j = s_sb[i];
    const uint32_t g = s_off[j] + (i - s_cnt[j]);
    okey[g] = s_key[i];
    oval[g] = s_val[i];
  }
}

// The first kHeavyPar heavy sub-buckets of the list are split, and their first-level
// digit ranges reduced, by many workgroups (the phases of k_heavy: heavy_rows; heavy_layout,
// heavy_hist and heavy_starts; heavy_scatter; heavy_bigleaf; heavy_ranges); heavy_finish then
// sums up each one's entries and k_final gathers them from the ranges.  heavy_rest takes the
// other listed sub-buckets whole.  (In small builds teams do the same in one launch: heavy_team.)
// The first-level digits follow the rows: row r of a sub-bucket gets n_r digits (a
// power of two, none for a row without pairs), each covering 2^(colbits) / n_r columns,
// with n_r about kHvyShare times the row's share of the pairs, at most one digit per
// leaf width of columns, and at least 2^(colbits - 23) so that a digit is at most 2^23
// keys wide (split once more into leaves).  A row holding most pairs of its sub-bucket
// thus gets 2048 digits, leaf-wide up to 2^23 columns, which many workgroups reduce
// side by side.  The digits of all rows total at most kHvyShare + 256 + 256 =
// kHvyDigits.
constexpr int kHeavyPar = 64;
constexpr int kHvyDigits = 4096;  // first-level digits at most
constexpr uint32_t kHvyShare = 3584;
constexpr int kHvyRows = 256;  // rows of a sub-bucket at most
constexpr int kHvyWords = (kHvyDigits + 1) + kHvyDigits + 2 * kHvyRows + (kHvyRows + 1) + 4;
struct HeavyTable {
  uint32_t* st;     // [kHvyDigits + 1] digit starts (absolute pair positions)
  uint32_t* hist;   // [kHvyDigits] pairs of each digit, then the scatter's cursors
  uint32_t* ucnt;   // the same words once the scatter is done: the entries of each digit
                    // range (every range writes its own), then their offsets
  uint32_t* rpair;  // [kHvyRows] pairs of each row
  uint32_t* rsh;    // [kHvyRows] column shift of each row's digits
  uint32_t* rbase;  // [kHvyRows + 1] first digit of each row; rbase[kHvyRows] = digits
  uint32_t* meta;   // [4] digits; workgroups done (heavy_team) or chunks counted (heavy_hist)
  __device__ HeavyTable(uint32_t* hvy, uint32_t it) {
    st = hvy + (size_t)it * kHvyWords;
    hist = st + kHvyDigits + 1;
    ucnt = hist;
    rpair = hist + kHvyDigits;
    rsh = rpair + kHvyRows;
    rbase = rsh + kHvyRows;
    meta = rbase + kHvyRows + 1;
  }
  // words that k_begin clears, per table: rpair; for the teams meta[1]
  static constexpr int kRpairAt = 2 * kHvyDigits + 1, kTeamAt = kHvyWords - 3;
};

// first-level digit of key k (row k >> colbits) from the layout in LDS
__device__ __forceinline__ uint32_t heavy_digit(uint32_t k, int colbits, const uint32_t* s_rbase,
                                                const uint32_t* s_rsh) {
  const uint32_t r = k >> colbits;
  return s_rbase[r] + ((k & ((1u << colbits) - 1u)) >> s_rsh[r]);
}

// ------------------------------------------------------------------------ pass 3
// home slot of a packed key in a table of HT (a power of two) slots: the top bits of
// the key mixed by xor-shift, multiply by 2^32/phi, xor-shift.  A plain multiplicative
// hash lets the row bits (the key's top bits) and the columns of a naturally numbered
// grid interfere: on the 300^3 brick box it gave 1.9 probes per insert on average and
// runs of up to 15, against 1.1 and 4 for the mixed key (the reduce 1.9x slower)
template <int HT>
__device__ __forceinline__ uint32_t slot_hash(uint32_t k) {
  constexpr int bits = __builtin_ctz(HT);
  k ^= k >> 15;
  k *= 0x9E3779B1u;
  k ^= k >> 13;
  return k >> (32 - bits);
}

// One workgroup per sub-bucket g (rows [g << s2, ...)).  Writes its unique entries in
// CSR order to tcol/tval[sbb[g] + f], each row's first entry (relative to the
// sub-bucket) to rowoff, its total to usub[g].  A sub-bucket of more than 2^16 pairs
// or more distinct entries than the table holds is appended to list (count in *count) and
// left to k_heavy or, if the direct way's sub-buckets are wider, to k_pass3_parts.
// Sub-buckets run in their natural order: under a random numbering the lower-triangle
// pairs of a row grow with its id, so an even interleave keeps the XCDs balanced.
// With RES, each entry's residual (the exact sum minus its rounding) goes to tres too.
// (The grid has the two-level way's number of sub-buckets; where the direct way has fewer,
// the other workgroups return: about 0.4 ns each, against 20% slower code if a workgroup
// could take several in turn.)
constexpr int kPass3Threads = 256;

// a workgroup's table and the arrays that order its entries.  Once summed, each slot's value
// (and residual) is kept in place of its low chunk sum, which frees the high chunk sums for
// the columns grouped by row (one array fewer); a double with its double residual needs both
// words.  The per-row arrays are sized by the sub-bucket's rows at launch and the columns are
// grouped by row through cursors (no per-slot index within the row): 22.5 KB at 1024 slots,
// seven workgroups per CU; with a double's residuals 26.5 KB, of which six fit as long as 64 rows
// take no more than 512 bytes and the two words below none (1.8M tetrahedra in two
// groups: 91 -> 83 us)
template <typename V, int HT, bool RES>
struct Pass3Smem {
  static constexpr bool kSepCols = RES && sizeof(V) == 8;
  uint32_t* key;
  unsigned long long* lo;  // sum of low 48-bit chunks, then value (+ residual)
  unsigned long long* hi;  // sum of signed high chunks, then the columns
  uint16_t* slot;          // occupied slots, in insertion order
  uint32_t* lcol;          // columns of the slots, grouped by row
  uint32_t *rc, *cur;      // [1 << s2] entries per row; cursors, at last each row's end
  uint32_t *over, *nu;     // the table is full; occupied slots
  __device__ __forceinline__ void clear(int rows) const {
    for (int h = threadIdx.x; h < HT; h += kPass3Threads) {
      key[h] = kEmptyKey;
      lo[h] = 0ull;
      hi[h] = 0ull;
    }
    for (int r = threadIdx.x; r < rows; r += kPass3Threads) rc[r] = 0;
  }
};

// Stream n <= 2^16 pairs into the table: PER loads per lane in flight (indices clamped into
// the range; the empty asm keeps the compiler from sinking a load into the branch that first
// uses it).  A key that finds no slot sets *over, which ends the stream, and empties the table,
// whose sums are then not used: each further pair probing a full table to its end took 0.5 ms
// for 2000 pairs (a limit on the probes short of that costs the pairs of every other table:
// 20.25M tets 3.98 -> 4.01 ms).
// PART: only the pairs whose key >> part_shift is part.
template <bool PART, typename V, int HT, bool RES>
__device__ __forceinline__ void pass3_insert(const Pass3Smem<V, HT, RES>& sm, const uint32_t* kp, const V* vp,
                                             uint32_t n, int F, uint32_t part, int part_shift) {
  constexpr int NT = kPass3Threads, PER = 8;
  for (uint32_t j0 = 0; j0 < n; j0 += PER * NT) {
    uint32_t kk[PER];
    V vv[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const uint32_t j = j0 + u * NT + threadIdx.x;
      const uint32_t jc = (j < n ? j : 0u) & 0xffffu;
      kk[u] = kp[jc];
      vv[u] = vp[jc];
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) asm volatile("" : "+v"(kk[u]), "+v"(vv[u]));
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      if (j0 + u * NT + threadIdx.x >= n) continue;
      const uint32_t key = kk[u];
      if (PART && key >> part_shift != part) continue;
      // one compare-and-swap per probe: it returns the empty marker when this lane
      // took the slot, the key when the entry was there already, else another key
      uint32_t h = slot_hash<HT>(key);
      uint32_t k = atomicCAS(&sm.key[h], kEmptyKey, key);
      int probes = 0;
#pragma unroll 1
      while (k != kEmptyKey && k != key && ++probes < HT) {
        h = (h + 1) & (HT - 1);
        k = atomicCAS(&sm.key[h], kEmptyKey, key);
      }
      if (k != kEmptyKey && k != key) {
        *sm.over = 1;
#pragma unroll 1
        for (int i = 0; i < HT; ++i) sm.key[i] = kEmptyKey;
        continue;
      }
      uint64_t c0;
      int64_t c1;
      to_chunks(vv[u], F, c0, c1);
      // (a float within 2^23 of the largest is a multiple of 2^48: 20.25M tets, 671 -> 655 us)
      if (sizeof(V) == 8 || c0) atomicAdd(&sm.lo[h], (unsigned long long)c0);
      atomicAdd(&sm.hi[h], (unsigned long long)c1);
    }
    if (j0 + PER * NT < n && __hip_atomic_load(sm.over, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
  }
}

// rows of which 32 columns at a time are ranked: four at a time leave a long row waiting (1M
// tetrahedra of 5000 nodes, 1600 entries a row: pass 3 941 -> 690 us), 32 at a time rows of
// several components (1M bricks of three: 6.17 -> 6.36 ms)
constexpr uint32_t kLongRow = 128;

// The table's entries rounded, ordered by (row, col) and written from tcol / tval / tres
// [0, ...) on, and the first entries of rows [row_lo, row_hi), counted from u0, to rowoff.
// Returns their number.
template <typename V, int HT, bool RES>
__device__ __forceinline__ uint32_t pass3_emit(const Pass3Smem<V, HT, RES>& sm, int F, int colbits, int s2, uint32_t u0,
                                           int row_lo, int row_hi, int32_t* tcol, V* tval, V* tres,
                                           uint32_t* rowoff) {
  constexpr int NT = kPass3Threads;
  const uint32_t cmask = (1u << colbits) - 1;
  // list the occupied slots and count the entries of each row (once per entry here
  // rather than on the insertion path of every pair)
  for (int h = threadIdx.x; h < HT; h += NT) {
    const uint32_t k = sm.key[h];
    if (k != kEmptyKey) {
      sm.slot[atomicAdd(sm.nu, 1u)] = (uint16_t)h;
      atomicAdd(&sm.rc[k >> colbits], 1u);
    }
  }
  __syncthreads();
  // order the U entries by (row, col): the row counts scanned by one
  // wave while the others round each sum to its value, the entries grouped by row, then
  // ranked by column within their row
  const uint32_t U = *sm.nu;
  const int RB = 1 << s2;  // rows of a full sub-bucket (<= 256)
  for (uint32_t f = threadIdx.x < 64 ? U : threadIdx.x - 64; f < U; f += NT - 64) {
    const uint32_t h = sm.slot[f];
    uint64_t lo, hi;
    join48(sm.lo[h], (int64_t)sm.hi[h], lo, hi);
    const V hv = from_fixed_as<V>(lo, hi, F);
    if constexpr (sizeof(V) == 8) {
      sm.lo[h] = (unsigned long long)__double_as_longlong((double)hv);
      if constexpr (RES) sm.hi[h] = (unsigned long long)__double_as_longlong((double)fixed_residual<V>(lo, hi, F, hv));
    } else {
      const uint32_t rv = RES ? __float_as_uint((float)fixed_residual<V>(lo, hi, F, hv)) : 0u;
      sm.lo[h] = ((unsigned long long)rv << 32) | __float_as_uint((float)hv);
    }
  }
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    uint32_t v[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = lane * 4 + k;
      v[k] = r < RB ? sm.rc[r] : 0u;
      sum += v[k];
    }
    uint32_t x = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    uint32_t run = x - sum;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = lane * 4 + k;
      if (r < RB) sm.cur[r] = run;
      run += v[k];
    }
  }
  __syncthreads();
  for (uint32_t f = threadIdx.x; f < U; f += NT) {
    const uint32_t h = sm.slot[f];
    const uint32_t k = sm.key[h];
    sm.lcol[atomicAdd(&sm.cur[k >> colbits], 1u)] = k & cmask;
  }
  __syncthreads();
  for (uint32_t f = threadIdx.x; f < U; f += NT) {
    const uint32_t h = sm.slot[f];
    const uint32_t k = sm.key[h];
    const uint32_t row = k >> colbits, col = k & cmask;
    const uint32_t nr = sm.rc[row], ro = sm.cur[row] - nr;
    uint32_t rank = 0, q = 0;
    if (nr >= kLongRow)
#pragma unroll 1
      for (; q + 32 <= nr; q += 32) {
#pragma unroll
        for (int i = 0; i < 32; ++i) rank += (sm.lcol[ro + q + i] < col) ? 1u : 0u;
      }
#pragma unroll 4
    for (; q < nr; ++q) rank += (sm.lcol[ro + q] < col) ? 1u : 0u;
    const uint32_t pos = ro + rank;
    tcol[pos] = (int32_t)col;
    const unsigned long long w = sm.lo[h];
    if constexpr (sizeof(V) == 8) {
      tval[pos] = (V)__longlong_as_double((long long)w);
      if constexpr (RES) tres[pos] = (V)__longlong_as_double((long long)sm.hi[h]);
    } else {
      tval[pos] = (V)__uint_as_float((uint32_t)w);
      if constexpr (RES) tres[pos] = (V)__uint_as_float((uint32_t)(w >> 32));
    }
  }
  for (int r = row_lo + threadIdx.x; r < row_hi; r += NT) rowoff[r] = u0 + sm.cur[r] - sm.rc[r];
  return U;
}

template <typename V, int HT, bool RES = false>
__global__ __launch_bounds__(kPass3Threads) void k_pass3(uint32_t* __restrict__ ikey, V* __restrict__ ival,
                                               const uint32_t* __restrict__ sbb, const SubBuckets sub, int colbits,
                                               int64_t n_node,
                                               const uint32_t* __restrict__ emax, int32_t* __restrict__ tcol,
                                               V* __restrict__ tval, V* __restrict__ tres,
                                               uint32_t* __restrict__ rowoff, uint32_t* __restrict__ usub,
                                               uint32_t* __restrict__ list, uint32_t* __restrict__ count) {
  using SM = Pass3Smem<V, HT, RES>;
  __shared__ uint32_t s_key[HT];
  __shared__ unsigned long long s_lo[HT];
  __shared__ unsigned long long s_hi[HT];
  __shared__ uint16_t s_slot[HT];
  __shared__ uint32_t s_sep[SM::kSepCols ? HT : 2];
  uint32_t &s_over = s_sep[0], &s_nu = s_sep[1];  // (read before the columns are written)
  extern __shared__ uint32_t s_rows[];  // 2 << s2 words
  const int64_t g = blockIdx.x;
  const bool either = g < sub.nsub[1];
  if (!either && sub.pick()) return;  // (only the workgroups beyond the direct way's wait for its word here)
  const uint32_t beg = sbb[g], end = sbb[g + 1];
  SM sm{s_key, s_lo, s_hi, s_slot, SM::kSepCols ? s_sep : (uint32_t*)s_hi, s_rows, nullptr, &s_over, &s_nu};
  sm.clear(1 << (sub.s2[0] > sub.s2[1] ? sub.s2[0] : sub.s2[1]));
  const int s2 = sub.s2[either ? sub.pick() : 0];
  sm.cur = s_rows + (1 << s2);
  const int F = 1117 - (int)*emax;
  const int64_t r0 = g << s2;
  const int64_t rr = n_node - r0;
  const int R = rr <= 0 ? 0 : (rr < ((int64_t)1 << s2) ? (int)rr : (1 << s2));
  // more than 2^16 pairs could overflow the chunk sums: left to k_heavy
  if (threadIdx.x == 0) {
    s_over = (end - beg > (1u << 16)) ? 1u : 0u;
    s_nu = 0;
  }
  __syncthreads();
  if (!s_over) pass3_insert<false>(sm, ikey + beg, ival + beg, end - beg, F, 0u, 0);
  __syncthreads();
  if (s_over) {
    if (threadIdx.x == 0) list[atomicAdd(count, 1u)] = (uint32_t)g;
    return;
  }
  const uint32_t U =
      pass3_emit(sm, F, colbits, s2, 0u, 0, R, tcol + beg, tval + beg, RES ? tres + beg : nullptr, rowoff + r0);
  if (threadIdx.x == 0) usub[g] = U;
}

// The sub-buckets that k_pass3 listed, if the direct way's are the wider ones.  Those are
// sized for the mesh's average row: one whose rows are longer (rows of unlike length in
// ranges of ids) is reduced here in parts of the two-level way's width, each with the whole
// table; its pairs are read once per part.  What does not fit its table goes to ov_list,
// for k_heavy (a workgroup of which takes some 0.5 ms: a mesh of 216,000 bricks that share no
// node, all of it listed, took 128 ms).  In k_pass3 itself the parts made every sub-bucket
// slower (scalar registers: 27M bricks 13.3 -> 13.7 ms); the launch takes 4 us when nothing
// is listed.
constexpr int kPartsGroups = 2;   // workgroups per CU
template <typename V, int HT, bool RES = false>
__global__ __launch_bounds__(kPass3Threads) void k_pass3_parts(
    uint32_t* __restrict__ ikey, V* __restrict__ ival, const uint32_t* __restrict__ sbb, const SubBuckets sub,
    int colbits, int64_t n_node, const uint32_t* __restrict__ emax, int32_t* __restrict__ tcol, V* __restrict__ tval,
    V* __restrict__ tres, uint32_t* __restrict__ rowoff, uint32_t* __restrict__ usub,
    const uint32_t* __restrict__ list, const uint32_t* __restrict__ count, uint32_t* __restrict__ ov_list,
    uint32_t* __restrict__ ov_count) {
  using SM = Pass3Smem<V, HT, RES>;
  __shared__ uint32_t s_key[HT];
  __shared__ unsigned long long s_lo[HT];
  __shared__ unsigned long long s_hi[HT];
  __shared__ uint16_t s_slot[HT];
  __shared__ uint32_t s_sep[SM::kSepCols ? HT : 2];
  uint32_t &s_over = s_sep[0], &s_nu = s_sep[1];  // (read before the columns are written)
  extern __shared__ uint32_t s_rows[];  // 2 << s2 words
  const uint32_t n_list = *count;
  if (blockIdx.x >= n_list) return;
  const int s2 = sub.s2[sub.pick()], s2p = s2 < sub.s2[0] ? s2 : sub.s2[0], np = 1 << (s2 - s2p);
  const SM sm{s_key,  s_lo, s_hi, s_slot, SM::kSepCols ? s_sep : (uint32_t*)s_hi, s_rows, s_rows + (1 << s2),
              &s_over, &s_nu};
  const int F = 1117 - (int)*emax;
  for (uint32_t i = blockIdx.x; i < n_list; i += gridDim.x) {
    const int64_t g = list[i], r0 = g << s2;
    const uint32_t beg = sbb[g], end = sbb[g + 1];
    const int R = (int)min((int64_t)1 << s2, n_node - r0);
    uint32_t U = 0;
    int p = end - beg > (1u << 16) ? np + 1 : 0;  // (as k_pass3)
    for (; p < np; ++p) {
      __syncthreads();  // (the entries before are written)
      sm.clear(1 << s2);
      if (threadIdx.x == 0) {
        s_over = 0u;
        s_nu = 0;
      }
      __syncthreads();
      pass3_insert<true>(sm, ikey + beg, ival + beg, end - beg, F, (uint32_t)p, colbits + s2p);
      __syncthreads();
      if (s_over) break;
      const int lo = p << s2p, hi = lo + (1 << s2p) < R ? lo + (1 << s2p) : R;
      U += pass3_emit(sm, F, colbits, s2, U, lo, hi, tcol + beg + U, tval + beg + U, RES ? tres + beg + U : nullptr,
                      rowoff + r0);
    }
    if (threadIdx.x == 0) {
      if (p == np)
        usub[g] = U;
      else
        ov_list[atomicAdd(ov_count, 1u)] = (uint32_t)g;
    }
  }
}

// ------------------------------------------------------------ heavy sub-buckets
// A sub-bucket that overflows pass 3 (a node shared by very many elements: its row holds
// more distinct entries than an LDS table, or more than 2^16 pairs) is split by key into
// ranges of at most kLeafKeys keys, each summed into a direct-addressed LDS table.  The
// first kHeavyPar listed are split by the whole device (the tables above);
// each further one is reduced whole by one 1024-lane workgroup of heavy_rest:
//   - the key range [kmin, kmax] of the sub-bucket; a range wider than kLeafKeys is split
//     into at most 2048 digit ranges of 2^shift keys (a histogram, its scan and a
//     scatter into the other buffer, at the same place), twice at most for 31-bit keys;
//   - each leaf range (in key order) sums its pairs into a direct-addressed LDS table,
//     one slot per key, with the exact chunk sums of pass 3, carried into a third word
//     after every 2^16 pairs (so any number of pairs sums exactly); then the occupied
//     slots, in slot order = (row, col) order, are written after the entries before.
// Output as pass 3.  The pairs alternate between (ikey, ival) and (akey, aval), the
// pass-1 arrays, which also receive the output (tcol / tval): a leaf writes at most as
// many entries as it has pairs, so the output never reaches a pair not yet read.
constexpr int kLeafKeys = 4096, kHeavyThreads = 1024, kDigits = 2048;

struct HeavySmem {
  unsigned long long* lo;  // [kLeafKeys] sum of low 48-bit chunks
  long long* hi;           // [kLeafKeys] sum of signed high chunks (bits 48..)
  long long* top;          // [kLeafKeys] carries above bit 96
  uint8_t* occ;            // [kLeafKeys] 1 for an occupied slot (byte stores: no atomics)
  uint32_t* hist;          // [kDigits] digit counts, then cursors
  uint32_t* start;         // [2][kDigits + 1] digit starts of the two split levels
  uint32_t* rowcnt;        // [256] entries per row of the sub-bucket
  uint32_t* scan;          // [kHeavyThreads / 64 + 1]
  uint32_t* misc;          // [4]
  __device__ explicit HeavySmem(unsigned char* p) {
    lo = (unsigned long long*)p;
    hi = (long long*)(lo + kLeafKeys);
    top = hi + kLeafKeys;
    occ = (uint8_t*)(top + kLeafKeys);
    hist = (uint32_t*)(occ + kLeafKeys);
    start = hist + kDigits;
    rowcnt = start + 2 * (kDigits + 1);
    scan = rowcnt + 256;
    misc = scan + kHeavyThreads / 64 + 1;
  }
  static constexpr size_t bytes() {
    return (size_t)kLeafKeys * 25 + 4 * ((size_t)kDigits + 2 * (kDigits + 1) + 256 + kHeavyThreads / 64 + 1 + 4);
  }
};

// block-wide barrier after global stores that other waves of the workgroup read next:
// the barrier's workgroup-scope fence waits for the stores, and the waves of one
// workgroup share the compute unit's write-through vector cache (an agent-scope fence
// here would write back and invalidate the whole L2 at every call)
__device__ __forceinline__ void heavy_sync() { __syncthreads(); }

// Stream [a, b) of (key, value) pairs through f(key, value, ok), kHeavyPer pairs per lane
// in flight (indices clamped into the range; the empty asm keeps the loads ahead of the
// atomics that use them).  f is called by every lane in uniform control flow, ok telling
// whether its pair is in the range, so that f can combine the lanes of a wave.
// WITH_VAL = false reads the keys only.
constexpr int kHeavyPer = 8;
template <bool WITH_VAL, typename V, typename Fn>
__device__ __forceinline__ void heavy_stream(const uint32_t* key, const V* val, uint32_t a, uint32_t b, Fn f) {
  for (uint32_t i0 = a; i0 < b; i0 += kHeavyPer * kHeavyThreads) {
    uint32_t kk[kHeavyPer];
    V vv[kHeavyPer] = {};
#pragma unroll
    for (int u = 0; u < kHeavyPer; ++u) {
      const uint32_t i = i0 + u * kHeavyThreads + threadIdx.x;
      const uint32_t ic = i < b ? i : a;
      kk[u] = key[ic];
      if constexpr (WITH_VAL) vv[u] = val[ic];
    }
#pragma unroll
    for (int u = 0; u < kHeavyPer; ++u) {
      if constexpr (WITH_VAL)
        asm volatile("" : "+v"(kk[u]), "+v"(vv[u]));
      else
        asm volatile("" : "+v"(kk[u]));
    }
#pragma unroll
    for (int u = 0; u < kHeavyPer; ++u) f(kk[u], vv[u], i0 + u * kHeavyThreads + threadIdx.x < b);
  }
}

// A heavy node's diagonal (or one column of its row) can own most pairs of a range, and
// atomics on one LDS address serialise.  Each wave therefore takes its first lane's
// digit or slot as "hot": when more than one lane holds it, those lanes are combined into
// one atomic by the first lane (heavy_hot returns their mask, else 0).
__device__ __forceinline__ uint64_t heavy_hot(uint32_t x, bool ok, uint32_t& hot) {
  hot = __builtin_amdgcn_readfirstlane(x);
  const uint64_t m = __ballot(ok && x == hot);
  return __popcll(m) > 1 ? m : 0ull;
}

template <typename V>
__device__ void heavy_split(const HeavySmem& sm, const uint32_t* skey, const V* sval, uint32_t* dkey, V* dval,
                            uint32_t a, uint32_t b, uint32_t kmin, int shift, int nd, uint32_t* st) {
  const int lane = threadIdx.x & 63;
  for (int d = threadIdx.x; d < nd; d += kHeavyThreads) sm.hist[d] = 0;
  __syncthreads();
  heavy_stream<false>(skey, sval, a, b, [&](uint32_t k, V, bool ok) {
    const uint32_t d = (k - kmin) >> shift;
    uint32_t hot;
    const uint64_t m = heavy_hot(d, ok, hot);
    if (ok && !((m >> lane) & 1ull)) atomicAdd(&sm.hist[d], 1u);
    if (lane == 0 && m) atomicAdd(&sm.hist[hot], (uint32_t)__popcll(m));
  });
  __syncthreads();
  block_scan_array(sm.hist, nd, sm.scan);  // (ends with a barrier)
  for (int d = threadIdx.x; d < nd; d += kHeavyThreads) st[d] = a + sm.hist[d];
  if (threadIdx.x == 0) st[nd] = b;
  __syncthreads();
  heavy_stream<true>(skey, sval, a, b, [&](uint32_t k, V v, bool ok) {
    const uint32_t d = (k - kmin) >> shift;
    uint32_t hot;
    const uint64_t m = heavy_hot(d, ok, hot);
    uint32_t base = 0;
    if (lane == 0 && m) base = atomicAdd(&sm.hist[hot], (uint32_t)__popcll(m));
    base = __shfl(base, 0, 64);
    const bool mine = (m >> lane) & 1ull;
    uint32_t pos = 0;
    if (mine)
      pos = a + base + (uint32_t)__popcll(m & ((1ull << lane) - 1));
    else if (ok)
      pos = a + atomicAdd(&sm.hist[d], 1u);
    if (ok) {
      dkey[pos] = k;
      dval[pos] = v;
    }
  });
  heavy_sync();
}

// carry the low and high chunk sums of the occupied slots upward: lo < 2^48, hi < 2^48
__device__ __forceinline__ void heavy_normalise(const HeavySmem& sm) {
  constexpr unsigned long long M48 = (1ull << 48) - 1;
  for (int h = threadIdx.x; h < kLeafKeys; h += kHeavyThreads) {
    if (!sm.occ[h]) continue;
    const unsigned long long l = sm.lo[h];
    const long long x = sm.hi[h] + (long long)(l >> 48);
    sm.lo[h] = l & M48;
    sm.top[h] += x >> 48;  // arithmetic shift: floor division
    sm.hi[h] = (long long)((unsigned long long)x & M48);
  }
}

// pairs per round of a leaf: the carried sums (below 2^48) plus kRound chunks (below
// 2^48 unsigned, below 2^47 in magnitude signed) stay inside 64 bits
constexpr uint32_t kRound = 65532;

// the exact sums of the leaf's pairs [a, b) (keys in [kmin, kmin + kLeafKeys); PICK: of those
// with keys in [kmin, kmin + w), w <= kLeafKeys) into the LDS slots, carried after every round
// (lo, hi below 2^48; occ set)
template <typename V, bool PICK = false>
__device__ void heavy_leaf_sum(const HeavySmem& sm, const uint32_t* key, const V* val, uint32_t a, uint32_t b,
                               uint32_t kmin, int F, uint32_t w = kLeafKeys) {
  const int lane = threadIdx.x & 63;
  // the wave's kept slot: once a slot has been hot (held by more than one lane), the
  // lanes that meet it again while it is the wave's first lane's slot add its chunks to
  // their own sums, which are summed over the wave and added once, at the end of the
  // round (a key that owns most of the leaf, such as a heavy node's diagonal, then costs
  // two register additions per pair)
  for (uint32_t r = a; r < b; r += kRound) {
    const uint32_t re = b - r > kRound ? r + kRound : b;
    uint32_t kept = kEmptyKey;  // (uniform)
    unsigned long long k0 = 0ull;
    long long k1 = 0ll;
    const auto flush = [&]() {  // the kept sums over the wave, added to the kept slot
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
        k0 += __shfl_xor(k0, o, 64);
        k1 += __shfl_xor(k1, o, 64);
      }
      if (lane == 0) {
        atomicAdd(&sm.lo[kept], k0);
        atomicAdd((unsigned long long*)&sm.hi[kept], (unsigned long long)k1);
        sm.occ[kept] = 1;
      }
      k0 = 0ull;
      k1 = 0ll;
    };
    heavy_stream<true>(key, val, r, re, [&](uint32_t k, V v, bool ok) {
      const uint32_t h = k - kmin;
      if constexpr (PICK) ok = ok && h < w;
      uint64_t c0;
      int64_t c1;
      to_chunks(v, F, c0, c1);
      uint32_t hot;
      const uint64_t m = heavy_hot(h, ok, hot);
      const bool mine = (m >> lane) & 1ull;
      if (ok && !mine) {
        atomicAdd(&sm.lo[h], (unsigned long long)c0);
        atomicAdd((unsigned long long*)&sm.hi[h], (unsigned long long)c1);
        sm.occ[h] = 1;
      }
      if (m) {
        if (hot != kept) {  // (uniform) a new kept slot: the old one's sums go first
          if (kept != kEmptyKey) flush();
          kept = hot;
        }
        if (mine) {  // (64 lanes x 64 pairs of a round: the sums stay below 2^60)
          k0 += c0;
          k1 += c1;
        }
      }
    });
    if (kept != kEmptyKey) flush();
    __syncthreads();
    heavy_normalise(sm);
    __syncthreads();
  }
}

// the occupied LDS slots (carried sums) as entries, appended in key order at tcol /
// tval [u0 ...), the slots cleared; returns the number of entries
template <typename V, bool RES>
__device__ uint32_t heavy_leaf_emit(const HeavySmem& sm, uint32_t kmin, int F, int colbits, int32_t* tcol, V* tval,
                                    V* tres, uint32_t u0) {
  const int lane = threadIdx.x & 63;
  // the occupied slots in order: kLeafKeys / kHeavyThreads consecutive slots per lane
  constexpr int PL = kLeafKeys / kHeavyThreads;
  const int h0 = threadIdx.x * PL;
  static_assert(PL == 4, "four slot flags per lane are read as one word");
  const uint32_t fw = *(const uint32_t*)(sm.occ + h0);  // byte j: slot h0 + j
  const uint32_t bits = (fw & 1u) | ((fw >> 7) & 2u) | ((fw >> 14) & 4u) | ((fw >> 21) & 8u);
  uint32_t total;
  uint32_t pos = u0 + block_scan_u32(__popc(bits), sm.scan, &total);
  const uint32_t cmask = (1u << colbits) - 1;
#pragma unroll
  for (int j = 0; j < PL; ++j) {
    const bool occ = (bits >> j) & 1u;
    const int h = h0 + j;
    const uint32_t k = kmin + (uint32_t)h;
    // entries per row: a range spans few rows, so the lanes of a wave mostly share one
    uint32_t hot;
    const uint64_t m = heavy_hot(k >> colbits, occ, hot);
    if (occ && !((m >> lane) & 1ull)) atomicAdd(&sm.rowcnt[k >> colbits], 1u);
    if (lane == 0 && m) atomicAdd(&sm.rowcnt[hot], (uint32_t)__popcll(m));
    if (!occ) continue;
    // value = lo + hi 2^48 + top 2^96, lo and hi in [0, 2^48): as a 128-bit integer
    const unsigned long long l = sm.lo[h], x = (unsigned long long)sm.hi[h];
    const long long t = sm.top[h];
    const uint64_t qlo = l | (x << 48);
    const uint64_t qhi = (x >> 16) | ((uint64_t)t << 32);
    const V hv = from_fixed_as<V>(qlo, qhi, F);
    tcol[pos] = (int32_t)(k & cmask);
    tval[pos] = hv;
    if constexpr (RES) tres[pos] = fixed_residual<V>(qlo, qhi, F, hv);
    sm.lo[h] = 0ull;
    sm.hi[h] = 0ll;
    sm.top[h] = 0ll;
    ++pos;
  }
  __syncthreads();
  if (threadIdx.x < kLeafKeys / 4) ((uint32_t*)sm.occ)[threadIdx.x] = 0u;
  heavy_sync();
  return total;
}

// sums of the leaf's pairs [a, b) (keys in [kmin, kmin + kLeafKeys)), appended in key
// order at tcol / tval [u0 ...); returns the number of entries
template <typename V, bool RES>
__device__ uint32_t heavy_leaf(const HeavySmem& sm, const uint32_t* key, const V* val, uint32_t a, uint32_t b,
                               uint32_t kmin, int F, int colbits, int32_t* tcol, V* tval, V* tres, uint32_t u0) {
  heavy_leaf_sum<V>(sm, key, val, a, b, kmin, F);
  return heavy_leaf_emit<V, RES>(sm, kmin, F, colbits, tcol, tval, tres, u0);
}

// Leaves of the split sub-buckets (first-level digit ranges no wider than a leaf) with
// more than kBigLeafPairs pairs, such as the one holding a heavy node's diagonal, are
// summed by several workgroups: heavy_starts lists up to kBigLeaves of them, each
// workgroup of heavy_bigleaf sums one round (kRound pairs) of one of them into its LDS
// slots and adds the carried sums (lo, hi below 2^48, top) of its occupied slots into
// the leaf's accumulator with 64-bit atomics (exact: a leaf of fewer than 2^31 pairs has
// fewer than 2^16 rounds), and heavy_ranges carries the accumulated sums once
// more and writes the leaf's entries.  Leaves beyond the list are summed as the others.
constexpr int kBigLeaves = 8;
constexpr uint32_t kBigLeafPairs = 2 * kRound;
constexpr int kBigRec = 8;  // words per listed leaf: it, d0, a, b, k0
constexpr int kBigListWords = 8 + kBigRec * kBigLeaves;
constexpr int kBigAccWords = 7 * kLeafKeys;  // lo, hi, top (64-bit) and occ (32-bit) per slot
constexpr size_t kBigWords = kBigListWords + (size_t)kBigLeaves * kBigAccWords;
struct BigLeaves {
  uint32_t* list;  // [0] leaves listed (may exceed kBigLeaves), then the records
  __device__ explicit BigLeaves(uint32_t* hvy) : list(hvy + (size_t)kHeavyPar * kHvyWords) {}
  __device__ uint32_t count() const { return list[0] < (uint32_t)kBigLeaves ? list[0] : (uint32_t)kBigLeaves; }
  __device__ uint32_t* rec(uint32_t i) const { return list + 8 + kBigRec * i; }
  __device__ unsigned long long* lo(uint32_t i) const {
    return (unsigned long long*)(list + kBigListWords + (size_t)i * kBigAccWords);
  }
  __device__ unsigned long long* hi(uint32_t i) const { return lo(i) + kLeafKeys; }
  __device__ unsigned long long* top(uint32_t i) const { return lo(i) + 2 * kLeafKeys; }
  __device__ uint32_t* occ(uint32_t i) const { return (uint32_t*)(lo(i) + 3 * kLeafKeys); }
};
static_assert(((size_t)kHeavyPar * kHvyWords + kBigListWords) % 2 == 0, "the accumulators are 8-byte aligned");

// split width for a key range of w keys: 0 for a leaf, else the digit shift
__device__ __forceinline__ int heavy_shift(uint32_t w) {
  if (w <= (uint32_t)kLeafKeys) return 0;
  const int bits = 32 - __clz(w - 1);  // keys need `bits` bits
  return bits - 11 > 12 ? bits - 11 : 12;  // at most kDigits digits
}

// One first-level digit range [a, b) of a heavy sub-bucket, in (akey, aval), keys in
// [k0, k0 + w): a leaf, or split again into (ikey, ival) at the same place and its leaves
// summed in key order.  Entries written from tcol / tval / tres [u0 ...); returns their
// number.  The range's pairs are all read before any entry is written, and a range has
// at most as many entries as pairs.
template <typename V, bool RES>
__device__ uint32_t heavy_range(const HeavySmem& sm, uint32_t* ikey, V* ival, uint32_t* akey, V* aval, uint32_t a,
                                uint32_t b, uint32_t k0, uint32_t w, int F, int colbits, int32_t* tcol, V* tval,
                                V* tres, uint32_t u0) {
  const int sh1 = heavy_shift(w);
  if (sh1 == 0) return heavy_leaf<V, RES>(sm, akey, aval, a, b, k0, F, colbits, tcol, tval, tres, u0);
  const int nd1 = (int)((w - 1) >> sh1) + 1;
  uint32_t* st1 = sm.start + (kDigits + 1);
  heavy_split<V>(sm, akey, aval, ikey, ival, a, b, k0, sh1, nd1, st1);
  uint32_t U = 0;
  for (int d1 = 0; d1 < nd1; ++d1) {  // leaves (sh1 = 12 after a first split)
    const uint32_t a1 = st1[d1], b1 = st1[d1 + 1];
    if (a1 == b1) continue;
    U += heavy_leaf<V, RES>(sm, ikey, ival, a1, b1, k0 + ((uint32_t)d1 << sh1), F, colbits, tcol, tval, tres, u0 + U);
  }
  return U;
}

// What the phases of k_heavy share (the pair buffers alias the output, so nothing here
// carries __restrict__).
template <typename V>
struct HeavyArgs {
  uint32_t* ikey;  // the listed sub-buckets' pairs, then scratch
  V* ival;
  uint32_t* akey;  // the other pair buffer, then the output columns and values
  V* aval;
  V* tres;
  const uint32_t* sbb;
  SubBuckets sub;
  int s2, colbits;  // (s2: the way taken)
  int64_t n_node;
  int F;
  uint32_t* rowoff;
  uint32_t* usub;
  const uint32_t* ov_list;
  uint32_t n_over, npar;  // listed; of those, split by the whole device (the first npar)
  uint32_t* hvy;
};

// The listed sub-buckets after the first npar, one workgroup each
template <typename V, bool RES>
__device__ void heavy_rest(unsigned char* smem, const HeavyArgs<V>& A, uint32_t blk, uint32_t nblk) {
  const HeavySmem sm(smem);
  const uint32_t n_over = A.n_over;
  uint32_t *const ikey = A.ikey, *const akey = A.akey, *const rowoff = A.rowoff, *const usub = A.usub;
  V *const ival = A.ival, *const aval = A.aval, *const tres = A.tres;
  const uint32_t *const sbb = A.sbb, *const ov_list = A.ov_list;
  const int s2 = A.s2, colbits = A.colbits, F = A.F;
  if (A.npar + blk >= n_over) return;
  for (int h = threadIdx.x; h < kLeafKeys; h += kHeavyThreads) {
    sm.lo[h] = 0ull;
    sm.hi[h] = 0ll;
    sm.top[h] = 0ll;
  }
  if (threadIdx.x < kLeafKeys / 4) ((uint32_t*)sm.occ)[threadIdx.x] = 0u;
  int32_t* const tcol = (int32_t*)akey;
  for (uint32_t it = A.npar + blk; it < n_over; it += nblk) {
    const int64_t g = ov_list[it];
    const uint32_t beg = sbb[g], end = sbb[g + 1];
    const int64_t r0 = g << s2;
    const int R = (int)min((int64_t)1 << s2, A.n_node - r0);
    for (int r = threadIdx.x; r < 256; r += kHeavyThreads) sm.rowcnt[r] = 0u;
    // key range
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    heavy_stream<false>(ikey, ival, beg, end, [&](uint32_t k, V, bool ok) {
      mn = ok && k < mn ? k : mn;
      mx = ok && k > mx ? k : mx;
    });
    if (threadIdx.x < 2) sm.misc[threadIdx.x] = threadIdx.x == 0 ? 0xFFFFFFFFu : 0u;
    __syncthreads();
    atomicMin(&sm.misc[0], mn);
    atomicMax(&sm.misc[1], mx);
    __syncthreads();
    const uint32_t kmin = sm.misc[0], w0 = sm.misc[1] - kmin + 1;
    __syncthreads();
    uint32_t U = 0;
    const int sh0 = heavy_shift(w0);
    if (sh0 == 0) {
      U = heavy_leaf<V, RES>(sm, ikey, ival, beg, end, kmin, F, colbits, tcol + beg, aval + beg,
                             RES ? tres + beg : nullptr, 0);
    } else {
      const int nd0 = (int)((w0 - 1) >> sh0) + 1;
      uint32_t* st0 = sm.start;
      heavy_split<V>(sm, ikey, ival, akey, aval, beg, end, kmin, sh0, nd0, st0);
      for (int d0 = 0; d0 < nd0; ++d0) {
        const uint32_t a = st0[d0], b = st0[d0 + 1];
        if (a == b) continue;
        const uint32_t k0 = kmin + ((uint32_t)d0 << sh0);
        const uint32_t w1 = (1u << sh0) < (kmin + w0 - k0) ? (1u << sh0) : (kmin + w0 - k0);
        U += heavy_range<V, RES>(sm, ikey, ival, akey, aval, a, b, k0, w1, F, colbits, tcol + beg, aval + beg,
                                 RES ? tres + beg : nullptr, U);
      }
    }
    // row offsets within the sub-bucket
    if (threadIdx.x < 64) {
      const int lane = threadIdx.x;
      uint32_t v[4], sum = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int r = lane * 4 + k;
        v[k] = r < R ? sm.rowcnt[r] : 0u;
        sum += v[k];
      }
      uint32_t x = sum;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
      }
      uint32_t run = x - sum;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int r = lane * 4 + k;
        if (r < R) rowoff[r0 + r] = run;
        run += v[k];
      }
    }
    if (threadIdx.x == 0) usub[g] = U;
    heavy_sync();
  }
}

// ---- the split of the first kHeavyPar listed sub-buckets, by many workgroups.  Their
// pairs are cut into chunks of kSplitChunk (a sub-bucket's last chunk shorter); each
// workgroup takes chunks j = blockIdx.x, blockIdx.x + gridDim.x, ...  in list order.
constexpr uint32_t kSplitChunk = 8192;

// the listed sub-buckets' pair ranges and chunk prefix in LDS (npar <= kHeavyPar)
__device__ __forceinline__ void heavy_chunk_table(const uint32_t* sbb, const uint32_t* ov_list, uint32_t npar,
                                                  uint32_t* s_beg, uint32_t* s_end, uint32_t* s_c0) {
  if (threadIdx.x < 64) {
    const uint32_t it = threadIdx.x;
    uint32_t a = 0, b = 0;
    if (it < npar) {
      const uint32_t g = ov_list[it];
      a = sbb[g];
      b = sbb[g + 1];
    }
    const uint32_t nc = (b - a + kSplitChunk - 1) / kSplitChunk;
    uint32_t x = nc;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if ((int)it >= d) x += y;
    }
    s_beg[it] = a;
    s_end[it] = b;
    s_c0[it + 1] = x;
    if (it == 0) s_c0[0] = 0u;
  }
  __syncthreads();
}

// the sub-bucket of chunk j (j below the chunk total): the last it with s_c0[it] <= j
__device__ __forceinline__ uint32_t heavy_chunk_owner(const uint32_t* s_c0, uint32_t j) {
  uint32_t lo = 0, n = kHeavyPar;
#pragma unroll
  for (int s = 0; s < 6; ++s) {  // kHeavyPar = 2^6 candidates
    const uint32_t half = n >> 1;
    if (s_c0[lo + half] <= j) lo += half;
    n -= half;
  }
  return lo;
}

// Calls f(it, a, b) for each chunk [a, b) of this workgroup, it its sub-bucket's place
// in the list.  f is called by all threads and may use barriers.
template <typename Fn>
__device__ __forceinline__ void heavy_chunks(const uint32_t* sbb, const uint32_t* ov_list, uint32_t npar,
                                             uint32_t blk, uint32_t nblk, Fn f) {
  __shared__ uint32_t s_beg[kHeavyPar], s_end[kHeavyPar], s_c0[kHeavyPar + 1];
  heavy_chunk_table(sbb, ov_list, npar, s_beg, s_end, s_c0);
  const uint32_t nch = s_c0[kHeavyPar];
  for (uint32_t j = blk; j < nch; j += nblk) {
    const uint32_t it = heavy_chunk_owner(s_c0, j);
    const uint32_t a = s_beg[it] + (j - s_c0[it]) * kSplitChunk;
    const uint32_t b = s_end[it] - a > kSplitChunk ? a + kSplitChunk : s_end[it];
    f(it, a, b);
  }
}

// A wave's keys of one LDS counter combined (heavy_hot) into count[x(k)].
template <typename X>
__device__ __forceinline__ void heavy_count(const uint32_t* key, uint32_t a, uint32_t b, uint32_t* count, X x) {
  const int lane = threadIdx.x & 63;
  heavy_stream<false, uint32_t>(key, nullptr, a, b, [&](uint32_t k, uint32_t, bool ok) {
    const uint32_t d = ok ? x(k) : 0u;
    uint32_t hot;
    const uint64_t m = heavy_hot(d, ok, hot);
    if (ok && !((m >> lane) & 1ull)) atomicAdd(&count[d], 1u);
    if (lane == 0 && m) atomicAdd(&count[hot], (uint32_t)__popcll(m));
  });
}

// Pairs of each row of the split sub-buckets; their digit counts cleared
template <typename V>
__device__ void heavy_rows(unsigned char* smem, const HeavyArgs<V>& A, uint32_t blk, uint32_t nblk) {
  uint32_t* const s_rows = (uint32_t*)smem;  // [kHvyRows]
  const int colbits = A.colbits;
  for (uint32_t i = blk * kHeavyThreads + threadIdx.x; i < A.npar * (uint32_t)kHvyDigits; i += nblk * kHeavyThreads)
    HeavyTable(A.hvy, i / kHvyDigits).hist[i % kHvyDigits] = 0u;
  if (blk == 0 && threadIdx.x == 0) BigLeaves(A.hvy).list[0] = 0u;
  if (blk == 0 && threadIdx.x < A.npar) HeavyTable(A.hvy, threadIdx.x).meta[1] = 0u;
  heavy_chunks(A.sbb, A.ov_list, A.npar, blk, nblk, [&](uint32_t it, uint32_t a, uint32_t b) {
    for (int r = threadIdx.x; r < kHvyRows; r += kHeavyThreads) s_rows[r] = 0u;
    __syncthreads();
    heavy_count(A.ikey, a, b, s_rows, [&](uint32_t k) { return k >> colbits; });
    __syncthreads();
    const HeavyTable t(A.hvy, it);
    for (int r = threadIdx.x; r < kHvyRows; r += kHeavyThreads) {
      const uint32_t c = s_rows[r];
      if (c) atomicAdd(&t.rpair[r], c);
    }
    __syncthreads();
  });
}

// The digits of each row of a split sub-bucket (of n pairs) from its rows' pair counts,
// into LDS (s_rbase: kHvyRows + 1 words, s_rsh: kHvyRows, s_scan: kHeavyThreads / 64 + 1);
// `store`: to the table too.  Ends with a barrier.
__device__ __forceinline__ void heavy_layout(const HeavyTable& t, const uint32_t* rpair, uint64_t n, int colbits,
                                             bool store, uint32_t* s_rbase, uint32_t* s_rsh, uint32_t* s_scan) {
  const int r = threadIdx.x;
  const uint32_t c = r < kHvyRows ? rpair[r] : 0u;
  const int lg_max = colbits > 12 ? colbits - 12 : 0;  // digits no narrower than a leaf
  const int lg_min = colbits > 23 ? colbits - 23 : 0;  // nor wider than 2^23 keys
  int lg = 0;
  if (c) {
    const uint64_t q = (uint64_t)c * kHvyShare / n;
    lg = q > 1 ? 63 - __clzll((long long)q) : 0;
    lg = lg < lg_min ? lg_min : (lg > lg_max ? lg_max : lg);
  }
  const uint32_t nr = c ? 1u << lg : 0u;
  uint32_t total;
  const uint32_t base = block_scan_u32(nr, s_scan, &total);
  if (r < kHvyRows) {
    s_rbase[r] = base;
    s_rsh[r] = (uint32_t)(colbits - lg);
    if (store) {
      t.rbase[r] = base;
      t.rsh[r] = (uint32_t)(colbits - lg);
    }
  }
  if (r == 0) {
    s_rbase[kHvyRows] = total;
    if (store) {
      t.rbase[kHvyRows] = total;
      t.meta[0] = total;
    }
  }
  __syncthreads();
}

// a sub-bucket's digit layout into LDS (s_rbase: kHvyRows + 1 words, s_rsh: kHvyRows)
__device__ __forceinline__ void heavy_load_layout(const HeavyTable& t, uint32_t* s_rbase, uint32_t* s_rsh) {
  for (int r = threadIdx.x; r <= kHvyRows; r += blockDim.x) {
    s_rbase[r] = t.rbase[r];
    if (r < kHvyRows) s_rsh[r] = t.rsh[r];
  }
}

// the row of digit d: the last r with rbase[r] <= d
__device__ __forceinline__ uint32_t heavy_row(const uint32_t* rbase, uint32_t d) {
  uint32_t r = 0, n = kHvyRows;
#pragma unroll
  for (int s = 0; s < 8; ++s) {  // kHvyRows = 2^8 candidates
    const uint32_t half = n >> 1;
    if (rbase[r + half] <= d) r += half;
    n -= half;
  }
  return r;
}

// A split sub-bucket's digit starts (absolute pair positions) from its digit counts, which become
// the scatter's cursors; digit ranges no wider than a leaf with more than kBigLeafPairs pairs are
// listed as big leaves.  s_off: kHvyDigits words; s_rbase, s_rsh: the layout; s_scan as block_scan.
template <typename V>
__device__ __forceinline__ void heavy_starts(const HeavyArgs<V>& A, uint32_t it, uint32_t* s_off,
                                             const uint32_t* s_rbase, const uint32_t* s_rsh, uint32_t* s_scan) {
  const int colbits = A.colbits;
  uint32_t* const hvy = A.hvy;
  const HeavyTable t(hvy, it);
  const uint32_t nd = s_rbase[kHvyRows];
  const uint32_t g = A.ov_list[it];
  const uint32_t beg = A.sbb[g], end = A.sbb[g + 1];
  for (uint32_t d = threadIdx.x; d < nd; d += kHeavyThreads)
    s_off[d] = __hip_atomic_load(&t.hist[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  block_scan_array(s_off, (int)nd, s_scan);  // (ends with a barrier)
  const BigLeaves big(hvy);
  for (uint32_t d = threadIdx.x; d < nd; d += kHeavyThreads) {
    const uint32_t a = beg + s_off[d], b = d + 1 < nd ? beg + s_off[d + 1] : end;
    t.st[d] = a;
    t.hist[d] = a;
    if (b - a > kBigLeafPairs) {
      const uint32_t r = heavy_row(s_rbase, d), sh = s_rsh[r];
      if ((1u << sh) <= (uint32_t)kLeafKeys) {
        const uint32_t i = atomicAdd(big.list, 1u);
        if (i < (uint32_t)kBigLeaves) {
          uint32_t* const q = big.rec(i);
          q[0] = it;
          q[1] = d;
          q[2] = a;
          q[3] = b;
          q[4] = (r << colbits) + ((d - s_rbase[r]) << sh);
        }
      }
    }
  }
  if (threadIdx.x == 0) t.st[nd] = end;
}

// Pairs per first-level digit, summed over the chunks into the table's hist.  Every
// workgroup works out the digit layout from the row counts (a scan of 256 words: less
// than a launch of its own takes); the one with a sub-bucket's first chunk stores it, the
// last to finish a chunk of it turns the counts into starts.
template <typename V>
__device__ void heavy_hist(unsigned char* smem, const HeavyArgs<V>& A, uint32_t blk, uint32_t nblk) {
  uint32_t* const s_hist = (uint32_t*)smem;        // [kHvyDigits]
  uint32_t* const s_rbase = s_hist + kHvyDigits;   // [kHvyRows + 1]
  uint32_t* const s_rsh = s_rbase + kHvyRows + 1;  // [kHvyRows]
  uint32_t* const s_scan = s_rsh + kHvyRows;       // [kHeavyThreads / 64 + 1]
  __shared__ uint32_t s_last;
  const int colbits = A.colbits;
  heavy_chunks(A.sbb, A.ov_list, A.npar, blk, nblk, [&](uint32_t it, uint32_t a, uint32_t b) {
    const HeavyTable t(A.hvy, it);
    const uint32_t g = A.ov_list[it];
    for (int d = threadIdx.x; d < kHvyDigits; d += kHeavyThreads) s_hist[d] = 0u;
    heavy_layout(t, t.rpair, A.sbb[g + 1] - A.sbb[g], colbits, a == A.sbb[g], s_rbase, s_rsh, s_scan);
    const uint32_t nd = s_rbase[kHvyRows];
    heavy_count(A.ikey, a, b, s_hist, [&](uint32_t k) { return heavy_digit(k, colbits, s_rbase, s_rsh); });
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < nd; d += kHeavyThreads) {
      const uint32_t c = s_hist[d];
      if (c) atomicAdd(&t.hist[d], c);
    }
    const uint32_t n = A.sbb[g + 1] - A.sbb[g];
    // this thread's counts done before the arrival (as last_block_starts: nothing but the counts,
    // which are atomics, passes on; a fence's write-back of the L2 for each chunk took 0.12 ms of a
    // fan of 1M tetrahedra)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(&t.meta[1], 1u) == (n - 1) / kSplitChunk ? 1u : 0u;
    __syncthreads();
    if (s_last) heavy_starts<V>(A, it, s_hist, s_rbase, s_rsh, s_scan);
    __syncthreads();
  });
}

// Each chunk's pairs moved from (ikey, ival) to (akey, aval) in first-level digit
// order: the chunk's digit counts taken again, a block of each digit reserved from the
// table's cursors, then each pair placed in its digit's block
template <typename V>
__device__ void heavy_scatter(unsigned char* smem, const HeavyArgs<V>& A, uint32_t blk, uint32_t nblk) {
  uint32_t* const s_hist = (uint32_t*)smem;        // [kHvyDigits]
  uint32_t* const s_rbase = s_hist + kHvyDigits;   // [kHvyRows + 1]
  uint32_t* const s_rsh = s_rbase + kHvyRows + 1;  // [kHvyRows]
  const int colbits = A.colbits;
  uint32_t *const hvy = A.hvy, *const ikey = A.ikey, *const akey = A.akey;
  V *const ival = A.ival, *const aval = A.aval;
  const int lane = threadIdx.x & 63;
  {  // the big leaves' accumulators cleared (the next phase adds into them)
    const BigLeaves big(hvy);
    uint32_t* const acc = big.list + kBigListWords;
    const size_t nw = (size_t)big.count() * kBigAccWords;
    for (size_t w = (size_t)blk * kHeavyThreads + threadIdx.x; w < nw; w += (size_t)nblk * kHeavyThreads)
      acc[w] = 0u;
  }
  heavy_chunks(A.sbb, A.ov_list, A.npar, blk, nblk, [&](uint32_t it, uint32_t a, uint32_t b) {
    const HeavyTable t(hvy, it);
    heavy_load_layout(t, s_rbase, s_rsh);
    for (int d = threadIdx.x; d < kHvyDigits; d += kHeavyThreads) s_hist[d] = 0u;
    __syncthreads();
    const uint32_t nd = s_rbase[kHvyRows];
    heavy_count(ikey, a, b, s_hist, [&](uint32_t k) { return heavy_digit(k, colbits, s_rbase, s_rsh); });
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < nd; d += kHeavyThreads) {
      const uint32_t c = s_hist[d];
      s_hist[d] = c ? atomicAdd(&t.hist[d], c) : 0u;
    }
    __syncthreads();
    heavy_stream<true, V>(ikey, ival, a, b, [&](uint32_t k, V v, bool ok) {
      const uint32_t d = ok ? heavy_digit(k, colbits, s_rbase, s_rsh) : 0u;
      uint32_t hot;
      const uint64_t m = heavy_hot(d, ok, hot);
      uint32_t base = 0;
      if (lane == 0 && m) base = atomicAdd(&s_hist[hot], (uint32_t)__popcll(m));
      base = __shfl(base, 0, 64);
      const bool mine = (m >> lane) & 1ull;
      uint32_t pos = 0;
      if (mine)
        pos = base + (uint32_t)__popcll(m & ((1ull << lane) - 1));
      else if (ok)
        pos = atomicAdd(&s_hist[d], 1u);
      if (ok) {
        akey[pos] = k;
        aval[pos] = v;
      }
    });
    __syncthreads();
  });
}

// The rounds of the listed big leaves, one per workgroup at a time, added into
// their accumulators (each leaf's pairs in (akey, aval) [a, b), keys from k0)
template <typename V>
__device__ void heavy_bigleaf(unsigned char* smem, const HeavyArgs<V>& A, uint32_t blk, uint32_t nblk) {
  const HeavySmem sm(smem);
  __shared__ uint32_t s_p0[kBigLeaves + 1];
  uint32_t* const hvy = A.hvy;
  const BigLeaves big(hvy);
  const uint32_t nbig = big.count();
  if (nbig == 0) return;
  if (threadIdx.x == 0) {
    uint32_t s = 0;
    for (uint32_t i = 0; i < nbig; ++i) {
      s_p0[i] = s;
      s += (big.rec(i)[3] - big.rec(i)[2] + kRound - 1) / kRound;
    }
    s_p0[nbig] = s;
  }
  for (int h = threadIdx.x; h < kLeafKeys; h += kHeavyThreads) {
    sm.lo[h] = 0ull;
    sm.hi[h] = 0ll;
    sm.top[h] = 0ll;
  }
  if (threadIdx.x < kLeafKeys / 4) ((uint32_t*)sm.occ)[threadIdx.x] = 0u;
  __syncthreads();
  for (uint32_t p = blk; p < s_p0[nbig]; p += nblk) {
    uint32_t i = 0;
    while (i + 1 < nbig && s_p0[i + 1] <= p) ++i;
    const uint32_t* const q = big.rec(i);
    const uint32_t a = q[2] + (p - s_p0[i]) * kRound;
    const uint32_t b = q[3] - a > kRound ? a + kRound : q[3];
    heavy_leaf_sum<V>(sm, A.akey, A.aval, a, b, q[4], A.F);
    unsigned long long* const glo = big.lo(i);
    unsigned long long* const ghi = big.hi(i);
    unsigned long long* const gtop = big.top(i);
    uint32_t* const gocc = big.occ(i);
    for (int h = threadIdx.x; h < kLeafKeys; h += kHeavyThreads) {
      if (!sm.occ[h]) continue;
      atomicAdd(&glo[h], sm.lo[h]);
      atomicAdd(&ghi[h], (unsigned long long)sm.hi[h]);
      atomicAdd(&gtop[h], (unsigned long long)sm.top[h]);
      gocc[h] = 1u;
      sm.lo[h] = 0ull;
      sm.hi[h] = 0ll;
      sm.top[h] = 0ll;
    }
    __syncthreads();
    if (threadIdx.x < kLeafKeys / 4) ((uint32_t*)sm.occ)[threadIdx.x] = 0u;
    __syncthreads();
  }
}

// The first-level digit ranges of the first kHeavyPar listed sub-buckets, split
// by heavy_scatter: range d0 of sub-bucket it is reduced by workgroup d0 mod nblk, its
// entries written from its own first pair's place (its pairs all read before; other
// workgroups read other ranges), its entry count recorded in the table.
template <typename V, bool RES>
__device__ void heavy_ranges(unsigned char* smem, const HeavyArgs<V>& A, uint32_t blk, uint32_t nblk) {
  const HeavySmem sm(smem);
  const uint32_t npar = A.npar;
  const int colbits = A.colbits, F = A.F;
  uint32_t *const hvy = A.hvy, *const ikey = A.ikey, *const akey = A.akey;
  V *const ival = A.ival, *const aval = A.aval, *const tres = A.tres;
  for (int h = threadIdx.x; h < kLeafKeys; h += kHeavyThreads) {
    sm.lo[h] = 0ull;
    sm.hi[h] = 0ll;
    sm.top[h] = 0ll;
  }
  if (threadIdx.x < kLeafKeys / 4) ((uint32_t*)sm.occ)[threadIdx.x] = 0u;
  for (int r = threadIdx.x; r < 256; r += kHeavyThreads) sm.rowcnt[r] = 0u;
  __syncthreads();
  int32_t* const tcol = (int32_t*)akey;
  // the layout of the sub-bucket in hand, in the first of the two split-start arrays
  // (heavy_range uses the second)
  uint32_t* const s_rbase = sm.start;
  uint32_t* const s_rsh = sm.start + kHvyRows + 1;
  static_assert(2 * kHvyRows + 1 <= kDigits + 1, "the row layout fits one split-start array");
  // the big leaves (summed by heavy_bigleaf): their sub-bucket and digit
  __shared__ uint32_t s_big[2 * kBigLeaves];
  const BigLeaves big(hvy);
  const uint32_t nbig = big.count();
  if (threadIdx.x < nbig) {
    s_big[2 * threadIdx.x] = big.rec(threadIdx.x)[0];
    s_big[2 * threadIdx.x + 1] = big.rec(threadIdx.x)[1];
  }
  for (uint32_t it = 0; it < npar; ++it) {
    const HeavyTable t(hvy, it);
    heavy_load_layout(t, s_rbase, s_rsh);
    __syncthreads();
    const uint32_t nd0 = s_rbase[kHvyRows];
    for (uint32_t d0 = blk; d0 < nd0; d0 += nblk) {
      const uint32_t a = t.st[d0], b = t.st[d0 + 1];
      if (a == b) {  // (its count word still holds the scatter's cursor)
        if (threadIdx.x == 0) t.ucnt[d0] = 0u;
        continue;
      }
      const uint32_t r = heavy_row(s_rbase, d0);
      const uint32_t sh = s_rsh[r];
      const uint32_t k0 = (r << colbits) + ((d0 - s_rbase[r]) << sh);
      uint32_t bi = nbig;
      for (uint32_t i = 0; i < nbig; ++i)
        if (s_big[2 * i] == it && s_big[2 * i + 1] == d0) bi = i;
      uint32_t U;
      if (bi < nbig) {  // summed already: its accumulated sums carried once more
        const unsigned long long* const glo = big.lo(bi);
        const unsigned long long* const ghi = big.hi(bi);
        const unsigned long long* const gtop = big.top(bi);
        const uint32_t* const gocc = big.occ(bi);
        for (int h = threadIdx.x; h < kLeafKeys; h += kHeavyThreads) {
          if (!gocc[h]) continue;
          sm.lo[h] = glo[h];
          sm.hi[h] = (long long)ghi[h];
          sm.top[h] = (long long)gtop[h];
          sm.occ[h] = 1;
        }
        __syncthreads();
        heavy_normalise(sm);
        __syncthreads();
        U = heavy_leaf_emit<V, RES>(sm, k0, F, colbits, tcol + a, aval + a, RES ? tres + a : nullptr, 0);
      } else {
        U = heavy_range<V, RES>(sm, ikey, ival, akey, aval, a, b, k0, 1u << sh, F, colbits, tcol + a, aval + a,
                                RES ? tres + a : nullptr, 0);
      }
      if (threadIdx.x == 0) t.ucnt[d0] = U;
    }
    __syncthreads();  // (the next layout overwrites this one)
  }
}

// last index d in [0, n) with off[d] <= f (off nondecreasing, off[0] <= f)
template <typename P>
__device__ __forceinline__ uint32_t heavy_find(P off, uint32_t n, uint32_t f) {
  uint32_t lo = 0;
  while (n > 1) {
    const uint32_t half = n >> 1;
    if (off[lo + half] <= f) lo += half;
    n -= half;
  }
  return lo;
}

constexpr uint32_t kFinalWave = 4096;  // entries one wavefront of k_final copies
constexpr uint32_t kFinalHeavyGrid = 256;  // workgroups of k_final copying heavy sub-buckets

// Per sub-bucket of the table, its ranges' entry counts replaced by their
// offsets (k_final gathers the entries from the ranges through them), the row offsets
// within the sub-bucket and its entry count.  A sub-bucket of at most kFinalWave entries,
// which k_final copies as one run from its first pair's place, has them moved there: each
// thread reads its entries, and writes them after a barrier.
constexpr int kFinishThreads = kHeavyThreads;
template <typename V, bool RES>
__device__ void heavy_finish(unsigned char* smem, const HeavyArgs<V>& A, uint32_t it) {
  uint32_t* const s_off = (uint32_t*)smem;      // [kHvyDigits]
  uint32_t* const s_scan = s_off + kHvyDigits;  // [kFinishThreads / 64 + 1]
  if (it >= A.npar) return;
  uint32_t *const akey = A.akey, *const rowoff = A.rowoff, *const usub = A.usub;
  V *const aval = A.aval, *const tres = A.tres;
  const int s2 = A.s2;
  const int64_t n_node = A.n_node;
  const HeavyTable t(A.hvy, it);
  const uint32_t nd0 = t.meta[0];
  const int64_t g = A.ov_list[it];
  const uint32_t beg = A.sbb[g];
  for (uint32_t d = threadIdx.x; d < nd0; d += kFinishThreads) s_off[d] = t.ucnt[d];
  __syncthreads();
  const uint32_t U = block_scan_array(s_off, (int)nd0, s_scan);  // (ends with a barrier)
  for (uint32_t d = threadIdx.x; d < nd0; d += kFinishThreads) t.ucnt[d] = s_off[d];
  int32_t* const tcol = (int32_t*)akey;
  if (U <= kFinalWave) {
    constexpr int PER = kFinalWave / kFinishThreads;
    int32_t c[PER];
    V v[PER], e[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const uint32_t f = j * kFinishThreads + threadIdx.x;
      if (f >= U) continue;
      const uint32_t d = heavy_find(s_off, nd0, f);
      const uint32_t src = t.st[d] + (f - s_off[d]);
      c[j] = tcol[src];
      v[j] = aval[src];
      if constexpr (RES) e[j] = tres[src];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const uint32_t f = j * kFinishThreads + threadIdx.x;
      if (f >= U) continue;
      tcol[beg + f] = c[j];
      aval[beg + f] = v[j];
      if constexpr (RES) tres[beg + f] = e[j];
    }
  }
  // a row's entries start where its first digit's do
  const int64_t r0 = g << s2;
  const int R = (int)min((int64_t)1 << s2, n_node - r0);
  for (int r = threadIdx.x; r < R; r += kFinishThreads) {
    const uint32_t d = t.rbase[r];
    rowoff[r0 + r] = d < nd0 ? s_off[d] : U;
  }
  if (threadIdx.x == 0) usub[g] = U;
}

// A build of at most kHeavySplitPairs pairs, in the one launch that it makes: each of the first
// kHeavyPar listed sub-buckets is reduced by a team of workgroups, with no workgroup waiting
// for another.  Every member works out the digit layout and the digits' pair counts itself
// (two reads of at most 2^16 keys); a digit's member then sums it straight from the
// unpartitioned pairs, keeping those of the digit, and writes its entries where the digit's
// pairs would start.  The last member to finish turns the entry counts into offsets
// (heavy_finish).  One workgroup for a whole sub-bucket (heavy_rest) took 5 us for each of the
// 264 or more leaves of a fan's: 500 tetrahedra around a node 0.78 ms in all, ten fans of 650
// 1.7 ms.
template <typename V, bool RES>
__device__ void heavy_team(unsigned char* smem, const HeavyArgs<V>& A, uint32_t blk, uint32_t nblk) {
  const HeavySmem sm(smem);
  // (the words of heavy_split, which a team does not use)
  uint32_t* const s_start = sm.hist;                    // [kHvyDigits + 1] pairs before each digit
  uint32_t* const s_rbase = s_start + kHvyDigits + 1;   // [kHvyRows + 1]
  uint32_t* const s_rsh = s_rbase + kHvyRows + 1;       // [kHvyRows]
  uint32_t* const s_rows = s_rsh + kHvyRows;            // [kHvyRows]
  static_assert(kHvyDigits + 1 + 3 * kHvyRows + 1 <= kDigits + 2 * (kDigits + 1), "a team's words fit");
  __shared__ uint32_t s_last;
  const uint32_t team = nblk / A.npar, it = blk % A.npar, member = blk / A.npar;
  if (member >= team) return;
  const int colbits = A.colbits;
  const uint32_t g = A.ov_list[it], beg = A.sbb[g], end = A.sbb[g + 1];
  const HeavyTable t(A.hvy, it);
  for (int h = threadIdx.x; h < kLeafKeys; h += kHeavyThreads) {
    sm.lo[h] = 0ull;
    sm.hi[h] = 0ll;
    sm.top[h] = 0ll;
  }
  if (threadIdx.x < kLeafKeys / 4) ((uint32_t*)sm.occ)[threadIdx.x] = 0u;
  for (int d = threadIdx.x; d <= kHvyDigits; d += kHeavyThreads) s_start[d] = 0u;
  if (threadIdx.x < kHvyRows) s_rows[threadIdx.x] = 0u;
  __syncthreads();
  heavy_count(A.ikey, beg, end, s_rows, [&](uint32_t k) { return k >> colbits; });
  __syncthreads();
  heavy_layout(t, s_rows, end - beg, colbits, member == 0, s_rbase, s_rsh, sm.scan);
  const uint32_t nd = s_rbase[kHvyRows];
  heavy_count(A.ikey, beg, end, s_start, [&](uint32_t k) { return heavy_digit(k, colbits, s_rbase, s_rsh); });
  __syncthreads();
  block_scan_array(s_start, (int)nd + 1, sm.scan);  // (ends with a barrier)
  if (member == 0)
    for (uint32_t d = threadIdx.x; d <= nd; d += kHeavyThreads) t.st[d] = beg + s_start[d];
  int32_t* const tcol = (int32_t*)A.akey;
  for (uint32_t d = member; d < nd; d += team) {
    const uint32_t a = beg + s_start[d];
    uint32_t U = 0;
    if (s_start[d + 1] > s_start[d]) {
      const uint32_t r = heavy_row(s_rbase, d), sh = s_rsh[r], w = 1u << sh;
      const uint32_t k0 = (r << colbits) + ((d - s_rbase[r]) << sh);
      // leaves of the digit (one, unless the mesh has very many nodes), from its keys found next
      for (uint32_t at = 0; at < w;) {
        if (w > (uint32_t)kLeafKeys) {
          uint32_t mn = w;
          heavy_stream<false>(A.ikey, A.ival, beg, end, [&](uint32_t k, V, bool ok) {
            const uint32_t x = k - k0;
            mn = ok && x >= at && x < mn ? x : mn;
          });
          if (threadIdx.x == 0) sm.misc[0] = w;
          __syncthreads();
          if (mn < w) atomicMin(&sm.misc[0], mn);
          __syncthreads();
          at = sm.misc[0];
          __syncthreads();
          if (at >= w) break;
        }
        const uint32_t n = w - at < (uint32_t)kLeafKeys ? w - at : (uint32_t)kLeafKeys;
        heavy_leaf_sum<V, true>(sm, A.ikey, A.ival, beg, end, k0 + at, A.F, n);
        U += heavy_leaf_emit<V, RES>(sm, k0 + at, A.F, colbits, tcol + a, A.aval + a, RES ? A.tres + a : nullptr, U);
        at += n;
      }
    }
    if (threadIdx.x == 0) t.ucnt[d] = U;
  }
  __threadfence();  // this thread's entries and counts before the arrival
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomicAdd(&t.meta[1], 1u) == team - 1 ? 1u : 0u;
  __syncthreads();
  if (!s_last) return;
  __threadfence();
  heavy_finish<V, RES>(smem, A, it);
}

// The sub-buckets listed by pass 3, one kernel per phase; with none listed every workgroup
// returns at once.  At most `par` of them are split by the whole device; a build of at most
// 2^16 pairs launches one phase alone, whose workgroups form teams (heavy_team).  The others'
// phases are separate launches: one kernel
// that hands their workgroups out as tickets in order, each phase waiting for the one
// before, did not finish on a batch with two heavy rows.
enum HeavyPhase { kHeavyRowsPhase, kHeavyHistPhase, kHeavyScatterPhase, kHeavyBigPhase,
                  kHeavyRangesPhase, kHeavyFinishPhase, kHeavyTeamPhase };
constexpr int64_t kHeavySplitPairs = 1 << 16;
constexpr int kScanHere = 16384;  // sub-buckets whose entry counts the last phase scans itself

__device__ __forceinline__ void scan_counts(uint32_t* usub, int n, uint32_t* ubase, int64_t* nnz,
                                            uint32_t* s_scan) {
  constexpr int PER = 4;
  uint32_t carry = 0;
  for (int b0 = 0; b0 < n; b0 += PER * (int)blockDim.x) {
    const int b = b0 + PER * threadIdx.x;
    uint32_t v[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      v[i] = b + i < n ? __hip_atomic_load(&usub[b + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
      sum += v[i];
    }
    uint32_t total;
    uint32_t off = carry + block_scan_u32(sum, s_scan, &total);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (b + i < n) ubase[b + i] = off;
      off += v[i];
    }
    carry += total;
  }
  if (threadIdx.x == 0) {
    ubase[n] = carry;
    *nnz = carry;
  }
}

// SCAN (the last launch): the entry counts of few sub-buckets (ubase not null) scanned too,
// by the last workgroup to finish, or by the first if none is listed.
template <typename V, bool RES, HeavyPhase PHASE, bool SCAN = false>
__global__ __launch_bounds__(kHeavyThreads) void k_heavy(HeavyArgs<V> A, const uint32_t* __restrict__ emax,
                                                       const uint32_t* __restrict__ n_over, uint32_t par,
                                                       uint32_t* done, uint32_t* ubase, int64_t* nnz) {
  extern __shared__ __align__(16) unsigned char smem[];
  A.n_over = *n_over;
  if (!SCAN && A.n_over == 0) return;
  const int taken = A.sub.pick(), nsub = A.sub.nsub[taken];
  A.s2 = A.sub.s2[taken];
  if (A.n_over == 0) {
    if constexpr (SCAN)
      if (ubase && blockIdx.x == 0) scan_counts(A.usub, nsub, ubase, nnz, (uint32_t*)smem);
    return;
  }
  A.npar = A.n_over < par ? A.n_over : par;
  A.F = 1117 - (int)*emax;
  const uint32_t blk = blockIdx.x, nblk = gridDim.x;
  if constexpr (PHASE == kHeavyRowsPhase) heavy_rows<V>(smem, A, blk, nblk);
  if constexpr (PHASE == kHeavyHistPhase) heavy_hist<V>(smem, A, blk, nblk);
  if constexpr (PHASE == kHeavyScatterPhase) heavy_scatter<V>(smem, A, blk, nblk);
  if constexpr (PHASE == kHeavyBigPhase) heavy_bigleaf<V>(smem, A, blk, nblk);
  if constexpr (PHASE == kHeavyRangesPhase) {
    heavy_ranges<V, RES>(smem, A, blk, nblk);
    __syncthreads();
    heavy_rest<V, RES>(smem, A, blk, nblk);
  }
  if constexpr (PHASE == kHeavyFinishPhase) heavy_finish<V, RES>(smem, A, blk);
  if constexpr (PHASE == kHeavyTeamPhase) {
    heavy_team<V, RES>(smem, A, blk, nblk);
    __syncthreads();
    heavy_rest<V, RES>(smem, A, blk, nblk);
  }
  if constexpr (SCAN) {
    if (!ubase) return;
    __shared__ uint32_t s_last;
    __threadfence();  // this thread's counts before the arrival
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(done, 1u) == gridDim.x - 1 ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    scan_counts(A.usub, nsub, ubase, nnz, (uint32_t*)smem);
  }
}

// ------------------------------------------------------------------ many entry counts
// ubase[0 .. nsub] = exclusive scan of usub over the sub-buckets of the way taken, in two
// kernels (chunk sums, then each chunk with the sums before it)
static __global__ __launch_bounds__(kScanThreads) void k_scan_partials(const int32_t* __restrict__ usub,
                                                                       const SubBuckets sub,
                                                                       int32_t* __restrict__ part) {
  const int64_t n = sub.nsub[sub.pick()];
  if ((int64_t)blockIdx.x * kScanChunk < n) scan_chunk_sum(usub, n, part);
}

static __global__ __launch_bounds__(kScanThreads) void k_scan_down(const int32_t* __restrict__ usub,
                                                                   const SubBuckets sub,
                                                                   const int32_t* __restrict__ part,
                                                                   int32_t* __restrict__ ubase,
                                                                   int64_t* __restrict__ nnz) {
  const int64_t n = sub.nsub[sub.pick()];
  if ((int64_t)blockIdx.x * kScanChunk < n) scan_chunk_down(usub, n, part, ubase, nullptr, nnz);
}

// ------------------------------------------------------------------------- final
// A batch of meshes built as one block-diagonal matrix (kb_batch.hpp): each mesh's rows
// and columns are written in its own numbering.  node_off null: one mesh.
struct BatchRows {
  const int64_t* node_off;  // [n_mesh + 1]
  int64_t n_mesh;
  const uint32_t* flags;    // set: the offsets failed their check and are not read
};

// the last mesh m with node_off[m] <= i, by a whole wave: 64 candidates at a time
__device__ __forceinline__ int64_t wave_owner(const int64_t* __restrict__ off, int64_t n, int64_t i) {
  const int lane = threadIdx.x & 63;
  int64_t lo = 0;
  while (n > 1) {
    const int64_t step = (n + 63) / 64, at = lo + lane * step;
    const int k = __popcll(__ballot(lane * step < n && off[at] <= i)) - 1;  // (off[lo] <= i)
    lo += k * step;
    n = n - k * step < step ? n - k * step : step;
  }
  return lo;
}

// position of node i's first entry in the union matrix (i = n_node: the number of entries)
__device__ __forceinline__ int64_t row_start(const uint32_t* __restrict__ ubase, const uint32_t* __restrict__ rowoff,
                                             int s2, int64_t n_node, int64_t nsub, int64_t i) {
  return i >= n_node ? (int64_t)ubase[nsub] : (int64_t)ubase[i >> s2] + rowoff[i];
}

// The entries of the sub-buckets that one wavefront does not copy (more than kFinalWave:
// only a heavy sub-bucket, listed by pass 3, can hold more than a pass-3 table), copied
// by nblk workgroups in chunks of 1024: from the sub-bucket's first pair's place on, or,
// for the first `par` listed, from the digit ranges that hold them (entry f of the
// range d whose entry offset is the last at or below f, at the range's start plus f minus
// that offset).  With GROUPED each entry's row is found by a binary search of the
// sub-bucket's row offsets.
template <typename V, bool GROUPED, bool BATCH>
__device__ __forceinline__ void final_heavy(const uint32_t* __restrict__ sbb, const uint32_t* __restrict__ ubase,
                                            const int32_t* __restrict__ tcol, const V* __restrict__ tval,
                                            const V* __restrict__ tres, const uint32_t* __restrict__ rowoff, int s2,
                                            int64_t n_node, int64_t nsub, const uint32_t* __restrict__ ov_list,
                                            const uint32_t* __restrict__ ov_count, const uint32_t* __restrict__ hvy,
                                            int32_t* __restrict__ col_idx, V* __restrict__ vals, V* __restrict__ res,
                                            int32_t* __restrict__ rows, int64_t cap, const BatchRows& batch,
                                            uint32_t par, uint32_t blk, uint32_t nblk) {
  __shared__ uint32_t s_off[kHvyDigits];  // entry offsets of the ranges
  const uint32_t n_over = *ov_count;
  if (n_over == 0 || (int64_t)ubase[nsub] > cap) return;
  for (uint32_t it = 0; it < n_over; ++it) {
    const int64_t g = ov_list[it];
    const uint32_t base = ubase[g], U = ubase[g + 1] - base;
    if (U <= kFinalWave) continue;
    const uint32_t beg = sbb[g];
    const bool ranged = it < par;
    const HeavyTable t(const_cast<uint32_t*>(hvy), ranged ? it : 0u);
    const uint32_t nd0 = ranged ? t.meta[0] : 0u;
    if (ranged) {
      __syncthreads();  // (the previous sub-bucket's offsets are no longer read)
      for (uint32_t d = threadIdx.x; d < nd0; d += blockDim.x) s_off[d] = t.ucnt[d];
      __syncthreads();
    }
    const int64_t r0 = g << s2;
    const int R = (int)min((int64_t)1 << s2, n_node - r0);
    for (uint32_t c = blk * 1024u; c < U; c += nblk * 1024u) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t f = c + j * 256 + threadIdx.x;
        if (f >= U) continue;
        uint32_t src = beg + f;
        if (ranged) {
          const uint32_t d = heavy_find(s_off, nd0, f);
          src = t.st[d] + (f - s_off[d]);
        }
        int32_t col = tcol[src];
        vals[base + f] = tval[src];
        if constexpr (GROUPED || BATCH) {
          int lo = 0, hi = R - 1;  // last row whose first entry is at or before f
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (rowoff[r0 + mid] <= f)
              lo = mid;
            else
              hi = mid - 1;
          }
          if constexpr (GROUPED) {
            res[base + f] = tres[src];
            rows[base + f] = (int32_t)(r0 + lo);
          } else {  // the row's mesh: the last with node_off <= row
            int64_t m = 0, n = batch.n_mesh;
            while (n > 1) {
              const int64_t half = n >> 1;
              if (batch.node_off[m + half] <= r0 + lo) m += half;
              n -= half;
            }
            col -= (int32_t)batch.node_off[m];
          }
        }
        col_idx[base + f] = col;
      }
    }
  }
}

// One wavefront per sub-bucket g: its entries copied to their final place ubase[g],
// its rows' row_ptr = ubase[g] + local row offset.
// GROUPED (running sums of a grouped build): also each entry's residual (tres -> res)
// and its row (rows), the form in which the next group's pass reads them back.
// BATCH: columns and row pointers of each mesh in its own numbering, as they are copied (a
// second pass over the columns took 0.96 of the 256-brick batch's 7.3 ms).
// The last kFinalHeavyGrid workgroups copy the larger sub-buckets (final_heavy).
template <typename V, bool GROUPED = false, bool BATCH = false>
__global__ __launch_bounds__(256) void k_final(const uint32_t* __restrict__ sbb, const uint32_t* __restrict__ ubase,
                                               const int32_t* __restrict__ tcol, const V* __restrict__ tval,
                                               const V* __restrict__ tres, const uint32_t* __restrict__ rowoff,
                                               const SubBuckets sub, int64_t n_node, int32_t* __restrict__ row_ptr,
                                               int32_t* __restrict__ col_idx, V* __restrict__ vals,
                                               V* __restrict__ res, int32_t* __restrict__ rows, int64_t cap,
                                               uint32_t* __restrict__ status, const uint32_t* __restrict__ ov_list,
                                               const uint32_t* __restrict__ ov_count,
                                               const uint32_t* __restrict__ hvy, uint32_t par, const BatchRows batch) {
  const uint32_t n_wave = gridDim.x - kFinalHeavyGrid;
  const int way = sub.pick(), s2 = sub.s2[way];
  const int64_t nsub = sub.nsub[way];
  if (BATCH && *batch.flags) {  // no element was kept: empty rows for every mesh
    const int64_t n = n_node + batch.n_mesh;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
      row_ptr[i] = 0;
    return;
  }
  if (blockIdx.x >= n_wave) {
    final_heavy<V, GROUPED, BATCH>(sbb, ubase, tcol, tval, tres, rowoff, s2, n_node, nsub, ov_list, ov_count, hvy,
                                   col_idx, vals, res, rows, cap, batch, par, blockIdx.x - n_wave, kFinalHeavyGrid);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int64_t nnz = ubase[nsub];
  const int64_t g = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
  if (g >= nsub) return;
  const uint32_t base = ubase[g], U = ubase[g + 1] - base;
  const int64_t r0 = g << s2;
  const int R = (int)min((int64_t)1 << s2, n_node - r0);
  if constexpr (BATCH) {
    if (nnz > cap && g == 0 && lane == 0) raise_flag(status, KB_F_CAPACITY);
    if (R <= 0) return;
    const uint32_t src = sbb[g];
    const bool copy = nnz <= cap && U <= kFinalWave;  // (larger: a heavy sub-bucket, final_heavy)
    // the sub-bucket's rows mesh by mesh
    int64_t m = wave_owner(batch.node_off, batch.n_mesh, r0);
    for (int64_t a = r0; a < r0 + R; ++m) {
      const int64_t n0 = batch.node_off[m], n1 = batch.node_off[m + 1];
      const int64_t b = n1 < r0 + R ? n1 : r0 + R;
      if (b <= a) continue;  // (a mesh without nodes)
      const uint32_t f0 = rowoff[a], f1 = b < r0 + R ? rowoff[b] : U;
      if (copy)
        for (uint32_t f = f0 + lane; f < f1; f += 64) {
          col_idx[base + f] = tcol[src + f] - (int32_t)n0;
          vals[base + f] = tval[src + f];
        }
      const int64_t first = row_start(ubase, rowoff, s2, n_node, nsub, n0);
      for (int64_t r = a + lane; r < b; r += 64) row_ptr[r + m] = (int32_t)(base + rowoff[r] - first);
      a = b;
    }
    return;
  }
  if (nnz <= cap && U <= kFinalWave) {  // (larger: a heavy sub-bucket, final_heavy)
    const uint32_t src = sbb[g];
    for (uint32_t f = lane; f < U; f += 64) {
      col_idx[base + f] = tcol[src + f];
      vals[base + f] = tval[src + f];
      if constexpr (GROUPED) res[base + f] = tres[src + f];
    }
    if constexpr (GROUPED) {
      for (int r = lane; r < R; r += 64) {
        const uint32_t k1 = r + 1 < R ? rowoff[r0 + r + 1] : U;
        for (uint32_t k = rowoff[r0 + r]; k < k1; ++k) rows[base + k] = (int32_t)(r0 + r);
      }
    }
  } else if (nnz > cap && g == 0 && lane == 0) {
    raise_flag(status, KB_F_CAPACITY);
  }
  for (int r = lane; r < R; r += 64) row_ptr[r0 + r] = (int32_t)(base + rowoff[r0 + r]);
  if (g == nsub - 1 && lane == 0) row_ptr[n_node] = (int32_t)nnz;
}

}  // namespace kb
