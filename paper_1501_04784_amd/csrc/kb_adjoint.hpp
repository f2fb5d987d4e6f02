// kb_adjoint.hpp -- adjoint of the construction: gradients of L = sum W_ij K_ij.
//
// Not part of the paper; derived from Eq. 7-9.  Per element, with S the symmetric
// nen x nen matrix S_aa = W(E_a, E_a), S_ab = S_ba = W(pair a, b) / 2 (so the element's
// share of L is S : k_e), A = adj(J), G = A dN (so B = G / |J|) and P = G S G^T at
// each integration point (weight w):
//   dL/dc_e  = sum_q w tr(P) / |J|                        (k_e is linear in c),
//   dL/dX_a += c sum_q w / |J|^2 (tr(P) G_a - 2 P G_a)    (G_a = column a of G),
// the second from d|J| = |J| tr(J^{-1} dJ), d(J^{-1}) = -J^{-1} dJ J^{-1}, dJ = dN dX;
// it is c w |J| B^T (tr(M) I - 2 M) with M = B S B^T, written in terms of G.
// All arithmetic is FP64.
//
// Node gradients are sums over the elements at each node.  They are accumulated as the
// same exact fixed-point integers as the assembly (scale from the largest exponent of
// all element contributions; two 64-bit integer chunks per value), so the result does not
// depend on the order of the additions: bitwise deterministic, and exact.  The corners are
// partitioned by node bucket first, so each bucket's sums are formed in one workgroup's LDS:
//   k_adjoint_count   each corner's place within its bucket, and the bucket starts
//   k_adjoint_elems   the gradients, one 32-byte record per corner at its place
//   k_adjoint_reduce  a bucket's records summed, rounded once, written
// Adding each workgroup's node sums to global accumulators instead (64-bit atomics: 27
// G/s, and a node's six words from every workgroup that touches it) took 278 us of the
// 64^3 bricks' 489 us.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kb_assemble.hpp"
#include "kb_element.hpp"
#include "kb_kernels.hpp"
#include "kbuild.h"

namespace kb {

// position of (row, col) in a lower CSR with ascending columns, or -1.  The search is
// confined to [0, nnz), the length of col_idx: a row range outside it (a row pointer
// that does not belong to this col_idx) also gives -1.
__device__ __forceinline__ int64_t csr_position(const int32_t* __restrict__ row_ptr,
                                                const int32_t* __restrict__ col_idx, int64_t nnz, int32_t row,
                                                int32_t col) {
  int64_t lo = row_ptr[row], hi = (int64_t)row_ptr[row + 1] - 1;
  if (lo < 0 || hi >= nnz || lo > hi + 1) return -1;
  while (lo <= hi) {
    const int64_t mid = (lo + hi) >> 1;
    const int32_t c = col_idx[mid];
    if (c == col) return mid;
    if (c < col)
      lo = mid + 1;
    else
      hi = mid - 1;
  }
  return -1;
}

// one integration point: P = G S G^T from G (3 x NEN) and the lower triangle of S;
// adds w tr(P) / det to *gc and c w / det^2 (tr(P) G_a - 2 P G_a) to D[a]
template <int NEN, typename SMat>
__device__ __forceinline__ void adjoint_point(const double (&G)[3][NEN], const SMat& S,
                                              double det, double w, double c, double* gc, double (&D)[NEN][3]) {
  // T = S G^T (NEN x 3), then P = G T (3 x 3)
  double P[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll
  for (int a = 0; a < NEN; ++a) {
    double t0 = 0.0, t1 = 0.0, t2 = 0.0;
#pragma unroll
    for (int b = 0; b < NEN; ++b) {
      const double s = a >= b ? S[lidx(a, b)] : S[lidx(b, a)];
      t0 += s * G[0][b];
      t1 += s * G[1][b];
      t2 += s * G[2][b];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      P[i][0] += G[i][a] * t0;
      P[i][1] += G[i][a] * t1;
      P[i][2] += G[i][a] * t2;
    }
  }
  const double tr = P[0][0] + P[1][1] + P[2][2];
  const double inv = 1.0 / det;
  *gc += w * tr * inv;
  const double f = c * w * inv * inv;
#pragma unroll
  for (int a = 0; a < NEN; ++a)
#pragma unroll
    for (int i = 0; i < 3; ++i)
      D[a][i] += f * (tr * G[i][a] - 2.0 * (P[i][0] * G[0][a] + P[i][1] * G[1][a] + P[i][2] * G[2][a]));
}

// ---- corners by node bucket (node >> bits) ------------------------------------------
// at least 2^6 nodes a bucket, at most 2^10 (48 KB of LDS sums); about 512 buckets between
constexpr int kAdjMinBits = 6, kAdjMaxBits = 10, kAdjBuckets = 512;
constexpr int kAdjArray = 8192;           // buckets counted in an LDS array, else in the slot hash
constexpr int kAdjPer = 4;                // elements per lane of k_adjoint_count
// records per workgroup of k_adjoint_reduce at most: above the 24 a node of a box's tetrahedra
// times the nodes of a bucket, and below the kRound that sums inside 64 bits
constexpr uint32_t kAdjChunk = 32768;
static_assert(kAdjChunk <= kRound, "a chunk's sums stay inside 64 bits");

constexpr int kAdjAcc = 9;                // global words per node: low, high and top sums of x, y, z
constexpr int kAdjHot = 32;               // lanes of a wave with one node from which they are combined

constexpr int kAdjElemThreads = 128;

struct AdjointRecord {
  double g[3];
  uint64_t node;  // within its bucket
};

// head: [0] largest exponent, [1] workgroups done, [2] buckets of more than kAdjChunk
// records, [3] workgroups they need beyond one each.  big: (bucket, first of those
// workgroups, workgroups done) per such bucket.
static __global__ __launch_bounds__(256) void k_adjoint_begin(uint32_t* __restrict__ status,
                                                              uint32_t* __restrict__ head,
                                                              uint32_t* __restrict__ cnt, int64_t nb) {
  if (blockIdx.x == 0) {
    if (threadIdx.x < KB_STATUS_WORDS) status[threadIdx.x] = 0u;
    if (threadIdx.x < 4) head[threadIdx.x] = 0u;
  }
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nb; i += (int64_t)gridDim.x * blockDim.x)
    cnt[i] = 0u;
}

// rel[e * NEN + a]: corner a's place within its node's bucket.  A workgroup counts its
// elements' corners per bucket in LDS (one atomic per run of an element's corners in one
// bucket), takes its places in each bucket with one global atomic, whose result is where
// its corners start.  The last workgroup turns the counts into the bucket starts
// start[0 .. nb] and lists the buckets of more than kAdjChunk corners.  An element that
// fails its connectivity check has no places.
template <int NEN>
__global__ __launch_bounds__(256) void k_adjoint_count(const int32_t* __restrict__ conn, int64_t n_elem,
                                                       int64_t n_node, int bits, int nb, uint32_t* cnt,
                                                       uint32_t* __restrict__ start, uint32_t* __restrict__ rel,
                                                       uint32_t* head, uint32_t* __restrict__ big) {
  extern __shared__ uint32_t s_w[];  // counts, then bases (and keys of the hash)
  const bool array = nb <= kAdjArray;
  TileSlots<true> sl(s_w, s_w + kSlotsHash, array ? kDirect : kAsk, 0, 0, bits, nb);
  sl.clear(blockDim.x);
  __syncthreads();
  const int64_t e0 = blockIdx.x * (int64_t)blockDim.x * kAdjPer;
  uint32_t q[kAdjPer][NEN];
  bool ok[kAdjPer];
#pragma unroll
  for (int u = 0; u < kAdjPer; ++u) {
    const int64_t e = e0 + u * blockDim.x + threadIdx.x;
    ok[u] = false;
    if (e >= n_elem) continue;
    int32_t E[NEN];
    load_conn<NEN>(conn, e, E);
    ok[u] = check_conn<NEN>(E, n_node) == 0;
    if (!ok[u]) continue;
    const int one[NEN] = {};  // (reserve_rows takes rank + 1 places a row: one each)
    reserve_rows<NEN, 0>(sl, E, one, q[u]);
#pragma unroll
    for (int a = 0; a < NEN; ++a)  // no slot: the place taken at once
      if (q[u][a] == kNoSlot) rel[e * NEN + a] = atomicAdd(&cnt[E[a] >> bits], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < sl.n; b += blockDim.x) {
    const uint32_t c = sl.cnt[b];
    if (c) sl.cnt[b] = atomicAdd(&cnt[sl.hash ? sl.key[b] : (uint32_t)b], c);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kAdjPer; ++u) {
    const int64_t e = e0 + u * blockDim.x + threadIdx.x;
    if (!ok[u]) continue;
#pragma unroll
    for (int a = 0; a < NEN; ++a)
      if (q[u][a] != kNoSlot) rel[e * NEN + a] = sl.cnt[q[u][a] >> 16] + (q[u][a] & 0xFFFFu);
  }
  // bucket starts, and the buckets that need several workgroups
  __shared__ uint32_t s_scan[8], s_last;
  __syncthreads();  // (the additions to cnt have returned their results: last_block_starts)
  if (threadIdx.x == 0) s_last = atomicAdd(&head[1], 1u) == gridDim.x - 1 ? 1u : 0u;
  __syncthreads();
  if (!s_last) return;
  constexpr int PER = 4;
  uint32_t carry = 0;
  for (int b0 = 0; b0 < nb; b0 += PER * blockDim.x) {
    const int b = b0 + PER * threadIdx.x;
    uint32_t v[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      v[i] = b + i < nb ? __hip_atomic_load(&cnt[b + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
      sum += v[i];
    }
    uint32_t total;
    uint32_t off = carry + block_scan_u32(sum, s_scan, &total);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (b + i < nb) start[b + i] = off;
      off += v[i];
      if (v[i] > kAdjChunk) {
        uint32_t* const w = big + 3 * atomicAdd(&head[2], 1u);
        w[0] = (uint32_t)(b + i);
        w[1] = atomicAdd(&head[3], (v[i] - 1) / kAdjChunk);
        w[2] = 0u;
      }
    }
    carry += total;
  }
  if (threadIdx.x == 0) start[nb] = carry;
}

// The weights of an element's pairs as S (off-diagonal pairs at half weight).  All
// off-diagonal positions are searched for in lockstep, one step of every search per
// iteration, so the loads of a step are in flight together (one search after the other
// waited for about 100 loads in a row: 195 us for the 64^3 bricks).  A diagonal entry
// is the last of its row.  Returns KB_F_INDEX if an entry is missing (its weight is 0).
template <int NEN, typename SMat>
__device__ __forceinline__ uint32_t pair_weights(const int32_t* __restrict__ row_ptr,
                                                 const int32_t* __restrict__ col_idx, int64_t nnz,
                                                 const double* __restrict__ w, const int32_t (&E)[NEN],
                                                 SMat& S) {
  constexpr int NP = NEN * (NEN - 1) / 2;
  uint32_t f = 0;
  if (nnz == 0) {
#pragma unroll
    for (int p = 0; p < ElemTraits<NEN>::T; ++p) S[p] = 0.0;
    return KB_F_INDEX;
  }
  // each row's entries [lo, lo + n); n = 0 for a range outside [0, nnz)
  uint32_t lo[NEN], n[NEN], longest = 0;
#pragma unroll
  for (int a = 0; a < NEN; ++a) {
    const int64_t l = row_ptr[E[a]], h = row_ptr[E[a] + 1];
    const bool ok = l >= 0 && h <= nnz && l < h;
    lo[a] = ok ? (uint32_t)l : 0u;
    n[a] = ok ? (uint32_t)(h - l) : 0u;
    longest = n[a] > longest ? n[a] : longest;
  }
  uint32_t at[NP], len[NP];
  bool none[NP];
#pragma unroll
  for (int a = 1; a < NEN; ++a)
#pragma unroll
    for (int b = 0; b < a; ++b) {
      const int p = a * (a - 1) / 2 + b;
      const bool up = E[a] > E[b];
      at[p] = up ? lo[a] : lo[b];
      len[p] = up ? n[a] : n[b];
      none[p] = len[p] == 0;
    }
  // the last entry at or before the column, from `len` candidates
  for (uint32_t m = longest; m > 1; m -= m >> 1) {
    int32_t c[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) c[p] = col_idx[at[p] + (len[p] >> 1)];
#pragma unroll
    for (int a = 1; a < NEN; ++a)
#pragma unroll
      for (int b = 0; b < a; ++b) {
        const int p = a * (a - 1) / 2 + b;
        const uint32_t half = len[p] >> 1;
        at[p] += c[p] <= (E[a] > E[b] ? E[b] : E[a]) ? half : 0u;
        len[p] -= half;
      }
  }
#pragma unroll
  for (int a = 1; a < NEN; ++a)
#pragma unroll
    for (int b = 0; b < a; ++b) {
      const int p = a * (a - 1) / 2 + b;
      const bool found = !none[p] && col_idx[at[p]] == (E[a] > E[b] ? E[b] : E[a]);
      const double v = w[at[p]];
      S[lidx(a, b)] = found ? 0.5 * v : 0.0;
      f |= found ? 0u : KB_F_INDEX;
    }
#pragma unroll
  for (int a = 0; a < NEN; ++a) {
    int64_t k = (int64_t)lo[a] + n[a] - 1;
    if (n[a] == 0)
      k = -1;
    else if (col_idx[k] != E[a])  // (a pattern with columns past the diagonal)
      k = csr_position(row_ptr, col_idx, nnz, E[a], E[a]);
    S[lidx(a, a)] = k < 0 ? 0.0 : w[k];
    f |= k < 0 ? KB_F_INDEX : 0u;
  }
  return f;
}

// Per element (one per lane): dL/dc_e into grad_coef, the nen x 3 coordinate gradients as
// records at their corners' places, the largest exponent of those into head[0].
template <int NEN>
__global__ __launch_bounds__(kAdjElemThreads) void k_adjoint_elems(const int32_t* __restrict__ conn,
                                                       const double* __restrict__ coords,
                                                       const double* __restrict__ coef, int64_t n_elem,
                                                       int64_t n_node, const int32_t* __restrict__ row_ptr,
                                                       const int32_t* __restrict__ col_idx, int64_t nnz,
                                                       const double* __restrict__ w,
                                                       double* __restrict__ grad_coef, int bits,
                                                       const uint32_t* __restrict__ start,
                                                       const uint32_t* __restrict__ rel,
                                                       AdjointRecord* __restrict__ rec,
                                                       unsigned long long* __restrict__ acc,
                                                       uint32_t* __restrict__ head, const uint32_t* __restrict__ big,
                                                       uint32_t* __restrict__ status) {
  __shared__ uint32_t s_emax;
  if (threadIdx.x == 0) s_emax = 0;
  __syncthreads();
  // the global sums (kAdjAcc words a node) of the buckets that several workgroups reduce, in
  // the order of their list
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < ((int64_t)kAdjAcc * head[2]) << bits;
       j += (int64_t)gridDim.x * blockDim.x)
    acc[j] = 0ull;
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  uint32_t em = 0;
  if (e < n_elem) {
    int32_t E[NEN];
    load_conn<NEN>(conn, e, E);
    uint32_t f = check_conn<NEN>(E, n_node);
    const bool placed = f == 0;
    double D[NEN][3];
#pragma unroll
    for (int a = 0; a < NEN; ++a) D[a][0] = D[a][1] = D[a][2] = 0.0;
    double gc = 0.0;
    if (!f) {
      double S[ElemTraits<NEN>::T];
      f |= pair_weights<NEN>(row_ptr, col_idx, nnz, w, E, S);
      double X[NEN][3];
      double X0[3] = {coords[(int64_t)E[0] * 3], coords[(int64_t)E[0] * 3 + 1], coords[(int64_t)E[0] * 3 + 2]};
#pragma unroll
      for (int a = 0; a < NEN; ++a)
#pragma unroll
        for (int j = 0; j < 3; ++j) X[a][j] = a ? coords[(int64_t)E[a] * 3 + j] - X0[j] : 0.0;
      const double c = coef[e];
      if constexpr (NEN == 8) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          double J[3][3];
#pragma unroll
          for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
              double s = 0.0;
#pragma unroll
              for (int a = 1; a < 8; ++a) s += hex_dN(q, i, a) * X[a][j];
              J[i][j] = s;
            }
          double A[3][3];
          const double det = adjugate(J, A);
          if (!(det > 0.0)) f |= KB_F_INVERTED;
          double G[3][8];
#pragma unroll
          for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int a = 0; a < 8; ++a) G[i][a] = A[i][0] * hex_dN(q, 0, a) + A[i][1] * hex_dN(q, 1, a) +
                                                  A[i][2] * hex_dN(q, 2, a);
          adjoint_point<8>(G, S, det, 1.0, c, &gc, D);
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        double J[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int j = 0; j < 3; ++j) J[i][j] = X[i + 1][j];
        double A[3][3];
        const double det = adjugate(J, A);
        if (!(det > 0.0)) f |= KB_F_INVERTED;
        double G[3][4];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          G[i][1] = A[i][0];
          G[i][2] = A[i][1];
          G[i][3] = A[i][2];
          G[i][0] = -(A[i][0] + A[i][1] + A[i][2]);
        }
        adjoint_point<4>(G, S, det, 1.0 / 6.0, c, &gc, D);
      }
    }
    // a degenerate or inverted element, or non-finite input, gives non-finite gradients:
    // flagged, and their node contributions are dropped (the exact sums take 0 for them)
    bool finite = isfinite(gc);
#pragma unroll
    for (int a = 0; a < NEN; ++a)
#pragma unroll
      for (int j = 0; j < 3; ++j) finite = finite && isfinite(D[a][j]);
    if (!finite) f |= KB_F_NONFINITE;
    if (f) raise_flag(status, f);
    grad_coef[e] = gc;
#pragma unroll
    for (int a = 0; a < NEN; ++a)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const double v = D[a][j];
        const uint32_t ep = (uint32_t)biased_exponent(v);
        em = (ep > em && ep < 0x7FF) ? ep : em;
      }
    if (placed) {
#pragma unroll
      for (int a = 0; a < NEN; ++a)
        rec[start[E[a] >> bits] + rel[e * NEN + a]] =
            AdjointRecord{{D[a][0], D[a][1], D[a][2]}, (uint64_t)(E[a] & ((1 << bits) - 1))};
    }
  }
  if (em) atomicMax(&s_emax, em);
  __syncthreads();
  if (threadIdx.x == 0 && s_emax) atomicMax(&head[0], s_emax);
}

// A bucket's records summed per node in LDS and its nodes' gradients written: workgroup b
// takes bucket b (its first kAdjChunk records).  Further records of a larger bucket (a
// node of very many elements) go to workgroups nb, nb + 1, ...; all of that bucket's
// workgroups then add their sums to global ones, and the last to finish writes them.
// Where most lanes of a wave hold one node (a node of thousands of elements), they add to their
// own registers instead, which meet once per node: LDS atomics on one address take their turns
// (60,000 tetrahedra around a node: 335 us in all, 109 with sums by 512 corners and global
// atomics).
constexpr int kAdjThreads = 1024;
constexpr unsigned long long kMask48 = (1ull << 48) - 1;
static __global__ __launch_bounds__(kAdjThreads) void k_adjoint_reduce(
    const AdjointRecord* __restrict__ rec, const uint32_t* __restrict__ start, int64_t n_node, int bits, int nb,
    const uint32_t* __restrict__ head, uint32_t* big, unsigned long long* acc, double* __restrict__ grad_coords) {
  extern __shared__ unsigned long long s_acc[];  // [6][1 << bits]: low and high chunk sums of x, y, z
  __shared__ uint32_t s_last;
  const int N = 1 << bits, F = 1117 - (int)head[0];
  int b = blockIdx.x;
  uint32_t* entry = nullptr;  // the bucket's entry in the list of large ones
  uint32_t chunk = 0;
  const uint32_t n_big = head[2];
  if (b >= nb) {
    const uint32_t x = (uint32_t)(b - nb);
    if (x >= head[3]) return;
    for (uint32_t i = 0; i < n_big; ++i) {
      const uint32_t g = big[3 * i], f0 = big[3 * i + 1], extra = (start[g + 1] - start[g] - 1) / kAdjChunk;
      if (x >= f0 && x < f0 + extra) {
        b = (int)g;
        chunk = 1 + x - f0;
        entry = big + 3 * i;
      }
    }
  } else {
    for (uint32_t i = 0; i < n_big; ++i)
      if (big[3 * i] == (uint32_t)b) entry = big + 3 * i;
  }
  for (int h = threadIdx.x; h < 6 * N; h += kAdjThreads) s_acc[h] = 0ull;
  __syncthreads();
  const uint32_t i0 = start[b] + chunk * kAdjChunk, end = start[b + 1];
  const uint32_t i1 = end - i0 > kAdjChunk ? i0 + kAdjChunk : end;
  uint32_t kept = kEmptyKey;  // (uniform over the wave) the node that k0, k1 are sums of
  unsigned long long k0[3] = {0ull, 0ull, 0ull};
  long long k1[3] = {0ll, 0ll, 0ll};
  const int lane = threadIdx.x & 63;
  const auto flush = [&] {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
        k0[j] += __shfl_xor(k0[j], o, 64);
        k1[j] += __shfl_xor(k1[j], o, 64);
      }
      if (lane == 0) {
        atomicAdd(&s_acc[2 * j * N + (int)kept], k0[j]);
        atomicAdd(&s_acc[(2 * j + 1) * N + (int)kept], (unsigned long long)k1[j]);
      }
      k0[j] = 0ull;
      k1[j] = 0ll;
    }
  };
  for (uint32_t ib = i0; ib < i1; ib += kAdjThreads) {
    const uint32_t i = ib + threadIdx.x;
    const bool ok = i < i1;
    const AdjointRecord r = rec[ok ? i : i0];
    const uint32_t node = (uint32_t)r.node, hot = __builtin_amdgcn_readfirstlane(node);
    const bool many = __popcll(__ballot(ok && node == hot)) >= kAdjHot;  // (uniform over the wave)
    if (many && kept != hot) {
      if (kept != kEmptyKey) flush();
      kept = hot;
    }
    if (many && ok && node == hot) {  // (32 records a lane: below 2^53)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        uint64_t c0;
        int64_t c1;
        to_chunks(r.g[j], F, c0, c1);
        k0[j] += c0;
        k1[j] += c1;
      }
    } else if (ok) {
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        uint64_t c0;
        int64_t c1;
        to_chunks(r.g[j], F, c0, c1);
        if (c0) atomicAdd(&s_acc[2 * j * N + (int)node], (unsigned long long)c0);
        if (c1) atomicAdd(&s_acc[(2 * j + 1) * N + (int)node], (unsigned long long)c1);
      }
    }
  }
  if (kept != kEmptyKey) flush();
  __syncthreads();
  const int64_t n0 = (int64_t)b << bits;
  const int nn = n_node - n0 < N ? (int)(n_node - n0) : N;
  if (entry) {
    // each pair of chunk sums carried into three words, so any number of workgroups adds up
    unsigned long long* const sums = acc + (((int64_t)(entry - big) / 3 * kAdjAcc) << bits);
    for (int h = threadIdx.x; h < 3 * nn; h += kAdjThreads) {
      const int j = h / nn, i = h - j * nn;
      const unsigned long long lo = s_acc[2 * j * N + i];
      const long long hi = (long long)s_acc[(2 * j + 1) * N + i] + (long long)(lo >> 48);
      unsigned long long* const q = sums + i * kAdjAcc + 3 * j;
      if (lo & kMask48) atomicAdd(&q[0], lo & kMask48);
      if (hi) {
        atomicAdd(&q[1], (unsigned long long)hi & kMask48);
        atomicAdd(&q[2], (unsigned long long)(hi >> 48));
      }
    }
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(&entry[2], 1u) == (end - start[b] - 1) / kAdjChunk ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    for (int h = threadIdx.x; h < 3 * nn; h += kAdjThreads) {
      uint64_t q[3];
#pragma unroll
      for (int k = 0; k < 3; ++k)
        q[k] = __hip_atomic_load(&sums[3 * h + k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      q[1] += q[0] >> 48;  // (low and high sums: below 2^48 times 2^16 workgroups)
      q[2] += q[1] >> 48;
      grad_coords[3 * n0 + h] = from_fixed((q[0] & kMask48) | q[1] << 48, (q[1] & kMask48) >> 16 | q[2] << 32, F);
    }
    return;
  }
  for (int h = threadIdx.x; h < 3 * nn; h += kAdjThreads) {
    const int i = h / 3, j = h - 3 * i;
    uint64_t lo, hi;
    join48(s_acc[2 * j * N + i], (int64_t)s_acc[(2 * j + 1) * N + i], lo, hi);
    grad_coords[3 * n0 + h] = from_fixed(lo, hi, F);
  }
}

}  // namespace kb
