// kb_kernels.hpp -- gfx950 kernels of the lower-triangular stiffness build.
//
// Shared pieces: connectivity checks, node ranks, device-wide int32 scan, the
// per-element integration wrapper (precision modes, FP64 fallback, flags) and the
// element-major integration kernel.  The assembly kernels are in kb_assemble.hpp.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kb_element.hpp"
#include "kbuild.h"

namespace kb {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanChunk = kScanThreads * kScanItems;

__device__ __forceinline__ void raise_flag(uint32_t* status, uint32_t f) { atomicOr(status, f); }

// Workgroups are dispatched round-robin over the 8 XCDs (workgroup b runs on XCD b % 8).
// Map b to a work item so that each XCD takes one contiguous range of the n items: the
// runs that neighbouring items write next to each other then meet in the same L2.
constexpr int kXcds = 8;
__device__ __forceinline__ int64_t xcd_item(int64_t b, int64_t n) {
  const int64_t x = b % kXcds, i = b / kXcds, full = n / kXcds, rem = n % kXcds;
  return x * full + (x < rem ? x : rem) + i;
}

template <int NEN>
__device__ __forceinline__ void load_conn(const int32_t* __restrict__ conn, int64_t e, int32_t (&E)[NEN]) {
#pragma unroll
  for (int a = 0; a < NEN; ++a) E[a] = conn[e * NEN + a];
}

// KB_F_INDEX / KB_F_REPEAT bits of one element
template <int NEN>
__device__ __forceinline__ uint32_t check_conn(const int32_t (&E)[NEN], int64_t n_node) {
  uint32_t f = 0;
#pragma unroll
  for (int a = 0; a < NEN; ++a)
    if (E[a] < 0 || (int64_t)E[a] >= n_node) f |= KB_F_INDEX;
#pragma unroll
  for (int a = 0; a < NEN; ++a)
#pragma unroll
    for (int b = 0; b < a; ++b)
      if (E[a] == E[b]) f |= KB_F_REPEAT;
  return f;
}

// rank of each node among the element's (distinct) ids
template <int NEN>
__device__ __forceinline__ void node_ranks(const int32_t (&E)[NEN], int (&r)[NEN]) {
#pragma unroll
  for (int a = 0; a < NEN; ++a) {
    int s = 0;
#pragma unroll
    for (int b = 0; b < NEN; ++b) s += (E[b] < E[a]) ? 1 : 0;
    r[a] = s;
  }
}

// ---------------------------------------------------------------- several DOFs
// Connectivity of the DOF view of a mesh with dof components per node: entry a*dof+i
// of element e is the global DOF dof*E[a]+i.  An id outside [0, n_node) maps to ids
// outside [0, dof*n_node) (a negative one stays negative; distinct ids stay distinct
// below 2^31/dof in magnitude), so the pipeline flags the element as the node ids would.
static __global__ __launch_bounds__(256) void k_dof_conn(const int32_t* __restrict__ conn, int64_t n, int dof,
                                                  int32_t* __restrict__ dconn) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t v = conn[t];
    for (int i = 0; i < dof; ++i) {
      int64_t w = dof * v + i;
      w = w > INT32_MAX ? INT32_MAX : (w < INT32_MIN ? INT32_MIN : w);
      dconn[t * dof + i] = (int32_t)w;
    }
  }
}

// ------------------------------------------------------------------------- fill
static __global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

static __global__ void k_init_status(uint32_t* __restrict__ status, int64_t* __restrict__ nnz) {
  if (threadIdx.x < KB_STATUS_WORDS) status[threadIdx.x] = 0u;
  if (threadIdx.x == 0 && nnz) *nnz = 0;
}

// --------------------------------------------------------------------- scan (int32)
// block-wide exclusive scan of one value per thread; returns the block total in *total
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t* smem_waves, int32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
  int32_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    int32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) smem_waves[wave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t s = 0;
    for (int w = 0; w < nwaves; ++w) {
      int32_t t = smem_waves[w];
      smem_waves[w] = s;
      s += t;
    }
    smem_waves[nwaves] = s;
  }
  __syncthreads();
  const int32_t r = x - v + smem_waves[wave];
  *total = smem_waves[nwaves];
  __syncthreads();
  return r;
}

// sum of in[] over this workgroup's chunk of kScanChunk entries -> part[blockIdx.x]
__device__ __forceinline__ void scan_chunk_sum(const int32_t* __restrict__ in, int64_t n, int32_t* __restrict__ part) {
  __shared__ int32_t sw[kScanThreads / 64 + 1];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
  int32_t s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i)
    if (base + i < n) s += in[base + i];
  int32_t total;
  block_exclusive_scan(s, sw, &total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// out[0..n] = exclusive scan of in[0..n) (out[n] = total), this workgroup's chunk: the
// chunk sums before it are added up here, so no kernel in between scans them.  also (in
// itself, or null) gets out[0..n); total64 optional
__device__ __forceinline__ void scan_chunk_down(const int32_t* in, int64_t n, const int32_t* __restrict__ part,
                                                int32_t* __restrict__ out, int32_t* also,
                                                int64_t* __restrict__ total64) {
  __shared__ int32_t sw[kScanThreads / 64 + 1];
  int32_t before = 0;
  for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kScanThreads) before += part[i];
  int32_t prefix;
  block_exclusive_scan(before, sw, &prefix);
  const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
  int32_t v[kScanItems];
  int32_t s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    v[i] = (base + i < n) ? in[base + i] : 0;
    s += v[i];
  }
  int32_t total;
  int32_t off = block_exclusive_scan(s, sw, &total) + prefix;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    if (base + i < n) {
      out[base + i] = off;
      if (also) also[base + i] = off;
    }
    off += v[i];
  }
  if ((int64_t)(blockIdx.x + 1) * kScanChunk >= n && threadIdx.x == 0) {
    const int32_t grand = prefix + total;
    out[n] = grand;
    if (total64) *total64 = grand;
  }
}

// n == 0: out[0] = 0 (optional)
static __global__ void k_scan_empty(int32_t* __restrict__ out, int64_t* __restrict__ total64) {
  if (out) out[0] = 0;
  if (total64) *total64 = 0;
}

// --------------------------------------------------------------------- integrate
enum class Prec { F64, F32, F32FB };

template <Prec P>
struct PrecTraits;
template <>
struct PrecTraits<Prec::F64> {
  using V = double;
};
template <>
struct PrecTraits<Prec::F32> {
  using V = float;
};
template <>
struct PrecTraits<Prec::F32FB> {
  using V = float;
};

// Node coordinate sources: [n][3] as given, or padded [n][4] (one aligned 32-byte
// record per node, so each random gather touches a single cache line).
struct NodesXYZ {
  const double* __restrict__ p;
  __device__ __forceinline__ void get(int32_t n, double (&x)[3]) const {
    const double* q = p + (int64_t)n * 3;
    x[0] = q[0];
    x[1] = q[1];
    x[2] = q[2];
  }
};
struct NodesPadded {
  const double4* __restrict__ p;
  __device__ __forceinline__ void get(int32_t n, double (&x)[3]) const {
    const double4 v = p[n];
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
  }
};

// Coordinates of the element's nodes, gathered once into registers.
template <int NEN, typename NODES>
__device__ __forceinline__ void gather_nodes(const NODES& nodes, const int32_t (&E)[NEN], double (&Xn)[NEN][3]) {
#pragma unroll
  for (int a = 0; a < NEN; ++a) nodes.get(E[a], Xn[a]);
}

// An element's integrals (without c); relative(X) fills in its node coordinates relative to
// node 0.  What the Jacobian of a brick's stiffness is made of is formed in FP64 whatever
// the precision, as in element_values_pair, and rounded once (from corner differences rounded
// to FP32 the integrals of bricks ten times as long as wide were off by 1.18e-7 rms, not
// 0.98e-7).  With FP32 geometry an ill-conditioned element is integrated again with its
// Jacobian, determinant and adjugate in FP64 and counted in *fb.  Returns false if some
// determinant is not > 0.
template <int NEN, Prec P, Op OP, typename Fn>
__device__ __forceinline__ bool element_integrals(const Fn& relative, float tau,
                                                  typename PrecTraits<P>::V (&k)[ElemTraits<NEN>::T], uint32_t* fb) {
  constexpr bool kModal = NEN == 8 && OP == Op::Stiffness;
  constexpr int N = kModal ? kModes : NEN;
  const auto geometry = [&](double (&G)[N][3]) {
    if constexpr (kModal) {
      double X[NEN][3];
      relative(X);
      corner_modes(X, G);
    } else {
      relative(G);
    }
  };
  const auto wide = [&] {
    using V = typename PrecTraits<P>::V;
    double G[N][3];
    geometry(G);
    if constexpr (kModal)
      return hex_integrate<double, V, false>(G, k, 0.0, nullptr);
    else
      return integrate<NEN, double, V, false, OP>(G, k, 0.0, nullptr);
  };
  if constexpr (P == Prec::F64) {
    return wide();
  } else {
    float F[N][3];
    {
      double G[N][3];
      geometry(G);
#pragma unroll
      for (int a = 0; a < N; ++a)
#pragma unroll
        for (int j = 0; j < 3; ++j) F[a][j] = (float)G[a][j];
    }
    bool need_fb = false, ok;
    if constexpr (kModal)
      ok = hex_integrate<float, float, P == Prec::F32FB>(F, k, tau, &need_fb);
    else
      ok = integrate<NEN, float, float, P == Prec::F32FB, OP>(F, k, tau, &need_fb);
    if constexpr (P == Prec::F32FB) {
      if (need_fb) {
        ok = wide();
        *fb += 1;
      }
    }
    return ok;
  }
}

// Integrate one element of coefficient c into k (value type V, c applied).  Adds flag bits to
// *f and counts a fallback in *fb.
template <int NEN, Prec P, Op OP, typename Fn>
__device__ __forceinline__ void element_values_of(const Fn& relative, double c, float tau,
                                                  typename PrecTraits<P>::V (&k)[ElemTraits<NEN>::T], uint32_t* f,
                                                  uint32_t* fb) {
  constexpr int T = ElemTraits<NEN>::T;
  using V = typename PrecTraits<P>::V;
  const bool ok = element_integrals<NEN, P, OP>(relative, tau, k, fb);
  bool finite = true;
#pragma unroll
  for (int p = 0; p < T; ++p) {
    k[p] = (V)(c * (double)k[p]);
    finite = finite && isfinite(k[p]);
  }
  if (!ok) *f |= KB_F_INVERTED;
  if (!finite) *f |= KB_F_NONFINITE;
}

// from its gathered node coordinates Xn
template <int NEN, Prec P, Op OP = Op::Stiffness>
__device__ __forceinline__ void element_values_at(const double (&Xn)[NEN][3], double c, float tau,
                                                  typename PrecTraits<P>::V (&k)[ElemTraits<NEN>::T], uint32_t* f,
                                                  uint32_t* fb) {
  const auto relative = [&](double (&X)[NEN][3]) {
#pragma unroll
    for (int a = 0; a < NEN; ++a)
#pragma unroll
      for (int j = 0; j < 3; ++j) X[a][j] = a ? Xn[a][j] - Xn[0][j] : 0.0;
  };
  element_values_of<NEN, P, OP>(relative, c, tau, k, f, fb);
}

// gathering its nodes (again for a fallback, which needs fewer registers than to keep them).
// E must be valid.
template <int NEN, Prec P, typename NODES, Op OP = Op::Stiffness>
__device__ __forceinline__ void element_values(const NODES& nodes, const double* __restrict__ coef, int64_t e,
                                               const int32_t (&E)[NEN], float tau,
                                               typename PrecTraits<P>::V (&k)[ElemTraits<NEN>::T], uint32_t* f,
                                               uint32_t* fb) {
  double X0[3];
  nodes.get(E[0], X0);
  const double c = coef[e];
  const auto relative = [&](double (&X)[NEN][3]) {
    X[0][0] = X[0][1] = X[0][2] = 0.0;
#pragma unroll
    for (int a = 1; a < NEN; ++a) {
      nodes.get(E[a], X[a]);
#pragma unroll
      for (int j = 0; j < 3; ++j) X[a][j] -= X0[j];
    }
  };
  element_values_of<NEN, P, OP>(relative, c, tau, k, f, fb);
}

// Lane h of a pair gathers nodes 4h .. 4h+3 of its brick (a branch per half keeps every
// index into E a constant).
template <typename NODES>
__device__ __forceinline__ void gather_pair(const NODES& nodes, const int32_t (&E)[8], int h, double (&xo)[4][3]) {
  if (h) {
#pragma unroll
    for (int a = 0; a < 4; ++a) nodes.get(E[4 + a], xo[a]);
  } else {
#pragma unroll
    for (int a = 0; a < 4; ++a) nodes.get(E[a], xo[a]);
  }
}

// A brick of coefficient c integrated by a lane pair (lanes 2i and 2i+1; h = lane & 1)
// from the nodes gather_pair brought: each lane forms its face's part of the mode
// coefficients from the coordinates relative to node 0, in FP64; the parts are exchanged,
// and each lane integrates the four points of its half of the rule.  Lane h ends with
// rows 4h .. 4h+3, k[a][b] = k_(4h+a, b).  Both lanes of a pair must be active together.
// An ill-conditioned point in either half gives the element FP64 geometry (counted by h = 0).
template <Prec P>
__device__ __forceinline__ void element_values_pair(const double (&xo)[4][3], double c, float tau, int h,
                                                    typename PrecTraits<P>::V (&k)[4][8], uint32_t* f, uint32_t* fb) {
  static_assert(P != Prec::F64, "one lane per brick in FP64 (k_pass1_two)");
  using V = typename PrecTraits<P>::V;
  const double sg = h ? 1.0 : -1.0;
  double Cd[kModes][3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const double other = pair_other(xo[0][j]), x0 = h ? other : xo[0][j];
    double own[4], o[4];
    half_modes(xo[0][j] - x0, xo[1][j] - x0, xo[2][j] - x0, xo[3][j] - x0, own);
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = pair_other(own[i]);
    Cd[0][j] = own[1] + o[1];
    Cd[1][j] = own[2] + o[2];
    Cd[2][j] = sg * (own[0] - o[0]);  // (t = +1) - (t = -1)
    Cd[3][j] = own[3] + o[3];
    Cd[4][j] = sg * (own[2] - o[2]);
    Cd[5][j] = sg * (own[1] - o[1]);
    Cd[6][j] = sg * (own[3] - o[3]);
  }
  float C[kModes][3];
#pragma unroll
  for (int m = 0; m < kModes; ++m)
#pragma unroll
    for (int j = 0; j < 3; ++j) C[m][j] = (float)Cd[m][j];
  V M[4][6];
  bool need_fb = false;
  bool ok = half_points<float, float, P == Prec::F32FB>(C, M, tau, &need_fb, h);
  if constexpr (P == Prec::F32FB) {
    const int other = pair_other((int)need_fb);  // (outside any branch: both lanes take part)
    if (need_fb || other) {  // the element: both halves with FP64 geometry
      ok = half_points<double, float, false>(Cd, M, 0.0, nullptr, h);
      if (h == 0) *fb += 1;
    }
  }
  half_matrix<V>(M, k, h);
  bool finite = true;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      k[a][b] = (V)(c * (double)k[a][b]);
      finite = finite && isfinite(k[a][b]);
    }
  if (!ok) *f |= KB_F_INVERTED;
  if (!finite) *f |= KB_F_NONFINITE;
}

template <int NEN, Prec P, Op OP = Op::Stiffness>
__global__ __launch_bounds__(256) void k_integrate_store(const int32_t* __restrict__ conn,
                                                         const double* __restrict__ coords,
                                                         const double* __restrict__ coef, int64_t n_elem,
                                                         int64_t n_node, float tau,
                                                         typename PrecTraits<P>::V* __restrict__ out,
                                                         uint32_t* __restrict__ status) {
  constexpr int T = ElemTraits<NEN>::T;
  using V = typename PrecTraits<P>::V;
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= n_elem) return;
  int32_t E[NEN];
  load_conn<NEN>(conn, e, E);
  uint32_t f = check_conn<NEN>(E, n_node);
  V k[T];
  uint32_t fb = 0;
  if (f) {
#pragma unroll
    for (int p = 0; p < T; ++p) k[p] = V(0);
  } else {
    element_values<NEN, P, NodesXYZ, OP>(NodesXYZ{coords}, coef, e, E, tau, k, &f, &fb);
  }
#pragma unroll
  for (int p = 0; p < T; ++p) out[e * T + p] = k[p];
  if (f) raise_flag(status, f);
  if (fb) atomicAdd(&status[1], fb);
}

}  // namespace kb
