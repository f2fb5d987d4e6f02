// kb_element.hpp -- per-lane element integration for gfx950 (one element per lane).
//
// Lower triangle of k_e = c * sum_q W_q |J_q| B_q^T B_q (Eq. 7-9), computed as in the
// per-thread pipeline of Section 3 / Alg. 2: J = dN X, |J| by the 3x3 determinant
// formula, J^{-1} by the 3x3 adjugate formula, B = J^{-1} dN, lower triangle only.
//
// Arithmetic form used here (same mathematics, fewer operations):
//   A = adj(J) (so J^{-1} = A / |J|),  G = A dN  (so B = G / |J|),
//   W |J| B^T B = (W / |J|) G^T G = dN^T M dN,  M = (W / |J|) A^T A  (3 x 3).
// X holds node coordinates minus those of local node 0 (translation does not change
// J), formed in FP64 before any conversion, so FP32 geometry never suffers the
// cancellation of absolute coordinates.
//
// Shape-function derivatives at the integration points are compile-time constants:
// every loop over points and nodes is fully unrolled, so they become instruction
// literals instead of table loads.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

namespace kb {

// ---- brick: natural corner signs (corner order of the C ABI) ----------------------
__host__ __device__ constexpr int hex_sign(int a, int dir) {
  // dir 0: r, 1: s, 2: t
  return dir == 0 ? ((a == 1 || a == 2 || a == 5 || a == 6) ? 1 : -1)
       : dir == 1 ? ((a == 2 || a == 3 || a == 6 || a == 7) ? 1 : -1)
                  : (a >= 4 ? 1 : -1);
}

// 1/sqrt(3): abscissa of the two-point Gauss-Legendre rule (weights 1).
constexpr double kGauss2 = 0.57735026918962576450914878050195746;

// natural coordinate of integration point q (0..7) along dir: q = 4 i + 2 j + k
__host__ __device__ constexpr double hex_qp(int q, int dir) {
  return ((dir == 0 ? (q >> 2) : dir == 1 ? (q >> 1) : q) & 1) ? kGauss2 : -kGauss2;
}

// dN_a / d xi_dir of the trilinear brick at point q:
//   d/dr N_a = r_a (1 + s_a s)(1 + t_a t) / 8, and cyclically.
__host__ __device__ constexpr double hex_dN(int q, int dir, int a) {
  const double r = hex_qp(q, 0), s = hex_qp(q, 1), t = hex_qp(q, 2);
  const double ra = hex_sign(a, 0), sa = hex_sign(a, 1), ta = hex_sign(a, 2);
  return dir == 0 ? ra * (1.0 + sa * s) * (1.0 + ta * t) / 8.0
       : dir == 1 ? (1.0 + ra * r) * sa * (1.0 + ta * t) / 8.0
                  : (1.0 + ra * r) * (1.0 + sa * s) * ta / 8.0;
}

__host__ __device__ constexpr int lidx(int a, int b) { return a * (a + 1) / 2 + b; }

template <typename T>
__device__ __forceinline__ T kabs(T x) {
  return x < T(0) ? -x : x;
}

// adjugate A of J (J^{-1} = A / det) and det J
template <typename T>
__device__ __forceinline__ T adjugate(const T (&J)[3][3], T (&A)[3][3]) {
  A[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
  A[0][1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
  A[0][2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
  A[1][0] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
  A[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
  A[1][2] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
  A[2][0] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
  A[2][1] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
  A[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
  return J[0][0] * A[0][0] + J[0][1] * A[1][0] + J[0][2] * A[2][0];
}

// Estimated infinity-norm condition number ||J|| ||J^{-1}|| = ||J|| ||A|| / |det|,
// tested without division: returns true if ||J|| ||A|| > tau |det| (or det is not finite/positive).
template <typename T>
__device__ __forceinline__ bool ill_conditioned(const T (&J)[3][3], const T (&A)[3][3], T det, T tau) {
  T nj = T(0), na = T(0);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    T sj = kabs(J[i][0]) + kabs(J[i][1]) + kabs(J[i][2]);
    T sa = kabs(A[i][0]) + kabs(A[i][1]) + kabs(A[i][2]);
    nj = sj > nj ? sj : nj;
    na = sa > na ? sa : na;
  }
  return !(nj * na <= tau * det);
}

// ---- brick in the basis of its modes ---------------------------------------------------
// The trilinear functions are spanned by 1 and the modes r, s, t, rs, st, tr, rst, and a
// corner's shape function is the sum of all eight times its signs / 8, so corner values
// and mode coefficients are one Walsh transform apart (24 additions for 8 values).  In
// modes, the derivatives at an integration point are single products of its coordinates
// (+-g): J takes 8 additions an entry for all points together, and
//   k_mn = sum_q dphi_m^T M(q) dphi_n
// needs only the Walsh sums of M's six entries over the eight points.  About 1200
// operations a brick against 2400 with G^T G formed corner by corner at every point, and
// rigid translation drops out exactly.
// The 1/8 of the shape functions is in the mode coefficients, so that J is the Jacobian and
// its determinant and 1 / det span FP32's range as they do corner by corner (with J 8 times
// the Jacobian a brick of side 1.8e12 had det = infinity and k = 0); the 1/64 of k's two
// gradients is in its entries in modes (kModalScale).  Both are powers of two.
constexpr double kModalScale = 1.0 / 64.0;
constexpr int kModes = 7;

// d phi_m / d xi_i as a set of coordinates multiplied together (bits: r 1, s 2, t 4), or -1
__host__ __device__ constexpr int mode_set(int m) {  // the mode itself
  return m == 0 ? 1 : m == 1 ? 2 : m == 2 ? 4 : m == 3 ? 3 : m == 4 ? 6 : m == 5 ? 5 : 7;
}
__host__ __device__ constexpr int mode_grad(int m, int i) {
  return (mode_set(m) >> i & 1) ? mode_set(m) & ~(1 << i) : -1;
}
__host__ __device__ constexpr int mode_degree(int m) { return m < 3 ? 0 : m < 6 ? 1 : 2; }
__host__ __device__ constexpr int sym3(int i, int j) {  // entry of M: 00 01 02 11 12 22
  return i > j ? sym3(j, i) : i == 0 ? j : i == 1 ? 2 + j : 5;
}
// g^d
__host__ __device__ constexpr double gauss_power(int d) {
  return d == 0 ? 1.0 : d == 1 ? kGauss2 : d == 2 ? 1.0 / 3.0 : d == 3 ? kGauss2 / 3.0 : 1.0 / 9.0;
}

// mode coefficients of a field with values x[8] at the corners: C[7], modes r s t rs st tr
// rst.  half_modes: the part of the four corners of one face t = const (sum, r, s, rs).
template <typename T>
__device__ __forceinline__ void half_modes(T x0, T x1, T x2, T x3, T (&h)[4]) {
  const T p0 = x1 + x0, m0 = x1 - x0, p1 = x2 + x3, m1 = x2 - x3;
  h[0] = T(0.125) * (p0 + p1);
  h[1] = T(0.125) * (m0 + m1);
  h[2] = T(0.125) * (p1 - p0);
  h[3] = T(0.125) * (m1 - m0);
}
template <typename T>
__device__ __forceinline__ void corner_modes(const T (&X)[8][3], T (&C)[kModes][3]) {
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    T b[4], u[4];
    half_modes(X[0][j], X[1][j], X[2][j], X[3][j], b);
    half_modes(X[4][j], X[5][j], X[6][j], X[7][j], u);
    C[0][j] = u[1] + b[1];
    C[1][j] = u[2] + b[2];
    C[2][j] = u[0] - b[0];
    C[3][j] = u[3] + b[3];
    C[4][j] = u[2] - b[2];
    C[5][j] = u[1] - b[1];
    C[6][j] = u[3] - b[3];
  }
}

// A^T A / det of one point (A = adj J, geometry GT; M in AT); returns det > 0,
// and sets *need_fb for an ill-conditioned J if CHECK
template <typename GT, typename AT, bool CHECK>
__device__ __forceinline__ bool point_metric(const GT (&J)[3][3], GT tau, bool* need_fb, AT (&M)[6]) {
  GT A[3][3];
  const GT det = adjugate(J, A);
  if (CHECK) {
    if (ill_conditioned(J, A, det, tau)) *need_fb = true;
  }
  const AT f = AT(GT(1) / det);
  AT B[3][3];  // f A: the scale of 1 / length, so that no product leaves the range of AT
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) B[i][j] = f * AT(A[i][j]);
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = i; j < 3; ++j)
      M[sym3(i, j)] = B[0][i] * AT(A[0][j]) + B[1][i] * AT(A[1][j]) + B[2][i] * AT(A[2][j]);
  return det > GT(0);
}

// k in modes from the Walsh sums W[ij][c] = sum_q M_ij(q) sign_c(q).  (Templates rather
// than loops: which terms an entry has must be known before the arrays become registers.)
// the first term 3 i + j >= from of entry (m, n) with both derivatives non-zero, or 9
__host__ __device__ constexpr int mode_term(int m, int n, int from) {
  for (int t = from; t < 9; ++t)
    if (mode_grad(m, t / 3) >= 0 && mode_grad(n, t % 3) >= 0) return t;
  return 9;
}
template <int M, int N, int TERM, typename AT>
__device__ __forceinline__ AT modal_sum(const AT (&W)[6][8]) {
  constexpr int i = TERM / 3, j = TERM % 3, next = mode_term(M, N, TERM + 1);
  constexpr int ij = sym3(i, j), c = mode_grad(M, i) ^ mode_grad(N, j);
  if constexpr (next < 9)
    return W[ij][c] + modal_sum<M, N, next>(W);
  else
    return W[ij][c];
}
template <int MN, typename AT>
__device__ __forceinline__ void modal_entry(const AT (&W)[6][8], AT (&K)[kModes][kModes]) {
  constexpr int m = MN / kModes, n = MN % kModes;
  if constexpr (n <= m) {
    constexpr int d = mode_degree(m) + mode_degree(n);
    const AT s = AT(kModalScale * gauss_power(d)) * modal_sum<m, n, mode_term(m, n, 0)>(W);
    K[m][n] = s;
    K[n][m] = s;
  }
}
template <typename AT, int... MN>
__device__ __forceinline__ void modal_entries(const AT (&W)[6][8], AT (&K)[kModes][kModes],
                                              std::integer_sequence<int, MN...>) {
  (modal_entry<MN>(W, K), ...);
}
template <typename AT>
__device__ __forceinline__ void modal_matrix(const AT (&W)[6][8], AT (&K)[kModes][kModes]) {
  modal_entries(W, K, std::make_integer_sequence<int, kModes * kModes>{});
}

// corner values of a field given by its mode coefficients (no constant): all eight, or
// those of the face t = sign
template <typename T>
__device__ __forceinline__ void face_values(T r, T s, T rs, T c, T (&v)[4]) {
  const T a = c - r, b = c + r, d = s - rs, e = s + rs;  // s = -1: a - d ..., s = +1: a + d ...
  v[0] = a - d;
  v[1] = b - e;
  v[2] = b + e;
  v[3] = a + d;
}
template <typename T>
__device__ __forceinline__ void corner_values(const T (&c)[kModes], T (&v)[8]) {
  T lo[4], hi[4];
  face_values(c[0] - c[5], c[1] - c[4], c[3] - c[6], -c[2], lo);
  face_values(c[0] + c[5], c[1] + c[4], c[3] + c[6], c[2], hi);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = lo[i];
    v[4 + i] = hi[i];
  }
}

// four-point Walsh transform over the signs of two coordinates: x[2 i + j] at (-+, -+)[i][j]
// -> sum, first, second, product
template <typename T>
__device__ __forceinline__ void walsh4(T x0, T x1, T x2, T x3, T& one, T& a, T& b, T& ab) {
  const T p = x0 + x1, q = x2 + x3, d = x1 - x0, e = x3 - x2;
  one = p + q;
  a = q - p;
  b = d + e;
  ab = e - d;
}

// ---- brick, one precision for geometry (GT) and one for M / accumulation (AT) ----------
// C: mode coefficients of the node coordinates (corner_modes).  k[36]: lower triangle of
// the element integral (without c).  Returns false if some det is not > 0.  If CHECK,
// *need_fb is set when a point's Jacobian is ill-conditioned.
template <typename GT, typename AT, bool CHECK>
__device__ __forceinline__ bool hex_integrate(const GT (&C)[kModes][3], AT (&k)[36], GT tau, bool* need_fb) {
  bool ok = true;
  AT W[6][8];
#pragma unroll
  for (int ri = 0; ri < 2; ++ri) {  // the four points of each r, their sums, then both together
    AT w[6][4];
    AT P[4][6];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const GT r = ri ? GT(kGauss2) : -GT(kGauss2), s = p >= 2 ? GT(kGauss2) : -GT(kGauss2),
               u = (p & 1) ? GT(kGauss2) : -GT(kGauss2);
      GT J[3][3];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        J[0][j] = (C[0][j] + s * C[3][j]) + u * (C[5][j] + s * C[6][j]);
        J[1][j] = (C[1][j] + r * C[3][j]) + u * (C[4][j] + r * C[6][j]);
        J[2][j] = (C[2][j] + r * C[5][j]) + s * (C[4][j] + r * C[6][j]);
      }
      ok = point_metric<GT, AT, CHECK>(J, tau, need_fb, P[p]) && ok;
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) walsh4(P[0][i], P[1][i], P[2][i], P[3][i], w[i][0], w[i][1], w[i][2], w[i][3]);
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) {  // c: 1, s, t, st; W's sets: r 1, s 2, t 4
        if (ri == 0) {
          W[i][2 * c] = w[i][c];
        } else {
          const AT lo = W[i][2 * c];
          W[i][2 * c] = w[i][c] + lo;
          W[i][2 * c + 1] = w[i][c] - lo;
        }
      }
    __builtin_amdgcn_sched_barrier(0);
  }
  AT K[kModes][kModes];
  modal_matrix(W, K);
  AT R[kModes][8];  // rows in modes, columns at the corners
#pragma unroll
  for (int m = 0; m < kModes; ++m) corner_values(K[m], R[m]);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    AT c[kModes], v[8];
#pragma unroll
    for (int m = 0; m < kModes; ++m) c[m] = R[m][b];
    corner_values(c, v);
#pragma unroll
    for (int a = 0; a < 8; ++a)
      if (a >= b) k[lidx(a, b)] = v[a];
  }
  return ok;
}

// value of the other lane of a pair (lanes 2i and 2i + 1), both active
__device__ __forceinline__ int pair_other(int x) {
  return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, false);  // quad_perm [1 0 3 2]
}
__device__ __forceinline__ float pair_other(float x) { return __int_as_float(pair_other(__float_as_int(x))); }
__device__ __forceinline__ double pair_other(double x) {
  const int lo = pair_other(__double2loint(x)), hi = pair_other(__double2hiint(x));
  return __hiloint2double(hi, lo);
}

// Two lanes sharing one brick: lane h has the points of r = -g (h = 0) or +g (h = 1).
// half_points: their metrics P from the mode coefficients C; as point_metric for the four.
template <typename GT, typename AT, bool CHECK>
__device__ __forceinline__ bool half_points(const GT (&C)[kModes][3], AT (&P)[4][6], GT tau, bool* need_fb, int h) {
  const GT r = h ? GT(kGauss2) : -GT(kGauss2);
  bool ok = true;
  GT J1[2][3], J2[2][3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const GT v = GT(kGauss2) * (C[4][j] + r * C[6][j]), u1 = C[1][j] + r * C[3][j], u2 = C[2][j] + r * C[5][j];
    J1[0][j] = u1 - v;
    J1[1][j] = u1 + v;
    J2[0][j] = u2 - v;
    J2[1][j] = u2 + v;
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const GT s = p >= 2 ? GT(kGauss2) : -GT(kGauss2), u = (p & 1) ? GT(kGauss2) : -GT(kGauss2);
    GT J[3][3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      J[0][j] = (C[0][j] + s * C[3][j]) + u * (C[5][j] + s * C[6][j]);
      J[1][j] = J1[p & 1][j];
      J[2][j] = J2[p >> 1][j];
    }
    ok = point_metric<GT, AT, CHECK>(J, tau, need_fb, P[p]) && ok;
    __builtin_amdgcn_sched_barrier(0);
  }
  return ok;
}

// half_matrix: rows 4h .. 4h+3 of the element integral, k[a][b] = k_(4h+a, b), from the two
// lanes' metrics.  Both lanes of the pair are active.
template <typename AT>
__device__ __forceinline__ void half_matrix(const AT (&P)[4][6], AT (&k)[4][8], int h) {
  const AT sg = h ? AT(1) : AT(-1);
  AT W[6][8];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    AT w[4];
    walsh4(P[0][i], P[1][i], P[2][i], P[3][i], w[0], w[1], w[2], w[3]);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const AT o = pair_other(w[c]);
      W[i][2 * c] = w[c] + o;
      W[i][2 * c + 1] = sg * (w[c] - o);  // (r = +g) - (r = -g), the same in both lanes
    }
  }
  AT K[kModes][kModes];
  modal_matrix(W, K);
  // rows at the lane's face t = sg, columns at the corners
  AT R[4][kModes];  // [corner of the face][mode]
#pragma unroll
  for (int n = 0; n < kModes; ++n) {
    AT v[4];
    face_values(K[0][n] + sg * K[5][n], K[1][n] + sg * K[4][n], K[3][n] + sg * K[6][n], sg * K[2][n], v);
#pragma unroll
    for (int a = 0; a < 4; ++a) R[a][n] = v[a];
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) corner_values(R[a], k[a]);
  // one value per pair of corners, whichever of the two rows it is used in: the entry with
  // the larger corner first (rounding differs between the two orders of the transforms)
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const AT cross = pair_other(k[b][a]);  // lane 1's k_(4+b, a)
      if (b > a) {
        k[a][4 + b] = h ? k[b][4 + a] : cross;
        k[a][b] = h ? k[a][b] : k[b][a];
      } else {
        k[a][4 + b] = h ? k[a][4 + b] : cross;
      }
    }
}

// ---- tetrahedron: J rows are the edge vectors from node 0 (dN constant) -------------
// X[a][j] = x_j(node a) - x_j(node 0), a = 1..3.  One point, weight 1/6.
template <typename GT, typename AT, bool CHECK>
__device__ __forceinline__ bool tet_integrate(const GT (&X)[4][3], AT (&k)[10], GT tau, bool* need_fb) {
  GT J[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) J[i][j] = X[i + 1][j];
  GT A[3][3];
  const GT det = adjugate(J, A);
  if (CHECK) {
    if (ill_conditioned(J, A, det, tau)) *need_fb = true;
  }
  // G = A dN with dN = [[-1,1,0,0],[-1,0,1,0],[-1,0,0,1]]: column a >= 1 is A[:, a-1]
  AT G[3][4];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    G[i][1] = AT(A[i][0]);
    G[i][2] = AT(A[i][1]);
    G[i][3] = AT(A[i][2]);
    G[i][0] = -(G[i][1] + G[i][2] + G[i][3]);
  }
  const AT f = AT(GT(1) / (GT(6) * det));
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const AT g0 = f * G[0][a], g1 = f * G[1][a], g2 = f * G[2][a];
#pragma unroll
    for (int b = 0; b <= a; ++b) k[lidx(a, b)] = g0 * G[0][b] + g1 * G[1][b] + g2 * G[2][b];
  }
  return det > GT(0);
}

// ---- consistent mass matrix: m_ab = integral of N_a N_b (c applied by the caller) ------
// N_a at brick point q: (1 + r_a r)(1 + s_a s)(1 + t_a t) / 8
__host__ __device__ constexpr double hex_N(int q, int a) {
  return (1.0 + hex_sign(a, 0) * hex_qp(q, 0)) * (1.0 + hex_sign(a, 1) * hex_qp(q, 1)) *
         (1.0 + hex_sign(a, 2) * hex_qp(q, 2)) / 8.0;
}

// brick: sum over the 2x2x2 points of |J_q| N_a N_b (exact for affine bricks)
template <typename GT, typename AT, bool CHECK>
__device__ __forceinline__ bool hex_mass(const GT (&X)[8][3], AT (&m)[36], GT tau, bool* need_fb) {
  bool ok = true;
#pragma unroll
  for (int p = 0; p < 36; ++p) m[p] = AT(0);
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    GT J[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        GT s = GT(0);
#pragma unroll
        for (int a = 1; a < 8; ++a) s += GT(hex_dN(q, i, a)) * X[a][j];
        J[i][j] = s;
      }
    GT A[3][3];
    const GT det = adjugate(J, A);
    ok = ok && (det > GT(0));
    if (CHECK) {
      if (ill_conditioned(J, A, det, tau)) *need_fb = true;
    }
    const AT d = AT(det);
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
      for (int b = 0; b <= a; ++b) m[lidx(a, b)] += d * AT(hex_N(q, a) * hex_N(q, b));
    __builtin_amdgcn_sched_barrier(0);
  }
  return ok;
}

// tetrahedron: the exact integral of two barycentric coordinates, V (1 + delta_ab) / 20
// with V = |J| / 6
template <typename GT, typename AT, bool CHECK>
__device__ __forceinline__ bool tet_mass(const GT (&X)[4][3], AT (&m)[10], GT tau, bool* need_fb) {
  GT J[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) J[i][j] = X[i + 1][j];
  GT A[3][3];
  const GT det = adjugate(J, A);
  if (CHECK) {
    if (ill_conditioned(J, A, det, tau)) *need_fb = true;
  }
  const AT f = AT(det) / AT(120);
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) m[lidx(a, b)] = a == b ? AT(2) * f : f;
  return det > GT(0);
}

// packed lower-triangle entries of an element matrix of NEN rows (NEN = nodes times
// degrees of freedom per node)
template <int NEN>
struct ElemTraits {
  static constexpr int T = NEN * (NEN + 1) / 2;
};

// the element integrand: stiffness (Eq. 7-9) or consistent mass
enum class Op { Stiffness = 0, Mass = 1 };

// from the node coordinates relative to node 0 (the stiffness of bricks: hex_integrate)

template <int NEN, typename GT, typename AT, bool CHECK, Op OP = Op::Stiffness>
__device__ __forceinline__ bool integrate(const GT (&X)[NEN][3], AT (&k)[ElemTraits<NEN>::T], GT tau, bool* need_fb) {
  if constexpr (OP == Op::Mass) {
    if constexpr (NEN == 8)
      return hex_mass<GT, AT, CHECK>(X, k, tau, need_fb);
    else
      return tet_mass<GT, AT, CHECK>(X, k, tau, need_fb);
  } else {
    static_assert(NEN == 4, "bricks: hex_integrate, from their modes");
    return tet_integrate<GT, AT, CHECK>(X, k, tau, need_fb);
  }
}

}  // namespace kb
