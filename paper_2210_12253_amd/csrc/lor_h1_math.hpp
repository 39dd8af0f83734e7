// Per-subelement integration of the LOR H1 matrix on one trilinear subelement.
//
// Section 2.2: the LOR matrix is the Q1 stiffness + mass matrix of the refined
// mesh.  On a subelement with corner coordinates X_v (v = a + 2b + 4c at the
// reference corner (a,b,c) of [0,1]^3), with 2x2x2 Gauss points q (weight 1/8):
//
//   K_uv = kappa sum_q (1/8) det J (J^-T g_u).(J^-T g_v)
//        = sum_q sum_rc  G_rc(q) g_u,r(q) g_v,c(q),   G = (kappa / 8 det J) R R^T,
//   M_uv = beta sum_q (1/8) det J phi_u phi_v,
//
// where R has the rows r_0 = J_1 x J_2, r_1 = J_2 x J_0, r_2 = J_0 x J_1 (J_c the
// columns of J, so J^-1 = R / det J).  The reference gradients are tensor
// products, g_u,0 = l_a'(xi) l_b(eta) l_c(zeta) with l_0 = 1 - t, l_1 = t, so
// l' = -1 or +1.  Every entry therefore splits into 1D pieces:
//
//   M_uv  = TM[a+a'][b+b'][c+c']
//   (r,r) terms: s_a S0[b+b'][c+c'] + s_b S1[a+a'][c+c'] + s_c S2[a+a'][b+b']
//   (r,c) terms: sig_a sig_b' T01[a'][b][c+c'] + sig_b sig_a' T01[a][b'][c+c']  (and 02, 12)
//
// with s_a = +1 if a == a' else -1, sig_a = 2a - 1, and the factor tables
//   S0[B][C]  = sum_q G00(q) LL_B(eta_q) LL_C(zeta_q)        (LL_0 = l0^2, LL_1 = l0 l1, LL_2 = l1^2)
//   T01[x][y][C] = sum_q G01(q) l_x(xi_q) l_y(eta_q) LL_C(zeta_q)   ...
//   TM[A][B][C] = sum_q (beta det J / 8) LL_A LL_B LL_C.
// They are contracted one axis at a time (sum factorisation), so a subelement
// costs about 1.3k flops instead of ~2k for the direct 8x8 quadrature.
#pragma once

#include <hip/hip_runtime.h>

namespace lor {

// l_a(t_q) at the two Gauss points t_0 = (1 - 1/sqrt3)/2, t_1 = (1 + 1/sqrt3)/2.
constexpr double kGA = 0.78867513459481288225457439025098;  // l_0(t_0) = l_1(t_1)
constexpr double kGB = 0.21132486540518711774542560974902;  // l_1(t_0) = l_0(t_1)
constexpr double kGA2 = 0.62200846792814621558800373425063;  // kGA^2
constexpr double kGB2 = 0.04465819873852045107866293241604;  // kGB^2
constexpr double kSixth = 0.16666666666666666666666666666667;  // kGA * kGB

__host__ __device__ constexpr double L1(int a, int q) { return a == q ? kGA : kGB; }
// LL_A(t_q) for A = a + a' in {0, 1, 2}
__host__ __device__ constexpr double LL(int A, int q) {
  return A == 1 ? kSixth : ((A == 0) == (q == 0) ? kGA2 : kGB2);
}

// Index of the unordered corner pair (u <= v) among the 36 pairs, u-major.
__host__ __device__ constexpr int pair_index(int u, int v) {
  return u <= v ? (u * (15 - u)) / 2 + v : (v * (15 - v)) / 2 + u;
}

// 1/x from the hardware reciprocal estimate refined by Newton steps (two in
// FP64, one in FP32): within an ulp or two, far cheaper than IEEE division.
__device__ __forceinline__ double rcp_refined(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float rcp_refined(float x) {
  float r = __builtin_amdgcn_rcpf(x);
  const float e = __builtin_fmaf(-x, r, 1.0f);
  return __builtin_fmaf(r, e, r);
}

template <typename R>
struct H1Factors {
  R S0[3][3], S1[3][3], S2[3][3];
  R T01[2][2][3], T02[2][2][3], T12[2][2][3];
  R TM[3][3][3];
};

// Edge vectors of the trilinear subelement, formed in FP64 then rounded to R:
// ex[b][c] = X(1,b,c) - X(0,b,c), ey[a][c] = X(a,1,c) - X(a,0,c),
// ez[a][b] = X(a,b,1) - X(a,b,0).
template <typename R>
__device__ __forceinline__ void h1_edges(const double (&X)[8][3], R (&ex)[2][2][3], R (&ey)[2][2][3],
                                         R (&ez)[2][2][3]) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        ex[s][t][d] = static_cast<R>(X[1 + 2 * s + 4 * t][d] - X[0 + 2 * s + 4 * t][d]);
        ey[s][t][d] = static_cast<R>(X[s + 2 + 4 * t][d] - X[s + 4 * t][d]);
        ez[s][t][d] = static_cast<R>(X[s + 2 * t + 4][d] - X[s + 2 * t][d]);
      }
}

// Largest / smallest Jacobian determinant over the 8 corners (the triple
// product of the three edge vectors meeting at the corner).
template <typename R>
__device__ __forceinline__ void h1_corner_det_range(const R (&ex)[2][2][3], const R (&ey)[2][2][3],
                                                    const R (&ez)[2][2][3], R& dmin, R& dmax) {
  dmin = R(3.0e38);
  dmax = R(-3.0e38);
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const R* A = ex[b][c];
        const R* B = ey[a][c];
        const R* C = ez[a][b];
        const R d = A[0] * (B[1] * C[2] - B[2] * C[1]) + A[1] * (B[2] * C[0] - B[0] * C[2]) +
                    A[2] * (B[0] * C[1] - B[1] * C[0]);
        dmin = d < dmin ? d : dmin;
        dmax = d > dmax ? d : dmax;
      }
}

// Jacobian columns at the Gauss points: J_0 = dx/dxi depends on (eta, zeta)
// only and is the bilinear interpolant of the four x-edge vectors, etc.
// c0[q2][q3], c1[q1][q3], c2[q1][q2].
template <typename R>
__device__ __forceinline__ void jac_columns(const R (&ex)[2][2][3], const R (&ey)[2][2][3], const R (&ez)[2][2][3],
                                            R (&c0)[2][2][3], R (&c1)[2][2][3], R (&c2)[2][2][3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d)
#pragma unroll
    for (int qs = 0; qs < 2; ++qs) {
      const R m0x = R(L1(0, qs)) * ex[0][0][d] + R(L1(1, qs)) * ex[1][0][d];
      const R m1x = R(L1(0, qs)) * ex[0][1][d] + R(L1(1, qs)) * ex[1][1][d];
      const R m0y = R(L1(0, qs)) * ey[0][0][d] + R(L1(1, qs)) * ey[1][0][d];
      const R m1y = R(L1(0, qs)) * ey[0][1][d] + R(L1(1, qs)) * ey[1][1][d];
      const R m0z = R(L1(0, qs)) * ez[0][0][d] + R(L1(1, qs)) * ez[1][0][d];
      const R m1z = R(L1(0, qs)) * ez[0][1][d] + R(L1(1, qs)) * ez[1][1][d];
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        c0[qs][qt][d] = R(L1(0, qt)) * m0x + R(L1(1, qt)) * m1x;
        c1[qs][qt][d] = R(L1(0, qt)) * m0y + R(L1(1, qt)) * m1y;
        c2[qs][qt][d] = R(L1(0, qt)) * m0z + R(L1(1, qt)) * m1z;
      }
    }
}

// Contract the per-point metric values into the S and T factor tables.
//   H00[q2][q3] = sum_q1 G00,  H11[q1][q3] = sum_q2 G11,  H22[q1][q2] = sum_q3 G22,
//   Z01[x][q2][q3] = sum_q1 l_x(xi) G01,  Z02[x][q2][q3] = sum_q1 l_x(xi) G02,
//   G12q[q1][q2][q3] = G12 at every point.
template <typename R>
__device__ __forceinline__ void h1_contract_stiffness(const R (&H00)[2][2], const R (&H11)[2][2],
                                                      const R (&H22)[2][2], const R (&Z01)[2][2][2],
                                                      const R (&Z02)[2][2][2], const R (&G12q)[2][2][2],
                                                      H1Factors<R>& F) {
#pragma unroll
  for (int B = 0; B < 3; ++B) {
    R y0[2], y1[2], y2[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      y0[t] = R(LL(B, 0)) * H00[0][t] + R(LL(B, 1)) * H00[1][t];  // S0: eta -> B
      y1[t] = R(LL(B, 0)) * H11[0][t] + R(LL(B, 1)) * H11[1][t];  // S1: xi  -> B
      y2[t] = R(LL(B, 0)) * H22[0][t] + R(LL(B, 1)) * H22[1][t];  // S2: xi  -> B
    }
#pragma unroll
    for (int Cc = 0; Cc < 3; ++Cc) {
      F.S0[B][Cc] = R(LL(Cc, 0)) * y0[0] + R(LL(Cc, 1)) * y0[1];
      F.S1[B][Cc] = R(LL(Cc, 0)) * y1[0] + R(LL(Cc, 1)) * y1[1];
      F.S2[B][Cc] = R(LL(Cc, 0)) * y2[0] + R(LL(Cc, 1)) * y2[1];
    }
  }
#pragma unroll
  for (int x = 0; x < 2; ++x) {
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      // T01[x][y][C]: eta -> l_y, zeta -> LL_C
      const R t0 = R(L1(y, 0)) * Z01[x][0][0] + R(L1(y, 1)) * Z01[x][1][0];
      const R t1 = R(L1(y, 0)) * Z01[x][0][1] + R(L1(y, 1)) * Z01[x][1][1];
#pragma unroll
      for (int Cc = 0; Cc < 3; ++Cc) F.T01[x][y][Cc] = R(LL(Cc, 0)) * t0 + R(LL(Cc, 1)) * t1;
    }
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      // T02[x][z][B]: zeta -> l_z, eta -> LL_B
      const R t0 = R(L1(z, 0)) * Z02[x][0][0] + R(L1(z, 1)) * Z02[x][0][1];
      const R t1 = R(L1(z, 0)) * Z02[x][1][0] + R(L1(z, 1)) * Z02[x][1][1];
#pragma unroll
      for (int B = 0; B < 3; ++B) F.T02[x][z][B] = R(LL(B, 0)) * t0 + R(LL(B, 1)) * t1;
    }
  }
#pragma unroll
  for (int al = 0; al < 3; ++al) {
    R Z12[2][2];
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int t3 = 0; t3 < 2; ++t3)
        Z12[t2][t3] = R(LL(al, 0)) * G12q[0][t2][t3] + R(LL(al, 1)) * G12q[1][t2][t3];
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      // T12[y][z][A]: xi -> LL_A, eta -> l_y, zeta -> l_z
      const R t0 = R(L1(y, 0)) * Z12[0][0] + R(L1(y, 1)) * Z12[1][0];
      const R t1 = R(L1(y, 0)) * Z12[0][1] + R(L1(y, 1)) * Z12[1][1];
#pragma unroll
      for (int z = 0; z < 2; ++z) F.T12[y][z][al] = R(L1(z, 0)) * t0 + R(L1(z, 1)) * t1;
    }
  }
}

// mass: TM[A][B][C] = sum_q D(q) LL_A(xi) LL_B(eta) LL_C(zeta)
template <typename R>
__device__ __forceinline__ void h1_contract_mass(const R (&Dq)[2][2][2], R (&TM)[3][3][3]) {
#pragma unroll
  for (int al = 0; al < 3; ++al) {
    R U[2][2];
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int t3 = 0; t3 < 2; ++t3) U[t2][t3] = R(LL(al, 0)) * Dq[0][t2][t3] + R(LL(al, 1)) * Dq[1][t2][t3];
#pragma unroll
    for (int B = 0; B < 3; ++B) {
      const R t0 = R(LL(B, 0)) * U[0][0] + R(LL(B, 1)) * U[1][0];
      const R t1 = R(LL(B, 0)) * U[0][1] + R(LL(B, 1)) * U[1][1];
#pragma unroll
      for (int Cc = 0; Cc < 3; ++Cc) TM[al][B][Cc] = R(LL(Cc, 0)) * t0 + R(LL(Cc, 1)) * t1;
    }
  }
}

// Factor tables of one subelement; returns false if det J <= 0 at a Gauss point.
template <typename R>
__device__ __forceinline__ bool h1_factors(const R (&ex)[2][2][3], const R (&ey)[2][2][3],
                                           const R (&ez)[2][2][3], R kap, R bet, H1Factors<R>& F) {
  R c0[2][2][3], c1[2][2][3], c2[2][2][3];
  jac_columns<R>(ex, ey, ez, c0, c1, c2);
  R H00[2][2] = {}, H11[2][2] = {}, H22[2][2] = {};
  R Z01[2][2][2] = {}, Z02[2][2][2] = {};
  R G12q[2][2][2], Dq[2][2][2];  // per Gauss point (q1, q2, q3): G_12 and beta det J / 8
  bool ok = true;
  const R wk = R(0.125) * kap;
  const R wb = R(0.125) * bet;
#pragma unroll
  for (int q3 = 0; q3 < 2; ++q3)
#pragma unroll
    for (int q2 = 0; q2 < 2; ++q2)
#pragma unroll
      for (int q1 = 0; q1 < 2; ++q1) {
        const R* A = c0[q2][q3];
        const R* B = c1[q1][q3];
        const R* C = c2[q1][q2];
        R r0[3], r1[3], r2[3];
        r0[0] = B[1] * C[2] - B[2] * C[1];
        r0[1] = B[2] * C[0] - B[0] * C[2];
        r0[2] = B[0] * C[1] - B[1] * C[0];
        r1[0] = C[1] * A[2] - C[2] * A[1];
        r1[1] = C[2] * A[0] - C[0] * A[2];
        r1[2] = C[0] * A[1] - C[1] * A[0];
        r2[0] = A[1] * B[2] - A[2] * B[1];
        r2[1] = A[2] * B[0] - A[0] * B[2];
        r2[2] = A[0] * B[1] - A[1] * B[0];
        const R det = A[0] * r0[0] + A[1] * r0[1] + A[2] * r0[2];
        ok = ok && (det > R(0));
        const R f = wk * rcp_refined(det);
        H00[q2][q3] += f * (r0[0] * r0[0] + r0[1] * r0[1] + r0[2] * r0[2]);
        H11[q1][q3] += f * (r1[0] * r1[0] + r1[1] * r1[1] + r1[2] * r1[2]);
        H22[q1][q2] += f * (r2[0] * r2[0] + r2[1] * r2[1] + r2[2] * r2[2]);
        const R g01 = f * (r0[0] * r1[0] + r0[1] * r1[1] + r0[2] * r1[2]);
        const R g02 = f * (r0[0] * r2[0] + r0[1] * r2[1] + r0[2] * r2[2]);
        G12q[q1][q2][q3] = f * (r1[0] * r2[0] + r1[1] * r2[1] + r1[2] * r2[2]);
        Dq[q1][q2][q3] = wb * det;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          Z01[x][q2][q3] += R(L1(x, q1)) * g01;
          Z02[x][q2][q3] += R(L1(x, q1)) * g02;
        }
      }
  h1_contract_stiffness<R>(H00, H11, H22, Z01, Z02, G12q, F);
  h1_contract_mass<R>(Dq, F.TM);
  return ok;
}

// Entry (u, v) of K + M from the factor tables.
template <typename R>
__device__ __forceinline__ R h1_entry(const H1Factors<R>& F, int u, int v) {
  const int a = u & 1, b = (u >> 1) & 1, c = (u >> 2) & 1;
  const int a2 = v & 1, b2 = (v >> 1) & 1, c2 = (v >> 2) & 1;
  const int A = a + a2, B = b + b2, C = c + c2;
  const R sa = R(2 * a - 1), sb = R(2 * b - 1), sc = R(2 * c - 1);
  const R sa2 = R(2 * a2 - 1), sb2 = R(2 * b2 - 1), sc2 = R(2 * c2 - 1);
  R val = F.TM[A][B][C];
  val += (a == a2 ? R(1) : R(-1)) * F.S0[B][C];
  val += (b == b2 ? R(1) : R(-1)) * F.S1[A][C];
  val += (c == c2 ? R(1) : R(-1)) * F.S2[A][B];
  val += sa * sb2 * F.T01[a2][b][C] + sb * sa2 * F.T01[a][b2][C];
  val += sa * sc2 * F.T02[a2][c][B] + sc * sa2 * F.T02[a][c2][B];
  val += sb * sc2 * F.T12[b2][c][A] + sc * sb2 * F.T12[b][c2][A];
  return val;
}

// --------------------------------------------------------------- whole cell
//
// All 36 entries of a cell, from the Walsh moments of the point values.  The
// value kernels on box lattices and the coloured kernel are bound by FP64 (or
// FP32) instruction issue, so the operation count decides: about 950 here
// against 1330 for factor tables and entries one by one (h1_factors,
// h1_entry).  At a Gauss point the coordinate along an axis is (1 + s / sqrt3) / 2
// with s = -1 or +1, so with sig_a = 2a - 1
//   l_a      = (1 + sig_a s / sqrt3) / 2,
//   l_a l_a' = {2 - sqrt3 s, 1, 2 + sqrt3 s} / 6  for a + a' = 0, 1, 2
// (s^2 = 1): only the moments m_ijk = sum_q s1^i s2^j s3^k f(q) with i, j, k in
// {0, 1} of each metric value f are needed, and they cost additions only.
//   * an axis contracted with l l' turns (m_0, m_1) into three values (walsh3);
//   * the two mixed terms of a pair of axes (x, y) together are, with
//     A = 3 m_00, P = sqrt3 m_10, Q = sqrt3 m_01, W = m_11 (m_ij over x and y),
//       a = a', b = b':    W + sig_a Q + sig_b P + sig_a sig_b A
//       a = a', b != b':  -W - sig_a Q
//       a != a', b = b':  -W - sig_b P
//       both differ:       W - sig_a sig_b A
//     (sums over a row vanish, as they must for a stiffness matrix);
//   * everything contracted with l_c l_c' (xx, yy, xy and mass: H[k], ten
//     values per moment k along z) is added up before that last contraction,
//     and the rest depends on (a + a', b + b') only, with one sign per c, c'
//     (B9 for zz and the even part of xz, yz; C9 for the odd part), except for
//     an antisymmetric part where c != c'.
// The scale of the columns and all constant factors are folded into the
// coefficients of the point values.

constexpr double kSqrt3 = 1.7320508075688772935274463415059;
constexpr double kGR = 0.26794919243112270647255365849413;  // kGB / kGA = 2 - sqrt3

// (m_0, m_1) -> the three values of l l' (times 6)
template <typename R>
__device__ __forceinline__ void walsh3(R m0, R m1, R (&o)[3]) {
  const R t = m0 + m0;
  o[0] = t - R(kSqrt3) * m1;
  o[1] = m0;
  o[2] = t + R(kSqrt3) * m1;
}

// Jacobian columns at the Gauss points, divided by kGA^2 (one fused
// multiply-add per value and axis).
template <typename R>
__device__ __forceinline__ void scaled_columns(const R (&e)[2][2][3], R (&c)[2][2][3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const R m00 = e[0][0][d] + R(kGR) * e[1][0][d], m10 = R(kGR) * e[0][0][d] + e[1][0][d];
    const R m01 = e[0][1][d] + R(kGR) * e[1][1][d], m11 = R(kGR) * e[0][1][d] + e[1][1][d];
    c[0][0][d] = m00 + R(kGR) * m01;
    c[0][1][d] = R(kGR) * m00 + m01;
    c[1][0][d] = m10 + R(kGR) * m11;
    c[1][1][d] = R(kGR) * m10 + m11;
  }
}

// c x with the constant's rounding to R made up for (rounded once, it would be
// the same relative error in every entry).
template <typename R>
__device__ __forceinline__ R scale_by(double c, R x) {
  if constexpr (sizeof(R) == 8) {
    return c * x;
  } else {
    const R hi = static_cast<R>(c), lo = static_cast<R>(c - static_cast<double>(hi));
    return __builtin_fmaf(lo, x, hi * x);
  }
}

// Entries of K + M of one cell from its edge vectors, entry (u, v), u <= v,
// handed to st(pair_index(u, v), value).  Returns false if det J <= 0 at a
// Gauss point.
template <typename R, typename St>
__device__ __forceinline__ bool h1_cell(const R (&ex)[2][2][3], const R (&ey)[2][2][3], const R (&ez)[2][2][3], R kap,
                                        R bet, const St& st) {
  R c0[2][2][3], c1[2][2][3], c2[2][2][3];
  scaled_columns<R>(ex, c0);
  scaled_columns<R>(ey, c1);
  scaled_columns<R>(ez, c2);
  // columns are J / kGA2: det J = kGA2^3 det, r_a . r_b / det J = kGA2 (r_a . r_b / det)
  const R wk = scale_by<R>(0.125 * kGA2 / 36.0, kap);
  const R wb = scale_by<R>(0.125 * kGA2 * kGA2 * kGA2 / 216.0, bet);
  bool ok = true;
  // moments: xx[j][k], yy[i][k], zz[i][j]; xy, xz, yz, dd [i][j][k]
  R xx[2][2], yy[2][2], zz[2][2] = {}, xy[2][2][2], xz[2][2][2], yz[2][2][2], dd[2][2][2];
#pragma unroll
  for (int q3 = 0; q3 < 2; ++q3) {
    // moments over s1 and s2 at this s3
    R pxx[2], pyy[2] = {}, pxy[2][2], pxz[2][2], pyz[2][2], pdd[2][2];
    R hxx[2], hxy[2][2], hxz[2][2], hyz[2][2], hdd[2][2], hzz[2][2];
#pragma unroll
    for (int q2 = 0; q2 < 2; ++q2) {
      R g[2][7];  // 00, 11, 22, 01, 02, 12, det at q1 = 0, 1
#pragma unroll
      for (int q1 = 0; q1 < 2; ++q1) {
        const R* A = c0[q2][q3];
        const R* B = c1[q1][q3];
        const R* C = c2[q1][q2];
        R r0[3], r1[3], r2[3];
        r0[0] = B[1] * C[2] - B[2] * C[1];
        r0[1] = B[2] * C[0] - B[0] * C[2];
        r0[2] = B[0] * C[1] - B[1] * C[0];
        r1[0] = C[1] * A[2] - C[2] * A[1];
        r1[1] = C[2] * A[0] - C[0] * A[2];
        r1[2] = C[0] * A[1] - C[1] * A[0];
        r2[0] = A[1] * B[2] - A[2] * B[1];
        r2[1] = A[2] * B[0] - A[0] * B[2];
        r2[2] = A[0] * B[1] - A[1] * B[0];
        const R det = A[0] * r0[0] + A[1] * r0[1] + A[2] * r0[2];
        ok = ok && (det > R(0));
        const R f = wk * rcp_refined(det);
        g[q1][0] = f * (r0[0] * r0[0] + r0[1] * r0[1] + r0[2] * r0[2]);
        g[q1][1] = f * (r1[0] * r1[0] + r1[1] * r1[1] + r1[2] * r1[2]);
        g[q1][2] = f * (r2[0] * r2[0] + r2[1] * r2[1] + r2[2] * r2[2]);
        g[q1][3] = f * (r0[0] * r1[0] + r0[1] * r1[1] + r0[2] * r1[2]);
        g[q1][4] = f * (r0[0] * r2[0] + r0[1] * r2[1] + r0[2] * r2[2]);
        g[q1][5] = f * (r1[0] * r2[0] + r1[1] * r2[1] + r1[2] * r2[2]);
        g[q1][6] = wb * det;
      }
      hxx[q2] = g[1][0] + g[0][0];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        auto sd = [&](int m) { return i == 0 ? g[1][m] + g[0][m] : g[1][m] - g[0][m]; };
        pyy[i] = q2 == 0 ? sd(1) : pyy[i] + sd(1);
        hzz[q2][i] = sd(2);
        hxy[q2][i] = sd(3);
        hxz[q2][i] = sd(4);
        hyz[q2][i] = sd(5);
        hdd[q2][i] = sd(6);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      auto sd = [&](R a, R b) { return j == 0 ? b + a : b - a; };  // a at s2 = -1, b at s2 = +1
      pxx[j] = sd(hxx[0], hxx[1]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        pxy[i][j] = sd(hxy[0][i], hxy[1][i]);
        pxz[i][j] = sd(hxz[0][i], hxz[1][i]);
        pyz[i][j] = sd(hyz[0][i], hyz[1][i]);
        pdd[i][j] = sd(hdd[0][i], hdd[1][i]);
        const R z = sd(hzz[0][i], hzz[1][i]);
        zz[i][j] = q3 == 0 ? z : zz[i][j] + z;
      }
    }
    // moments over s3: at q3 = 0 the values are parked in [0], at q3 = 1 combined
    auto fold = [&](R& m0, R& m1, R v) {
      if (q3 == 0) {
        m0 = v;
      } else {
        m1 = v - m0;
        m0 = v + m0;
      }
    };
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      fold(xx[j][0], xx[j][1], pxx[j]);
      fold(yy[j][0], yy[j][1], pyy[j]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fold(xy[i][j][0], xy[i][j][1], pxy[i][j]);
        fold(xz[i][j][0], xz[i][j][1], pxz[i][j]);
        fold(yz[i][j][0], yz[i][j][1], pyz[i][j]);
        fold(dd[i][j][0], dd[i][j][1], pdd[i][j]);
      }
    }
  }

  // H[k]: xx + yy + xy + mass per moment k along z, for the ten pairs of
  // (a, b) corners: 0..3 the corner a + 2b with itself, 4 + a: b differs,
  // 6 + b: a differs, 8: (0,0)-(1,1), 9: (1,0)-(0,1)
  R H[2][10];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    R M[3][3];  // [A][B]
    {
      R t0[3], t1[3];
      walsh3<R>(dd[0][0][k], dd[1][0][k], t0);
      walsh3<R>(dd[0][1][k], dd[1][1][k], t1);
#pragma unroll
      for (int A = 0; A < 3; ++A) walsh3<R>(t0[A], t1[A], M[A]);
    }
    R S0[3], S1[3];
    walsh3<R>(xx[0][k], xx[1][k], S0);  // [B]
    walsh3<R>(yy[0][k], yy[1][k], S1);  // [A]
    const R A = R(3) * xy[0][0][k], P = R(kSqrt3) * xy[1][0][k], Q = R(kSqrt3) * xy[0][1][k], W = xy[1][1][k];
    const R WpA = W + A, WmA = W - A, QpP = Q + P, QmP = Q - P;
    H[k][0] = (M[0][0] + S0[0] + S1[0]) + (WpA - QpP);
    H[k][3] = (M[2][2] + S0[2] + S1[2]) + (WpA + QpP);
    H[k][1] = (M[2][0] + S0[0] + S1[2]) + (WmA + QmP);
    H[k][2] = (M[0][2] + S0[2] + S1[0]) + (WmA - QmP);
    H[k][4] = (M[0][1] + S0[1] - S1[0]) - (W - Q);
    H[k][5] = (M[2][1] + S0[1] - S1[2]) - (W + Q);
    H[k][6] = (M[1][0] - S0[0] + S1[1]) - (W - P);
    H[k][7] = (M[1][2] - S0[2] + S1[1]) - (W + P);
    const R m11 = M[1][1] - S0[1] - S1[1];
    H[k][8] = m11 + WmA;
    H[k][9] = m11 + WpA;
  }
  // zz and the xz, yz terms: even part B9, odd part C9 per (A, B), and the
  // antisymmetric values XA[B] (a differs) and YA[A] (b differs)
  R B9[3][3], C9[3][3], XA[3], YA[3];
  {
    R t0[3], t1[3];
    walsh3<R>(zz[0][0], zz[1][0], t0);
    walsh3<R>(zz[0][1], zz[1][1], t1);
#pragma unroll
    for (int A = 0; A < 3; ++A) walsh3<R>(t0[A], t1[A], B9[A]);
    R P[3], Q[3], W[3];
    walsh3<R>(R(3) * xz[0][0][0], R(3) * xz[0][1][0], XA);
    walsh3<R>(R(kSqrt3) * xz[1][0][0], R(kSqrt3) * xz[1][1][0], P);
    walsh3<R>(R(kSqrt3) * xz[0][0][1], R(kSqrt3) * xz[0][1][1], Q);
    walsh3<R>(xz[1][0][1], xz[1][1][1], W);
#pragma unroll
    for (int B = 0; B < 3; ++B) {
      B9[0][B] += W[B] - Q[B];
      B9[1][B] -= W[B];
      B9[2][B] += W[B] + Q[B];
      C9[0][B] = P[B] - XA[B];
      C9[1][B] = -P[B];
      C9[2][B] = P[B] + XA[B];
    }
    walsh3<R>(R(3) * yz[0][0][0], R(3) * yz[1][0][0], YA);
    walsh3<R>(R(kSqrt3) * yz[0][1][0], R(kSqrt3) * yz[1][1][0], P);
    walsh3<R>(R(kSqrt3) * yz[0][0][1], R(kSqrt3) * yz[1][0][1], Q);
    walsh3<R>(yz[0][1][1], yz[1][1][1], W);
#pragma unroll
    for (int A = 0; A < 3; ++A) {
      B9[A][0] += W[A] - Q[A];
      B9[A][1] -= W[A];
      B9[A][2] += W[A] + Q[A];
      C9[A][0] += P[A] - YA[A];
      C9[A][1] -= P[A];
      C9[A][2] += P[A] + YA[A];
    }
  }
  // contraction along z and the entries
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int m = n; m < 4; ++m) {
      const int a = n & 1, b = n >> 1, a2 = m & 1, b2 = m >> 1;
      const int h = n == m ? n : a == a2 ? 4 + a : b == b2 ? 6 + b : n == 0 ? 8 : 9;
      const R even = B9[a + a2][b + b2];
      const R U = R(2) * H[0][h] + even;
      const R V = H[0][h] - even;
      const R O = R(kSqrt3) * H[1][h] + C9[a + a2][b + b2];
      st(pair_index(n, m), U - O);
      st(pair_index(n + 4, m + 4), U + O);
      if (n == m) {
        st(pair_index(n, n + 4), V);
      } else {
        // u = n at c = 0, v = m at c = 1 adds sig_a XA[B] + sig_b YA[A] where
        // the corners differ; u = m, v = n subtracts it
        R Z = R(0);
        if (a != a2 && b != b2)
          Z = (a ? XA[1] : -XA[1]) + (b ? YA[1] : -YA[1]);
        else if (a != a2)
          Z = a ? XA[b + b2] : -XA[b + b2];
        else
          Z = b ? YA[a + a2] : -YA[a + a2];
        st(pair_index(n, m + 4), V + Z);
        st(pair_index(m, n + 4), V - Z);
      }
    }
  return ok;
}

}  // namespace lor
