// The 2D reconstruction of one wave's row (Section 2.2, Steps 1-3): stencils from
// the LDS ring of rows, characteristic fields and their polynomials, shared by
// the 2D stage kernels.
#pragma once

#include "hwenou_internal.hpp"

namespace hwenou {

constexpr int kCols = 66;  // LDS columns: strip*62 - 2 .. strip*62 + 63

__device__ __forceinline__ double g3w(int g) { return g == 1 ? G3W1 : G3W0; }
__device__ __forceinline__ double g3x(int g) { return g == 0 ? -G3S : (g == 1 ? 0.0 : G3S); }

// Primitive quantities at the cell average shared by both sweeps.
struct Prim {
  double u, v, c, ci, H, b1, b2, q2;
};

template <class TR>
__device__ __forceinline__ Prim make_prim(double gm1, const double (&U)[4]) {
  Prim p;
  const double rinv = rcp_w<TR>(U[0]);
  p.u = U[1] * rinv;
  p.v = U[2] * rinv;
  p.q2 = p.u * p.u + p.v * p.v;
  const double pr = gm1 * (U[3] - 0.5 * U[0] * p.q2);
  const double c2 = (gm1 + 1.0) * pr * rinv;
  p.ci = rsq_w<TR>(c2);
  p.c = c2 * p.ci;
  p.H = (U[3] + pr) * rinv;
  p.b1 = gm1 * (p.ci * p.ci);
  p.b2 = 0.5 * p.b1 * p.q2;
  return p;
}

// The same quantities at the Roe average of two cell averages (the
// per-interface bases): sqrt(rho)-weighted velocity and total enthalpy,
// c^2 = (gamma - 1)(H - q^2 / 2).  The arguments come in a fixed order (the
// lower or left cell first), so the two cells that share an interface form
// bitwise the same basis.
template <class TR>
__device__ __forceinline__ Prim make_prim_roe(double gm1, const double (&UL)[4],
                                              const double (&UR)[4]) {
  Prim p;
  const double il = rsq_w<TR>(UL[0]), ir = rsq_w<TR>(UR[0]);  // 1/sqrt(rho)
  const double sl = UL[0] * il, sr = UR[0] * ir;                 // sqrt(rho)
  const double w = rcp_w<TR>(sl + sr);
  p.u = (UL[1] * il + UR[1] * ir) * w;
  p.v = (UL[2] * il + UR[2] * ir) * w;
  p.q2 = p.u * p.u + p.v * p.v;
  // sqrt(rho) H = (E + p) / sqrt(rho), with p = (gamma - 1)(E - |m|^2 / (2 rho))
  const double hl = (UL[3] + gm1 * (UL[3] - 0.5 * (UL[1] * UL[1] + UL[2] * UL[2]) * il * il)) * il;
  const double hr = (UR[3] + gm1 * (UR[3] - 0.5 * (UR[1] * UR[1] + UR[2] * UR[2]) * ir * ir)) * ir;
  p.H = (hl + hr) * w;
  const double c2 = gm1 * (p.H - 0.5 * p.q2);
  p.ci = rsq_w<TR>(c2);
  p.c = c2 * p.ci;
  p.b1 = gm1 * (p.ci * p.ci);
  p.b2 = 0.5 * p.b1 * p.q2;
  return p;
}

// Row k of the left eigenvectors of the Euler flux Jacobian in direction DIR
// (ideal gas), normalised to the right eigenvectors
// x: R = [(1,u-c,v,H-uc), (1,u,v,q^2/2), (0,0,1,v), (1,u+c,v,H+uc)]
// y: R = [(1,u,v-c,H-vc), (1,u,v,q^2/2), (0,1,0,u), (1,u,v+c,H+vc)]
template <int DIR>
__device__ __forceinline__ void eig_row(const Prim& p, int k, double (&l)[4]) {
  const double un = DIR == 0 ? p.u : p.v;  // normal velocity
  const double ut = DIR == 0 ? p.v : p.u;  // tangential velocity
  constexpr int n = DIR == 0 ? 1 : 2, t = DIR == 0 ? 2 : 1;
  if (k == 0 || k == 3) {
    const double s = k == 0 ? 1.0 : -1.0;
    l[0] = 0.5 * (p.b2 + s * un * p.ci);
    l[n] = -0.5 * (p.b1 * un + s * p.ci);
    l[t] = -0.5 * p.b1 * ut;
    l[3] = 0.5 * p.b1;
  } else if (k == 1) {
    l[0] = 1.0 - p.b2;
    l[n] = p.b1 * un;
    l[t] = p.b1 * ut;
    l[3] = -p.b1;
  } else {
    l[0] = -ut;
    l[n] = 0.0;
    l[t] = 1.0;
    l[3] = 0.0;
  }
}

template <int NC, class TM, int ROWS = 3>
struct RowBuf {
  double u[ROWS][NC][kCols];      // cell averages of the ring's rows
  double m[ROWS][2][NC][kCols];   // x and y moments (widened once on store)
};

// Loads rows of an instance into registers (RowRegs) and stores them into the
// ring's columns 0..65.  Lane l loads column l of the 3 NC planes.  The row's
// two columns beyond: in FP64 one value to a lane (lane 2 q + c takes column
// 64 + c of plane q), which costs one register and one load and store instead
// of 3 NC (2048^2: 2.07 -> 1.99 ms per Runge-Kutta step, with the first four
// rows of a run loaded together, which the registers allow then).  In the mixed
// form, whose planes have two types, lanes 0 and 1 load their column of every
// plane (the other way took 3% longer on long runs: 64 grids of 256^2 to 1024^2
// 9.77 instead of 9.38 ms per step).
template <int NC, class TM>
struct RowRegs {  // mixed
  double u[NC], u1[NC];
  TM m[2][NC], m1[2][NC];
};
template <int NC>
struct RowRegs<NC, double> {
  double u[NC];
  double m[2][NC];
  double x;
};

template <int NC, class TM>
struct RowLoader {  // mixed
  const double* u_in;
  const TM* m_in;
  long long plane;
  int lane;
  unsigned ou, om, ou1, om1;  // byte offsets of this lane's columns in a row

  // gx0, gx1: grid columns of ring columns `lane` and 64 + (lane & 1)
  __device__ __forceinline__ RowLoader(const double* u, const TM* m, long long plane_, int lane_,
                                       int gx0, int gx1)
      : u_in(u), m_in(m), plane(plane_), lane(lane_), ou((unsigned)gx0 * 8u),
        om((unsigned)gx0 * (unsigned)sizeof(TM)), ou1((unsigned)gx1 * 8u),
        om1((unsigned)gx1 * (unsigned)sizeof(TM)) {}
  // base: first cell of the row in a plane
  __device__ __forceinline__ void load(long long base, RowRegs<NC, TM>& R) const {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const double* pu = u_in + (k * plane + base);
      const TM* pv = m_in + (k * plane + base);
      const TM* pw = m_in + ((NC + k) * plane + base);
      R.u[k] = load_at(pu, ou);
      R.m[0][k] = load_at(pv, om);
      R.m[1][k] = load_at(pw, om);
      if (lane < 2) {
        R.u1[k] = load_at(pu, ou1);
        R.m1[0][k] = load_at(pv, om1);
        R.m1[1][k] = load_at(pw, om1);
      }
    }
  }
  template <int ROWS>
  __device__ __forceinline__ void store(RowBuf<NC, TM, ROWS>& B, int slot,
                                        const RowRegs<NC, TM>& R) const {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      B.u[slot][k][lane] = R.u[k];
      B.m[slot][0][k][lane] = (double)R.m[0][k];
      B.m[slot][1][k][lane] = (double)R.m[1][k];
      if (lane < 2) {
        B.u[slot][k][64 + lane] = R.u1[k];
        B.m[slot][0][k][64 + lane] = (double)R.m1[0][k];
        B.m[slot][1][k][64 + lane] = (double)R.m1[1][k];
      }
    }
  }
};
template <int NC>
struct RowLoader<NC, double> {
  const double* u_in;
  const double* m_in;
  long long plane;
  int lane;
  unsigned ou;
  const char* extra;  // this lane's value of the last two columns, in row 0

  __device__ __forceinline__ RowLoader(const double* u, const double* m, long long plane_,
                                       int lane_, int gx0, int gx1)
      : u_in(u), m_in(m), plane(plane_), lane(lane_) {
    ou = (unsigned)gx0 * 8u;
    const int q = lane >> 1;
    extra = q < NC ? reinterpret_cast<const char*>(u_in + (q * plane + gx1))
                   : reinterpret_cast<const char*>(m_in + ((q - NC) * plane + gx1));
  }
  __device__ __forceinline__ void load(long long base, RowRegs<NC, double>& R) const {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      R.u[k] = load_at(u_in + (k * plane + base), ou);
      R.m[0][k] = load_at(m_in + (k * plane + base), ou);
      R.m[1][k] = load_at(m_in + ((NC + k) * plane + base), ou);
    }
    R.x = 0.0;
    if (lane < 6 * NC) R.x = *reinterpret_cast<const double*>(extra + base * 8);
  }
  template <int ROWS>
  __device__ __forceinline__ void store(RowBuf<NC, double, ROWS>& B, int slot,
                                        const RowRegs<NC, double>& R) const {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      B.u[slot][k][lane] = R.u[k];
      B.m[slot][0][k][lane] = R.m[0][k];
      B.m[slot][1][k][lane] = R.m[1][k];
    }
    if (lane < 6 * NC) {
      const int q = lane >> 1, c = 64 + (lane & 1);
      double* to = q < NC ? &B.u[slot][0][0] + q * kCols + c
                          : &B.m[slot][0][0][0] + (q - NC) * kCols + c;
      *to = R.x;
    }
  }
};

// The 17 stencil values of field/component data around lane column `l`
// (LDS columns l, l+1, l+2; ring slots sb, sc, st for rows j-1, j, j+1).
template <int NC, class TM, int ROWS>
__device__ __forceinline__ void read_stencil(const RowBuf<NC, TM, ROWS>& B, int sb, int sc, int st, int l,
                                             int k, Sten2& S) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    S.u[a] = B.u[sb][k][l + a];
    S.u[3 + a] = B.u[sc][k][l + a];
    S.u[6 + a] = B.u[st][k][l + a];
  }
  S.v[0] = B.m[sb][0][k][l + 1];
  S.v[1] = B.m[sc][0][k][l];
  S.v[2] = B.m[sc][0][k][l + 2];
  S.v[3] = B.m[st][0][k][l + 1];
  S.w[0] = B.m[sb][1][k][l + 1];
  S.w[1] = B.m[sc][1][k][l];
  S.w[2] = B.m[sc][1][k][l + 2];
  S.w[3] = B.m[st][1][k][l + 1];
}

// What the reconstruction of one scalar field needs of its stencil, linear in
// it: the coefficients of p0 and the values at cells 2, 4, 5, 6, 8.
struct Field {
  double c[15], x[5];
};

// The FP64 stage's results are the same bits from every kernel that computes a
// cell (one wave or a pair of waves per run).  What the compiler fuses into one
// rounding depends on the code around, so the steps of the FP64 reconstruction
// end in values it cannot see through (pin: no instruction), and the mapping's
// sums of products say which product is fused (mad).  The mixed kernels, of
// which there is one per cell, spill with mad as fma.
template <class T, int N>
__device__ __forceinline__ void pin(T (&x)[N]) {
  if constexpr (sizeof(T) == 8) {
#pragma unroll
    for (int n = 0; n < N; ++n) asm("" : "+v"(x[n]));
  }
}
template <class T, int M, int N>
__device__ __forceinline__ void pin(T (&x)[M][N]) {
#pragma unroll
  for (int m = 0; m < M; ++m) pin(x[m]);
}
template <class T>
__device__ __forceinline__ T mad(T a, T b, T c) {
  if constexpr (sizeof(T) == 8)
    return fma(a, b, c);
  else
    return a * b + c;
}

template <class TR>
__device__ __forceinline__ void make_field(const Sten2& S, Field& F) {
  p0_coeffs_2d<TR>(S, F.c);
  F.x[0] = S.u[1];
  F.x[1] = S.u[3];
  F.x[2] = S.u[4];
  F.x[3] = S.u[5];
  F.x[4] = S.u[7];
  if constexpr (sizeof(TR) == 8) {
    pin(F.c);
    pin(F.x);
  }
}

// F = A + s B
__device__ __forceinline__ void add_fields(const Field& A, double s, const Field& B, Field& F) {
#pragma unroll
  for (int n = 0; n < 15; ++n) F.c[n] = fma(s, B.c[n], A.c[n]);
#pragma unroll
  for (int n = 0; n < 5; ++n) F.x[n] = fma(s, B.x[n], A.x[n]);
  pin(F.c);
  pin(F.x);
}

// Scalar HWENO reconstruction of one field -> combined coefficients
template <class TR, bool SI, bool FOLD = false>
__device__ __forceinline__ void recon_field(const SchemeParams& P, const Field& F, TR (&C)[15],
                                            double* a_out = nullptr) {
  const double u5 = F.x[2];
  const double asum = fabs(F.x[0]) + fabs(F.x[1]) + fabs(u5) + fabs(F.x[3]) + fabs(F.x[4]);
  hweno_2d<TR, SI, FOLD>(P, F.c, u5, u5 - F.x[1], F.x[3] - u5, u5 - F.x[0], F.x[4] - u5, asum, C,
                         a_out);
  if constexpr (sizeof(TR) == 8) {
    pin(C);
    if constexpr (FOLD) asm("" : "+v"(*a_out));
  }
}

// S += s * (stencil of component k); first = true: S = s * (...)
template <bool FIRST, int NC, class TM>
__device__ __forceinline__ void add_stencil(double s, const Sten2& A, Sten2& S) {
#pragma unroll
  for (int q = 0; q < 9; ++q) S.u[q] = FIRST ? s * A.u[q] : fma(s, A.u[q], S.u[q]);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    S.v[q] = FIRST ? s * A.v[q] : fma(s, A.v[q], S.v[q]);
    S.w[q] = FIRST ? s * A.w[q] : fma(s, A.w[q], S.w[q]);
  }
}

// Stencil of (component k) - s (density): the momentum relative to velocity s.
template <class TR, class TM, int ROWS>
__device__ __forceinline__ void relative_momentum(const RowBuf<4, TM, ROWS>& B, int sb, int sc, int st,
                                                  int l, int k, double s, Field& F) {
  Sten2 R, M;
  read_stencil<4, TM>(B, sb, sc, st, l, 0, R);
  read_stencil<4, TM>(B, sb, sc, st, l, k, M);
  add_stencil<false, 4, TM>(-s, R, M);
  make_field<TR>(M, F);
}

// One characteristic field K of the sweep in direction DIR, mixed form: project the
// stencil with row K of L and reconstruct.  Returns C (C[0..2] combined
// coefficients, C[3..14] p0 coefficients) and the factor a of p0.  The shear
// field (K = 2) has only two non-zero entries in its L row; they are used
// directly.
template <int DIR, int K, bool SI, class TR, class TM, int ROWS>
__device__ __forceinline__ void char_field(const SchemeParams& P, const Prim& pr,
                                           const RowBuf<4, TM, ROWS>& B, int sb, int sc, int st, int l,
                                           TR (&C)[15], double& a) {
  double lrow[4];
  eig_row<DIR>(pr, K, lrow);
  Sten2 W;
  if constexpr (K == 2) {
    // L row: -u_t at density, 1 at the tangential momentum
    constexpr int t = DIR == 0 ? 2 : 1;
    Sten2 S0, St;
    read_stencil<4, TM>(B, sb, sc, st, l, 0, S0);
    read_stencil<4, TM>(B, sb, sc, st, l, t, St);
    const double m0 = lrow[0];
#pragma unroll
    for (int q = 0; q < 9; ++q) W.u[q] = St.u[q] + m0 * S0.u[q];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      W.v[q] = St.v[q] + m0 * S0.v[q];
      W.w[q] = St.w[q] + m0 * S0.w[q];
    }
  } else {
#pragma unroll
    for (int q = 0; q < 9; ++q) W.u[q] = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) W.v[q] = W.w[q] = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      Sten2 S;
      read_stencil<4, TM>(B, sb, sc, st, l, m, S);
      const double lm = lrow[m];
#pragma unroll
      for (int q = 0; q < 9; ++q) W.u[q] += lm * S.u[q];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        W.v[q] += lm * S.v[q];
        W.w[q] += lm * S.w[q];
      }
    }
  }
  Field F;
  make_field<TR>(W, F);
  recon_field<TR, SI, true>(P, F, C, &a);
}

// Characteristic sweep in direction DIR: combined polynomials of the four
// fields mapped back to conserved variables, Cc[m][n] = sum_K R[m][K] P_K[n].
//
// Projection, FP64 form.  The left eigenvectors of the flux Jacobian are
//   l0 = P - N / (2c),  l1 = rho - 2 P,  l2 = T,  l3 = P + N / (2c)
// of the fields
//   P = (b2 rho - b1 (u m_x + v m_y - E)) / 2,
//   N = m_n - u_n rho,  T = m_t - u_t rho
// (normal and tangential momentum relative to the cell's velocity).  The
// coefficients of p0 are linear in the stencil, so they are formed for P, N, T
// and the density and combined; P does not depend on the direction and goes
// from the first sweep to the second through LDS (PARKP).  Per cell and both
// directions that is about 620 operations and 190 LDS reads of stencil values,
// where projecting each of the seven field-sweeps and forming its p0 takes 930
// and 270.  2048^2 grid: 2.20 -> 2.11 ms per Runge-Kutta step; 500 x 333 with
// per-interface bases: 320 -> 293 us.
// The mixed form projects field by field (char_field): its FP32 results are
// bound to the FP64 rounding in front of them (see p0_coeffs_2d).
// The entropy field (K = 1) has the same left row and right column in both
// directions: its polynomial is reconstructed once per cell, by the first
// sweep, and passed on through LDS (PARK: a second sweep follows).
//
// Mapping back.  Each field's polynomial P_K arrives as C with C[0..2]
// combined and C[3..14] still to be scaled by the factor a of its p0.  The
// right eigenvectors
//   r0 = (1, un - c, ut, H - un c), r1 = (1, un, ut, q^2/2),
//   r2 = (0, 0, 1, ut),             r3 = (1, un + c, ut, H + un c)
// (components: density, normal momentum, tangential momentum, energy) give
//   Cc_rho = S + P1,          S = P0 + P3,  D = P3 - P0,
//   Cc_n   = un Cc_rho + c D,
//   Cc_t   = ut Cc_rho + P2,
//   Cc_E   = H S + un c D + q^2/2 P1 + ut P2,
// so the fields are taken in the order 0, 3, 1, 2 and fold into S, D and
// then into Cc.  OVERLAP12: no scheduling barrier between fields 1 and 2
// (the FP64 split sweeps fit their registers without it and run 0.7% faster;
// the other kernels then spill or run slower).
template <int DIR, bool SI, bool PARK, bool PARKP, class TR, class TM, bool OVERLAP12 = false,
          int ROWS>
__device__ __forceinline__ void char_sweep(const SchemeParams& P, const Prim& pr,
                                           const RowBuf<4, TM, ROWS>& B, int sb, int sc, int st, int l,
                                           TR (&Cc)[4][15], TR (*c1buf)[64], double (*pbuf)[64],
                                           bool have_c1) {
  constexpr int nd = DIR == 0 ? 1 : 2, td = DIR == 0 ? 2 : 1;  // normal, tangential momentum
  const double un = DIR == 0 ? pr.u : pr.v, ut = DIR == 0 ? pr.v : pr.u;
  constexpr bool FIELDS = sizeof(TR) == 8;
  TR C[15], S[15], D[15];
  double a;
  Field FP;
  {
    Field FN, F;
    const double hc = 0.5 * pr.ci;
    if constexpr (!FIELDS) {
      char_field<DIR, 0, SI, TR, TM>(P, pr, B, sb, sc, st, l, C, a);
    } else if (!(PARKP && have_c1)) {
      Sten2 A, WP, WN;
      const double hb = 0.5 * pr.b1;
      read_stencil<4, TM>(B, sb, sc, st, l, 0, A);
      add_stencil<true, 4, TM>(0.5 * pr.b2, A, WP);
      read_stencil<4, TM>(B, sb, sc, st, l, nd, WN);
      add_stencil<false, 4, TM>(-hb * un, WN, WP);
      add_stencil<false, 4, TM>(-un, A, WN);
      read_stencil<4, TM>(B, sb, sc, st, l, td, A);
      add_stencil<false, 4, TM>(-hb * ut, A, WP);
      read_stencil<4, TM>(B, sb, sc, st, l, 3, A);
      add_stencil<false, 4, TM>(hb, A, WP);
      make_field<TR>(WP, FP);
      make_field<TR>(WN, FN);
      if constexpr (PARKP) {
#pragma unroll
        for (int n = 0; n < 15; ++n) pbuf[n][l] = FP.c[n];
#pragma unroll
        for (int n = 0; n < 5; ++n) pbuf[15 + n][l] = FP.x[n];
      }
    } else {
#pragma unroll
      for (int n = 0; n < 15; ++n) FP.c[n] = pbuf[n][l];
#pragma unroll
      for (int n = 0; n < 5; ++n) FP.x[n] = pbuf[15 + n][l];
      relative_momentum<TR, TM>(B, sb, sc, st, l, nd, un, FN);
    }
    if constexpr (FIELDS) {
      add_fields(FP, -hc, FN, F);
      recon_field<TR, SI, true>(P, F, C, &a);
    }
    {
      const TR a0 = (TR)a;
#pragma unroll
      for (int n = 0; n < 15; ++n) S[n] = n < 3 ? C[n] : a0 * C[n];  // P0
    }
    if constexpr (FIELDS) {
      // fields 0 and 3 one after the other: 1% faster than overlapped, which
      // took the registers of the stencil reads they used to share
      __builtin_amdgcn_sched_barrier(0);
      add_fields(FP, hc, FN, F);
      recon_field<TR, SI, true>(P, F, C, &a);
    } else {
      char_field<DIR, 3, SI, TR, TM>(P, pr, B, sb, sc, st, l, C, a);
    }
    {
      const TR a3 = (TR)a;
#pragma unroll
      for (int n = 0; n < 15; ++n) {
        const TR p0 = S[n];
        const TR f = n < 3 ? (TR)1 : a3;
        S[n] = mad(f, C[n], p0);
        D[n] = mad(f, C[n], -p0);
      }
    }
  }
  // scheduling barriers keep the later fields apart (bounds register pressure;
  // without them the compiler spills to scratch)
  __builtin_amdgcn_sched_barrier(0);
  {
    TR C1[15];
    double a1;
    if (!have_c1) {
      if constexpr (FIELDS) {
        Field FR;
        Sten2 A;
        read_stencil<4, TM>(B, sb, sc, st, l, 0, A);
        make_field<TR>(A, FR);
        if constexpr (PARKP) {
#pragma unroll
          for (int n = 0; n < 15; ++n) FP.c[n] = pbuf[n][l];
#pragma unroll
          for (int n = 0; n < 5; ++n) FP.x[n] = pbuf[15 + n][l];
        }
        add_fields(FR, -2.0, FP, FR);
        recon_field<TR, SI, true>(P, FR, C1, &a1);
      } else {
        char_field<DIR, 1, SI, TR, TM>(P, pr, B, sb, sc, st, l, C1, a1);
      }
      if constexpr (PARK) {  // parked in LDS for the other sweep
#pragma unroll
        for (int n = 0; n < 15; ++n) c1buf[n][l] = C1[n];
        c1buf[15][l] = (TR)a1;
      }
    } else {
#pragma unroll
      for (int n = 0; n < 15; ++n) C1[n] = c1buf[n][l];
      a1 = (double)c1buf[15][l];
    }
    const TR tun = (TR)un, tc = (TR)pr.c, tH = (TR)pr.H, tunc = (TR)(un * pr.c);
    const TR ta1 = (TR)a1, th = (TR)(0.5 * pr.q2), tha1 = (TR)(0.5 * pr.q2 * a1);
#pragma unroll
    for (int n = 0; n < 15; ++n) {
      const TR f1 = n < 3 ? (TR)1 : ta1, fh = n < 3 ? th : tha1;
      Cc[0][n] = mad(f1, C1[n], S[n]);
      Cc[nd][n] = mad(tun, Cc[0][n], tc * D[n]);
      Cc[3][n] = mad(fh, C1[n], mad(tunc, D[n], tH * S[n]));
    }
  }
  if constexpr (!OVERLAP12) __builtin_amdgcn_sched_barrier(0);
  {
    if constexpr (FIELDS) {
      Field FT;
      relative_momentum<TR, TM>(B, sb, sc, st, l, td, ut, FT);
      recon_field<TR, SI, true>(P, FT, C, &a);
    } else {
      char_field<DIR, 2, SI, TR, TM>(P, pr, B, sb, sc, st, l, C, a);
    }
    const TR tut = (TR)ut, a2 = (TR)a, uta2 = (TR)(ut * a);
#pragma unroll
    for (int n = 0; n < 15; ++n) {
      const TR f2 = n < 3 ? (TR)1 : a2, fu = n < 3 ? tut : uta2;
      Cc[td][n] = mad(f2, C[n], tut * Cc[0][n]);
      Cc[3][n] = mad(fu, C[n], Cc[3][n]);
    }
  }
}

}  // namespace hwenou
