// The 1D stage operator of one wave (Section 2.1), shared by the kernels that
// run one stage per launch and those that run whole Runge-Kutta steps: from a
// cell's 3-cell stencil to its right-hand sides and modified moment.  Lane l
// holds cell i, lane l - 1 cell i - 1; interface values and fluxes move
// between lanes by DPP shifts, and every interface flux is evaluated once, by
// the lane on its right.  The results are valid on the lanes whose two
// neighbours hold valid stencils.
#pragma once

#include "hwenou_internal.hpp"

namespace hwenou {

// A read of data that no kernel writes while a stage kernel runs (the work
// list, the instance records, the done flags, alpha and dt), through the
// constant address space and word by word, so that at a wave-uniform address
// it becomes a scalar load, which does not wait behind the wave's vector
// memory traffic.
template <class T>
__device__ __forceinline__ T load_invariant(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "records of whole 32-bit words");
  using Word = const __attribute__((address_space(4))) unsigned;
  Word* q = (Word*)p;
  unsigned v[sizeof(T) / 4];
#pragma unroll
  for (int k = 0; k < (int)(sizeof(T) / 4); ++k) v[k] = q[k];
  T r;
  __builtin_memcpy(&r, v, sizeof(T));
  return r;
}

// The boundary rule of bc_index (periodic wrap, transmissive copy, mirror
// image at a reflective wall) as selects, so that the lanes of a tile form
// their source cells without branching on their own indices.
__device__ __forceinline__ int source_cell(int i, int n, int bc_lo, int bc_hi, bool& mirrored) {
  const bool lo = i < 0, out = lo || i >= n;
  const int bc = lo ? bc_lo : bc_hi;
  const int wrap = lo ? i + n : i - n;
  const int mirror = lo ? -1 - i : 2 * n - 1 - i;
  const int edge = lo ? 0 : n - 1;
  mirrored = out && bc == BC_REFLECTIVE;
  const int j = bc == BC_PERIODIC ? wrap : (bc == BC_REFLECTIVE ? mirror : edge);
  return out ? j : i;
}

// Right-hand sides F1 (averages) and F2 (moments) of Eq. (2.3) and the
// modified moments vh of this lane's cell; idx = 1 / dx.
template <int EQ, bool CHAR, class TR, int NC>
__device__ __forceinline__ void cell_rhs_1d(const SchemeParams& P, const double (&Um)[NC],
                                            const double (&Uc)[NC], const double (&Up)[NC],
                                            const double (&Vm)[NC], const double (&Vp)[NC],
                                            TR alpha, double idx, double (&F1)[NC], TR (&F2)[NC],
                                            TR (&vh)[NC]) {
  // ---- reconstruction: point values at the 4 Gauss-Lobatto nodes, v^ ----
  TR pt[4][NC];
  if constexpr (EQ == EQ_EULER && CHAR) {
    // Characteristic fields of f' at the cell average: left rows
    //   l_0 = (b2 + u/c, -(b1 u + 1/c), b1) / 2,  l_1 = (1 - b2, b1 u, -b1),
    //   l_2 = (b2 - u/c, -(b1 u - 1/c), b1) / 2,
    // right columns r_0 = (1, u - c, H - u c), r_1 = (1, u, u^2/2),
    // r_2 = (1, u + c, H + u c), with b1 = (gamma - 1)/c^2, b2 = b1 u^2/2.
    // The point values and moment P_K of the fields map back as
    //   rho = S + P_1,  m = u rho + c D,  E = H S + u c D + u^2/2 P_1,
    // with S = P_0 + P_2 and D = P_2 - P_0 (in FP64), so no 3x3 matrix is
    // kept and fewer values are live while the fields are reconstructed.
    const double gm1 = P.gas_gamma - 1.0;
    const double rinv = rcp_w<TR>(Uc[0]);
    const double u = Uc[1] * rinv;
    const double pr = gm1 * (Uc[2] - 0.5 * Uc[1] * u);
    const double c2 = (gm1 + 1.0) * pr * rinv;
    const double ci = rsq_w<TR>(c2);
    const double c = c2 * ci;
    const double H = (Uc[2] + pr) * rinv;
    const double b1 = gm1 * (ci * ci);
    const double b2 = 0.5 * b1 * u * u;
    // one field: project with row (l0, l1, l2), reconstruct, evaluate
    auto field = [&](double l0, double l1, double l2, double (&q)[5]) {
      const double wm = l0 * Um[0] + l1 * Um[1] + l2 * Um[2];
      const double wc = l0 * Uc[0] + l1 * Uc[1] + l2 * Uc[2];
      const double wp = l0 * Up[0] + l1 * Up[1] + l2 * Up[2];
      const double vvm = l0 * Vm[0] + l1 * Vm[1] + l2 * Vm[2];
      const double vvp = l0 * Vp[0] + l1 * Vp[1] + l2 * Vp[2];
      double cf[5];
      p0_coeffs_1d(wm, wc, wp, vvm, vvp, cf);
      TR C[5], pts[4], qm;
      hweno_1d<TR>(P, cf, wc, wc - wm, wp - wc, fabs(wm), fabs(wc), fabs(wp), C);
      eval_1d<TR>(C, pts, qm);
#pragma unroll
      for (int g = 0; g < 4; ++g) q[g] = (double)pts[g];
      q[4] = (double)qm;
    };
    double S[5], D[5], Q[5];  // q[0..3] point values, q[4] the moment
    field(0.5 * (b2 + u * ci), -0.5 * (b1 * u + ci), 0.5 * b1, Q);
    field(0.5 * (b2 - u * ci), -0.5 * (b1 * u - ci), 0.5 * b1, S);
#pragma unroll
    for (int g = 0; g < 5; ++g) {
      D[g] = S[g] - Q[g];
      S[g] = S[g] + Q[g];
    }
    field(1.0 - b2, b1 * u, -b1, Q);
#pragma unroll
    for (int g = 0; g < 5; ++g) {
      const double rho = S[g] + Q[g];
      const TR mom = (TR)(u * rho + c * D[g]);
      const TR en = (TR)(H * S[g] + (u * c) * D[g] + (0.5 * u * u) * Q[g]);
      if (g < 4) {
        pt[g][0] = (TR)rho;
        pt[g][1] = mom;
        pt[g][2] = en;
      } else {
        vh[0] = (TR)rho;
        vh[1] = mom;
        vh[2] = en;
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      double c[5];
      p0_coeffs_1d(Um[k], Uc[k], Up[k], Vm[k], Vp[k], c);
      TR C[5];
      hweno_1d<TR>(P, c, Uc[k], Uc[k] - Um[k], Up[k] - Uc[k], fabs(Um[k]), fabs(Uc[k]),
                   fabs(Up[k]), C);
      TR q[4];
      eval_1d<TR>(C, q, vh[k]);
#pragma unroll
      for (int g = 0; g < 4; ++g) pt[g][k] = q[g];
    }
  }

  // ---- fluxes: the lane on the right of x_{i-1/2} evaluates it ----
  TR um[NC], up[NC], fl[NC], fr[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    um[k] = from_prev(pt[3][k]);
    up[k] = pt[0][k];
  }
  lf_flux2<EQ, NC, 0, TR>(P, um, up, alpha, fl);  // twice the flux
#pragma unroll
  for (int k = 0; k < NC; ++k) fr[k] = from_next(fl[k]);

  // volume term: Gauss-Lobatto quadrature of f over the cell
  TR vol[NC];
  {
    TR f[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) vol[k] = (TR)0;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      TR q[NC];
#pragma unroll
      for (int k = 0; k < NC; ++k) q[k] = pt[g][k];
      phys_flux<EQ, NC, 0, TR>(P, q, f);
      const TR wg = (TR)((g == 0 || g == 3) ? GL4W0 : GL4W1);
#pragma unroll
      for (int k = 0; k < NC; ++k) vol[k] += wg * f[k];
    }
  }

  // ---- semi-discrete right-hand sides ----
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    F1[k] = -((double)fr[k] - (double)fl[k]) * (0.5 * idx);
    F2[k] = -(fl[k] + fr[k]) * (TR)(0.25 * idx) + vol[k] * (TR)idx;
  }
}

}  // namespace hwenou
