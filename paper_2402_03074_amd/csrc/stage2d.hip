// One fused HWENO-U Runge-Kutta stage in 2D (Section 2.2): the true-2D
// quartic reconstruction on the 3x3 stencil (Step 1), smoothness indicators
// and scale-invariant weights (Steps 2-3), the modified moments v^, w^, the
// 21 point values, Lax-Friedrichs fluxes at the 3 Gauss points of every
// edge, the right-hand sides F1, F2, F3 of Eq. (2.16) and the modified
// SSP-RK3 update (Step 4).
//
// Euler: the reconstruction runs on local characteristic variables in two
// direction-split sweeps (Remark 2.2).  The y-sweep projects the stencil with
// the eigenvectors of g' at the cell average and yields the y-edge values,
// the interior values used for g, and w^; the x-sweep does the same with f'
// for the x-edges, f and v^.  Each characteristic field is reconstructed
// independently and the combined polynomials are mapped back to conserved
// variables before they are evaluated.  Scalar laws (and component-wise
// Euler) use one reconstruction for both directions.
//
// Mapping: a wave (one 64-thread block) marches a strip of 62 output columns
// upward, one row per step; lane l holds column strip*62 - 1 + l (lanes 0 and
// 63 only supply the neighbour columns' x-edge values).  The three stencil
// rows live in a ring of LDS rows shared by the wave; the row after next is
// prefetched into registers while the current row is computed.  x-interface
// values and fluxes move between lanes by shuffles.  The upper y-edge values
// of the previous row and that row's partially accumulated right-hand side
// stay in registers, so every flux is evaluated once and every row written
// once.  Waves take balanced runs of (strip, rows) from a per-wave work list:
// one persistent launch covers one large grid or many instances of uneven
// size.
#include <algorithm>

#include "field2d.hpp"

namespace hwenou {

// CHAR (Euler): 0 component-wise; 1 direction-split characteristic sweeps;
// 2 one reconstruction in x-characteristic variables for every output;
// 3 as 1, with the edge values at each interface reconstructed in the basis
// of the Roe average of the two cells that share it (three reconstructions
// per cell and direction: low interface, high interface, own average for the
// interior values and the moment).
// SI: scale-invariant weights compiled in (else the mode comes from P).
// ST: the Runge-Kutta stage (0, 1, 2), so that its coefficients and the
// stage-0-only stores are compiled in.
// One wave per block and one resident wave per SIMD (the row state needs
// 256 VGPRs plus 85-252 AGPRs).
template <int EQ, int CHAR, bool SI, int ST, class TR, class TM>
__global__ __launch_bounds__(64, 1) void stage2d_kernel(const StageArgs<TM> A) {
  constexpr int NC = EQ == EQ_EULER ? 4 : 1;
  constexpr bool PROJ = EQ == EQ_EULER && CHAR != 0;   // characteristic variables
  constexpr bool SPLIT = EQ == EQ_EULER && (CHAR == 1 || CHAR == 3);  // an x-direction sweep
  constexpr bool IFACE = EQ == EQ_EULER && CHAR == 3;  // interface bases for edge values
  __shared__ RowBuf<NC, TM> B;
  __shared__ TR c1buf[16][64];  // entropy-field polynomial shared by the two sweeps
  // p0 and cross values of the field P shared by the two sweeps
  __shared__ double pbuf[CHAR == 1 && EQ == EQ_EULER && sizeof(TR) == 8 ? 20 : 1][64];
  // per-interface bases: the edge values of the low and the high edge of the
  // current direction, parked while the cell's own basis is reconstructed
  __shared__ TR ebuf[IFACE ? 2 * 3 * NC : 1][64];
  const int lane = threadIdx.x;
  const int w = blockIdx.x;
  if (w >= A.n_waves) return;
  const SchemeParams& P = A.P;
  // out = ra * base + rb * (in + dt F)
  constexpr double ra = ST == 0 ? 0.0 : (ST == 1 ? 0.75 : 1.0 / 3.0);
  constexpr double rb = ST == 0 ? 1.0 : (ST == 1 ? 0.25 : 2.0 / 3.0);
  const long long plane = A.plane;
  const double gm1 = P.gas_gamma - 1.0;

  // the work list and the records of a run's instance are scalar loads
  const int it_end = load_invariant(A.work_ptr + w + 1);
  for (int it = load_invariant(A.work_ptr + w); it < it_end; ++it) {
    const WorkItem wk = load_invariant(A.work + it);
    const InstDev I = load_invariant(A.inst + wk.inst);
    double dt, alpha_x, alpha_y;
    if (A.ctl.run == nullptr) {
      dt = load_invariant(A.dt + wk.inst);
      alpha_x = load_invariant(A.alpha + 2 * wk.inst);
      alpha_y = load_invariant(A.alpha + 2 * wk.inst + 1);
    } else {
      const StepDt d = step_dt<2>(A.ctl, wk.inst, I);
      if (ST == 2 && wk.a == 0 && wk.b == 0 && lane == 0) write_step(A.ctl, wk.inst, d);
      if (d.done) continue;
      dt = uniform(d.dt);
      alpha_x = uniform(d.ax);
      alpha_y = uniform(d.ay);
    }
    const int nx = I.nx, ny = I.ny;
    const int c0 = wk.a * kStripWidth;
    int i = c0 - 1 + lane;
    if (i > nx) i = nx;
    const bool col_owner = lane >= 1 && lane <= kStripWidth && i < nx;
    // byte offsets of this lane's column in a row (clamped into the row, so
    // that loads need no lane mask; only owners store)
    const int ic = min(max(i, 0), nx - 1);
    const unsigned ou = (unsigned)ic * 8u, om = (unsigned)ic * (unsigned)sizeof(TM);
    const TR a1 = (TR)alpha_x, a2 = (TR)alpha_y;
    const double idx = uniform(1.0 / I.dx), idy = uniform(1.0 / I.dy);
    const int r0 = wk.b, r1 = wk.c;
    const double* u_in = A.u_in + I.offset;
    const TM* m_in = A.m_in + I.offset;

    // grid columns of the LDS columns this lane loads (clamped, then wrapped)
    const int gx0 = wrap_index(min(c0 - 2 + lane, nx + 1), nx, I.bc[0], I.bc[1]);
    const int gx1 = wrap_index(min(c0 + 62 + (lane & 1), nx + 1), nx, I.bc[0], I.bc[1]);
    const bool walls = EQ == EQ_EULER && (I.bc[0] == BC_REFLECTIVE || I.bc[1] == BC_REFLECTIVE ||
                                          I.bc[2] == BC_REFLECTIVE || I.bc[3] == BC_REFLECTIVE);
    const bool extra = lane < 2;
    // a row on its way to the ring
    const RowLoader<NC, TM> rows(u_in, m_in, plane, lane, gx0, gx1);
    auto fetch = [&](int row, RowRegs<NC, TM>& R) {
      rows.load((long long)wrap_index(row, ny, I.bc[2], I.bc[3]) * nx, R);
    };
    // Reflective walls: the stored cells of grid row `row` that are mirror
    // images (ghost columns beyond an x-wall, or the whole row beyond a
    // y-wall) get the signs of the mirror image: the wall-normal momentum
    // and the moments along the wall normal change sign (twice for the x-
    // moment of the x-momentum and the y-moment of the y-momentum).  Runs
    // after the row is in LDS, outside the register-heavy part of the row.
    auto mirror_row = [&](int slot, int row) {
      const bool my = (row < 0 && I.bc[2] == BC_REFLECTIVE) ||
                      (row >= ny && I.bc[3] == BC_REFLECTIVE);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        if (e == 1 && !extra) break;
        const int c = e == 0 ? c0 - 2 + lane : c0 + 62 + lane;  // grid column
        const bool mx = (c < 0 && I.bc[0] == BC_REFLECTIVE) ||
                        (c >= nx && I.bc[1] == BC_REFLECTIVE);
        if (!(mx || my)) continue;
        const int l = e == 0 ? lane : 64 + lane;
        double uu[NC], mm[2][NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          uu[k] = B.u[slot][k][l];
          mm[0][k] = B.m[slot][0][k][l];
          mm[1][k] = B.m[slot][1][k][l];
        }
        if (mx) mirror_cell<0, NC>(uu, mm, 2);
        if (my) mirror_cell<1, NC>(uu, mm, 2);
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          B.u[slot][k][l] = uu[k];
          B.m[slot][0][k][l] = mm[0][k];
          B.m[slot][1][k][l] = mm[1][k];
        }
      }
    };
    auto store = [&](int slot, int row, const RowRegs<NC, TM>& R) {
      rows.store(B, slot, R);
      if constexpr (EQ == EQ_EULER) {
        if (walls) mirror_row(slot, row);
      }
    };
    __syncthreads();  // the previous item's reads of B are complete
    // prologue: rows r0-2 .. r0 into ring slots 0..2, r0+1 into registers, all
    // four loaded together
    RowRegs<NC, TM> next;
    {
      RowRegs<NC, TM> R[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) fetch(r0 - 2 + q, R[q]);
      fetch(r0 + 1, next);
#pragma unroll
      for (int q = 0; q < 3; ++q) store(q, r0 - 2 + q, R[q]);
    }
    __syncthreads();

    // state carried from the row below (pending right-hand side of row j-1)
    TR yprev[3][NC];
    double F1p[NC];
    TR F2p[NC], F3p[NC], vhp[NC], whp[NC];
    double amax_x = 0.0, amax_y = 0.0;
    bool ok = true;

    int sb = 0, sc = 1, st = 2;  // ring slots of rows j-1, j, j+1
    for (int j = r0 - 1; j <= r1; ++j) {
      const bool row_out = j >= r0 && j < r1;
      const bool fin = j - 1 >= r0 && j - 1 < r1;  // row j-1 is finished in this step

      // base (u^n, v^n, w^n) of row j-1, loaded now and used after the y-sweep
      double ubase[NC];
      TM vbase[NC], wbase[NC];
      const long long orow = I.offset + (long long)(j - 1) * nx;  // row j-1
      if (ST != 0 && fin) {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          ubase[k] = load_at(A.u_base + (k * plane + orow), ou);
          vbase[k] = load_at(A.m_base + (k * plane + orow), om);
          wbase[k] = load_at(A.m_base + ((NC + k) * plane + orow), om);
        }
      }

      // ---- reconstruction of row j, y-direction ----
      TR Cc[NC][15];
      Prim pr;
      if constexpr (IFACE) {
        auto roe_rows = [&](int sl, int sr) {  // Roe basis of rows sl (below) and sr (above)
          double UL[4], UR[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            UL[k] = B.u[sl][k][lane + 1];
            UR[k] = B.u[sr][k][lane + 1];
          }
          return make_prim_roe<TR>(gm1, UL, UR);
        };
        // top edge, eta = +1/2, in the basis of y_{j+1/2}
        char_sweep<1, SI, false, false, TR, TM>(P, roe_rows(sc, st), B, sb, sc, st, lane, Cc, c1buf,
                                         pbuf, false);
#pragma unroll
        for (int G = 0; G < 3; ++G)
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            TR d[5], e0, e1, g0, g1, g2;
            restrict_xi_line<TR>(Cc[k], G, d);
            eval5<TR>(d, e0, e1, g0, g1, g2);
            ebuf[(3 + G) * NC + k][lane] = e1;
          }
        __builtin_amdgcn_sched_barrier(0);
        if (j >= r0) {
          // bottom edge, eta = -1/2, in the basis of y_{j-1/2}
          char_sweep<1, SI, false, false, TR, TM>(P, roe_rows(sb, sc), B, sb, sc, st, lane, Cc, c1buf,
                                           pbuf, false);
#pragma unroll
          for (int G = 0; G < 3; ++G)
#pragma unroll
            for (int k = 0; k < NC; ++k) {
              TR d[5], e0, e1, g0, g1, g2;
              restrict_xi_line<TR>(Cc[k], G, d);
              eval5<TR>(d, e0, e1, g0, g1, g2);
              ebuf[G * NC + k][lane] = e0;
            }
          __builtin_amdgcn_sched_barrier(0);
          // interior values and w^ in the cell's own basis
          double U5[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) U5[k] = B.u[sc][k][lane + 1];
          pr = make_prim<TR>(gm1, U5);
          char_sweep<1, SI, true, false, TR, TM>(P, pr, B, sb, sc, st, lane, Cc, c1buf, pbuf, false);
        }
      } else if constexpr (PROJ) {
        double U5[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) U5[k] = B.u[sc][k][lane + 1];
        pr = make_prim<TR>(gm1, U5);
        char_sweep<SPLIT ? 1 : 0, SI, SPLIT, SPLIT, TR, TM, SPLIT && SI && sizeof(TR) == 8>(
            P, pr, B, sb, sc, st, lane, Cc, c1buf, pbuf, false);
      } else {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          Sten2 S;
          Field F;
          read_stencil<NC, TM>(B, sb, sc, st, lane, k, S);
          make_field<TR>(S, F);
          recon_field<TR, SI>(P, F, Cc[k]);
        }
      }
      if constexpr (SPLIT && !IFACE) pin(Cc);
      // y-edges at (xi_G, -+1/2), interior values for g (and f when the
      // reconstruction is shared), y-fluxes at y_{j-1/2}
      TR F1n_s[NC], F2n[NC], F3n[NC];  // new row: bottom-flux terms
      double F1n[NC];
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        F1n[k] = 0.0;
        F2n[k] = (TR)0;
        F3n[k] = (TR)0;
        F1n_s[k] = (TR)0;
      }
      TR volf[NC], volg[NC];
#pragma unroll
      for (int k = 0; k < NC; ++k) volf[k] = volg[k] = (TR)0;
#pragma unroll
      for (int G = 0; G < 3; ++G) {
        const TR xg = (TR)g3x(G);
        TR ym[NC], yp[NC], in[3][NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          TR d[5];
          restrict_xi_line<TR>(Cc[k], G, d);
          eval5<TR>(d, ym[k], yp[k], in[0][k], in[1][k], in[2][k]);
          if constexpr (IFACE) {
            ym[k] = ebuf[G * NC + k][lane];
            yp[k] = ebuf[(3 + G) * NC + k][lane];
          }
        }
        if (row_out) {
#pragma unroll
          for (int H = 0; H < 3; ++H) {
            const TR wgt = (TR)(g3w(G) * g3w(H));
            TR g[NC];
            phys_flux<EQ, NC, 1, TR>(P, in[H], g);
#pragma unroll
            for (int k = 0; k < NC; ++k) volg[k] += wgt * g[k];
            if constexpr (!SPLIT) {
              TR f[NC];
              phys_flux<EQ, NC, 0, TR>(P, in[H], f);
#pragma unroll
              for (int k = 0; k < NC; ++k) volf[k] += wgt * f[k];
            }
          }
        }
        if (j >= r0) {
          // u- = row below at eta = +1/2, u+ = this row at eta = -1/2
          TR gb[NC];
          lf_flux2<EQ, NC, 1, TR>(P, yprev[G], ym, a2, gb);  // twice the flux
          const TR wg = (TR)(0.5 * g3w(G));
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            F1n_s[k] += wg * gb[k];       // sum_G w_G g_{G,j-1/2}
            if (G != 1) F2n[k] += wg * xg * gb[k];  // sum_G w_G xi_G g_{G,j-1/2} (xi_1 = 0)
          }
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) yprev[G][k] = yp[k];
      }
      if (j >= r0) {
        // the same sums close row j-1 (upper edge) and open row j (lower edge)
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          F1p[k] -= (double)F1n_s[k] * idy;
          F2p[k] -= F2n[k] * (TR)idy;
          F3p[k] -= F1n_s[k] * (TR)(0.5 * idy);
          F3n[k] = -F1n_s[k] * (TR)(0.5 * idy);
          F2n[k] = F2n[k] * (TR)idy;
        }
      }
      TR whn[NC];
#pragma unroll
      for (int k = 0; k < NC; ++k) whn[k] = qw_2d<TR>(Cc[k]);

      // ---- row j-1 is complete: Runge-Kutta update and store ----
      if (fin) {
        if (col_owner) {
          double Uo[NC];
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            const double uin = B.u[sb][k][lane + 1];
            const double ub = ST == 0 ? 0.0 : ubase[k];
            const double un = ra * ub + rb * (uin + dt * F1p[k]);
            TR vn, wn;
            if (ST == 0) {
              store_at(A.m_base + (k * plane + orow), om, (TM)vhp[k]);
              store_at(A.m_base + ((NC + k) * plane + orow), om, (TM)whp[k]);
              vn = vhp[k] + (TR)dt * F2p[k];
              wn = whp[k] + (TR)dt * F3p[k];
            } else {
              const TR vb = (TR)vbase[k];
              const TR wb = (TR)wbase[k];
              vn = (TR)ra * vb + (TR)rb * (vhp[k] + (TR)dt * F2p[k]);
              wn = (TR)ra * wb + (TR)rb * (whp[k] + (TR)dt * F3p[k]);
            }
            store_at(A.u_out + (k * plane + orow), ou, un);
            store_at(A.m_out + (k * plane + orow), om, (TM)vn);
            store_at(A.m_out + ((NC + k) * plane + orow), om, (TM)wn);
            Uo[k] = un;
          }
          if constexpr (ST == 2) {  // the wave speeds feed the next step's alpha
            double sx, sy;
            ok = wave_speeds<EQ, NC>(P, Uo, sx, sy) && ok;
            amax_x = fmax(amax_x, sx);
            amax_y = fmax(amax_y, sy);
          } else {
            ok = physical_state<EQ, NC>(Uo) && ok;
          }
        }
      }

      if (row_out) {
        // ---- x-direction reconstruction of row j ----
        if constexpr (IFACE) {
          auto roe_cols = [&](int cl) {  // Roe basis of columns cl (left) and cl + 1
            double UL[4], UR[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              UL[k] = B.u[sc][k][lane + cl];
              UR[k] = B.u[sc][k][lane + cl + 1];
            }
            return make_prim_roe<TR>(gm1, UL, UR);
          };
          // left edge, xi = -1/2, in the basis of x_{i-1/2}
          char_sweep<0, SI, false, false, TR, TM>(P, roe_cols(0), B, sb, sc, st, lane, Cc, c1buf,
                                           pbuf, false);
#pragma unroll
          for (int H = 0; H < 3; ++H)
#pragma unroll
            for (int k = 0; k < NC; ++k) {
              TR d[5], e0, e1, g0, g1, g2;
              restrict_eta_line<TR>(Cc[k], H, d);
              eval5<TR>(d, e0, e1, g0, g1, g2);
              ebuf[H * NC + k][lane] = e0;
            }
          __builtin_amdgcn_sched_barrier(0);
          // right edge, xi = +1/2, in the basis of x_{i+1/2}
          char_sweep<0, SI, false, false, TR, TM>(P, roe_cols(1), B, sb, sc, st, lane, Cc, c1buf,
                                           pbuf, false);
#pragma unroll
          for (int H = 0; H < 3; ++H)
#pragma unroll
            for (int k = 0; k < NC; ++k) {
              TR d[5], e0, e1, g0, g1, g2;
              restrict_eta_line<TR>(Cc[k], H, d);
              eval5<TR>(d, e0, e1, g0, g1, g2);
              ebuf[(3 + H) * NC + k][lane] = e1;
            }
          __builtin_amdgcn_sched_barrier(0);
          double U5[4];  // the own primitives again (cheaper than keeping them live)
#pragma unroll
          for (int k = 0; k < 4; ++k) U5[k] = B.u[sc][k][lane + 1];
          pr = make_prim<TR>(gm1, U5);
        }
        if constexpr (SPLIT)
          char_sweep<0, SI, false, !IFACE, TR, TM, !IFACE && SI && sizeof(TR) == 8>(P, pr, B, sb, sc, st, lane,
                                                                      Cc, c1buf, pbuf, true);
        if constexpr (SPLIT && !IFACE) pin(Cc);
        double F1x[NC];
        TR F2x[NC], F3x[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          F1x[k] = 0.0;
          F2x[k] = F3x[k] = (TR)0;
        }
#pragma unroll
        for (int H = 0; H < 3; ++H) {
          const TR yh = (TR)g3x(H);
          TR xm[NC], xp[NC], in[3][NC];
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            TR d[5];
            restrict_eta_line<TR>(Cc[k], H, d);
            eval5<TR>(d, xm[k], xp[k], in[0][k], in[1][k], in[2][k]);
            if constexpr (IFACE) {
              xm[k] = ebuf[H * NC + k][lane];
              xp[k] = ebuf[(3 + H) * NC + k][lane];
            }
          }
          if constexpr (SPLIT) {
#pragma unroll
            for (int G = 0; G < 3; ++G) {
              TR f[NC];
              phys_flux<EQ, NC, 0, TR>(P, in[G], f);
              const TR wgt = (TR)(g3w(G) * g3w(H));
#pragma unroll
              for (int k = 0; k < NC; ++k) volf[k] += wgt * f[k];
            }
          }
          // x_{i-1/2} at eta_H: u- = left lane at +1/2, u+ = this lane at -1/2
          TR um[NC], fl[NC], fr[NC];
#pragma unroll
          for (int k = 0; k < NC; ++k) um[k] = from_prev(xp[k]);
          lf_flux2<EQ, NC, 0, TR>(P, um, xm, a1, fl);  // twice the flux
#pragma unroll
          for (int k = 0; k < NC; ++k) fr[k] = from_next(fl[k]);
          const TR wg = (TR)(0.5 * g3w(H));
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            F1x[k] += (double)wg * ((double)fr[k] - (double)fl[k]);
            F2x[k] += wg * (fl[k] + fr[k]);
            if (H != 1) F3x[k] += wg * yh * (fr[k] - fl[k]);  // eta_1 = 0
          }
        }
        // pending right-hand side of row j
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          F1p[k] = -F1x[k] * idx + (double)F1n_s[k] * idy;
          F2p[k] = -F2x[k] * (TR)(0.5 * idx) + volf[k] * (TR)idx + F2n[k];
          F3p[k] = -F3x[k] * (TR)idx + volg[k] * (TR)idy + F3n[k];
          vhp[k] = qv_2d<TR>(Cc[k]);
          whp[k] = whn[k];
        }
      }

      // ---- advance the LDS ring: row j+2 from registers, prefetch j+3 ----
      __syncthreads();
      if (j + 2 <= r1 + 1) store(sb, j + 2, next);  // row j-1's slot takes row j+2
      if (j + 3 <= r1 + 1) fetch(j + 3, next);
      __syncthreads();
      const int s0 = sb;
      sb = sc;
      sc = st;
      st = s0;
    }
    if (!ok) atomicOr(&A.status[wk.inst], 1);
    if (ST == 2 && A.ctl.run != nullptr) {
      const double mx = wave_max(amax_x), my = wave_max(amax_y);
      if (lane == 0) {
        double* acc = A.ctl.acc_out + alpha_slot(wk.inst, blockIdx.x, A.ctl.slots);
        atomic_max_nonneg(acc, mx);
        atomic_max_nonneg(acc + 1, my);
      }
    }
  }
}

template <int EQ, int CHAR, bool SI, class TR, class TM>
static hipError_t launch(const void* args, int blocks, int threads, hipStream_t s) {
  const auto& a = *static_cast<const StageArgs<TM>*>(args);
  switch (a.stage) {
    case 0:
      hipLaunchKernelGGL((stage2d_kernel<EQ, CHAR, SI, 0, TR, TM>), dim3(blocks), dim3(threads), 0,
                         s, a);
      break;
    case 1:
      hipLaunchKernelGGL((stage2d_kernel<EQ, CHAR, SI, 1, TR, TM>), dim3(blocks), dim3(threads), 0,
                         s, a);
      break;
    default:
      hipLaunchKernelGGL((stage2d_kernel<EQ, CHAR, SI, 2, TR, TM>), dim3(blocks), dim3(threads), 0,
                         s, a);
  }
  return hipGetLastError();
}

template <bool SI, class TR>
static hipError_t launch_t(int eq, int char_mode, const void* args, int blocks, int threads,
                           hipStream_t s) {
  switch (eq) {
    case EQ_ADVECTION: return launch<EQ_ADVECTION, 0, SI, TR, TR>(args, blocks, threads, s);
    case EQ_BURGERS: return launch<EQ_BURGERS, 0, SI, TR, TR>(args, blocks, threads, s);
    default:
      if (char_mode == 3) return launch<EQ_EULER, 3, SI, TR, TR>(args, blocks, threads, s);
      if (char_mode == 2) return launch<EQ_EULER, 2, SI, TR, TR>(args, blocks, threads, s);
      return char_mode ? launch<EQ_EULER, 1, SI, TR, TR>(args, blocks, threads, s)
                       : launch<EQ_EULER, 0, SI, TR, TR>(args, blocks, threads, s);
  }
}

hipError_t launch_stage_2d(int eq, int char_mode, bool mixed, bool scale_invariant,
                           const void* args, int blocks, int threads, hipStream_t s) {
  if (scale_invariant)
    return mixed ? launch_t<true, float>(eq, char_mode, args, blocks, threads, s)
                 : launch_t<true, double>(eq, char_mode, args, blocks, threads, s);
  return mixed ? launch_t<false, float>(eq, char_mode, args, blocks, threads, s)
               : launch_t<false, double>(eq, char_mode, args, blocks, threads, s);
}

template <int EQ, int CHAR, bool SI, int ST, class TR>
static int occupancy_st(int threads) {
  int blocks = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &blocks, stage2d_kernel<EQ, CHAR, SI, ST, TR, TR>, threads, 0) != hipSuccess)
    return 0;
  return blocks;
}

// resident blocks per CU common to the three stage kernels
template <int EQ, int CHAR, bool SI, class TR>
static int occupancy(int threads) {
  return std::min(occupancy_st<EQ, CHAR, SI, 0, TR>(threads),
                  std::min(occupancy_st<EQ, CHAR, SI, 1, TR>(threads),
                           occupancy_st<EQ, CHAR, SI, 2, TR>(threads)));
}

template <bool SI, class TR>
static int occupancy_t(int eq, int char_mode, int threads) {
  switch (eq) {
    case EQ_ADVECTION: return occupancy<EQ_ADVECTION, 0, SI, TR>(threads);
    case EQ_BURGERS: return occupancy<EQ_BURGERS, 0, SI, TR>(threads);
    default:
      if (char_mode == 3) return occupancy<EQ_EULER, 3, SI, TR>(threads);
      if (char_mode == 2) return occupancy<EQ_EULER, 2, SI, TR>(threads);
      return char_mode ? occupancy<EQ_EULER, 1, SI, TR>(threads)
                       : occupancy<EQ_EULER, 0, SI, TR>(threads);
  }
}

int occupancy_stage_2d(int eq, int char_mode, bool mixed, bool scale_invariant, int threads) {
  if (scale_invariant)
    return mixed ? occupancy_t<true, float>(eq, char_mode, threads)
                 : occupancy_t<true, double>(eq, char_mode, threads);
  return mixed ? occupancy_t<false, float>(eq, char_mode, threads)
               : occupancy_t<false, double>(eq, char_mode, threads);
}

}  // namespace hwenou
