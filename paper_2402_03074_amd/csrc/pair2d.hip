// The 2D Euler stage in direction-split characteristic variables (the default
// mode), FP64, by pairs of waves: the same operator, strips, rows and work lists
// as stage2d.hip, with the two sweeps of a row on two waves of one block.
//
// What bounds it: a wave's row is one chain of dependent FP64 instructions (a
// SIMD holds one wave of 500 registers; VALU active ~75%), and a grid whose runs
// are a row or two leaves nothing else to overlap: its stage takes the start, the
// two boundary rows and the rows of one run, whatever the rest of the chip does.
// Two waves halve the chain: the y wave reconstructs in y and forms the y-fluxes,
// the x wave reconstructs in x, updates and stores.  Per row they exchange the
// entropy field's polynomial and the y wave's flux sums through LDS, and work one
// row apart, so that the x wave's update of a row runs beside the y wave's next
// sweep.  131 x 97 grid with walls: 760 -> 612 us per 10 Runge-Kutta steps.
// Two pairs per SIMD pair (256 registers) spill 500-1100 B per lane and are slower.
// In mixed precision one wave stays: there the two kernels' FP64 parts would have
// to be rounded alike by pin and mad, with which the one-wave kernels spill.
#include <algorithm>

#include "field2d.hpp"

namespace hwenou {

// LDS rows of the ring: the three of the current row's stencils and the one
// being loaded.
constexpr int kPairRows = 4;

using TR = double;
using TM = double;

// One sweep of a row.  DIR = 1 (the y wave) reconstructs the entropy field,
// hands it over through c1buf and takes the shear field last; DIR = 0 (the x
// wave) takes the shear field first and then the entropy field from c1buf.
// The barrier inside is the handover; both waves of a block meet it once per
// row.  See char_sweep for the fields.  The entropy field's p0 coefficients are
// formed by both waves (they are linear in P and the density, which both have);
// only its combined coefficients 0..2 and the factor change hands.
template <int DIR, bool SI>
__device__ __forceinline__ void pair_sweep(const SchemeParams& P, const Prim& pr,
                                           const RowBuf<4, TM, kPairRows>& B, int sb, int sc,
                                           int st, int l, TR (&Cc)[4][15], TR (*c1buf)[64]) {
  constexpr int nd = DIR == 0 ? 1 : 2, td = DIR == 0 ? 2 : 1;  // normal, tangential momentum
  const double un = DIR == 0 ? pr.u : pr.v, ut = DIR == 0 ? pr.v : pr.u;
  TR C[15], S[15], D[15], C1[15];
  double a, a1, a2;
  Field FP;
  {
    Field FN, F;
    const double hc = 0.5 * pr.ci;
    Sten2 W, WP, WN;
    const double hb = 0.5 * pr.b1;
    read_stencil<4, TM>(B, sb, sc, st, l, 0, W);
    add_stencil<true, 4, TM>(0.5 * pr.b2, W, WP);
    // P in one order on both waves, so that their entropy fields agree bitwise
    if constexpr (DIR == 1) {
      read_stencil<4, TM>(B, sb, sc, st, l, 2, WN);
      add_stencil<false, 4, TM>(-hb * pr.v, WN, WP);
      add_stencil<false, 4, TM>(-un, W, WN);
      read_stencil<4, TM>(B, sb, sc, st, l, 1, W);
      add_stencil<false, 4, TM>(-hb * pr.u, W, WP);
    } else {
      Sten2 T;
      read_stencil<4, TM>(B, sb, sc, st, l, 2, T);
      add_stencil<false, 4, TM>(-hb * pr.v, T, WP);
      read_stencil<4, TM>(B, sb, sc, st, l, 1, WN);
      add_stencil<false, 4, TM>(-hb * pr.u, WN, WP);
      add_stencil<false, 4, TM>(-un, W, WN);
    }
    read_stencil<4, TM>(B, sb, sc, st, l, 3, W);
    add_stencil<false, 4, TM>(hb, W, WP);
    make_field<TR>(WP, FP);
    make_field<TR>(WN, FN);
    __builtin_amdgcn_sched_barrier(0);
    add_fields(FP, -hc, FN, F);
    recon_field<TR, SI, true>(P, F, C, &a);
#pragma unroll
    for (int n = 0; n < 15; ++n) S[n] = n < 3 ? C[n] : a * C[n];  // P0
    __builtin_amdgcn_sched_barrier(0);
    add_fields(FP, hc, FN, F);
    recon_field<TR, SI, true>(P, F, C, &a);
#pragma unroll
    for (int n = 0; n < 15; ++n) {
      const TR p0 = S[n];
      const TR f = n < 3 ? 1.0 : a;
      S[n] = mad(f, C[n], p0);
      D[n] = mad(f, C[n], -p0);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  {
    Field FR;
    Sten2 W;
    read_stencil<4, TM>(B, sb, sc, st, l, 0, W);
    make_field<TR>(W, FR);
    add_fields(FR, -2.0, FP, FR);
    if constexpr (DIR == 1) {
      recon_field<TR, SI, true>(P, FR, C1, &a1);
    } else {
#pragma unroll
      for (int n = 0; n < 15; ++n) C1[n] = FR.c[n];
    }
  }
  auto shear = [&] {
    Field FT;
    relative_momentum<TR, TM>(B, sb, sc, st, l, td, ut, FT);
    recon_field<TR, SI, true>(P, FT, C, &a2);
  };
  if constexpr (DIR == 1) {
#pragma unroll
    for (int n = 0; n < 3; ++n) c1buf[n][l] = C1[n];
    c1buf[3][l] = a1;
    __syncthreads();
  } else {
    __builtin_amdgcn_sched_barrier(0);
    shear();
    __syncthreads();
#pragma unroll
    for (int n = 0; n < 3; ++n) C1[n] = c1buf[n][l];
    a1 = c1buf[3][l];
  }
  {
    const TR unc = un * pr.c, h = 0.5 * pr.q2, ha1 = 0.5 * pr.q2 * a1;
#pragma unroll
    for (int n = 0; n < 15; ++n) {
      const TR f1 = n < 3 ? 1.0 : a1, fh = n < 3 ? h : ha1;
      Cc[0][n] = mad(f1, C1[n], S[n]);
      Cc[nd][n] = mad(un, Cc[0][n], pr.c * D[n]);
      Cc[3][n] = mad(fh, C1[n], mad(unc, D[n], pr.H * S[n]));
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (DIR == 1) shear();
  {
    const TR uta2 = ut * a2;
#pragma unroll
    for (int n = 0; n < 15; ++n) {
      const TR f2 = n < 3 ? 1.0 : a2, fu = n < 3 ? ut : uta2;
      Cc[td][n] = mad(f2, C[n], ut * Cc[0][n]);
      Cc[3][n] = mad(fu, C[n], Cc[3][n]);
    }
  }
}

// SI, ST: as for the one-wave kernels.
template <bool SI, int ST>
__global__ __launch_bounds__(128, 1) void stage2d_pair_kernel(const StageArgs<double> A) {
  constexpr int NC = 4;
  __shared__ RowBuf<NC, TM, kPairRows> B;
  __shared__ double c1buf[4][64];
  __shared__ TR gbuf[4 * NC][64];  // what the y wave leaves of a row
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool ywave = wave == 0;
  const int w = blockIdx.x;
  if (w >= A.n_waves) return;
  const SchemeParams& P = A.P;
  // out = ra * base + rb * (in + dt F)
  constexpr double ra = ST == 0 ? 0.0 : (ST == 1 ? 0.75 : 1.0 / 3.0);
  constexpr double rb = ST == 0 ? 1.0 : (ST == 1 ? 0.25 : 2.0 / 3.0);
  const long long plane = A.plane;
  const double gm1 = P.gas_gamma - 1.0;

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
      if (ST == 2 && wk.a == 0 && wk.b == 0 && threadIdx.x == 64) write_step(A.ctl, wk.inst, d);
      if (d.done) continue;
      dt = uniform(d.dt);
      alpha_x = uniform(d.ax);
      alpha_y = uniform(d.ay);
    }
    const int nx = I.nx, ny = I.ny;
    const int c0 = wk.a * kStripWidth;
    const double idx = uniform(1.0 / I.dx), idy = uniform(1.0 / I.dy);
    const int r0 = wk.b, r1 = wk.c;
    const double* u_in = A.u_in + I.offset;
    const TM* m_in = A.m_in + I.offset;

    // a row's columns of the ring: this lane's, and for lanes 0-1 an extra one
    // (grid columns clamped, then wrapped)
    const int gx0 = wrap_index(min(c0 - 2 + lane, nx + 1), nx, I.bc[0], I.bc[1]);
    const int gx1 = wrap_index(min(c0 + 62 + (lane & 1), nx + 1), nx, I.bc[0], I.bc[1]);
    const bool walls = I.bc[0] == BC_REFLECTIVE || I.bc[1] == BC_REFLECTIVE ||
                       I.bc[2] == BC_REFLECTIVE || I.bc[3] == BC_REFLECTIVE;
    const bool extra = lane < 2;
    // a row on its way to the ring
    const RowLoader<NC, TM> rows(u_in, m_in, plane, lane, gx0, gx1);
    auto fetch = [&](int row, RowRegs<NC, TM>& R) {
      rows.load((long long)wrap_index(row, ny, I.bc[2], I.bc[3]) * nx, R);
    };
    // Cells beyond a reflective wall get the signs of the mirror image (see the
    // one-wave kernel).
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
      if (walls) mirror_row(slot, row);
    };
    auto prim = [&](int slot) {
      double U5[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) U5[k] = B.u[slot][k][lane + 1];
      return make_prim<TR>(gm1, U5);
    };
    // Row j is in ring slot (j - r0 + 2) mod 4.
    __syncthreads();  // the previous item's reads of B are complete
    RowRegs<NC, TM> next;  // the x wave's next row of the ring
    if (ywave) {
      RowRegs<NC, TM> a, b;
      fetch(r0 - 2, a);
      fetch(r0 - 1, b);
      store(0, r0 - 2, a);
      store(1, r0 - 1, b);
    } else {
      RowRegs<NC, TM> a;
      fetch(r0, a);
      fetch(r0 + 1, next);
      store(2, r0, a);
    }
    __syncthreads();

    // Two barriers per row: the entropy field's handover inside pair_sweep, and
    // the end of the row, after which the x wave reads what the y wave left in
    // gbuf (until the next handover) and the ring's new row is visible.
    if (ywave) {
      const TR a2 = (TR)alpha_y;
      TR yprev[3][NC];
      for (int j = r0 - 1; j <= r1; ++j) {
        const int q = j - r0 + 1;
        const int sb = q & 3, sc = (q + 1) & 3, st = (q + 2) & 3;
        const bool row_out = j >= r0 && j < r1;
        TR Cc[NC][15];
        pair_sweep<1, SI>(P, prim(sc), B, sb, sc, st, lane, Cc, c1buf);
        pin(Cc);
        // y-edges at (xi_G, -+1/2), interior values for g, y-fluxes at y_{j-1/2}
        TR F1n_s[NC], F2n[NC], volg[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) F1n_s[k] = F2n[k] = volg[k] = (TR)0;
#pragma unroll
        for (int G = 0; G < 3; ++G) {
          const TR xg = (TR)g3x(G);
          TR ym[NC], yp[NC], in[3][NC];
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            TR d[5];
            restrict_xi_line<TR>(Cc[k], G, d);
            eval5<TR>(d, ym[k], yp[k], in[0][k], in[1][k], in[2][k]);
          }
          if (row_out) {
#pragma unroll
            for (int H = 0; H < 3; ++H) {
              const TR wgt = (TR)(g3w(G) * g3w(H));
              TR g[NC];
              phys_flux<EQ_EULER, NC, 1, TR>(P, in[H], g);
#pragma unroll
              for (int k = 0; k < NC; ++k) volg[k] += wgt * g[k];
            }
          }
          if (j >= r0) {
            // u- = row below at eta = +1/2, u+ = this row at eta = -1/2
            TR gb[NC];
            lf_flux2<EQ_EULER, NC, 1, TR>(P, yprev[G], ym, a2, gb);  // twice the flux
            const TR wg = (TR)(0.5 * g3w(G));
#pragma unroll
            for (int k = 0; k < NC; ++k) {
              F1n_s[k] += wg * gb[k];                 // sum_G w_G g_{G,j-1/2}
              if (G != 1) F2n[k] += wg * xg * gb[k];  // sum_G w_G xi_G g_{G,j-1/2}
            }
          }
#pragma unroll
          for (int k = 0; k < NC; ++k) yprev[G][k] = yp[k];
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          gbuf[k][lane] = F1n_s[k];
          gbuf[NC + k][lane] = F2n[k];
          gbuf[2 * NC + k][lane] = volg[k];
          gbuf[3 * NC + k][lane] = qw_2d<TR>(Cc[k]);
        }
        __syncthreads();
      }
    } else {
      int i = c0 - 1 + lane;
      if (i > nx) i = nx;
      const bool col_owner = lane >= 1 && lane <= kStripWidth && i < nx;
      // byte offsets of this lane's column in a row (clamped into the row, so
      // that loads need no lane mask; only owners store)
      const int ic = min(max(i, 0), nx - 1);
      const unsigned ou = (unsigned)ic * 8u, om = (unsigned)ic * (unsigned)sizeof(TM);
      const TR a1 = (TR)alpha_x;
      double F1x[NC], F1p[NC];                  // x part of row j-1, pending sums of row j-2
      TR F2x[NC], F3x[NC], volf[NC], vh[NC];
      TR F2p[NC], F3p[NC], vhp[NC], whp[NC];
      double ubase[NC];
      TM vbase[NC], wbase[NC];
      // the base (u^n, v^n, w^n) of the row to be finished: a pass ahead where the
      // registers hold it
      constexpr bool kBaseEarly = ST != 0;
      auto load_base = [&](int row) {
        const long long brow = I.offset + (long long)row * nx;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          ubase[k] = load_at(A.u_base + (k * plane + brow), ou);
          vbase[k] = load_at(A.m_base + (k * plane + brow), om);
          wbase[k] = load_at(A.m_base + ((NC + k) * plane + brow), om);
        }
      };
      double amax_x = 0.0, amax_y = 0.0;
      bool ok = true;
      for (int j = r0 - 1; j <= r1 + 1; ++j) {
        const int q = j - r0 + 1;
        const int sb = q & 3, sc = (q + 1) & 3, st = (q + 2) & 3, sn = (q + 3) & 3;
        // ---- row j-1's y-fluxes have arrived: row j-2 is complete ----
        const bool fin = j - 2 >= r0;
        const long long orow = I.offset + (long long)(j - 2) * nx;
        if (ST != 0 && !kBaseEarly && fin) load_base(j - 2);
        if (j - 1 >= r0) {
          TR F1n_s[NC], F2n[NC], F3n[NC];
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            F1n_s[k] = gbuf[k][lane];
            F2n[k] = gbuf[NC + k][lane];
            // the same sums close row j-2 (upper edge) and open row j-1 (lower edge)
            F1p[k] -= (double)F1n_s[k] * idy;
            F2p[k] -= F2n[k] * (TR)idy;
            F3p[k] -= F1n_s[k] * (TR)(0.5 * idy);
            F3n[k] = -F1n_s[k] * (TR)(0.5 * idy);
            F2n[k] = F2n[k] * (TR)idy;
            // rounded here, as in the one-wave kernel, and not fused into the sums
            // below: the two kernels' results are the same bits
            asm("" : "+v"(F2n[k]), "+v"(F3n[k]));
          }
          if (fin && col_owner) {
            double Uo[NC];
#pragma unroll
            for (int k = 0; k < NC; ++k) {
              const double uin = B.u[sn][k][lane + 1];  // row j-2, before row j+2 takes its slot
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
              ok = wave_speeds<EQ_EULER, NC>(P, Uo, sx, sy) && ok;
              amax_x = fmax(amax_x, sx);
              amax_y = fmax(amax_y, sy);
            } else {
              ok = physical_state<EQ_EULER, NC>(Uo) && ok;
            }
          }
          if (j - 1 < r1) {
            // pending right-hand side of row j-1
#pragma unroll
            for (int k = 0; k < NC; ++k) {
              const TR volg = gbuf[2 * NC + k][lane];
              TR bottom = F1n_s[k];
              asm("" : "+v"(bottom));  // its product is formed again and fused, likewise
              F1p[k] = -F1x[k] * idx + (double)bottom * idy;
              F2p[k] = -F2x[k] * (TR)(0.5 * idx) + volf[k] * (TR)idx + F2n[k];
              F3p[k] = -F3x[k] * (TR)idx + volg * (TR)idy + F3n[k];
              vhp[k] = vh[k];
              whp[k] = gbuf[3 * NC + k][lane];
            }
          }
        }
        if (j + 2 <= r1 + 1) store(sn, j + 2, next);
        if (j > r1) break;
        // loads of the next pass
        if (j + 3 <= r1 + 1) fetch(j + 3, next);
        if (kBaseEarly && j - 1 >= r0) load_base(j - 1);
        if (j >= r0 && j < r1) {
          TR Cc[NC][15];
          pair_sweep<0, SI>(P, prim(sc), B, sb, sc, st, lane, Cc, c1buf);
          pin(Cc);
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            F1x[k] = 0.0;
            F2x[k] = F3x[k] = volf[k] = (TR)0;
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
            }
#pragma unroll
            for (int G = 0; G < 3; ++G) {
              TR f[NC];
              phys_flux<EQ_EULER, NC, 0, TR>(P, in[G], f);
              const TR wgt = (TR)(g3w(G) * g3w(H));
#pragma unroll
              for (int k = 0; k < NC; ++k) volf[k] += wgt * f[k];
            }
            // x_{i-1/2} at eta_H: u- = left lane at +1/2, u+ = this lane at -1/2
            TR um[NC], fl[NC], fr[NC];
#pragma unroll
            for (int k = 0; k < NC; ++k) um[k] = from_prev(xp[k]);
            lf_flux2<EQ_EULER, NC, 0, TR>(P, um, xm, a1, fl);  // twice the flux
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
#pragma unroll
          for (int k = 0; k < NC; ++k) vh[k] = qv_2d<TR>(Cc[k]);
        } else {
          __syncthreads();
        }
        __syncthreads();
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
}

template <bool SI>
static hipError_t launch(const StageArgs<double>& a, int blocks, hipStream_t s) {
  const dim3 grid(blocks), block(128);
  if (a.stage == 0)
    hipLaunchKernelGGL((stage2d_pair_kernel<SI, 0>), grid, block, 0, s, a);
  else if (a.stage == 1)
    hipLaunchKernelGGL((stage2d_pair_kernel<SI, 1>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((stage2d_pair_kernel<SI, 2>), grid, block, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_pair_2d(bool scale_invariant, const StageArgs<double>& args, int blocks,
                          hipStream_t s) {
  return scale_invariant ? launch<true>(args, blocks, s) : launch<false>(args, blocks, s);
}

}  // namespace hwenou
