// Whole Runge-Kutta steps in 1D (Section 2.1, Steps 1-4): one launch advances
// every instance by one step of the modified SSP-RK3 of Eq. (2.13), its dt and
// wave speed included.
//
// Mapping: one wave per 54-cell tile.  Lane l holds cell start - 5 + l through
// all three stages.  A stage's output at a cell reaches two cells to either
// side, so the valid lanes shrink by two per stage: 0..63 hold the input (the
// two cells beyond are loaded by the end lanes), 1..62, 3..60 and 5..58 the
// stage outputs, and lanes 5..58 own the tile's cells.  The stage values, the
// base (u^n, v^n) and the modified moments stay in registers: a step reads the
// state once and writes it once (96 bytes per cell and step for Euler in FP64
// against 408 with one stage per launch) for 64/54 instead of 64/62 of the
// arithmetic, and has one launch's latency instead of four.  Measured against
// one stage per launch (replayed from a graph), FP64 Euler: 512 grids of 256 to
// 65 536 cells 695 -> 455 us per step (bound by the VALU issue rate now, by
// memory latency before), one grid of 65 536 cells 27 -> 14 us, 801 cells
// 24 -> 10 us; 200 cells of advection 12.3 -> 4.6 us.
//
// Ghost cells: the stage outputs beyond a periodic side are recomputed from
// wrapped data, which is bitwise what the cells they image compute; beyond a
// transmissive or reflective side they are copies or mirror images of cells
// that the same wave holds (the two ghost cells that a boundary cell needs
// image the two cells next to the side, and those lie within the valid lanes
// of every tile that needs them), taken with a cross-lane read after each
// stage.  An instance with exactly one periodic side has no such rule (its
// wrapped cells depend on the other side's ghost cells) and runs one stage per
// launch.
#include <algorithm>

#include "tile1d.hpp"

namespace hwenou {

// Resident waves per SIMD the compiler must allow.  The FP64 characteristic
// kernel uses 165 VGPRs; held to 4 waves (128) it spills and a batch of 512
// grids takes 513 instead of 452 us per step.
template <int EQ, bool CHAR, class TR>
constexpr int min_waves_step1d() {
  return EQ == EQ_EULER ? 3 : 1;
}

template <int EQ, bool CHAR, class TR, int NC>
__device__ __forceinline__ void cell_rhs_1d(const SchemeParams& P, const double (&Um)[NC],
                                            const double (&Uc)[NC], const double (&Up)[NC],
                                            const double (&Vm)[NC], const double (&Vp)[NC],
                                            TR alpha_in, double idx, double (&F1)[NC],
                                            TR (&F2)[NC], TR (&vh)[NC]) {
#include "tile1d_terms.inc"
}

// Everything one stage of a tile needs from one lane to the next.
template <int EQ, bool CHAR, int ST, class TR, class TM, int NC>
__device__ __forceinline__ void rk_stage(const SchemeParams& P, double alpha_in, double idx, double dt,
                                         const double (&Uend)[NC], const TM (&Vend)[NC],
                                         bool edge_lo, bool edge_hi, double (&Uc)[NC],
                                         TM (&Vc)[NC], double (&Ub)[NC], TM (&Mb)[NC]) {
  constexpr double ra = ST == 0 ? 0.0 : (ST == 1 ? 0.75 : 1.0 / 3.0);
  constexpr double rb = ST == 0 ? 1.0 : (ST == 1 ? 0.25 : 2.0 / 3.0);
  double Um[NC], Up[NC], Vm[NC], Vp[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    Um[k] = from_prev(Uc[k]);
    Up[k] = from_next(Uc[k]);
    Vm[k] = (double)from_prev(Vc[k]);
    Vp[k] = (double)from_next(Vc[k]);
    if (ST == 0) {
      if (edge_lo) {
        Um[k] = Uend[k];
        Vm[k] = (double)Vend[k];
      }
      if (edge_hi) {
        Up[k] = Uend[k];
        Vp[k] = (double)Vend[k];
      }
    }
  }
  double F1[NC];
  TR F2[NC], vh[NC];
  cell_rhs_1d<EQ, CHAR, TR, NC>(P, Um, Uc, Up, Vm, Vp, (TR)alpha_in, idx, F1, F2, vh);
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const double ub = ST == 0 ? 0.0 : Ub[k];
    const double un = ra * ub + rb * (Uc[k] + dt * F1[k]);
    TR mn;
    if (ST == 0) {
      mn = vh[k] + (TR)dt * F2[k];
      Ub[k] = Uc[k];
      Mb[k] = (TM)vh[k];
    } else {
      const TR mb = (TR)Mb[k];
      mn = (TR)ra * mb + (TR)rb * (vh[k] + (TR)dt * F2[k]);
    }
    Uc[k] = un;
    Vc[k] = (TM)mn;
  }
}

// Ghost lanes beyond a transmissive or reflective side take the value of the
// lane whose cell they image.
template <int EQ, class TM, int NC>
__device__ __forceinline__ void ghost_lanes(int src, bool mirrored, double (&Uc)[NC],
                                            TM (&Vc)[NC]) {
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    Uc[k] = __shfl(Uc[k], src, 64);
    Vc[k] = __shfl(Vc[k], src, 64);
  }
  if constexpr (EQ == EQ_EULER) {
    if (mirrored) mirror_cell<0, NC>(Uc, reinterpret_cast<TM(*)[NC]>(Vc), 1);
  }
}

// One Runge-Kutta step of the tile that starts at cell `start`: load(cell, U, V)
// reads a cell of the input.  On return lanes with `owner` hold their cell i
// of the output in Uc, Vc; `ok` turns false where an owned stage output is not
// physical.
template <int EQ, bool CHAR, class TR, class TM, int NC, class Load>
__device__ __forceinline__ void tile_step(const SchemeParams& P, const InstDev& I, int start,
                                          int lane, double alpha_in, double idx, double dt,
                                          Load load, int& i, bool& owner, bool& ok,
                                          double (&Uc)[NC], TM (&Vc)[NC]) {
  const int n = I.nx;
  const bool periodic = I.bc[0] == BC_PERIODIC;
  // Cell of this lane, and the cell it reads.  Lanes further out than any
  // valid result reaches read some cell of the instance: past the last one
  // periodic lanes stop at n + 5, the others at the two ghost cells that
  // stencils of the instance's own cells use.
  i = start - 5 + lane;
  owner = lane >= 5 && lane < 5 + kStepWidth && i < n;
  int ic, ie;
  bool mir_c = false, mir_e = false;
  if (periodic) {
    const int last = n + 5;
    auto wrap = [n](int j) {
      j += j < 0 ? n : 0;
      j += j < 0 ? n : 0;
      j -= j >= n ? n : 0;
      j -= j >= n ? n : 0;
      return j;
    };
    ic = wrap(min(i, last));
    ie = wrap(min(lane == 0 ? i - 1 : i + 1, last));
  } else {
    auto clamp = [n](int j) { return min(max(j, -2), n + 1); };
    ic = source_cell(clamp(i), n, I.bc[0], I.bc[1], mir_c);
    ie = source_cell(clamp(lane == 0 ? i - 1 : i + 1), n, I.bc[0], I.bc[1], mir_e);
  }
  const bool edge_lo = lane == 0, edge_hi = lane == 63;
  double Uend[NC], Ub[NC];
  TM Vend[NC], Mb[NC];
  load(ic, Uc, Vc);
  if (edge_lo || edge_hi) load(ie, Uend, Vend);
  if constexpr (EQ == EQ_EULER) {
    if (mir_c) mirror_cell<0, NC>(Uc, reinterpret_cast<TM(*)[NC]>(Vc), 1);
    if (mir_e && (edge_lo || edge_hi))
      mirror_cell<0, NC>(Uend, reinterpret_cast<TM(*)[NC]>(Vend), 1);
  }
  // lane that holds the cell a ghost lane images (boundary tiles only)
  const bool ghosts = !periodic && (start < 5 || start + 58 >= n);
  const int src = min(max(ic - start + 5, 0), 63);

  rk_stage<EQ, CHAR, 0, TR, TM, NC>(P, alpha_in, idx, dt, Uend, Vend, edge_lo, edge_hi, Uc, Vc,
                                    Ub, Mb);
  if (owner) ok = physical_state<EQ, NC>(Uc) && ok;
  if (ghosts) ghost_lanes<EQ, TM, NC>(src, mir_c, Uc, Vc);
  rk_stage<EQ, CHAR, 1, TR, TM, NC>(P, alpha_in, idx, dt, Uend, Vend, false, false, Uc, Vc, Ub,
                                    Mb);
  if (owner) ok = physical_state<EQ, NC>(Uc) && ok;
  if (ghosts) ghost_lanes<EQ, TM, NC>(src, mir_c, Uc, Vc);
  rk_stage<EQ, CHAR, 2, TR, TM, NC>(P, alpha_in, idx, dt, Uend, Vend, false, false, Uc, Vc, Ub,
                                    Mb);
}

template <int EQ, bool CHAR, class TR, class TM>
__global__ __launch_bounds__(256, (min_waves_step1d<EQ, CHAR, TR>())) void step1d_kernel(
    const StepArgs<TM> A) {
  constexpr int NC = EQ == EQ_EULER ? 3 : 1;
  const int lane = threadIdx.x & 63;
  const int w =
      __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
  if (w >= A.n_waves) return;
  const SchemeParams& P = A.P;
  const long long plane = A.plane;

  // contiguous run of tiles
  const int it0 = (int)((long long)A.n_tiles * w / A.n_waves);
  const int it1 = (int)((long long)A.n_tiles * (w + 1) / A.n_waves);
  int inst = -1;
  InstDev I;
  StepDt sd;
  double dt = 0.0, alpha_in = 0.0, idx = 0.0;
  double mx = 0.0;   // wave speed of this wave's output cells of `inst`
  bool ok = true;
  auto flush = [&]() {  // hand over what the wave knows about instance `inst`
    if (inst < 0 || sd.done) return;
    const double m = wave_max_dpp(mx);
    if (lane == 63)
      atomic_max_nonneg(A.ctl.acc_out + alpha_slot(inst, w, A.ctl.slots), m);
    if (!ok) atomicOr(A.ctl.flag_out + inst, 1);
    mx = 0.0;
    ok = true;
  };
  for (int it = it0; it < it1; ++it) {
    const TileItem wk = load_invariant(A.tiles + it);
    if (wk.inst != inst) {
      flush();
      inst = wk.inst;
      I = load_invariant(A.inst + inst);
      sd = step_dt<1>(A.ctl, inst, I);
      dt = uniform(sd.dt);
      alpha_in = uniform(sd.ax);
      idx = uniform(1.0 / I.dx);
      if (wk.start == 0 && lane == 0) write_step(A.ctl, inst, sd);
    }
    if (sd.done) continue;
    const double* u = A.u_in + I.offset;
    const TM* m = A.m_in + I.offset;
    int i;
    bool owner;
    double Uc[NC];
    TM Vc[NC];
    tile_step<EQ, CHAR, TR, TM, NC>(
        P, I, wk.start, lane, alpha_in, idx, dt,
        [&](int c, double (&U)[NC], TM (&V)[NC]) {
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            U[k] = u[k * plane + c];
            V[k] = m[k * plane + c];
          }
        },
        i, owner, ok, Uc, Vc);
    if (owner) {
      const long long o = I.offset + i;
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        A.u_out[k * plane + o] = Uc[k];
        A.m_out[k * plane + o] = Vc[k];
      }
      double sx, sy;
      ok = wave_speeds<EQ, NC>(P, Uc, sx, sy) && ok;
      mx = fmax(mx, sx);
    }
  }
  flush();
}

// A run of steps of an instance that one block can hold (one tile per wave):
// the state stays in LDS from step to step, a step is its three stages, the
// exchange through LDS and one barrier, and the block takes the wave speed and
// forms the time step itself.  Such an instance is bound by the latency of the
// chain of launches otherwise: 200 cells of advection take 4.5 us per step with
// one launch per step and 1.5 us here.
template <int EQ, bool CHAR, class TR, class TM>
__global__ __launch_bounds__(64 * block_run_waves(EQ)) void block_run_kernel(
    const BlockRunArgs<TM> A) {
  constexpr int NC = EQ == EQ_EULER ? 3 : 1;
  constexpr int WAVES = block_run_waves(EQ), CELLS = WAVES * kStepWidth;
  __shared__ double Us[2][NC][CELLS];
  __shared__ TM Vs[2][NC][CELLS];
  __shared__ double speed[2][WAVES];
  __shared__ int bad[2][WAVES];
  const int inst = blockIdx.x, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int waves = blockDim.x >> 6;
  const InstDev I = load_invariant(A.inst + inst);
  const RunParams R = load_invariant(A.run);
  StepState s = A.st[inst];
  int flag = A.flag[inst];
  StepDt d;
  d.ax = A.acc[kAlphaStride * inst];
  d.ay = 0.0;
  const int n = I.nx, start = wave * kStepWidth;
  const bool active = start < n;
  const double idx = uniform(1.0 / I.dx);
  for (int c = threadIdx.x; c < n; c += blockDim.x) {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      Us[0][k][c] = A.u[k * A.plane + I.offset + c];
      Vs[0][k][c] = A.m[k * A.plane + I.offset + c];
    }
  }
  __syncthreads();
  int cur = 0;
  bool failed = false;
  for (int step = 0; step < A.steps; ++step) {
    step_rule<1>(R, I, s, flag, d);  // the same on every thread
    if (d.done) {
      failed = d.failed;
      break;
    }
    double mx = 0.0;
    bool ok = true;
    if (active) {
      int i;
      bool owner;
      double Uc[NC];
      TM Vc[NC];
      tile_step<EQ, CHAR, TR, TM, NC>(
          A.P, I, start, lane, uniform(d.ax), idx, uniform(d.dt),
          [&](int c, double (&U)[NC], TM (&V)[NC]) {
#pragma unroll
            for (int k = 0; k < NC; ++k) {
              U[k] = Us[cur][k][c];
              V[k] = Vs[cur][k][c];
            }
          },
          i, owner, ok, Uc, Vc);
      if (owner) {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          Us[cur ^ 1][k][i] = Uc[k];
          Vs[cur ^ 1][k][i] = Vc[k];
        }
        double sx, sy;
        ok = wave_speeds<EQ, NC>(A.P, Uc, sx, sy) && ok;
        mx = sx;
      }
    }
    // two sets of slots: a wave may write the next step's before the last wave
    // has read this one's
    const unsigned long long all_ok = __ballot(ok);
    mx = wave_max_dpp(fmax(0.0, mx));
    if (lane == 63) {
      speed[cur][wave] = mx;
      bad[cur][wave] = ~all_ok != 0;
    }
    __syncthreads();
    d.ax = 0.0;
    for (int w = 0; w < waves; ++w) {
      d.ax = fmax(d.ax, speed[cur][w]);
      flag |= bad[cur][w];
    }
    s.t += d.dt;
    s.steps += 1;
    cur ^= 1;
  }
  for (int c = threadIdx.x; c < n; c += blockDim.x) {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      A.u[k * A.plane + I.offset + c] = Us[cur][k][c];
      A.m[k * A.plane + I.offset + c] = Vs[cur][k][c];
    }
  }
  if (threadIdx.x == 0) {
    s.done = s.done || failed;
    A.st[inst] = s;
    A.flag[inst] = flag | (failed ? 1 : 0);
    A.acc[kAlphaStride * inst] = d.ax;
  }
}

template <int EQ, bool CHAR, class TR, class TM>
static hipError_t launch_block(const void* args, int n_inst, int waves, hipStream_t s) {
  const auto& a = *static_cast<const BlockRunArgs<TM>*>(args);
  hipLaunchKernelGGL((block_run_kernel<EQ, CHAR, TR, TM>), dim3(n_inst), dim3(64 * waves), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_block_run_1d(int eq, int char_mode, bool mixed, const void* args, int n_inst,
                               int waves, hipStream_t s) {
  if (waves > block_run_waves(eq)) return hipErrorInvalidValue;
  if (mixed) {
    switch (eq) {
      case EQ_ADVECTION:
        return launch_block<EQ_ADVECTION, false, float, float>(args, n_inst, waves, s);
      case EQ_BURGERS: return launch_block<EQ_BURGERS, false, float, float>(args, n_inst, waves, s);
      default:
        return char_mode ? launch_block<EQ_EULER, true, float, float>(args, n_inst, waves, s)
                         : launch_block<EQ_EULER, false, float, float>(args, n_inst, waves, s);
    }
  }
  switch (eq) {
    case EQ_ADVECTION:
      return launch_block<EQ_ADVECTION, false, double, double>(args, n_inst, waves, s);
    case EQ_BURGERS: return launch_block<EQ_BURGERS, false, double, double>(args, n_inst, waves, s);
    default:
      return char_mode ? launch_block<EQ_EULER, true, double, double>(args, n_inst, waves, s)
                       : launch_block<EQ_EULER, false, double, double>(args, n_inst, waves, s);
  }
}

template <int EQ, bool CHAR, class TR, class TM>
static hipError_t launch(const void* args, int waves, int threads, hipStream_t s) {
  const auto& a = *static_cast<const StepArgs<TM>*>(args);
  const int per = threads / 64;
  hipLaunchKernelGGL((step1d_kernel<EQ, CHAR, TR, TM>), dim3((waves + per - 1) / per),
                     dim3(threads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_step_1d(int eq, int char_mode, bool mixed, const void* args, int waves,
                          int threads, hipStream_t s) {
  if (mixed) {
    switch (eq) {
      case EQ_ADVECTION: return launch<EQ_ADVECTION, false, float, float>(args, waves, threads, s);
      case EQ_BURGERS: return launch<EQ_BURGERS, false, float, float>(args, waves, threads, s);
      default:
        return char_mode ? launch<EQ_EULER, true, float, float>(args, waves, threads, s)
                         : launch<EQ_EULER, false, float, float>(args, waves, threads, s);
    }
  }
  switch (eq) {
    case EQ_ADVECTION: return launch<EQ_ADVECTION, false, double, double>(args, waves, threads, s);
    case EQ_BURGERS: return launch<EQ_BURGERS, false, double, double>(args, waves, threads, s);
    default:
      return char_mode ? launch<EQ_EULER, true, double, double>(args, waves, threads, s)
                       : launch<EQ_EULER, false, double, double>(args, waves, threads, s);
  }
}

template <int EQ, bool CHAR, class TR, class TM>
static int occupancy(int threads) {
  int blocks = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, step1d_kernel<EQ, CHAR, TR, TM>,
                                                   threads, 0) != hipSuccess)
    return 0;
  return blocks;
}

int occupancy_step_1d(int eq, int char_mode, bool mixed, int threads) {
  if (mixed) {
    switch (eq) {
      case EQ_ADVECTION: return occupancy<EQ_ADVECTION, false, float, float>(threads);
      case EQ_BURGERS: return occupancy<EQ_BURGERS, false, float, float>(threads);
      default:
        return char_mode ? occupancy<EQ_EULER, true, float, float>(threads)
                         : occupancy<EQ_EULER, false, float, float>(threads);
    }
  }
  switch (eq) {
    case EQ_ADVECTION: return occupancy<EQ_ADVECTION, false, double, double>(threads);
    case EQ_BURGERS: return occupancy<EQ_BURGERS, false, double, double>(threads);
    default:
      return char_mode ? occupancy<EQ_EULER, true, double, double>(threads)
                       : occupancy<EQ_EULER, false, double, double>(threads);
  }
}

}  // namespace hwenou
