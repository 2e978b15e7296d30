// Internal interface between the host library (hwenou_api.cpp) and the
// kernel translation units.  Not part of the public C-ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "hwenou_device.hpp"

namespace hwenou {

// A read of data that no kernel writes while its kernel runs (the work
// list, the instance records, alpha and dt, what the step before left), through the
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

// One problem instance as the kernels see it.
struct InstDev {
  int nx, ny;        // cells (ny = 1 in 1D)
  int bc[4];         // x-lo, x-hi, y-lo, y-hi (BC_*)
  double dx, dy;     // mesh sizes
  long long offset;  // first cell of the instance in each component plane
};

// One work item.  1D: (inst, first cell of a 62-cell tile).  2D: (inst,
// strip, first row, end row) -- a strip is 62 output columns marched upward.
struct WorkItem {
  int inst, a, b, c;
};

// Lanes of a wave that produce output; lane 0 and lane 63 only reconstruct
// the neighbouring cells whose interface values the strip needs.
constexpr int kStripWidth = 62;

// The last stage reduces the wave speeds of its output into `slots`
// accumulators per instance (a power of two up to kAlphaSlots; the wave's
// index picks one), so that ~1000 waves ending together on one instance do
// not all serialise their atomics on one address.  Each accumulator (x and y
// wave speed) sits in a 128-byte line of its own (kAlphaStride doubles),
// since the atomics of one line are serialised as well; the next step takes
// the maximum of the slots.  Handles of many instances use fewer slots per
// instance: few waves end on any one instance at a time, and every wave of the
// next step reads all slots.
constexpr int kAlphaSlots = 16;
constexpr int kAlphaStride = 16;
__device__ __host__ __forceinline__ int alpha_slot(int inst, int wave, int slots) {
  return kAlphaStride * (inst * slots + (wave & (slots - 1)));
}

// Parameters of one hwenou_advance call, read by the time-step kernels from
// device memory so that a captured step graph stays valid across calls.
struct RunParams {
  double cfl, t_final;
  int max_steps;
};

// Whole steps in 1D (step1d.hip): a tile of kStepWidth owned cells, and an
// instance's time, step count and completion.
constexpr int kStepWidth = 54;
struct TileItem {
  int inst, start;
};
struct StepState {
  double t;
  int steps, done;
};

// The state of a run (one hwenou_advance call) that its kernels carry from
// step to step.  Time, step count, completion and failure flags alternate
// between two buffers, the wave-speed accumulators between four: every kernel
// of step p forms its instances' time step itself from what step p - 1 left,
// so that no wave reads what another wave of the same step writes, and a step
// has no kernel of its own for its bookkeeping.  One wave per instance writes
// the new time and step count and clears the accumulators of the next step.
struct StepControl {
  const RunParams* run;    // nullptr: the caller gives dt and alpha (hwenou_stage)
  const StepState* st_in;  // [n_inst]
  StepState* st_out;
  const int* flag_in;      // [n_inst]: non-physical states found before this step
  int* flag_out;           // [n_inst]: ... and by this step
  const double* acc_in;    // wave speeds of the input, [n_inst][slots][kAlphaStride]
  double* acc_out;         // wave speeds of the output (cleared by the step before)
  double* acc_zero;        // accumulators to clear for the next step
  int slots;
};

// What one step of an instance starts from: its time step and wave speeds, or
// that it is done.  It is when it has reached t_final or max_steps, or a
// kernel has flagged one of its states as non-physical or non-finite (it
// stops after the step that failed, and its t and step count say where), or
// its wave speed is infinite (failed: to be flagged now).  The wave speeds are
// reduced with fmax, which drops NaN arguments, so a NaN state is caught by
// the flag, not by the wave speed.
struct StepDt {
  double dt, ax, ay;
  StepState s;
  bool done, failed;
};
template <int DIM>
__device__ __forceinline__ void step_rule(const RunParams& R, const InstDev& I, const StepState& s,
                                          int flag, StepDt& r) {  // r.ax, r.ay are given
  r.s = s;
  r.dt = 0.0;
  r.failed = false;
  r.done = s.done || flag || s.steps >= R.max_steps || s.t >= R.t_final * (1.0 - 1e-14);
  if (r.done) return;
  if (!isfinite(r.ax) || (DIM == 2 && !isfinite(r.ay))) {
    r.done = r.failed = true;
    return;
  }
  if (r.ax == 0.0 && (DIM == 1 || r.ay == 0.0))
    r.dt = R.t_final - s.t;  // zero wave speed: every flux vanishes, the CFL bound is infinite
  else if (DIM == 1)
    r.dt = R.cfl * I.dx / r.ax;
  else
    r.dt = R.cfl / (r.ax / I.dx + r.ay / I.dy);
  if (s.t + r.dt > R.t_final) r.dt = R.t_final - s.t;
}

template <int DIM>
__device__ __forceinline__ StepDt step_dt(const StepControl& A, int inst, const InstDev& I) {
  StepDt r;
  const RunParams R = load_invariant(A.run);
  const StepState s = load_invariant(A.st_in + inst);
  const int flag = load_invariant(A.flag_in + inst);
  struct Line {
    double x, y;
  };
  const double* acc = A.acc_in + kAlphaStride * inst * A.slots;
  if (A.slots == 1) {
    const Line l = load_invariant(reinterpret_cast<const Line*>(acc));
    r.ax = l.x;
    r.ay = l.y;
  } else {
    // all slot lines in one round of loads; the last one stands in for those
    // beyond this handle's slots
    Line l[kAlphaSlots];
#pragma unroll
    for (int q = 0; q < kAlphaSlots; ++q)
      l[q] = load_invariant(
          reinterpret_cast<const Line*>(acc + kAlphaStride * min(q, A.slots - 1)));
    r.ax = r.ay = 0.0;
#pragma unroll
    for (int q = 0; q < kAlphaSlots; ++q) {
      r.ax = fmax(r.ax, l[q].x);
      if (DIM == 2) r.ay = fmax(r.ay, l[q].y);
    }
  }
  step_rule<DIM>(R, I, s, flag, r);
  return r;
}

// Done by one lane per instance and step.
__device__ __forceinline__ void write_step(const StepControl& A, int inst, const StepDt& d) {
  A.st_out[inst] = {d.done ? d.s.t : d.s.t + d.dt, d.done ? d.s.steps : d.s.steps + 1,
                    d.done ? 1 : 0};
  if (d.failed) atomicOr(A.flag_out + inst, 1);
  for (int q = 0; q < A.slots; ++q) {
    double* line = A.acc_zero + kAlphaStride * (inst * A.slots + q);
    line[0] = line[1] = 0.0;
  }
}

template <class TM>
struct StepArgs {
  SchemeParams P;
  StepControl ctl;
  const InstDev* inst;
  const double* u_in;
  const TM* m_in;
  double* u_out;
  TM* m_out;
  long long plane;
  const TileItem* tiles;
  int n_tiles, n_waves;    // wave w takes tiles [n_tiles w / n_waves, n_tiles (w+1) / n_waves)
};

template <class TM>
struct StageArgs {
  SchemeParams P;
  const InstDev* inst;
  StepControl ctl;      // ctl.run == nullptr: not part of a run
  const double* dt;     // [n_inst], read outside a run and by the 1D kernels
  const double* alpha;  // [n_inst][2], likewise
  const int* done;      // [n_inst] or nullptr (1D kernels)
  const double* u_in;   // [nc][plane]
  const TM* m_in;       // [dim][nc][plane]
  const double* u_base; // u^n for stages 1, 2
  TM* m_base;           // v^_n (and w^_n): written by stage 0, read by stages 1, 2
  double* u_out;
  TM* m_out;
  int* status;          // [n_inst]: set to 1 on a non-physical or non-finite output
                        // (ctl.flag_out within a run)
  long long plane;      // cells per component plane
  const WorkItem* work;
  const int* work_ptr;  // wave w handles work[work_ptr[w] .. work_ptr[w+1])
  int n_waves;
  int stage;            // 0, 1, 2
};

// Host helpers shared by the entry points (hwenou_api.hip).
}  // namespace hwenou
struct hwenou_desc;
struct hwenou_inst;
namespace hwenou {
int check_desc(const hwenou_desc* d);                           // HWENOU_OK or an error code
int check_inst(const hwenou_desc* d, const hwenou_inst& inst);  // one instance's own checks
InstDev inst_dev(const hwenou_desc* d, const hwenou_inst& inst);
SchemeParams scheme_params(const hwenou_desc& d);

// kernel launchers (one per translation unit); return hipSuccess or the launch error.
// char_mode (Euler): 0 component-wise, 1 direction-split characteristic, 2 single
// x-projection (the same as 1 in 1D)
hipError_t launch_stage_1d(int eq, int char_mode, bool mixed, const void* args, int blocks,
                           int threads, hipStream_t s);
// scale_invariant: the default weights, compiled into their own 2D kernels
hipError_t launch_stage_2d(int eq, int char_mode, bool mixed, bool scale_invariant,
                           const void* args, int blocks, int threads, hipStream_t s);

// the same stage, direction-split characteristic Euler in FP64, by pairs of waves
// (pair2d.hip)
hipError_t launch_pair_2d(bool scale_invariant, const StageArgs<double>& args, int blocks,
                          hipStream_t s);

// Whether a 2D handle's stages run by pairs of waves (two resident per compute
// unit, against four single waves): `total` strip-rows over all grids, of which
// the largest has `strips` strips of `ny` rows.  With r rows per run a stage
// takes about 34 + 35 r us per Runge-Kutta step by single waves and 40 + 19 r by
// pairs, whose runs are up to twice as long, since half as many are in flight.
// So pairs win where rounding to whole rows leaves them less than twice the rows
// of a single wave, and runs are short.  Measured, single waves / pairs (rows per
// run), us per step: 60 x 60 70 / 56 (1 / 1), 131 x 97 76 / 61 (1 / 1),
// 900 x 100 113 / 103 (2 / 3), 256 x 256 110 / 99 (2 / 3), 500 x 200 115 / 119
// (2 / 4), 400 x 300 142 / 135 (3 / 5), 512 x 512 201 / 221 (5 / 10), 6 grids of
// 40^2 to 150^2 85 / 108 (1 / 2), 24 grids of 60^2 109 / 97 (2 / 3).
constexpr int kPairMaxRows = 5;
inline bool use_pairs_2d(int eq, int char_mode, bool mixed, long long total, int strips, int ny,
                         int n_cu) {
  if (eq != EQ_EULER || char_mode != 1 || mixed) return false;
  const bool several = total > (long long)strips * ny;
  const auto rows = [&](long long runs) {
    if (several) return (total + runs - 1) / runs;  // several grids: equal runs
    const long long per_strip = std::max(1LL, runs / strips);
    return (ny + per_strip - 1) / per_strip;
  };
  const long long pair = rows(2LL * n_cu);
  return pair <= kPairMaxRows && pair < 2 * rows(4LL * n_cu);
}

// resident blocks per compute unit of a stage kernel at `threads` per block
int occupancy_stage_1d(int eq, int char_mode, bool mixed, int threads);
int occupancy_stage_2d(int eq, int char_mode, bool mixed, bool scale_invariant, int threads);

// Runs of whole 1D steps in one launch, one block per instance.
template <class TM>
struct BlockRunArgs {
  SchemeParams P;
  const InstDev* inst;
  const RunParams* run;
  double* u;
  TM* m;
  StepState* st;     // [n_inst], read and written
  int* flag;         // [n_inst], likewise
  double* acc;       // [n_inst][kAlphaStride]: wave speed of the state, likewise
  long long plane;
  int n_inst, steps; // at most `steps` steps per launch
};
// Waves of a block that holds an instance, one tile per wave.  All tiles share
// one CU's four SIMDs there, where a launch per step gives each tile its own, so
// the line lies where a SIMD gets its third tile for Euler and not before the
// block is full for the scalar laws.  Measured, launch per step / run of steps,
// us per 12 steps: Euler characteristic 4 tiles 113 / 78, 8 tiles 119 / 114,
// 12 tiles 120 / 158; component-wise (4 steps) 47 / 38, 50 / 48, 50 / 60;
// Burgers (20 steps) 8 tiles 120 / 67, 16 tiles 124 / 105.
constexpr int block_run_waves(int eq) { return eq == EQ_EULER ? 8 : 16; }
hipError_t launch_block_run_1d(int eq, int char_mode, bool mixed, const void* args, int n_inst,
                               int waves, hipStream_t s);

// whole Runge-Kutta steps in 1D, one per launch; args: StepArgs<float or double>
hipError_t launch_step_1d(int eq, int char_mode, bool mixed, const void* args, int waves,
                          int threads, hipStream_t s);
int occupancy_step_1d(int eq, int char_mode, bool mixed, int threads);

// auxiliary kernels
// Blocks of the wave-speed reduction of an instance of n cells, at most `most`.
constexpr int kSpeedThreads = 1024;
constexpr int kSpeedCells = 8 * kSpeedThreads;  // per block, up to 512 blocks per instance
constexpr int kSpeedBlocks = 512;
__device__ __host__ __forceinline__ int speed_blocks(long long n, int most) {
  const long long b = (n + kSpeedCells - 1) / kSpeedCells;
  return b < most ? (int)b : most;
}
struct AuxArgs {
  SchemeParams P;
  int eq, dim, n_inst;
  const InstDev* inst;
  long long plane;
  const double* u;       // [nc][plane]
  double* alpha;         // [n_inst][alpha_stride]: x and y wave speed first
  int alpha_stride;
  double* part;          // [n_inst][part_blocks][2] partial maxima
  int part_blocks;       // speed_blocks of the largest instance
  int* status;           // [n_inst]: 1 once the instance left the physical states
};
hipError_t launch_max_wavespeed(const AuxArgs& a, hipStream_t s);

// One step's time steps, wave speeds and completion into arrays, for the 1D
// kernels that run one stage per launch.
struct ControlArgs {
  StepControl ctl;
  const InstDev* inst;
  int n_inst;
  double *dt, *alpha;
  int* done;
};
hipError_t launch_step_control(const ControlArgs& a, hipStream_t s);

// Start, polls and end of a run.
struct RunArgs {
  RunParams R;
  RunParams* run;          // device copy of R
  int n_inst, slots, nc, mom_planes, mom_elem;
  StepState* st[2];
  int* flag[2];
  double* acc[4];
  int last;                // buffer (0, 1) the last step wrote
  // whole 1D steps (tiles != nullptr): what brings the state home
  const double* u_odd;     // scratch state that odd steps write
  const void* m_odd;
  double* u;
  void* m;
  const InstDev* inst;
  long long plane;
  const TileItem* tiles;
  int n_tiles;
  int* status;             // [n_inst] device status flags
  double* t_host;          // pinned host results
  int *steps_host, *status_host, *running_host;
};
hipError_t launch_run_begin(const RunArgs& a, hipStream_t s);
hipError_t launch_run_poll(const RunArgs& a, hipStream_t s);
hipError_t launch_run_end(const RunArgs& a, hipStream_t s);

}  // namespace hwenou
