// Internal interface between the host library (hwenou_api.cpp) and the
// kernel translation units.  Not part of the public C-ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hwenou_device.hpp"

namespace hwenou {

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
// since the atomics of one line are serialised as well; the finish kernel
// takes the maximum of the slots.  Handles of many instances use fewer slots
// per instance: few waves end on any one instance at a time, and the finish
// kernel's loop over the slots grows with their number.
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

// What one step of an instance starts from: its time step and wave speed, or
// that it is done.  It is when it has reached t_final or max_steps, or a
// kernel has flagged one of its states as non-physical or non-finite (it
// stops after the step that failed, and its t and step count say where), or
// its wave speed is infinite (failed: to be flagged now).  The same rule as
// set_step of the one-stage path.
struct StepDt {
  double dt, alpha;
  bool done, failed;
};
__device__ __forceinline__ StepDt step_dt(const RunParams& R, double dx, const StepState& s,
                                          int flag, double ax) {
  StepDt r;
  r.alpha = ax;
  r.dt = 0.0;
  r.failed = false;
  r.done = s.done || flag || s.steps >= R.max_steps || s.t >= R.t_final * (1.0 - 1e-14);
  if (r.done) return r;
  if (!isfinite(ax)) {
    r.done = r.failed = true;
    return r;
  }
  // zero wave speed: every flux vanishes, the CFL bound is infinite
  r.dt = ax == 0.0 ? R.t_final - s.t : R.cfl * dx / ax;
  if (s.t + r.dt > R.t_final) r.dt = R.t_final - s.t;
  return r;
}

template <class TM>
struct StepArgs {
  SchemeParams P;
  const InstDev* inst;
  const RunParams* run;
  const double* u_in;
  const TM* m_in;
  double* u_out;
  TM* m_out;
  const StepState* st_in;  // [n_inst], written by the step before
  StepState* st_out;
  const int* flag_in;      // [n_inst]: non-physical states found before this step
  int* flag_out;           // [n_inst]: ... and by this step
  const double* acc_in;    // wave speeds of the input, [n_inst][slots][kAlphaStride]
  double* acc_out;         // wave speeds of the output (cleared by the step before)
  double* acc_zero;        // accumulators to clear for the next step
  int slots;
  long long plane;
  const TileItem* tiles;
  int n_tiles, n_waves;    // wave w takes tiles [n_tiles w / n_waves, n_tiles (w+1) / n_waves)
};

template <class TM>
struct StageArgs {
  SchemeParams P;
  const InstDev* inst;
  const double* dt;     // [n_inst]
  const double* alpha;  // [n_inst][2]
  const int* done;      // [n_inst] or nullptr
  const double* u_in;   // [nc][plane]
  const TM* m_in;       // [dim][nc][plane]
  const double* u_base; // u^n for stages 1, 2
  TM* m_base;           // v^_n (and w^_n): written by stage 0, read by stages 1, 2
  double* u_out;
  TM* m_out;
  double* alpha_next;   // [n_inst][alpha_slots][kAlphaStride] or nullptr: max wave speed of
                        // the output (x, y in the first two doubles of each slot)
  int alpha_slots;      // accumulators per instance (power of two, <= kAlphaSlots)
  int* status;          // [n_inst]: set to 1 on a non-physical or non-finite output
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

// resident blocks per compute unit of a stage kernel at `threads` per block
int occupancy_stage_1d(int eq, int char_mode, bool mixed, int threads);
int occupancy_stage_2d(int eq, int char_mode, bool mixed, bool scale_invariant, int threads);

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
  double* dt;            // [n_inst]
  double* t;             // [n_inst]
  int* steps;            // [n_inst]
  int* done;             // [n_inst]
  int* status;           // [n_inst]: 1 once the instance left the physical states
  double* alpha_next;    // [n_inst][alpha_slots][kAlphaStride]
  int alpha_slots;
  const RunParams* run;  // CFL number, final time, step limit
  int* all_done;         // 1 when every instance is done
};
hipError_t launch_max_wavespeed(const AuxArgs& a, hipStream_t s);
hipError_t launch_dt(const AuxArgs& a, hipStream_t s);
hipError_t launch_finish(const AuxArgs& a, hipStream_t s);

// Start and end of a run of whole 1D steps.
struct RunArgs {
  RunParams R;
  RunParams* run;          // device copy of R
  int n_inst, slots, nc, mom_planes, mom_elem;
  StepState* st[2];
  int* flag[2];
  double* acc[4];
  int last;                // buffer (0, 1) the last step wrote
  // end of the run
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
