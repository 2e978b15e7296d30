// Auxiliary kernels of the time loop: the maximum wave speed
// alpha = max |f'(u)| over the cell averages (Section 2.1, used by the
// Lax-Friedrichs flux and the CFL condition), the per-instance time step
// dt = min(CFL dx / alpha, T - t) in 1D and CFL / (alpha_1/dx + alpha_2/dy)
// in 2D, and the per-step bookkeeping of t, the step count and completion.
// All per-instance state lives on the device so that whole steps can be
// replayed from a captured graph without host synchronisation.
#include <algorithm>

#include "hwenou_internal.hpp"

namespace hwenou {

// Largest wave speed of every instance, by blocks of kSpeedCells cells.  The
// kernel is bound by reading the averages: a block has 16 waves and each thread
// loads the cells of a round together, so that a large grid keeps every CU's
// loads in flight.  An instance of one block writes its result; the blocks of
// a larger one leave partial maxima, which the second kernel combines.
// Neither needs cleared memory or atomics (which serialise on the result's
// line: 256 waves took 7.7 us on any grid).  2048^2 cells 130 -> 32 us, 3001 cells
// (one block, one launch) 9.4 -> 4.6 us, 512 grids of 256 to 65 536 cells
// 133 -> 90 us.
template <int EQ, int NC>
__global__ __launch_bounds__(kSpeedThreads) void max_wavespeed_kernel(const AuxArgs A) {
  __shared__ double red[2][kSpeedThreads / 64];
  const int inst = blockIdx.y;
  const InstDev I = A.inst[inst];
  const long long n = (long long)I.nx * I.ny;
  const int blocks = speed_blocks(n, A.part_blocks);
  if ((int)blockIdx.x >= blocks) return;
  const double* u = A.u + I.offset;
  double mx = 0.0, my = 0.0;
  bool ok = true;
  constexpr int R = 4;  // cells per thread and round
  const long long stride = (long long)blocks * kSpeedThreads;
  for (long long c = (long long)blockIdx.x * kSpeedThreads + threadIdx.x; c < n; c += R * stride) {
    double U[R][NC];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const long long cr = c + r * stride < n ? c + r * stride : c;  // past the end: again cell c
#pragma unroll
      for (int k = 0; k < NC; ++k) U[r][k] = u[k * A.plane + cr];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      double sx, sy;
      ok = wave_speeds<EQ, NC>(A.P, U[r], sx, sy) && ok;
      mx = fmax(mx, sx);
      my = fmax(my, sy);
    }
  }
  if (!ok) atomicOr(&A.status[inst], 1);
  mx = wave_max_dpp(mx);
  my = wave_max_dpp(my);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) {
    red[0][wave] = mx;
    red[1][wave] = my;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double m = red[threadIdx.x][0];
#pragma unroll
    for (int w = 1; w < kSpeedThreads / 64; ++w) m = fmax(m, red[threadIdx.x][w]);
    if (blocks == 1)
      A.alpha[(long long)A.alpha_stride * inst + threadIdx.x] = m;
    else
      A.part[2 * ((long long)inst * A.part_blocks + blockIdx.x) + threadIdx.x] = m;
  }
}

__global__ __launch_bounds__(64) void combine_wavespeed_kernel(const AuxArgs A) {
  const int inst = blockIdx.x;
  const InstDev I = A.inst[inst];
  const int blocks = speed_blocks((long long)I.nx * I.ny, A.part_blocks);
  if (blocks == 1) return;
  const double* part = A.part + 2 * (long long)inst * A.part_blocks;
  double mx = 0.0, my = 0.0;
  for (int b = threadIdx.x; b < blocks; b += 64) {
    mx = fmax(mx, part[2 * b]);
    my = fmax(my, part[2 * b + 1]);
  }
  mx = wave_max_dpp(mx);
  my = wave_max_dpp(my);
  if (threadIdx.x == 63) {
    double* out = A.alpha + (long long)A.alpha_stride * inst;
    out[0] = mx;
    out[1] = my;
  }
}

hipError_t launch_max_wavespeed(const AuxArgs& a, hipStream_t s) {
  const dim3 grid(a.part_blocks, a.n_inst), block(kSpeedThreads);
  if (a.eq == EQ_ADVECTION)
    hipLaunchKernelGGL((max_wavespeed_kernel<EQ_ADVECTION, 1>), grid, block, 0, s, a);
  else if (a.eq == EQ_BURGERS)
    hipLaunchKernelGGL((max_wavespeed_kernel<EQ_BURGERS, 1>), grid, block, 0, s, a);
  else if (a.dim == 1)
    hipLaunchKernelGGL((max_wavespeed_kernel<EQ_EULER, 3>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((max_wavespeed_kernel<EQ_EULER, 4>), grid, block, 0, s, a);
  if (a.part_blocks > 1)
    hipLaunchKernelGGL(combine_wavespeed_kernel, dim3(a.n_inst), dim3(64), 0, s, a);
  return hipGetLastError();
}

// Time step of instance k for the step that starts at time t after `steps`
// steps, from its wave speeds (ax, ay); marks the instance done when it has
// reached t_final or max_steps, or when a kernel has flagged one of its
// states as non-physical or non-finite (dt = 0 then: the instance stops at
// the step that failed, and its t and step count say where).  The wave
// speeds are reduced with fmax, which drops NaN arguments, so a NaN state is
// caught by the flag, not by alpha.  The caller passes the values it has
// loaded, so that each step's bookkeeping costs one round of loads.  Returns
// whether the instance is done.
__device__ bool set_step(const AuxArgs& A, int k, const InstDev& I, const RunParams& R, bool done,
                         double t, int steps, int status, double ax, double ay) {
  const bool finished = done || steps >= R.max_steps || t >= R.t_final * (1.0 - 1e-14);
  if (finished || status) {
    A.done[k] = 1;
    A.dt[k] = 0.0;
    return true;
  }
  if (A.dim == 1) ay = 0.0;
  if (!isfinite(ax) || !isfinite(ay)) {  // infinite wave speed: stop and report it
    A.done[k] = 1;
    A.dt[k] = 0.0;
    atomicOr(&A.status[k], 1);
    return true;
  }
  double dt;
  if (ax == 0.0 && ay == 0.0)
    dt = R.t_final - t;  // zero wave speed: every flux vanishes, the CFL bound is infinite
  else if (A.dim == 1)
    dt = R.cfl * I.dx / ax;
  else
    dt = R.cfl / (ax / I.dx + ay / I.dy);
  if (t + dt > R.t_final) dt = R.t_final - t;
  A.dt[k] = dt;
  return false;
}

// Before the first step: its time step, and the reset of the wave-speed
// accumulators that the last stage of the step fills.
__global__ __launch_bounds__(256) void dt_kernel(const AuxArgs A) {
  for (int k = threadIdx.x; k < A.n_inst * A.alpha_slots; k += blockDim.x) {
    A.alpha_next[kAlphaStride * k] = 0.0;
    A.alpha_next[kAlphaStride * k + 1] = 0.0;
  }
  for (int k = threadIdx.x; k < A.n_inst; k += blockDim.x)
    set_step(A, k, A.inst[k], *A.run, A.done[k] != 0, A.t[k], A.steps[k], A.status[k],
             A.alpha[2 * k], A.alpha[2 * k + 1]);
}

// End of a step: advance t and the step count, take the new wave speed,
// reset its accumulator, set the next step's time step, and count the
// instances still running (read by the host every few steps).  Everything
// an instance needs is loaded up front, in one round of loads.
__global__ __launch_bounds__(256) void finish_kernel(const AuxArgs A) {
  __shared__ int running;
  if (threadIdx.x == 0) running = 0;
  __syncthreads();
  int mine = 0;
  const RunParams R = *A.run;
  for (int k = threadIdx.x; k < A.n_inst; k += blockDim.x) {
    double* acc = A.alpha_next + alpha_slot(k, 0, A.alpha_slots);
    const bool done = A.done[k] != 0;
    double t = A.t[k];
    const double dt = A.dt[k];
    int steps = A.steps[k];
    const int status = A.status[k];
    const InstDev I = A.inst[k];
    // every slot line of the allocation is loaded at once (in bounds: the
    // array holds kAlphaSlots lines per instance), and those beyond this
    // instance's slots count as zero (the wave speeds are non-negative)
    double sx[kAlphaSlots], sy[kAlphaSlots];
#pragma unroll
    for (int s = 0; s < kAlphaSlots; ++s) {
      sx[s] = acc[kAlphaStride * s];
      sy[s] = acc[kAlphaStride * s + 1];
    }
    double ax, ay;
    if (!done) {
      t += dt;
      steps += 1;
      ax = sx[0];
      ay = sy[0];
#pragma unroll
      for (int s = 1; s < kAlphaSlots; ++s) {
        const bool own = s < A.alpha_slots;
        ax = fmax(ax, own ? sx[s] : 0.0);
        ay = fmax(ay, own ? sy[s] : 0.0);
      }
      A.t[k] = t;
      A.steps[k] = steps;
      A.alpha[2 * k] = ax;
      A.alpha[2 * k + 1] = ay;
    } else {
      ax = ay = 0.0;  // unused: a done instance stays done
    }
#pragma unroll
    for (int s = 0; s < kAlphaSlots; ++s) {
      if (s < A.alpha_slots) {
        acc[kAlphaStride * s] = 0.0;
        acc[kAlphaStride * s + 1] = 0.0;
      }
    }
    if (!set_step(A, k, I, R, done, t, steps, status, ax, ay)) mine = 1;
  }
  if (mine) atomicOr(&running, 1);
  __syncthreads();
  if (threadIdx.x == 0) A.all_done[0] = running ? 0 : 1;
}

hipError_t launch_dt(const AuxArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(dt_kernel, dim3(1), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_finish(const AuxArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Start of a run of whole 1D steps: the call's parameters, zero time and step
// count, no flags, and zero wave-speed accumulators.
__global__ __launch_bounds__(256) void run_begin_kernel(const RunArgs A) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x, nt = gridDim.x * blockDim.x;
  if (t == 0) *A.run = A.R;
  for (int k = t; k < A.n_inst; k += nt) {
    A.st[0][k] = {0.0, 0, 0};
    A.flag[0][k] = 0;
    A.flag[1][k] = 0;
  }
  for (int k = t; k < A.n_inst * A.slots; k += nt)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      A.acc[b][kAlphaStride * k] = 0.0;
      A.acc[b][kAlphaStride * k + 1] = 0.0;
    }
}

// Between chunks of steps: whether any instance would take another step.
__global__ __launch_bounds__(256) void run_poll_kernel(const RunArgs A) {
  __shared__ int running;
  if (threadIdx.x == 0) running = 0;
  __syncthreads();
  const RunParams R = *A.run;
  int mine = 0;
  for (int k = threadIdx.x; k < A.n_inst; k += blockDim.x) {
    const StepState s = A.st[A.last][k];
    if (!(s.done || A.flag[A.last][k] || s.steps >= R.max_steps ||
          s.t >= R.t_final * (1.0 - 1e-14)))
      mine = 1;
  }
  if (mine) atomicOr(&running, 1);
  __syncthreads();
  if (threadIdx.x == 0) *A.running_host = running;
}

// End of a run: the state of an instance that stopped after an odd number of
// steps is in the scratch buffers and goes back to the caller's arrays; time,
// step count and status go to the pinned host arrays.  One wave per tile.
template <class TM>
__global__ __launch_bounds__(256) void run_end_kernel(const RunArgs A) {
  const int lane = threadIdx.x & 63, per = blockDim.x >> 6;
  const TM* m_odd = static_cast<const TM*>(A.m_odd);
  TM* m = static_cast<TM*>(A.m);
  for (int it = blockIdx.x * per + (threadIdx.x >> 6); it < A.n_tiles; it += gridDim.x * per) {
    const TileItem wk = A.tiles[it];
    const StepState s = A.st[A.last][wk.inst];
    const InstDev I = A.inst[wk.inst];
    if (s.steps & 1) {
      const int i = wk.start + lane;
      if (lane < kStepWidth && i < I.nx) {
        const long long o = I.offset + i;
        for (int k = 0; k < A.nc; ++k) A.u[k * A.plane + o] = A.u_odd[k * A.plane + o];
        for (int k = 0; k < A.mom_planes; ++k) m[k * A.plane + o] = m_odd[k * A.plane + o];
      }
    }
    if (wk.start == 0 && lane == 0) {
      const int f = A.flag[0][wk.inst] | A.flag[1][wk.inst];
      A.status[wk.inst] = f;
      A.t_host[wk.inst] = s.t;
      A.steps_host[wk.inst] = s.steps;
      A.status_host[wk.inst] = f;
    }
  }
}

hipError_t launch_run_begin(const RunArgs& a, hipStream_t s) {
  const int blocks = std::min(256, (a.n_inst * a.slots + 255) / 256);
  hipLaunchKernelGGL(run_begin_kernel, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_run_poll(const RunArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(run_poll_kernel, dim3(1), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_run_end(const RunArgs& a, hipStream_t s) {
  const int blocks = std::min(2048, (a.n_tiles + 3) / 4);
  if (a.mom_elem == 4)
    hipLaunchKernelGGL(run_end_kernel<float>, dim3(blocks), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(run_end_kernel<double>, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace hwenou
