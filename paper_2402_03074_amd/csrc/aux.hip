// Auxiliary kernels of the time loop: the maximum wave speed
// alpha = max |f'(u)| over the cell averages (Section 2.1, used by the
// Lax-Friedrichs flux and the CFL condition), and the start, polls and end of
// a run of steps.  The steps themselves form their time step
// dt = min(CFL dx / alpha, T - t) in 1D and CFL / (alpha_1/dx + alpha_2/dy) in
// 2D in the stage kernels (step_dt).  All per-instance state lives on the
// device, so steps follow each other without host synchronisation.
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

// Start of a run: the call's parameters, zero time and step
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

__global__ __launch_bounds__(256) void step_control_kernel(const ControlArgs A) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < A.n_inst; k += gridDim.x * blockDim.x) {
    const StepDt d = step_dt<1>(A.ctl, k, A.inst[k]);
    write_step(A.ctl, k, d);
    A.dt[k] = d.dt;
    A.alpha[2 * k] = d.ax;
    A.alpha[2 * k + 1] = 0.0;
    A.done[k] = d.done;
  }
}

hipError_t launch_step_control(const ControlArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(step_control_kernel, dim3(std::min(256, (a.n_inst + 255) / 256)), dim3(256), 0,
                     s, a);
  return hipGetLastError();
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

// Time, step count and status of an instance, into the pinned host arrays.
__device__ __forceinline__ void report(const RunArgs& A, int inst, const StepState& s) {
  const int f = A.flag[0][inst] | A.flag[1][inst];
  A.status[inst] = f;
  A.t_host[inst] = s.t;
  A.steps_host[inst] = s.steps;
  A.status_host[inst] = f;
}

__global__ __launch_bounds__(256) void run_end_kernel(const RunArgs A) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < A.n_inst; k += gridDim.x * blockDim.x)
    report(A, k, A.st[A.last][k]);
}

// End of a run of whole 1D steps: the state of an instance that stopped after
// an odd number of steps is in the scratch buffers and goes back to the
// caller's arrays.  One wave per tile.
template <class TM>
__global__ __launch_bounds__(256) void run_end_tiles_kernel(const RunArgs A) {
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
    if (wk.start == 0 && lane == 0) report(A, wk.inst, s);
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
  if (a.tiles == nullptr)
    hipLaunchKernelGGL(run_end_kernel, dim3(std::min(256, (a.n_inst + 255) / 256)), dim3(256), 0,
                       s, a);
  else if (a.mom_elem == 4)
    hipLaunchKernelGGL(run_end_tiles_kernel<float>, dim3(blocks), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(run_end_tiles_kernel<double>, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace hwenou
