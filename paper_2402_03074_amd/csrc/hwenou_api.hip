// Host side of libhwenou.so: handle management, work lists of the
// persistent stage launches, the stage entry point and the graph-replayed
// time loop.  See include/hwenou.h for the contract of every call.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/hwenou.h"
#include "hwenou_internal.hpp"

using namespace hwenou;

namespace {

thread_local char g_hip_error[256] = "";

int hip_fail(hipError_t e, const char* what) {
  std::snprintf(g_hip_error, sizeof g_hip_error, "HIP error in %s: %s", what,
                hipGetErrorString(e));
  return HWENOU_EHIP;
}

#define HIPCHK(call)                               \
  do {                                             \
    hipError_t e_ = (call);                        \
    if (e_ != hipSuccess) return hip_fail(e_, #call); \
  } while (0)

}  // namespace

struct hwenou_handle {
  hwenou_desc desc;
  int n_inst = 0;
  int dim = 1, nc = 1;
  bool mixed = false;
  long long plane = 0;
  size_t mom_elem = 8;
  hipStream_t stream = nullptr;      // caller's stream
  hipStream_t own = nullptr;         // capture stream, and the autotuner's
  hipEvent_t ev_in = nullptr;
  hipEvent_t ev_poll[2] = {nullptr, nullptr};
  std::vector<hwenou_inst> inst;
  // per-instance device records and state, in one allocation
  void* d_arena = nullptr;
  InstDev* d_inst = nullptr;
  TileItem* d_tiles = nullptr;       // whole-step tiles (1D)
  int* d_status = nullptr;
  double *d_alpha = nullptr, *d_dt = nullptr;  // the autotuner's and the one-stage 1D steps'
  int* d_done = nullptr;
  RunParams* d_run = nullptr;        // parameters of the current hwenou_advance call
  StepState* d_state = nullptr;      // [2][n_inst]
  int* d_flag = nullptr;             // [2][n_inst]
  double* d_part = nullptr;          // partial maxima of the wave-speed reduction
  int part_blocks = 1;
  double* d_acc = nullptr;           // [4][n_inst][slots][kAlphaStride], with the work lists
  size_t acc_lines = 0;              // n_inst * slots it has room for
  // pinned host results of a run
  double* h_t = nullptr;             // [n_inst]
  int *h_steps = nullptr, *h_status = nullptr;  // [n_inst]
  int* h_running = nullptr;          // [2]: whether any instance runs on, last two chunks
  // the graph of kGraphSteps steps of hwenou_advance (one stage per launch),
  // kept while the state pointers and the work lists stay the same
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  const void *g_ubar = nullptr, *g_mom = nullptr;
  // scratch of the time loop and the stage base, in one allocation
  void* d_scratch = nullptr;
  void* m_base = nullptr;            // v^_n (w^_n) [dim][nc][plane]
  double *s1u = nullptr, *s2u = nullptr;
  void *s1m = nullptr, *s2m = nullptr;
  const double* u_base = nullptr;    // recorded by stage 0
  // whole steps in one launch (1D; step1d.hip): usable when every instance has
  // two periodic sides or none
  bool whole_steps = false;
  int n_tiles = 0, step_waves = 0;
  // runs of whole steps in one launch, a block of this many waves per instance
  // (0: not for this handle)
  int block_waves = 0;
  // work lists
  int waves_per_cu = 0, rows_per_item = 0;
  int n_cu = 256;
  int n_xcd = 8;  // chiplets, each with its own L2
  int slots = 1;  // wave-speed accumulators per instance
  WorkItem* d_work = nullptr;        // with d_work_ptr behind it
  int* d_work_ptr = nullptr;
  int n_waves = 0;      // runs; of pairs of waves if `pairs`
  bool pairs = false;   // 2D: a pair of waves per run
  bool work_dirty = true;
};

namespace {

int dalloc(void** p, size_t bytes) {
  *p = nullptr;
  hipError_t e = hipMalloc(p, bytes ? bytes : 1);
  if (e == hipErrorOutOfMemory) return HWENOU_ENOMEM;
  if (e != hipSuccess) return hip_fail(e, "hipMalloc");
  return HWENOU_OK;
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

constexpr int kStepThreads = 256;  // block of the whole-step 1D kernel

// Steps per graph replay where a step is three launches; the rest of a call's
// steps are launched one by one.  A multiple of four, the number of
// accumulator buffers that the steps rotate through.
constexpr int kGraphSteps = 8;

void drop_graph(hwenou_handle* h) {
  if (h->exec) (void)hipGraphExecDestroy(h->exec);
  if (h->graph) (void)hipGraphDestroy(h->graph);
  h->exec = nullptr;
  h->graph = nullptr;
  h->g_ubar = h->g_mom = nullptr;
}

void free_handle(hwenou_handle* h) {
  if (!h) return;
  drop_graph(h);
  for (void* p : {h->d_arena, h->d_scratch, (void*)h->d_work, (void*)h->d_acc})
    if (p) (void)hipFree(p);
  if (h->h_t) (void)hipHostFree(h->h_t);
  for (hipEvent_t e : {h->ev_poll[0], h->ev_poll[1], h->ev_in})
    if (e) (void)hipEventDestroy(e);
  if (h->own) (void)hipStreamDestroy(h->own);
  delete h;
}

// Order the waves' runs for the chiplets.  The hardware hands the blocks of a
// launch to the XCDs in turn (block b to XCD b mod n_xcd), and every XCD has
// an L2 of its own.  The 2D work lists put runs that read the same cache
// lines next to each other (one grid: the strips of one band; many
// instances: consecutive rows of a strip, then the neighbouring strip), and
// here each XCD receives one contiguous range of the list.  For one grid the
// waves of neighbouring strips in a band then start together, march in step
// and share the columns at their common edge (the two-column halos and the
// cache lines a row segment straddles) through one L2, which fetches them
// from HBM once instead of once per XCD.
void xcd_order(std::vector<WorkItem>& items, std::vector<int>& ptr, int n_xcd) {
  const int nw = (int)ptr.size() - 1;
  if (n_xcd <= 1 || nw <= n_xcd) return;
  std::vector<int> run_of_block(nw);
  int r = 0;
  for (int x = 0; x < n_xcd; ++x)
    for (int b = x; b < nw; b += n_xcd) run_of_block[b] = r++;
  std::vector<WorkItem> it2;
  std::vector<int> p2;
  it2.reserve(items.size());
  p2.reserve(ptr.size());
  p2.push_back(0);
  for (int b = 0; b < nw; ++b) {
    const int q = run_of_block[b];
    for (int i = ptr[q]; i < ptr[q + 1]; ++i) it2.push_back(items[i]);
    p2.push_back((int)it2.size());
  }
  items.swap(it2);
  ptr.swap(p2);
}

// Build the per-wave work lists.
//  1D: tiles of kStripWidth cells; tiles are dealt out in contiguous runs.
//  2D, one grid (automatic shape): strips of kStripWidth columns, every strip
//      cut at the same rows into as many runs as fit the resident waves.
//  2D otherwise: the total strip-rows of all instances are split into equal
//      runs, one per wave, so every wave marches about the same number of
//      rows (a run that crosses the end of a strip continues at the bottom of
//      the next one).
// Also sets the number of wave-speed accumulators per instance.
int build_work(hwenou_handle* h) {
  drop_graph(h);  // the captured step graph holds the old work lists
  std::vector<WorkItem> items;
  std::vector<int> ptr;
  // a pair of waves per run, unless the caller has set the launch shape
  h->pairs = false;
  if (h->dim == 2 && h->waves_per_cu <= 0 && h->rows_per_item <= 0) {
    long long total = 0;
    int strips = 0, ny = 0;
    for (const hwenou_inst& I : h->inst) {
      const int ns = (I.nx + kStripWidth - 1) / kStripWidth;
      total += (long long)ns * I.ny;
      if ((long long)ns * I.ny > (long long)strips * ny) {
        strips = ns;
        ny = I.ny;
      }
    }
    h->pairs = use_pairs_2d(h->desc.eq, h->desc.char_decomp, h->mixed, total, strips, ny, h->n_cu);
  }
  // default: as many waves per compute unit as can be resident at once
  int wpc = h->pairs ? 2 : h->waves_per_cu;
  if (wpc <= 0) {
    const int chr = h->desc.eq == HWENOU_EQ_EULER ? h->desc.char_decomp : 0;
    const bool si = h->desc.weights == HWENOU_W_SCALE_INVARIANT;
    if (h->dim == 1)
      wpc = 4 * occupancy_stage_1d(h->desc.eq, chr, h->mixed, 256);
    else
      wpc = occupancy_stage_2d(h->desc.eq, chr, h->mixed, si, 64);
    if (wpc <= 0) wpc = 4;
  }
  const long long target_waves = (long long)h->n_cu * wpc;
  if (h->dim == 1) {
    std::vector<WorkItem> tiles;
    for (int k = 0; k < h->n_inst; ++k)
      for (int s = 0; s < h->inst[k].nx; s += kStripWidth) tiles.push_back({k, s, 0, 0});
    const long long nt = (long long)tiles.size();
    const long long nw = std::max<long long>(1, std::min<long long>(nt, target_waves));
    ptr.push_back(0);
    for (long long w = 0; w < nw; ++w) {
      const long long b = nt * (w + 1) / nw;
      ptr.push_back((int)b);
    }
    items = tiles;
  } else if (h->n_inst == 1 && h->rows_per_item <= 0) {
    // One grid: every strip is cut at the same rows into `q` runs of near-
    // equal length, and the runs are listed band by band.  The waves of one
    // band start together at the same row and march in step, so neighbouring
    // strips read their shared columns at the same time.
    const int ny = h->inst[0].ny;
    const int ns = (h->inst[0].nx + kStripWidth - 1) / kStripWidth;
    // The fewest rows per run that keep the runs within the resident waves, down
    // to one: a wave's time is that of its rows plus about 1.5 more (its two
    // boundary rows run the y-sweep, and the LDS ring is filled first), so a
    // grid too small to fill the SIMDs is fastest cut as short as it goes, and
    // no shorter than its longest run (400 x 300, component-wise: 107 us per
    // step in 100 runs of 3 rows per strip, 112 in 146 runs of 2 or 3).
    // Against runs of at least 4 rows, per Runge-Kutta step: 131 x 97 cells
    // (Euler, FP64) 204 -> 93 us, 240 x 240 (Burgers) 46 -> 34 us, 500 x 333
    // (Euler, per-interface bases) 433 -> 320 us.
    const long long fit = std::min<long long>(std::max<long long>(1, target_waves / ns), ny);
    const long long rows = (ny + fit - 1) / fit;
    const long long q = (ny + rows - 1) / rows;
    ptr.push_back(0);
    for (long long b = 0; b < q; ++b) {
      const int r0 = (int)(ny * b / q), r1 = (int)(ny * (b + 1) / q);
      for (int s = 0; s < ns; ++s) {
        items.push_back({0, s, r0, r1});
        ptr.push_back((int)items.size());
      }
    }
    xcd_order(items, ptr, h->n_xcd);
  } else {
    struct Strip {
      int inst, strip, rows;
    };
    std::vector<Strip> strips;
    long long total = 0;
    for (int k = 0; k < h->n_inst; ++k) {
      const int ns = (h->inst[k].nx + kStripWidth - 1) / kStripWidth;
      for (int s = 0; s < ns; ++s) {
        strips.push_back({k, s, h->inst[k].ny});
        total += h->inst[k].ny;
      }
    }
    // (a given shape has at least 4 rows per run)
    const long long per = h->rows_per_item > 0
                              ? std::max(h->rows_per_item, 4)
                              : std::max<long long>(1, (total + target_waves - 1) / target_waves);
    ptr.push_back(0);
    long long used = 0;  // rows assigned to the current wave
    for (const Strip& s : strips) {
      int r = 0;
      while (r < s.rows) {
        const int take = (int)std::min<long long>(s.rows - r, per - used);
        items.push_back({s.inst, s.strip, r, r + take});
        r += take;
        used += take;
        if (used == per) {
          ptr.push_back((int)items.size());
          used = 0;
        }
      }
    }
    if (used > 0) ptr.push_back((int)items.size());
    xcd_order(items, ptr, h->n_xcd);
  }
  h->n_waves = (int)ptr.size() - 1;
  // waves on the busiest instance, for the number of wave-speed accumulators:
  // one per 64 of them, a power of two from 1 to kAlphaSlots
  int busiest = 0;
  if (h->whole_steps) {
    int w = h->waves_per_cu;
    if (w <= 0) {
      const int chr = h->desc.eq == HWENOU_EQ_EULER ? h->desc.char_decomp : 0;
      w = kStepThreads / 64 * occupancy_step_1d(h->desc.eq, chr, h->mixed, kStepThreads);
      if (w <= 0) w = 4;
    }
    h->step_waves = (int)std::min<long long>(h->n_tiles, (long long)h->n_cu * w);
    for (const hwenou_inst& I : h->inst) {
      const long long nt = (I.nx + kStepWidth - 1) / kStepWidth;
      busiest = std::max(busiest, (int)(nt * h->step_waves / h->n_tiles) + 1);
    }
  } else {
    std::vector<int> waves(h->n_inst, 0), last(h->n_inst, -1);
    for (int w = 0; w < h->n_waves; ++w)
      for (int i = ptr[w]; i < ptr[w + 1]; ++i) {
        const int k = items[i].inst;
        if (last[k] != w) {
          last[k] = w;
          ++waves[k];
        }
      }
    busiest = waves.empty() ? 0 : *std::max_element(waves.begin(), waves.end());
  }
  h->slots = 1;
  while (h->slots < kAlphaSlots && 64 * h->slots < busiest) h->slots *= 2;
  if (h->acc_lines < (size_t)h->n_inst * h->slots) {
    if (h->d_acc) (void)hipFree(h->d_acc);
    h->d_acc = nullptr;
    h->acc_lines = (size_t)h->n_inst * h->slots;
    void* q = nullptr;
    const int rc = dalloc(&q, 4 * h->acc_lines * kAlphaStride * sizeof(double));
    if (rc) {
      h->acc_lines = 0;
      return rc;
    }
    h->d_acc = static_cast<double*>(q);
  }
  if (h->d_work) (void)hipFree(h->d_work);
  h->d_work = nullptr;
  h->d_work_ptr = nullptr;
  const size_t item_bytes = items.size() * sizeof(WorkItem), ptr_bytes = ptr.size() * sizeof(int);
  void* q = nullptr;
  const int rc = dalloc(&q, item_bytes + ptr_bytes);
  if (rc) return rc;
  h->d_work = static_cast<WorkItem*>(q);
  h->d_work_ptr = reinterpret_cast<int*>(static_cast<char*>(q) + item_bytes);
  std::vector<char> lists(item_bytes + ptr_bytes);
  std::memcpy(lists.data(), items.data(), item_bytes);
  std::memcpy(lists.data() + item_bytes, ptr.data(), ptr_bytes);
  HIPCHK(hipMemcpy(q, lists.data(), lists.size(), hipMemcpyHostToDevice));
  h->work_dirty = false;
  return HWENOU_OK;
}

}  // namespace

SchemeParams hwenou::scheme_params(const hwenou_desc& d) {
  SchemeParams P;
  P.adv_x = d.adv[0];
  P.adv_y = d.adv[1];
  P.gas_gamma = d.gas_gamma;
  P.gamma_low = d.gamma_low;
  P.eps = d.eps;
  P.ave_mul = d.weights == HWENOU_W_ZQ ? 0.0 : 1.0;
  P.ave_add = d.weights == HWENOU_W_ZQ ? 1.0 : 0.0;
  P.nonlin = d.weights == HWENOU_W_LINEAR ? 0.0 : 1.0;
  return P;
}

namespace {

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// One stage launch: with the caller's dt and alpha (ctl.run == nullptr; flags
// go to d_status), or as part of a run.
int launch_stage(hwenou_handle* h, int s, const double* dt, const double* alpha,
                 const StepControl& ctl, const double* u_in, const void* m_in, double* u_out,
                 void* m_out, hipStream_t st) {
  if (h->work_dirty) {
    int rc = build_work(h);
    if (rc) return rc;
  }
  const SchemeParams P = scheme_params(h->desc);
  const int chr = h->desc.eq == HWENOU_EQ_EULER ? h->desc.char_decomp : 0;
  const bool si = h->desc.weights == HWENOU_W_SCALE_INVARIANT;
  hipError_t e;
  auto fill = [&](auto& A, auto* mi, auto* mo, auto* mb) {
    A.P = P;
    A.inst = h->d_inst;
    A.ctl = ctl;
    A.dt = dt;
    A.alpha = alpha;
    A.done = ctl.run && h->dim == 1 ? h->d_done : nullptr;
    A.u_in = u_in;
    A.m_in = mi;
    A.u_base = h->u_base;
    A.m_base = mb;
    A.u_out = u_out;
    A.m_out = mo;
    A.status = ctl.run ? ctl.flag_out : h->d_status;
    A.plane = h->plane;
    A.work = h->d_work;
    A.work_ptr = h->d_work_ptr;
    A.n_waves = h->n_waves;
    A.stage = s;
  };
  if (h->mixed) {
    StageArgs<float> A{};
    fill(A, static_cast<const float*>(m_in), static_cast<float*>(m_out),
         static_cast<float*>(h->m_base));
    if (h->dim == 1)
      e = launch_stage_1d(h->desc.eq, chr, true, &A, (h->n_waves + 3) / 4, 256, st);
    else
      e = launch_stage_2d(h->desc.eq, chr, true, si, &A, h->n_waves, 64, st);
  } else {
    StageArgs<double> A{};
    fill(A, static_cast<const double*>(m_in), static_cast<double*>(m_out),
         static_cast<double*>(h->m_base));
    if (h->dim == 1)
      e = launch_stage_1d(h->desc.eq, chr, false, &A, (h->n_waves + 3) / 4, 256, st);
    else
      e = h->pairs ? launch_pair_2d(si, A, h->n_waves, st)
                   : launch_stage_2d(h->desc.eq, chr, false, si, &A, h->n_waves, 64, st);
  }
  if (e != hipSuccess) return hip_fail(e, "stage kernel launch");
  return HWENOU_OK;
}

AuxArgs aux_args(hwenou_handle* h, const double* u) {
  AuxArgs a{};
  a.P = scheme_params(h->desc);
  a.eq = h->desc.eq;
  a.dim = h->dim;
  a.n_inst = h->n_inst;
  a.inst = h->d_inst;
  a.plane = h->plane;
  a.u = u;
  a.alpha = h->d_alpha;
  a.alpha_stride = 2;
  a.part = h->d_part;
  a.part_blocks = h->part_blocks;
  a.status = h->d_status;
  return a;
}

}  // namespace

namespace hwenou {

int check_desc(const hwenou_desc* d) {
  if (!d) return HWENOU_EINVAL;
  if (d->dim != 1 && d->dim != 2) return HWENOU_EINVAL;
  if (d->eq < HWENOU_EQ_ADVECTION || d->eq > HWENOU_EQ_EULER) return HWENOU_EINVAL;
  if (d->precision != HWENOU_FP64 && d->precision != HWENOU_MIXED) return HWENOU_EINVAL;
  if (d->weights < HWENOU_W_SCALE_INVARIANT || d->weights > HWENOU_W_LINEAR) return HWENOU_EINVAL;
  if (d->char_decomp < HWENOU_CHAR_COMPONENT || d->char_decomp > HWENOU_CHAR_INTERFACE)
    return HWENOU_EINVAL;
  if (d->char_decomp == HWENOU_CHAR_INTERFACE && d->eq == HWENOU_EQ_EULER && d->dim != 2)
    return HWENOU_EINVAL;
  if (!(d->gamma_low > 0.0) || d->gamma_low * (d->dim == 1 ? 2 : 4) >= 1.0) return HWENOU_EINVAL;
  if (!(d->eps >= 0.0)) return HWENOU_EINVAL;
  if (d->eq == HWENOU_EQ_EULER && !(d->gas_gamma > 1.0)) return HWENOU_EINVAL;
  return HWENOU_OK;
}

int check_inst(const hwenou_desc* d, const hwenou_inst& I) {
  const int ny = d->dim == 1 ? 1 : I.ny;
  if (I.nx < 3 || (d->dim == 2 && ny < 3)) return HWENOU_EINVAL;
  if (!(I.x1 > I.x0) || (d->dim == 2 && !(I.y1 > I.y0))) return HWENOU_EINVAL;
  for (int s = 0; s < 2 * d->dim; ++s)
    if (I.bc[s] != HWENOU_BC_PERIODIC && I.bc[s] != HWENOU_BC_TRANSMISSIVE &&
        !(I.bc[s] == HWENOU_BC_REFLECTIVE && d->eq == HWENOU_EQ_EULER))
      return HWENOU_EINVAL;
  if (I.offset < 0) return HWENOU_EINVAL;
  const long long n = (long long)I.nx * ny;
  if (n > (1LL << 29)) return HWENOU_EUNSUPPORTED;  // 32-bit byte offsets in the kernels
  return HWENOU_OK;
}

InstDev inst_dev(const hwenou_desc* d, const hwenou_inst& I) {
  InstDev r;
  r.nx = I.nx;
  r.ny = d->dim == 1 ? 1 : I.ny;
  for (int s = 0; s < 4; ++s) r.bc[s] = (s < 2 * d->dim) ? I.bc[s] : HWENOU_BC_PERIODIC;
  r.dx = (I.x1 - I.x0) / I.nx;
  r.dy = d->dim == 1 ? 1.0 : (I.y1 - I.y0) / I.ny;
  r.offset = I.offset;
  return r;
}

}  // namespace hwenou

extern "C" {

const char* hwenou_strerror(int code) {
  switch (code) {
    case HWENOU_OK: return "success";
    case HWENOU_EINVAL: return "invalid argument";
    case HWENOU_ENOMEM: return "out of device memory";
    case HWENOU_EHIP: return g_hip_error[0] ? g_hip_error : "HIP error";
    case HWENOU_ENONPHYSICAL: return "non-physical state (rho <= 0, p <= 0 or non-finite)";
    case HWENOU_EUNSUPPORTED: return "unsupported configuration";
    case HWENOU_ESCRATCH:
      return "instance too large for the fixed scratch of hwenou_step_noalloc "
             "(HWENOU_NOALLOC_MAX_BYTES)";
    default: return "unknown error code";
  }
}


int hwenou_create(const hwenou_desc* d, int n_inst, const hwenou_inst* inst, void* stream,
                  hwenou_handle** out) {
  if (!out) return HWENOU_EINVAL;
  *out = nullptr;
  if (!d || !inst || n_inst < 1) return HWENOU_EINVAL;
  int rc0 = check_desc(d);
  if (rc0) return rc0;
  // instances: sizes, domains, boundary conditions, non-overlapping ranges
  std::vector<std::pair<long long, long long>> ranges;
  long long plane = 0;
  for (int k = 0; k < n_inst; ++k) {
    const hwenou_inst& I = inst[k];
    if ((rc0 = check_inst(d, I))) return rc0;
    const long long n = (long long)I.nx * (d->dim == 1 ? 1 : I.ny);
    ranges.push_back({I.offset, I.offset + n});
    plane = std::max(plane, (long long)(I.offset + n));
  }
  std::sort(ranges.begin(), ranges.end());
  for (size_t k = 1; k < ranges.size(); ++k)
    if (ranges[k].first < ranges[k - 1].second) return HWENOU_EINVAL;

  hwenou_handle* h = new hwenou_handle();
  h->desc = *d;
  if (d->dim == 1) {
    h->desc.adv[1] = 0.0;
  }
  h->n_inst = n_inst;
  h->dim = d->dim;
  h->nc = d->eq == HWENOU_EQ_EULER ? d->dim + 2 : 1;
  h->mixed = d->precision == HWENOU_MIXED;
  h->mom_elem = h->mixed ? 4 : 8;
  h->plane = plane;
  h->stream = static_cast<hipStream_t>(stream);
  h->inst.assign(inst, inst + n_inst);
  int dev = 0;
  hipDeviceProp_t prop;
  int rc = HWENOU_OK;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipGetDeviceProperties(&prop, dev);
  if (e != hipSuccess) {
    free_handle(h);
    return hip_fail(e, "hipGetDeviceProperties");
  }
  h->n_cu = prop.multiProcessorCount;
  {
    int nx = 0;
    if (hipDeviceGetAttribute(&nx, hipDeviceAttributeNumberOfXccs, dev) == hipSuccess && nx > 0)
      h->n_xcd = nx;
  }

  // records: instances, whole-step tiles, status (uploaded); the rest is written
  // by the calls that use it
  std::vector<TileItem> tiles;
  if (d->dim == 1) {
    h->whole_steps = true;
    for (int k = 0; k < n_inst; ++k)
      if ((inst[k].bc[0] == HWENOU_BC_PERIODIC) != (inst[k].bc[1] == HWENOU_BC_PERIODIC))
        h->whole_steps = false;
  }
  if (h->whole_steps)
    for (int k = 0; k < n_inst; ++k)
      for (int s = 0; s < inst[k].nx; s += kStepWidth) tiles.push_back({k, s});
  h->n_tiles = (int)tiles.size();
  // One block per instance where a block can hold the largest and every block
  // has a CU of its own: beyond that a launch per step spreads the tiles of
  // uneven instances more evenly.
  if (h->whole_steps && n_inst <= h->n_cu) {
    int most = 0;
    for (int k = 0; k < n_inst; ++k)
      most = std::max(most, (inst[k].nx + kStepWidth - 1) / kStepWidth);
    if (most <= block_run_waves(d->eq)) h->block_waves = most;
  }
  for (int k = 0; k < n_inst; ++k)
    h->part_blocks = std::max(
        h->part_blocks, speed_blocks((long long)inst[k].nx * (d->dim == 1 ? 1 : inst[k].ny),
                                     kSpeedBlocks));
  const size_t n = n_inst;
  size_t at = 0;
  auto place = [&at](size_t bytes) {
    const size_t o = at;
    at += align256(bytes);
    return o;
  };
  const size_t o_inst = place(n * sizeof(InstDev)), o_tiles = place(tiles.size() * sizeof(TileItem)),
               o_status = place(n * sizeof(int));
  std::vector<char> records(at, 0);
  for (int k = 0; k < n_inst; ++k) {
    const InstDev I = inst_dev(d, inst[k]);
    std::memcpy(records.data() + o_inst + k * sizeof(InstDev), &I, sizeof I);
  }
  if (!tiles.empty())
    std::memcpy(records.data() + o_tiles, tiles.data(), tiles.size() * sizeof(TileItem));
  const size_t o_alpha = place(2 * n * sizeof(double)), o_dt = place(n * sizeof(double)),
               o_done = place(n * sizeof(int)),
               o_run = place(sizeof(RunParams)), o_state = place(2 * n * sizeof(StepState)),
               o_flag = place(2 * n * sizeof(int)),
               o_part = place(2 * n * h->part_blocks * sizeof(double));
  const size_t arena_bytes = at;
  // scratch: the stored modified moments and the stage buffers (whole steps
  // alternate between the caller's arrays and one stage buffer)
  const size_t mom_bytes = (size_t)h->dim * h->nc * plane * h->mom_elem;
  const size_t u_bytes = (size_t)h->nc * plane * sizeof(double);
  at = 0;
  const size_t o_base = place(mom_bytes), o_s1u = place(u_bytes), o_s1m = place(mom_bytes);
  const size_t o_s2u = h->whole_steps ? 0 : place(u_bytes);
  const size_t o_s2m = h->whole_steps ? 0 : place(mom_bytes);
  if ((rc = dalloc(&h->d_arena, arena_bytes)) || (rc = dalloc(&h->d_scratch, at))) {
    free_handle(h);
    return rc;
  }
  char* arena = static_cast<char*>(h->d_arena);
  h->d_inst = reinterpret_cast<InstDev*>(arena + o_inst);
  h->d_tiles = reinterpret_cast<TileItem*>(arena + o_tiles);
  h->d_status = reinterpret_cast<int*>(arena + o_status);
  h->d_alpha = reinterpret_cast<double*>(arena + o_alpha);
  h->d_dt = reinterpret_cast<double*>(arena + o_dt);
  h->d_done = reinterpret_cast<int*>(arena + o_done);
  h->d_run = reinterpret_cast<RunParams*>(arena + o_run);
  h->d_state = reinterpret_cast<StepState*>(arena + o_state);
  h->d_flag = reinterpret_cast<int*>(arena + o_flag);
  h->d_part = reinterpret_cast<double*>(arena + o_part);
  char* scratch = static_cast<char*>(h->d_scratch);
  h->m_base = scratch + o_base;
  h->s1u = reinterpret_cast<double*>(scratch + o_s1u);
  h->s1m = scratch + o_s1m;
  if (!h->whole_steps) {
    h->s2u = reinterpret_cast<double*>(scratch + o_s2u);
    h->s2m = scratch + o_s2m;
  }
  auto chk = [&](hipError_t e2, const char* what) {
    if (e2 != hipSuccess) {
      rc = hip_fail(e2, what);
      return false;
    }
    return true;
  };
  if (!chk(hipHostMalloc(reinterpret_cast<void**>(&h->h_t),
                         n * (sizeof(double) + 2 * sizeof(int)) + 2 * sizeof(int)),
           "hipHostMalloc") ||
      !chk(hipMemcpy(arena, records.data(), records.size(), hipMemcpyHostToDevice), "hipMemcpy") ||
      !chk(hipEventCreateWithFlags(&h->ev_poll[0], hipEventDisableTiming), "hipEventCreate") ||
      !chk(hipEventCreateWithFlags(&h->ev_poll[1], hipEventDisableTiming), "hipEventCreate") ||
      !chk(hipEventCreateWithFlags(&h->ev_in, hipEventDisableTiming), "hipEventCreate") ||
      !chk(hipStreamCreateWithFlags(&h->own, hipStreamNonBlocking), "hipStreamCreate")) {
    free_handle(h);
    return rc;
  }
  h->h_steps = reinterpret_cast<int*>(h->h_t + n);
  h->h_status = h->h_steps + n;
  h->h_running = h->h_status + n;
  rc = build_work(h);
  if (rc) {
    free_handle(h);
    return rc;
  }
  *out = h;
  return HWENOU_OK;
}

int hwenou_destroy(hwenou_handle* h) {
  if (!h) return HWENOU_EINVAL;
  (void)hipStreamSynchronize(h->stream);
  (void)hipStreamSynchronize(h->own);
  free_handle(h);
  return HWENOU_OK;
}

int hwenou_set_launch(hwenou_handle* h, int waves_per_cu, int rows_per_item) {
  if (!h || waves_per_cu < 1 || waves_per_cu > 32 || rows_per_item < 0) return HWENOU_EINVAL;
  h->waves_per_cu = waves_per_cu;
  h->rows_per_item = rows_per_item;
  h->work_dirty = true;
  return HWENOU_OK;
}

int hwenou_autotune(hwenou_handle* h, const double* ubar, const void* mom, int reps,
                    int* waves_per_cu, int* rows_per_item) {
  if (!h || !ubar || !mom || reps < 1 || !aligned(ubar, 8) || !aligned(mom, h->mom_elem))
    return HWENOU_EINVAL;
  const int chr = h->desc.eq == HWENOU_EQ_EULER ? h->desc.char_decomp : 0;
  const bool si = h->desc.weights == HWENOU_W_SCALE_INVARIANT;
  const int occ = h->dim == 1 ? 4 * occupancy_stage_1d(h->desc.eq, chr, h->mixed, 256)
                              : occupancy_stage_2d(h->desc.eq, chr, h->mixed, si, 64);
  const int base = occ > 0 ? occ : 4;
  std::vector<int> wpcs;
  for (int f : {1, 2, 4}) {
    const int w = std::min(32, base * f);
    if (std::find(wpcs.begin(), wpcs.end(), w) == wpcs.end()) wpcs.push_back(w);
  }
  if (base > 1) wpcs.push_back(std::max(1, base / 2));
  std::vector<int> rows = h->dim == 1 ? std::vector<int>{0} : std::vector<int>{0, 16, 32, 64};
  hipStream_t st = h->own;
  HIPCHK(hipEventRecord(h->ev_in, h->stream));
  HIPCHK(hipStreamWaitEvent(st, h->ev_in, 0));
  HIPCHK(hipMemsetAsync(h->d_dt, 0, h->n_inst * sizeof(double), st));
  AuxArgs a = aux_args(h, ubar);
  hipError_t e = launch_max_wavespeed(a, st);
  if (e != hipSuccess) return hip_fail(e, "max_wavespeed launch");
  hipEvent_t t0, t1;
  HIPCHK(hipEventCreate(&t0));
  HIPCHK(hipEventCreate(&t1));
  const int save_w = h->waves_per_cu, save_r = h->rows_per_item;
  float best = 1e30f;
  int bw = save_w, br = save_r;
  int rc = HWENOU_OK;
  for (int w : wpcs) {
    for (int r : rows) {
      h->waves_per_cu = w;
      h->rows_per_item = r;
      h->work_dirty = true;
      if ((rc = build_work(h))) break;
      std::vector<float> ts;
      for (int k = 0; k <= reps && !rc; ++k) {  // first launch warms up
        if (hipEventRecord(t0, st) != hipSuccess) rc = HWENOU_EHIP;
        if (!rc)
          rc = launch_stage(h, 0, h->d_dt, h->d_alpha, {}, ubar, mom, h->s1u, h->s1m, st);
        if (!rc && hipEventRecord(t1, st) != hipSuccess) rc = HWENOU_EHIP;
        if (!rc && hipEventSynchronize(t1) != hipSuccess) rc = HWENOU_EHIP;
        float ms = 0.f;
        if (!rc && hipEventElapsedTime(&ms, t0, t1) != hipSuccess) rc = HWENOU_EHIP;
        if (!rc && k > 0) ts.push_back(ms);
      }
      if (rc) break;
      std::sort(ts.begin(), ts.end());
      const float med = ts[ts.size() / 2];
      if (med < best) {
        best = med;
        bw = w;
        br = r;
      }
    }
    if (rc) break;
  }
  (void)hipEventDestroy(t0);
  (void)hipEventDestroy(t1);
  h->waves_per_cu = rc ? save_w : bw;
  h->rows_per_item = rc ? save_r : br;
  h->work_dirty = true;
  h->u_base = nullptr;  // the timed stage-0 launches overwrote the stored v^n
  if (rc) return rc == HWENOU_EHIP ? hip_fail(hipGetLastError(), "autotune timing") : rc;
  HIPCHK(hipStreamSynchronize(st));
  if (waves_per_cu) *waves_per_cu = bw;
  if (rows_per_item) *rows_per_item = br;
  return HWENOU_OK;
}

int hwenou_max_wavespeed(hwenou_handle* h, const double* ubar, double* alpha_dev) {
  if (!h || !ubar || !alpha_dev || !aligned(ubar, 8) || !aligned(alpha_dev, 8))
    return HWENOU_EINVAL;
  AuxArgs a = aux_args(h, ubar);
  a.alpha = alpha_dev;
  hipError_t e = launch_max_wavespeed(a, h->stream);
  if (e != hipSuccess) return hip_fail(e, "max_wavespeed launch");
  return HWENOU_OK;
}

int hwenou_stage(hwenou_handle* h, int s, const double* dt_dev, const double* alpha_dev,
                 const double* ubar_in, const void* mom_in, double* ubar_out, void* mom_out) {
  if (!h || s < 0 || s > 2 || !dt_dev || !alpha_dev || !ubar_in || !mom_in || !ubar_out ||
      !mom_out)
    return HWENOU_EINVAL;
  if (!aligned(ubar_in, 8) || !aligned(ubar_out, 8) || !aligned(mom_in, h->mom_elem) ||
      !aligned(mom_out, h->mom_elem) || !aligned(dt_dev, 8) || !aligned(alpha_dev, 8))
    return HWENOU_EINVAL;
  if (ubar_in == ubar_out || mom_in == mom_out) return HWENOU_EINVAL;
  if (s == 0) h->u_base = ubar_in;
  if (s > 0 && h->u_base == nullptr) return HWENOU_EINVAL;
  return launch_stage(h, s, dt_dev, alpha_dev, {}, ubar_in, mom_in, ubar_out, mom_out, h->stream);
}

int hwenou_inst_status(hwenou_handle* h, int* flags) {
  if (!h) return HWENOU_EINVAL;
  std::vector<int> st(h->n_inst);
  HIPCHK(hipStreamSynchronize(h->stream));
  HIPCHK(hipStreamSynchronize(h->own));
  HIPCHK(hipMemcpy(st.data(), h->d_status, h->n_inst * sizeof(int), hipMemcpyDeviceToHost));
  HIPCHK(hipMemset(h->d_status, 0, h->n_inst * sizeof(int)));
  int any = 0;
  for (int k = 0; k < h->n_inst; ++k) {
    if (flags) flags[k] = st[k] & 1;
    any |= st[k] & 1;
  }
  return any ? HWENOU_ENONPHYSICAL : HWENOU_OK;
}

int hwenou_status(hwenou_handle* h) { return hwenou_inst_status(h, nullptr); }

}  // extern "C"

namespace {

// Control record of the p-th step of a run: the buffers it reads and leaves.
StepControl step_control(hwenou_handle* h, int p) {
  const size_t n = h->n_inst, lines = n * h->slots * kAlphaStride;
  StepControl c;
  c.run = h->d_run;
  c.st_in = h->d_state + (p & 1) * n;
  c.st_out = h->d_state + ((p + 1) & 1) * n;
  c.flag_in = h->d_flag + (p & 1) * n;
  c.flag_out = h->d_flag + ((p + 1) & 1) * n;
  c.acc_in = h->d_acc + (p & 3) * lines;
  c.acc_out = h->d_acc + ((p + 1) & 3) * lines;
  c.acc_zero = h->d_acc + ((p + 2) & 3) * lines;
  c.slots = h->slots;
  return c;
}

// The p-th step of a run as one launch; the state alternates between the
// caller's arrays and a stage buffer.
template <class TM>
int whole_step(hwenou_handle* h, double* ubar, void* mom, int p, hipStream_t st) {
  StepArgs<TM> A{};
  A.P = scheme_params(h->desc);
  A.ctl = step_control(h, p);
  A.inst = h->d_inst;
  A.u_in = p & 1 ? h->s1u : ubar;
  A.m_in = static_cast<const TM*>(p & 1 ? h->s1m : mom);
  A.u_out = p & 1 ? ubar : h->s1u;
  A.m_out = static_cast<TM*>(p & 1 ? mom : h->s1m);
  A.plane = h->plane;
  A.tiles = h->d_tiles;
  A.n_tiles = h->n_tiles;
  A.n_waves = h->step_waves;
  const int chr = h->desc.eq == HWENOU_EQ_EULER ? h->desc.char_decomp : 0;
  const hipError_t e =
      launch_step_1d(h->desc.eq, chr, h->mixed, &A, h->step_waves, kStepThreads, st);
  return e == hipSuccess ? HWENOU_OK : hip_fail(e, "step kernel launch");
}

// Up to `steps` steps of a run in one launch, the state held by one block per
// instance from step to step; the run's state stays in its first buffers.
template <class TM>
int block_run(hwenou_handle* h, double* ubar, void* mom, int steps, hipStream_t st) {
  BlockRunArgs<TM> A{};
  A.P = scheme_params(h->desc);
  A.inst = h->d_inst;
  A.run = h->d_run;
  A.u = ubar;
  A.m = static_cast<TM*>(mom);
  A.st = h->d_state;
  A.flag = h->d_flag;
  A.acc = h->d_acc;
  A.plane = h->plane;
  A.n_inst = h->n_inst;
  A.steps = steps;
  const int chr = h->desc.eq == HWENOU_EQ_EULER ? h->desc.char_decomp : 0;
  const hipError_t e =
      launch_block_run_1d(h->desc.eq, chr, h->mixed, &A, h->n_inst, h->block_waves, st);
  return e == hipSuccess ? HWENOU_OK : hip_fail(e, "run kernel launch");
}

// The p-th step of a run: one launch, or one per stage with the last stage
// writing into the caller's arrays.
int launch_step(hwenou_handle* h, double* ubar, void* mom, int p, hipStream_t st) {
  if (h->whole_steps)
    return h->mixed ? whole_step<float>(h, ubar, mom, p, st)
                    : whole_step<double>(h, ubar, mom, p, st);
  const StepControl c = step_control(h, p);
  if (h->dim == 1) {
    const hipError_t e = launch_step_control(
        {c, h->d_inst, h->n_inst, h->d_dt, h->d_alpha, h->d_done}, st);
    if (e != hipSuccess) return hip_fail(e, "step_control launch");
  }
  h->u_base = ubar;
  int rc = launch_stage(h, 0, h->d_dt, h->d_alpha, c, ubar, mom, h->s1u, h->s1m, st);
  if (!rc) rc = launch_stage(h, 1, h->d_dt, h->d_alpha, c, h->s1u, h->s1m, h->s2u, h->s2m, st);
  if (!rc) rc = launch_stage(h, 2, h->d_dt, h->d_alpha, c, h->s2u, h->s2m, ubar, mom, st);
  return rc;
}

// The graph of kGraphSteps steps that start at a multiple of it.
int capture_steps(hwenou_handle* h, double* ubar, void* mom) {
  drop_graph(h);
  HIPCHK(hipStreamBeginCapture(h->own, hipStreamCaptureModeThreadLocal));
  int rc = HWENOU_OK;
  for (int p = 0; p < kGraphSteps && !rc; ++p) rc = launch_step(h, ubar, mom, p, h->own);
  hipError_t e = hipStreamEndCapture(h->own, &h->graph);
  if (!rc && e != hipSuccess) rc = hip_fail(e, "hipStreamEndCapture");
  if (!rc && (e = hipGraphInstantiate(&h->exec, h->graph, nullptr, nullptr, 0)) != hipSuccess) {
    h->exec = nullptr;
    rc = hip_fail(e, "hipGraphInstantiate");
  }
  if (rc) {
    drop_graph(h);
    return rc;
  }
  h->g_ubar = ubar;
  h->g_mom = mom;
  return HWENOU_OK;
}

}  // namespace

extern "C" {

int hwenou_advance(hwenou_handle* h, double* ubar, void* mom, double cfl, double t_final,
                   int max_steps, double* t_out, int* steps_out) {
  if (!h || !ubar || !mom || !(cfl > 0.0) || !(t_final >= 0.0) || max_steps < 0)
    return HWENOU_EINVAL;
  if (!aligned(ubar, 8) || !aligned(mom, h->mom_elem)) return HWENOU_EINVAL;
  int rc = HWENOU_OK;
  if (h->work_dirty && (rc = build_work(h))) return rc;
  hipStream_t st = h->stream;
  const int n = h->n_inst;
  // a run begins with one kernel that resets its state, and the wave speed of
  // the initial averages
  RunArgs r{};
  r.R = {cfl, t_final, max_steps};
  r.run = h->d_run;
  r.n_inst = n;
  r.slots = h->slots;
  r.nc = r.mom_planes = h->nc;
  r.mom_elem = (int)h->mom_elem;
  for (int b = 0; b < 2; ++b) {
    r.st[b] = h->d_state + (size_t)b * n;
    r.flag[b] = h->d_flag + (size_t)b * n;
  }
  for (int b = 0; b < 4; ++b) r.acc[b] = h->d_acc + (size_t)b * n * h->slots * kAlphaStride;
  r.last = 0;
  r.u_odd = h->s1u;
  r.m_odd = h->s1m;
  r.u = ubar;
  r.m = mom;
  r.inst = h->d_inst;
  r.plane = h->plane;
  r.tiles = h->whole_steps && !h->block_waves ? h->d_tiles : nullptr;
  r.n_tiles = h->n_tiles;
  r.status = h->d_status;
  r.t_host = h->h_t;
  r.steps_host = h->h_steps;
  r.status_host = h->h_status;
  r.running_host = nullptr;
  hipError_t e = launch_run_begin(r, st);
  if (e != hipSuccess) return hip_fail(e, "run_begin launch");
  AuxArgs a = aux_args(h, ubar);
  a.alpha = r.acc[0];
  a.alpha_stride = kAlphaStride * h->slots;
  a.status = r.flag[0];
  e = launch_max_wavespeed(a, st);
  if (e != hipSuccess) return hip_fail(e, "max_wavespeed launch");

  // Steps in chunks of growing length.  Between chunks the device writes to a
  // pinned slot whether any instance runs on, and the host waits only for the
  // answer of the chunk before, so the device never idles.  Steps after every
  // instance is done are no-ops.
  int launched = 0, chunk = h->block_waves ? 1024 : 64, slot = 0, prev = -1;
  while (launched < max_steps && !rc) {
    const int k = std::min(chunk, max_steps - launched);
    int q = 0;
    if (h->block_waves) {
      rc = h->mixed ? block_run<float>(h, ubar, mom, k, st) : block_run<double>(h, ubar, mom, k, st);
      q = k;
    } else if (!h->whole_steps && k >= kGraphSteps) {
      if (h->exec == nullptr || h->g_ubar != ubar || h->g_mom != mom)
        rc = capture_steps(h, ubar, mom);
      for (; q + kGraphSteps <= k && !rc; q += kGraphSteps)
        if ((e = hipGraphLaunch(h->exec, st)) != hipSuccess) rc = hip_fail(e, "graph replay");
    }
    for (; q < k && !rc; ++q) rc = launch_step(h, ubar, mom, launched + q, st);
    if (rc) break;
    launched += k;
    if (launched == max_steps) break;
    r.last = h->block_waves ? 0 : launched & 1;
    r.running_host = h->h_running + slot;
    if ((e = launch_run_poll(r, st)) == hipSuccess) e = hipEventRecord(h->ev_poll[slot], st);
    if (e == hipSuccess && prev >= 0) e = hipEventSynchronize(h->ev_poll[prev]);
    if (e != hipSuccess) {
      rc = hip_fail(e, "poll");
      break;
    }
    if (prev >= 0 && !h->h_running[prev]) break;
    prev = slot;
    slot ^= 1;
    chunk = std::min(2 * chunk, h->block_waves ? 4096 : 512);
  }
  h->u_base = nullptr;  // the steps' stage-0 launches overwrote the stored v^n
  if (rc) return rc;
  // and ends with one that brings its results home
  r.last = h->block_waves ? 0 : launched & 1;
  if ((e = launch_run_end(r, st)) != hipSuccess) return hip_fail(e, "run_end launch");
  HIPCHK(hipStreamSynchronize(st));
  if (t_out) std::memcpy(t_out, h->h_t, n * sizeof(double));
  if (steps_out) std::memcpy(steps_out, h->h_steps, n * sizeof(int));
  for (int k = 0; k < n; ++k)
    if (h->h_status[k] & 1) return HWENOU_ENONPHYSICAL;
  return HWENOU_OK;
}

}  // extern "C"
