// Least-cost feasible configuration per cell (Section IV-B "Scale-up/down": filter what
// violates the SLO, then take the minimum energy), one wavefront per cell striding the
// configuration axis, then the per-window totals of the objective (Eq. 1 sums over the
// pools).  cost = energy + idle_cost_weight * n * power(load 0) * window.
#include <algorithm>

#include "dyn_mixed.h"

namespace {

// Four waves: blocks of 16 (10 us instead of 11 at 487 windows of 15 classes) waited until the kernels of other streams that
// fill the device were through (the plan beside an evaluation 949 us, 204 so).
constexpr int kWavesPerBlock = 4;
constexpr int32_t kNone = 0x7FFFFFFF;

// In the place of an energy: no feasible configuration (a NaN with bits of its own, so that an energy that is NaN still counts as one).
__device__ __forceinline__ double none_mark() { return __longlong_as_double(0x7FF8A5C3E1D20F47ll); }
__device__ __forceinline__ bool is_none(double e) { return __double_as_longlong(e) == 0x7FF8A5C3E1D20F47ll; }

// Least-cost feasible candidate of one cell by one wave: first each lane over its rows, kRowsInFlight loaded at a time, then over
// the lanes.
constexpr int kRowsInFlight = 8;
struct Best { double cost, e; int32_t k; };

// candidates [k0, k1); `idle_cost`: their idle terms, from k0 on (IDLE)
template <bool IDLE>
__device__ __forceinline__ void best_of_rows(const SelectArgs& a, int64_t cell, int k0, int k1, const double* idle_cost, int lane, Best* best) {
  const double* e_row = a.energy + (size_t)cell * a.K;
  const uint8_t* f_row = a.flags + (size_t)cell * a.K;
  for (int at = k0 + lane; at < k1; at += kRowsInFlight * DYN_WAVE) {
    double e[kRowsInFlight];
    uint32_t fl[kRowsInFlight];
#pragma unroll
    for (int r = 0; r < kRowsInFlight; ++r) {
      const int k = min(at + r * DYN_WAVE, k1 - 1);
      e[r] = e_row[k];
      fl[r] = f_row[k];
    }
#pragma unroll
    for (int r = 0; r < kRowsInFlight; ++r) {
      const int k = at + r * DYN_WAVE;
      const double cost = IDLE ? e[r] + idle_cost[min(k, k1 - 1) - k0] : e[r];
      // first feasible candidate, or strictly cheaper than the best so far (k ascending per lane)
      if (k < k1 && (fl[r] & DYN_F_FEASIBLE) && (best->k == kNone || cost < best->cost)) *best = {cost, e[r], k};
    }
  }
}

// wave minimum of (cost, k): lower cost wins, equal cost -> lower index; lanes without a
// feasible candidate carry k = kNone and lose every comparison against a real candidate
__device__ __forceinline__ void best_of_lanes(Best* best) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const double oc = __shfl_xor(best->cost, d, DYN_WAVE);
    const double oe = __shfl_xor(best->e, d, DYN_WAVE);
    const int32_t ok = __shfl_xor(best->k, d, DYN_WAVE);
    const bool take = (ok != kNone) && (best->k == kNone || oc < best->cost || (oc == best->cost && ok < best->k));
    if (take) *best = {oc, oe, ok};
  }
}

__device__ __forceinline__ void store_best(const SelectArgs& a, int64_t cell, const Best& best) {
  a.sel[cell] = best.k == kNone ? -1 : best.k;
  a.sel_energy[cell] = best.e;    // +inf when nothing is feasible
  a.sel_cost[cell] = best.cost;
}

__device__ __forceinline__ void window_total(const double* s_e, int G, double* energy, int32_t* infeasible);

// A block per window: a wave per class in turn, then the window's totals in class order.
__global__ __launch_bounds__(kWavesPerBlock* DYN_WAVE) void select_window_kernel(SelectArgs a) {
  extern __shared__ double s_e[];          // [G] selected energy, or none_mark()
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE);
  const int w = blockIdx.x;
  for (int g = wave; g < a.G; g += kWavesPerBlock) {
    const int64_t cell = (int64_t)w * a.G + g;
    Best best = {__builtin_inf(), __builtin_inf(), kNone};
    best_of_rows<false>(a, cell, 0, a.K, nullptr, lane, &best);
    best_of_lanes(&best);
    if (lane == 0) {
      store_best(a, cell, best);
      s_e[g] = best.k != kNone ? best.e : none_mark();
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) window_total(s_e, a.G, &a.win_energy[w], &a.win_inf[w]);
}

// A block per class and four windows, a wave per window.  The idle terms of the class's candidates are the same in every
// window: the block forms them once, a chunk of candidates at a time, in LDS (formed by every lane of every cell they
// were most of what the kernel loaded: 487 windows, 15 classes, 429 candidates 19 us,
// 11 us so).
constexpr int kIdleChunk = 2048;
template <bool IDLE>
__global__ __launch_bounds__(kWavesPerBlock* DYN_WAVE) void select_kernel(SelectArgs a) {
  extern __shared__ double s_idle[];       // [min(K, kIdleChunk)]
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE);
  const int g = (int)(blockIdx.x % (unsigned)a.G), w = (int)(blockIdx.x / (unsigned)a.G) * kWavesPerBlock + wave;
  const int64_t cell = (int64_t)w * a.G + g;
  Best best = {__builtin_inf(), __builtin_inf(), kNone};
  for (int k0 = 0; k0 < a.K; k0 += kIdleChunk) {
    const int k1 = min(k0 + kIdleChunk, a.K);
    if (IDLE) {
      __syncthreads();
      const double* pw0_row = a.pw0 + (size_t)g * a.n_tp_f;
      for (int k = k0 + threadIdx.x; k < k1; k += blockDim.x) {
        const DevCfg c = a.cfg[k];
        const double pw0 = (c.u != 0.0) ? (1.0 - c.u) * pw0_row[c.row_lo] + c.u * pw0_row[c.row_hi]
                                        : pw0_row[c.row_lo];
        s_idle[k - k0] = a.idle_w * ((c.nd * pw0) * a.window_s);
      }
      __syncthreads();
    }
    if (w < a.n_window) best_of_rows<IDLE>(a, cell, k0, k1, s_idle, lane, &best);
  }
  if (w >= a.n_window) return;
  best_of_lanes(&best);
  if (lane == 0) store_best(a, cell, best);
}

// Sum of the selected energies of a window in class order, and how many classes have none.
__device__ __forceinline__ void window_total(const double* s_e, int G, double* energy, int32_t* infeasible) {
  double e = 0.0;
  int32_t ninf = 0;
  int g = 0;
  for (; g + 8 <= G; g += 8) {             // operands first, then the additions in class order
    double v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = s_e[g + q];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (is_none(v[q])) ++ninf; else e += v[q];
    }
  }
  for (; g < G; ++g) {
    const double v = s_e[g];
    if (is_none(v)) ++ninf; else e += v;
  }
  *energy = e;
  *infeasible = ninf;
}

// A block sums `per` windows: their cells go to LDS in one coalesced sweep, rows of `stride` doubles (odd: the threads that
// sum read different banks).  per == 0: a thread per window reads its cells itself (classes beyond one block's LDS).
__global__ __launch_bounds__(256) void window_totals_kernel(const int32_t* __restrict__ sel, const double* __restrict__ sel_energy,
                                                            int32_t n_window, int32_t G, int32_t per, int32_t stride, double* __restrict__ win_energy,
                                                            int32_t* __restrict__ win_inf) {
  extern __shared__ double s_e[];
  if (per == 0) {
    const int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= n_window) return;
    double e = 0.0;
    int32_t ninf = 0;
    for (int g = 0; g < G; ++g) {  // fixed order: g ascending
      const size_t c = (size_t)w * G + g;
      if (sel[c] >= 0) e += sel_energy[c]; else ++ninf;
    }
    win_energy[w] = e;
    win_inf[w] = ninf;
    return;
  }
  const int w0 = blockIdx.x * per, n = min(per, n_window - w0), cells = n * G;
  const size_t c0 = (size_t)w0 * G;
  for (int q0 = threadIdx.x; q0 < cells; q0 += 4 * 256) {
    int32_t k[4];
    double e[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = min(q0 + r * 256, cells - 1);
      k[r] = sel[c0 + q];
      e[r] = sel_energy[c0 + q];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = q0 + r * 256;
      if (q < cells) s_e[q / G * stride + q % G] = k[r] >= 0 ? e[r] : none_mark();
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < n) window_total(s_e + threadIdx.x * stride, G, &win_energy[w0 + threadIdx.x], &win_inf[w0 + threadIdx.x]);
}

// Fused path: every cell has n_used partial records in ascending configuration order; a
// strict "<" scan keeps the lowest index among equal costs.  One block per window when the
// classes of a window fit a block: the class results go through LDS and thread 0 adds them
// in class order.
__device__ __forceinline__ void scan_partials(const SelPart* __restrict__ p, int n, double* bc, double* be, int32_t* bk) {
  double c = __builtin_inf(), e = __builtin_inf();
  int32_t k = -1;
  int i = 0;
  if (n <= 16) {                 // the usual case: every record in flight at once, compared in candidate order
    SelPart q[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      q[j].k = -1;
      if (j < n) q[j] = p[j];
    }
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (q[j].k >= 0 && (k < 0 || q[j].cost < c)) { c = q[j].cost; e = q[j].energy; k = q[j].k; }
    *bc = c; *be = e; *bk = k;
    return;
  }
  for (; i + 4 <= n; i += 4) {   // four independent loads in flight, compared in candidate order
    const SelPart q0 = p[i], q1 = p[i + 1], q2 = p[i + 2], q3 = p[i + 3];
    if (q0.k >= 0 && (k < 0 || q0.cost < c)) { c = q0.cost; e = q0.energy; k = q0.k; }
    if (q1.k >= 0 && (k < 0 || q1.cost < c)) { c = q1.cost; e = q1.energy; k = q1.k; }
    if (q2.k >= 0 && (k < 0 || q2.cost < c)) { c = q2.cost; e = q2.energy; k = q2.k; }
    if (q3.k >= 0 && (k < 0 || q3.cost < c)) { c = q3.cost; e = q3.energy; k = q3.k; }
  }
  for (; i < n; ++i) {
    const SelPart q = p[i];
    if (q.k >= 0 && (k < 0 || q.cost < c)) { c = q.cost; e = q.energy; k = q.k; }
  }
  *bc = c; *be = e; *bk = k;
}

__global__ __launch_bounds__(256) void finish_kernel(FinishArgs a) {
  extern __shared__ double s_e[];          // [G] selected energy, or none_mark()
  const int w = blockIdx.x;
  for (int g = threadIdx.x; g < a.G; g += blockDim.x) {
    const size_t cell = (size_t)w * a.G + g;
    double bc, be;
    int32_t bk;
    scan_partials(a.part + cell * (size_t)a.n_wslot, a.n_used, &bc, &be, &bk);
    a.sel[cell] = bk;
    a.sel_energy[cell] = be;
    a.sel_cost[cell] = bc;
    s_e[g] = bk >= 0 ? be : none_mark();
  }
  __syncthreads();
  if (threadIdx.x == 0) window_total(s_e, a.G, &a.win_energy[w], &a.win_inf[w]);
}

__global__ __launch_bounds__(256) void finish_cells_kernel(FinishArgs a) {   // classes beyond one block's LDS
  const int64_t cells = (int64_t)a.n_window * a.G;
  const int64_t cell = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= cells) return;
  double bc, be;
  int32_t bk;
  scan_partials(a.part + (size_t)cell * a.n_wslot, a.n_used, &bc, &be, &bk);
  a.sel[cell] = bk;
  a.sel_energy[cell] = be;
  a.sel_cost[cell] = bc;
}

}  // namespace

hipError_t dyn_launch_window_totals(const int32_t* sel, const double* sel_energy, int32_t n_window, int32_t G,
                                    double* win_energy, int32_t* win_inf, hipStream_t s) {
  DynTimed timed(DYN_K_TOTALS, s);
  const int stride = G | 1;
  const int per = stride <= 4096 ? std::min(64, 4096 / stride) : 0;   // windows a block sums
  const int each = per ? per : 256;
  hipLaunchKernelGGL(window_totals_kernel, dim3((unsigned)((n_window + each - 1) / each)), dim3(256), (size_t)per * stride * sizeof(double), s, sel,
                     sel_energy, n_window, G, per, stride, win_energy, win_inf);
  return hipGetLastError();
}

hipError_t dyn_launch_finish(const FinishArgs& a, hipStream_t s) {
  if (a.G <= 4096) {
    DynTimed timed(DYN_K_SELECT, s);
    hipLaunchKernelGGL(finish_kernel, dim3((unsigned)a.n_window), dim3(a.G <= 64 ? 64 : 256), (size_t)a.G * sizeof(double),
                       s, a);
    return hipGetLastError();
  }
  const int64_t cells = (int64_t)a.n_window * a.G;
  {
    DynTimed timed(DYN_K_SELECT, s);
    hipLaunchKernelGGL(finish_cells_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, s, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return dyn_launch_window_totals(a.sel, a.sel_energy, a.n_window, a.G, a.win_energy, a.win_inf, s);
}

// Without an idle term a block per window sums up as it selects, which saves a launch, where its waves have few classes each or
// the windows fill the device all the same.  Measured (us of the whole plan, a block per window and two kernels): 2016 windows of 20
// classes 364, 377; 300 of 25 298, 292; 256 of 100 281, 254.  With an idle term a block takes one class of several windows.
hipError_t dyn_launch_select(const SelectArgs& a, hipStream_t s) {
  const bool idle = a.idle_w != 0.0;
  if (!idle && a.G <= 4096 && (a.n_window >= 1024 || a.G <= 2 * kWavesPerBlock)) {
    DynTimed timed(DYN_K_SELECT, s);
    hipLaunchKernelGGL(select_window_kernel, dim3((unsigned)a.n_window), dim3(kWavesPerBlock * DYN_WAVE), (size_t)a.G * sizeof(double), s, a);
    return hipGetLastError();
  }
  {
    DynTimed timed(DYN_K_SELECT, s);
    const dim3 grid((unsigned)((int64_t)a.G * ((a.n_window + kWavesPerBlock - 1) / kWavesPerBlock))), block(kWavesPerBlock * DYN_WAVE);
    const size_t lds = (size_t)std::min(a.K, kIdleChunk) * sizeof(double);
    if (idle) hipLaunchKernelGGL(select_kernel<true>, grid, block, lds, s, a);
    else hipLaunchKernelGGL(select_kernel<false>, grid, block, 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return dyn_launch_window_totals(a.sel, a.sel_energy, a.n_window, a.G, a.win_energy, a.win_inf, s);
}
