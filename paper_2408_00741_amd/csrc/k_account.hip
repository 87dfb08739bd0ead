// Cost and carbon of a selection (Section VI "Cost and Carbon Emission"): per window the GPUs in
// use by the selected configurations, their price, the energy bill and the operational CO2 at the
// window's carbon intensity; totals in window order.
#include "dyn_account.h"

namespace {

// One thread per window.  GPUs = sum over the classes with a selection of n_inst x tp.
__global__ __launch_bounds__(128) void account_kernel(AccountArgs a) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= a.n_window) return;
  int64_t used = 0;
  uint32_t bad = 0;
  for (int g = 0; g < a.G; ++g) {
    const int32_t k = a.sel[(size_t)w * a.G + g];
    if (k >= a.K) bad = 1;                                 // not a candidate of the list: counted as no selection
    else if (k >= 0) used += a.cfg[k].gpus;
  }
  const double hours = ((double)used * a.window_s) / 3600.0;
  const double kwh = a.window_energy[w] / 3.6e6;
  a.gpus[w] = used;
  a.gpu_cost[w] = hours * a.gpu_hour_price;
  a.energy_cost[w] = kwh * a.kwh_price;
  a.carbon_g[w] = kwh * a.carbon[w];
  a.hours[w] = hours;
  a.servers[w] = (double)((used + a.gpus_per_server - 1) / a.gpus_per_server);
  if (bad) atomicOr(a.status, DYN_WS_BAD_REQUEST);
}

// t + x[0] + x[1] + ... in order; x in LDS, readable up to the next multiple of 16.  16 values in flight while 16 are added.
__device__ __forceinline__ double add_in_order(double t, const double* x, int n) {
  constexpr int N = 16;
  double v[N];
#pragma unroll
  for (int q = 0; q < N; ++q) v[q] = x[q];
  int at = 0;
  for (; at + N < n; at += N) {
    double next[N];
#pragma unroll
    for (int q = 0; q < N; ++q) next[q] = x[at + N + q];
#pragma unroll
    for (int q = 0; q < N; ++q) t += v[q];
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] = next[q];
  }
#pragma unroll
  for (int q = 0; q < N; ++q)
    if (at + q < n) t += v[q];
  return t;
}

// Totals in window order from 0: a wave per total, five independent sequential sums.  The chain of additions bounds it; the values
// come through LDS, the next while these are added (one at a time from memory they cost 82 ns a window).
constexpr int kTotalsChunk = 512;
__global__ __launch_bounds__(5 * DYN_WAVE) void account_totals_kernel(AccountArgs a) {
  __shared__ double s_x[5][kTotalsChunk];
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = threadIdx.x / DYN_WAVE;
  const double* x = wave == 0 ? a.hours : wave == 1 ? a.gpu_cost : wave == 2 ? a.energy_cost : wave == 3 ? a.carbon_g : a.servers;
  constexpr int kEach = kTotalsChunk / DYN_WAVE;
  double v[kEach], t = 0.0;
  auto load = [&](int w0) {
#pragma unroll
    for (int r = 0; r < kEach; ++r) v[r] = x[min(w0 + r * DYN_WAVE + lane, a.n_window - 1)];
  };
  load(0);
  for (int w = 0; w < a.n_window; w += kTotalsChunk) {
#pragma unroll
    for (int r = 0; r < kEach; ++r) s_x[wave][r * DYN_WAVE + lane] = v[r];
    __syncthreads();
    load(min(w + kTotalsChunk, a.n_window - 1));
    t = add_in_order(t, s_x[wave], min(kTotalsChunk, a.n_window - w));
    __syncthreads();
  }
  if (lane == 0) a.totals[wave] = t;
}

// Everything in one block, header included, where the cells are few: the launches would cost more than the work.  Four waves and
// 13 KB, so that the block fits beside what other streams run (16 waves and 49 KB waited until an evaluation was through: 60
// windows of 9 classes 792 us beside one, 23 so).  What bounds it: the latency of the selections, eight in flight per thread,
// and the chain of additions, five of them in five lanes.  Beyond 1024 windows the chain alone is as long as the
// kernels below take.  Measured (us; one launch, three without their gaps): 60 windows of 9 classes 3.2, 7.6; 487 of 15 12.9, 14.0;
// 1 of 16 384 17, 2757; 1440 of 9 28.6, 23.4; 1820 of 9 36.1, 27.7.
constexpr int kOneBlock = 256;                   // threads, and windows at a time
constexpr int64_t kOneBlockCells = 16384;
constexpr int32_t kOneBlockWindows = 1024;
__global__ __launch_bounds__(kOneBlock) void account_one_kernel(AccountArgs a, WsHeader* header) {
  constexpr int kAhead = 8, kRow = kOneBlock + 1;   // a row's first value lies in another bank than the next one's
  __shared__ unsigned long long s_used[kOneBlock];
  __shared__ double s_v[5 * kRow];
  __shared__ uint32_t s_bad;
  const int tid = threadIdx.x;
  if (tid == 0) s_bad = 0u;
  double t = 0.0;
  for (int w0 = 0; w0 < a.n_window; w0 += kOneBlock) {
    const int n = min(kOneBlock, a.n_window - w0), cells = n * a.G;
    s_used[tid] = 0ull;
    const bool in = tid < n;
    const double energy = in ? a.window_energy[w0 + tid] : 0.0, carbon = in ? a.carbon[w0 + tid] : 0.0;
    __syncthreads();
    const int32_t* sel = a.sel + (size_t)w0 * a.G;
    for (int c0 = tid; c0 < cells; c0 += kAhead * kOneBlock) {
      int32_t k[kAhead], gpus[kAhead];
#pragma unroll
      for (int q = 0; q < kAhead; ++q) k[q] = sel[min(c0 + q * kOneBlock, cells - 1)];
#pragma unroll
      for (int q = 0; q < kAhead; ++q) gpus[q] = a.cfg[k[q] >= 0 && k[q] < a.K ? k[q] : 0].gpus;
#pragma unroll
      for (int q = 0; q < kAhead; ++q) {
        const int c = c0 + q * kOneBlock;
        if (c >= cells) continue;
        if (k[q] >= a.K) s_bad = 1u;               // not a candidate of the list: counted as no selection
        else if (k[q] >= 0) atomicAdd(&s_used[c / a.G], (unsigned long long)gpus[q]);
      }
    }
    __syncthreads();
    if (in) {
      const int w = w0 + tid;
      const int64_t used = (int64_t)s_used[tid];
      const double hours = ((double)used * a.window_s) / 3600.0;
      const double kwh = energy / 3.6e6;
      a.gpus[w] = used;
      a.gpu_cost[w] = s_v[1 * kRow + tid] = hours * a.gpu_hour_price;
      a.energy_cost[w] = s_v[2 * kRow + tid] = kwh * a.kwh_price;
      a.carbon_g[w] = s_v[3 * kRow + tid] = kwh * carbon;
      s_v[tid] = hours;
      s_v[4 * kRow + tid] = (double)((used + a.gpus_per_server - 1) / a.gpus_per_server);
    }
    __syncthreads();
    if (tid < 5) t = add_in_order(t, s_v + tid * kRow, n);
  }
  if (tid < 5) a.totals[tid] = t;
  if (tid == 0) {
    header->status = s_bad ? DYN_WS_BAD_REQUEST : 0u;
    header->kind = DYN_WS_KIND_WORD;
    header->cells = 0;
  }
}

__global__ void account_header_kernel(WsHeader* header) {
  header->status = 0u;
  header->kind = DYN_WS_KIND_WORD;
  header->cells = 0;
}

}  // namespace

hipError_t dyn_launch_account(const AccountArgs& a, WsHeader* header, hipStream_t s) {
  DynTimed timed(DYN_K_TOTALS, s);
  if (a.n_window <= kOneBlockWindows && (int64_t)a.n_window * a.G <= kOneBlockCells) {
    hipLaunchKernelGGL(account_one_kernel, dim3(1), dim3(kOneBlock), 0, s, a, header);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(account_header_kernel, dim3(1), dim3(1), 0, s, header);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(account_kernel, dim3((unsigned)((a.n_window + 127) / 128)), dim3(128), 0, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(account_totals_kernel, dim3(1), dim3(5 * DYN_WAVE), 0, s, a);
  return hipGetLastError();
}
