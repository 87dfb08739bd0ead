// Selection with transition overheads between consecutive windows (Section IV-B "Accounting for
// the overheads"; Table VI lists the re-sharding overheads between layouts): per class the
// sequence of configurations with the least  sum_w cost(w, k_w) + sum_w transition[layout(k_{w-1})]
// [layout(k_w)], found window by window.  The step from one window to the next is factored
// through the layouts: the cheapest way to arrive in layout l' is the least over source
// layouts l of (least total ending in l) + transition[l][l'] - equal to the least over all
// predecessors because rounded addition is monotone.
//
// Two routes.  Up to 64 layouts (further down): a parallel pre-pass reduces every (window, class) to
// its layouts' least costs, one block per class walks the windows with a lane per layout keeping least
// totals only, and the predecessors and the trace-back are taken afterwards, in parallel over the windows.
// More layouts (next): one block per class walks the windows in time order (the recurrence is
// sequential, so the time per window is what counts).  The candidates are visited in an order sorted by layout
// (built on the host), a fixed number per thread, their costs loaded one window ahead; per
// window: (A) totals of the sequences ending in each candidate, (B) one thread per layout takes
// the least of its contiguous run of candidates, (C) the cheapest arrival in every layout of
// the next window, the source layouts split over several threads per destination and the
// partial results combined; four LDS-only barriers per window.  Predecessors are kept per (window,
// destination layout) in the workspace and traced back at the end in runs of windows staged
// through LDS.
#include <algorithm>

#include "dyn_path.h"
#include "dyn_device.h"
static_assert(DYN_PATH_MAX_CONFIGS == 256 * 8, "candidates are held in registers, a fixed number per thread");

namespace {

constexpr int kThreads = 256;
constexpr int kRun = 64;                                   // windows traced back per LDS stage
constexpr int kPerThread = 8;                              // candidates per thread: K <= kThreads * kPerThread
constexpr int kParts = 4;                                  // threads per destination layout in the arrival step

// Barrier that orders LDS traffic only: it does not wait for the global loads of the next window's
// costs (or the predecessor stores), which __syncthreads() would do at every step of the walk.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// lower total wins, then the lower candidate index
__device__ __forceinline__ bool beats(double v, int k, double bv, int bk) { return v < bv || (v == bv && k < bk); }

// LDS: [V by sorted position: K doubles] [transition, transposed [to][from]: NL*NL doubles] [M: NL doubles]
//      [B: NL doubles] [partial arrivals: kParts*NL doubles] [arg: NL ints] [partial args: kParts*NL ints]
//      [segment starts: NL+1 ints] [trace-back stage: kRun*NL ints] [selection of the run: kRun ints]
//      [layout of candidate k: K u16] [candidate at sorted position: K u16]
__global__ __launch_bounds__(kThreads) void path_kernel(PathArgs a) {
  extern __shared__ double smem[];
  const int g = blockIdx.x;
  const int K = a.K, NL = a.n_layout, NW = a.n_window, G = a.G;
  double* s_v = smem;
  double* s_t = s_v + K;
  double* s_m = s_t + (NL + 1) * NL;
  double* s_b = s_m + NL;
  double* s_pv = s_b + NL;                                 // [kParts][NL + 1]
  int32_t* s_arg = (int32_t*)(s_pv + kParts * (NL + 1));
  int32_t* s_pk = s_arg + NL;                              // [kParts][NL + 1]
  int32_t* s_seg = s_pk + kParts * (NL + 1);               // [NL + 1]
  int32_t* s_bp = s_seg + NL + 1;                          // [kRun][NL]
  int32_t* s_sel = s_bp + kRun * NL;                       // [kRun]
  uint16_t* s_lay = (uint16_t*)(s_sel + kRun);             // [K]
  uint16_t* s_ord = s_lay + K;                             // [K]
  __shared__ int s_gap;

  for (int i = threadIdx.x; i < NL * NL; i += kThreads) {  // transposed: a destination's sources are contiguous
    const int from = i / NL, to = i - from * NL;
    s_t[to * NL + from] = a.transition[i];
  }
  for (int i = threadIdx.x; i < NL; i += kThreads) s_t[NL * NL + i] = 0.0;   // destination "end of the sequence"
  for (int k = threadIdx.x; k < K; k += kThreads) { s_lay[k] = (uint16_t)a.layout[k]; s_ord[k] = (uint16_t)a.order[k]; }
  for (int l = threadIdx.x; l <= NL; l += kThreads) s_seg[l] = a.seg_start[l];
  int32_t* bp = a.pred + (size_t)g * NW * NL;              // [NW][NL]: predecessor when window w is entered in layout l
  int32_t* kend = a.kend + (size_t)g * NW;                 // [NW]: best end of a sequence at w, -1 for a window without a feasible candidate
  const double* pw0_row = a.pw0 + (size_t)g * a.n_tp_f;
  const double inf = __builtin_inf();
  __syncthreads();

  // this thread's candidates: sorted positions p = threadIdx.x + i * kThreads
  int my_k[kPerThread], my_l[kPerThread];
  double idle_k[kPerThread];                               // idle term (0 adds nothing)
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    const int p = threadIdx.x + i * kThreads;
    my_k[i] = p < K ? (int)s_ord[p] : -1;
    my_l[i] = p < K ? (int)s_lay[my_k[i]] : 0;
    idle_k[i] = 0.0;
    if (p < K && a.idle_w != 0.0) {
      const DevCfg cf = a.cfg[my_k[i]];
      const double pw0 = (cf.u != 0.0) ? (1.0 - cf.u) * pw0_row[cf.row_lo] + cf.u * pw0_row[cf.row_hi] : pw0_row[cf.row_lo];
      idle_k[i] = a.idle_w * ((cf.nd * pw0) * a.window_s);
    }
  }
  // cost of this thread's candidates in window w (+inf where not feasible)
  auto load_costs = [&](int w, double (&c)[kPerThread]) {
    const size_t row = ((size_t)w * G + g) * K;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      c[i] = inf;
      if (my_k[i] >= 0 && w < NW) {                        // both loads are issued before either is looked at
        const uint8_t fl = a.flags[row + my_k[i]];
        const double e = a.energy[row + my_k[i]];
        c[i] = (fl & DYN_F_FEASIBLE) ? e + idle_k[i] : inf;
      }
    }
  };
  // arrival step: thread (destination ld, part) takes the source layouts ls = part, part + n_part, ...
  const int n_part = (NL + 1) * kParts <= kThreads ? kParts : ((NL + 1) * 2 <= kThreads ? 2 : 1);
  const int c_ld = threadIdx.x % (NL + 1), c_part = threadIdx.x / (NL + 1);
  const bool c_on = c_part < n_part;
  const bool keeper = threadIdx.x == NL;                   // combines the "end" destination and keeps the class's total

  double total = 0.0, prev_end = 0.0;                      // keeper only
  bool first = true, prev_gap = true;
  double cur[kPerThread], nxt[kPerThread];
  load_costs(0, cur);
  for (int w = 0; w < NW; ++w) {
    load_costs(w + 1, nxt);                                // in flight while this window is processed
    // (A) totals of the sequences that end in window w with each candidate
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const int p = threadIdx.x + i * kThreads;
      if (p < K) s_v[p] = (first || !(cur[i] < inf)) ? cur[i] : s_b[my_l[i]] + cur[i];
    }
    lds_barrier();
    // (B) least total per layout, lowest candidate among equals (a layout's candidates ascend with the position)
    for (int l = threadIdx.x; l < NL; l += kThreads) {
      double bv = inf;
      int bk = 0x7FFFFFFF;
      const int p1 = s_seg[l + 1];
#pragma unroll 4
      for (int p = s_seg[l]; p < p1; ++p) {
        const double v = s_v[p];
        if (v < bv) { bv = v; bk = (int)s_ord[p]; }
      }
      s_m[l] = bv;
      s_arg[l] = bk;
    }
    lds_barrier();
    // (C) cheapest arrival in every layout of the next window and where it comes from; destination NL stands
    // for "the sequence ends here" (no transition): the window's best end
    if (c_on) {
      double bv = inf;
      int bk = 0x7FFFFFFF;
      const double* trow = s_t + c_ld * NL;                // row NL of the transposed table is all zero
#pragma unroll 4
      for (int ls = c_part; ls < NL; ls += n_part) {
        const double cand = s_m[ls] + trow[ls];            // +inf: nothing ends in ls
        const int ak = s_arg[ls];
        if (beats(cand, ak, bv, bk)) { bv = cand; bk = ak; }
      }
      s_pv[c_part * (NL + 1) + c_ld] = bv;
      s_pk[c_part * (NL + 1) + c_ld] = bk;
    }
    lds_barrier();
    if (threadIdx.x <= NL) {
      double bv = s_pv[threadIdx.x];
      int bk = s_pk[threadIdx.x];
      for (int q = 1; q < n_part; ++q) {
        const double v = s_pv[q * (NL + 1) + threadIdx.x];
        const int k = s_pk[q * (NL + 1) + threadIdx.x];
        if (beats(v, k, bv, bk)) { bv = v; bk = k; }
      }
      if (threadIdx.x < NL) {
        s_b[threadIdx.x] = bv;                             // read by (A) of the next window, after the barrier below
        if (w + 1 < NW) bp[(size_t)(w + 1) * NL + threadIdx.x] = bk;   // not read if this window turns out to have no end
      } else {                                             // the keeper of the class's total
        const bool gap_w = !(bv < inf);
        s_gap = gap_w ? 1 : 0;
        kend[w] = gap_w ? -1 : bk;
        if (gap_w && !prev_gap) total += prev_end;         // the sequence before the gap is complete
        prev_end = bv;
        prev_gap = gap_w;
      }
    }
    lds_barrier();
    const bool gap = s_gap != 0;
    first = gap;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) cur[i] = nxt[i];
  }
  if (keeper) {
    if (!prev_gap) total += prev_end;
    a.path_cost[g] = total;
  }
  // make this block's predecessor records visible to its own later loads
  __threadfence();
  __syncthreads();

  // trace back, a run of windows at a time from the end; carry = candidate chosen in the window after the run
  int carry = -1;                                          // thread 0 only: -1 = the next window starts a sequence
  for (int hi = NW; hi > 0; hi -= kRun) {
    const int lo = hi > kRun ? hi - kRun : 0;
    // predecessor records of the windows lo+1 .. hi (row i = window lo+1+i; window NW does not exist)
    const int n_row = (hi < NW ? hi : NW - 1) - lo;
    for (int i = threadIdx.x; i < n_row * NL; i += kThreads)
      s_bp[i] = __hip_atomic_load(&bp[(size_t)(lo + 1) * NL + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int i = threadIdx.x; i < hi - lo; i += kThreads)
      s_sel[i] = __hip_atomic_load(&kend[lo + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = hi - 1; w >= lo; --w) {
        const int ke = s_sel[w - lo];
        int k;
        if (ke < 0) k = -1;                                // no feasible candidate in this window
        else if (carry < 0) k = ke;                        // last window of a sequence: its best end
        else k = s_bp[(w - lo) * NL + s_lay[carry]];       // predecessor of the next window's choice
        s_sel[w - lo] = k;
        carry = k;
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < hi - lo; i += kThreads) {
      const int k = s_sel[i];
      const size_t cell = (size_t)(lo + i) * G + g;
      a.sel[cell] = k;
      a.sel_energy[cell] = k >= 0 ? a.energy[cell * K + k] : inf;
    }
    __syncthreads();
  }
}


// ---- up to 64 layouts ----------------------------------------------------------------------------
// The step through the layouts needs, per window, only the least cost of every layout and the
// candidate that has it (adding a layout's arrival total to its candidates' costs keeps their
// order: rounded addition is monotone).  Those are independent of the recurrence:
// path_min_kernel takes them for all windows at once.  The recurrence itself only needs minima:
// path_chain_kernel walks the windows and keeps, per (window, layout), the least total of the
// sequences that end there.  Which source and candidate reach a minimum is not part
// of the recurrence; path_pred_kernel recomputes the same rounded sums from the stored totals for all
// windows in parallel and records the predecessors (least total, then lowest candidate), and
// the two path_trace kernels follow them back, all runs of windows at once.  Where sequences end, and the classes'
// totals, come out of those kernels too.  What the walk costs is the latency of one window's step, so the step holds nothing else.
// thread = (cell, layout): least cost among the layout's candidates, lowest candidate among equals
__global__ __launch_bounds__(256) void path_min_kernel(PathArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int NL = a.n_layout, K = a.K;
  if (i >= (int64_t)a.n_window * a.G * NL) return;
  const int64_t cell = i / NL;
  const int l = (int)(i - cell * NL);
  const int g = (int)(cell % a.G);
  const double* pw0_row = a.pw0 + (size_t)g * a.n_tp_f;
  const size_t row = (size_t)cell * K;
  double bv = __builtin_inf();
  int bk = 0x7FFFFFFF;
  const int p1 = a.seg_start[l + 1];
  for (int p = a.seg_start[l]; p < p1; ++p) {               // candidates of a layout ascend with the position
    const int k = a.order[p];
    const uint8_t fl = a.flags[row + k];
    double c = a.energy[row + k];
    if (a.idle_w != 0.0) {
      const DevCfg cf = a.cfg[k];
      const double pw0 = (cf.u != 0.0) ? (1.0 - cf.u) * pw0_row[cf.row_lo] + cf.u * pw0_row[cf.row_hi] : pw0_row[cf.row_lo];
      c = c + a.idle_w * ((cf.nd * pw0) * a.window_s);
    }
    if ((fl & DYN_F_FEASIBLE) && c < bv) { bv = c; bk = k; }
  }
  a.min_cost[i] = bv;
  a.min_k[i] = bk;
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {   // lane must be wave-uniform
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Lane Q of each row of 16 lanes, in all of the row's lanes.
template <int Q>
__device__ __forceinline__ double row_lane_f64(double v) {
  return __longlong_as_double(__builtin_amdgcn_update_dpp((long long)0, __double_as_longlong(v), 0x150 + Q, 0xF, 0xF, true));   // row_newbcast
}
// Smaller of two values that are not NaN, for a lane exchange right after it: the wait states that an exchange of a just
// written register needs are part of the block (the compiler would quiet both operands first).
__device__ __forceinline__ double min_then_swap(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2\n\ts_nop 1" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// Least value over the four rows of 16 lanes, position by position, in all rows.
__device__ __forceinline__ double rows_min_f64(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const auto l16 = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
  const auto h16 = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  const double m = min_then_swap(__longlong_as_double((long long)(((uint64_t)h16[0] << 32) | l16[0])),
                                 __longlong_as_double((long long)(((uint64_t)h16[1] << 32) | l16[1])));
  const uint64_t x = (uint64_t)__double_as_longlong(m);
  const auto l32 = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
  const auto h32 = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(x >> 32), false, false);
  return min_then_swap(__longlong_as_double((long long)(((uint64_t)h32[0] << 32) | l32[0])),
                       __longlong_as_double((long long)(((uint64_t)h32[1] << 32) | l32[1])));
}
// m[q] = (lane q of the row's v) + t[q], q = Q .. N - 1
template <int Q, int N>
__device__ __forceinline__ void add_sources(double v, const double (&t)[N], double (&m)[N]) {
  if constexpr (Q < N) {
    m[Q] = row_lane_f64<Q>(v) + t[Q];
    add_sources<Q + 1, N>(v, t, m);
  }
}

// The walk.  One block per class, a wave per 16 destination layouts; each of its four rows of 16 lanes takes a quarter of
// the source layouts (SPL = LMAX / 4), lane p of a row the destination p of the wave, with its SPL entries of the overhead
// table in registers.  Per window a lane reads one total of the window before from LDS (lane q of row r: source
// r * SPL + q), the row's totals reach all its lanes by DPP broadcasts, and the rows' partial minima meet by lane swaps.
// Row i holds the least costs of window i of a run of four, adds them when it is that window's turn and writes the new
// totals to the other LDS buffer: one block barrier per window and nothing else between the waves.  Costs are loaded
// three runs ahead, totals stored once per run, a window per row.
// Bound: the latency of one window's chain (LDS read, SPL broadcasts and additions, minima, LDS write, barrier), 1440
// times in a row on the one-day workload; nothing of the chip's rates applies.  Sources split over waves, their totals
// by lane reads and the partial minima through LDS atomics: 0.41 us a window; sources read from LDS by every lane
// (n_layout^2 values a window through the LDS port): 0.27 us; this, with 48 layouts: 0.22 us (596 to 323 us for the day).
// totals[window][layout] (which may be min_cost itself) takes the least total of the sequences that end there (+inf: none).
// Begins at window w0 (a multiple of 16) with s_v[0] set; after every 16 windows `more` says whether to go on, and the windows walked come back.
// s_dump: a word for every one of the THREADS threads; waves beyond the layouts only keep step.
struct WalkOn {                                              // to the last window
  __device__ __forceinline__ bool more(int) { return true; }
};
template <int LMAX, int THREADS, typename More>
__device__ __forceinline__ int walk_whole(const PathArgs& a, int g, int w0, double (*s_v)[LMAX], double* s_dump, More& more) {
  constexpr int SPL = LMAX / 4;                              // sources per row
  static_assert(LMAX % 16 == 0 && LMAX <= 64, "a row of 16 lanes broadcasts its sources");
  int lane = threadIdx.x & (DYN_WAVE - 1), NL = a.n_layout;
  asm volatile("" : "+v"(lane), "+s"(NL));                   // inside a caller's loop: its addresses are not worth registers outside of it
  lane &= DYN_WAVE - 1;
  const int r = lane >> 4, p = lane & 15, d = (int)(threadIdx.x / DYN_WAVE) * 16 + p;   // row, place in it, destination
  const int src = r * SPL + min(p, SPL - 1);                 // the source whose total this lane reads
  const int NW = a.n_window, G = a.G;
  const double inf = __builtin_inf();
  const bool on = d < NL;
  double t[SPL];                                             // overhead of going from the row's source q to this lane's destination
#pragma unroll
  for (int q = 0; q < SPL; ++q) {
    const int ls = r * SPL + q;
    const double over = a.transition[(size_t)min(ls, NL - 1) * NL + (on ? d : 0)];
    t[q] = on && ls < NL ? over : inf;                       // layouts beyond NL never win
  }
  const size_t step = (size_t)G * NL, mine = (size_t)g * NL + (on ? d : 0);   // this destination in window w: [w * step + mine]
  double* tot = a.totals + mine + (size_t)(w0 + r) * step;   // of this row's window
  const double *next = a.min_cost + mine + (size_t)(w0 + r) * step, *last = a.min_cost + mine + (size_t)(NW - 1) * step;
  int next_w = w0 + r;
  // loaded by every lane, from the last window beyond the end: behind a branch the waits would take in later loads too
  auto cost = [&]() {
    const double x = *(next_w < NW ? next : last);
    next += 4 * step;
    next_w += 4;
    return x;
  };
  constexpr int kRuns = 4;                                   // runs per loop pass: their costs sit in registers of their own, since
  double c[kRuns];                                           // handing a value on that is still being loaded would wait for it
#pragma unroll
  for (int u = 0; u + 1 < kRuns; ++u) c[u] = cost();
  double* put[4];                                            // where a lane writes in window i of a run: no branch in the walk
#pragma unroll
  for (int i = 0; i < 4; ++i) put[i] = r == i && (THREADS == LMAX * 4 || d < LMAX) ? &s_v[(i & 1) ^ 1][d] : &s_dump[threadIdx.x];
#pragma unroll 1
  for (; w0 < NW; w0 += 4 * kRuns) {
#pragma unroll
    for (int u = 0; u < kRuns; ++u) {
      const int w = w0 + 4 * u + r;                          // this row's window
      c[(u + kRuns - 1) % kRuns] = cost();
      const bool has = on && w < NW;
      const double cw = has ? c[u] : inf;
      double keep = inf;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double v = s_v[i & 1][src];
        const bool alive = __ballot((int)(__double_as_longlong(v) >> 32) < 0x7FF00000) != 0;   // any total below +inf (the wave holds all of them)
        double m[SPL];
        add_sources<0, SPL>(v, t, m);
#pragma unroll
        for (int k = 1; k < SPL; k *= 2)
#pragma unroll
          for (int q = 0; q + k < SPL; q += 2 * k) m[q] = __builtin_fmin(m[q], m[q + k]);   // sums are never NaN here
        const double arrive = rows_min_f64(m[0]);
        // least total of the sequences that end in this window in this destination (row i: its window)
        const double now = (!alive || !(cw < inf)) ? cw : arrive + cw;
        *put[i] = now;                                       // the other rows' lanes write to a place of their own that nobody reads
        keep = r == i ? now : keep;
        lds_barrier();                                       // the window's only block barrier
      }
      if (has) *tot = keep;
      tot += 4 * step;
    }
    if (!more.more(w0 + 4 * kRuns)) return min(w0 + 4 * kRuns, NW);   // block-uniform
  }
  return NW;
}
template <int LMAX>
__global__ __launch_bounds__(LMAX * 4) void path_chain_kernel(PathArgs a) {
  __shared__ double s_v[2][LMAX];                            // least totals of the window before, two buffers in turn
  __shared__ double s_dump[LMAX * 4];
  if (threadIdx.x < LMAX) s_v[0][threadIdx.x] = __builtin_inf();   // before the first window: as after a window without a feasible candidate
  __syncthreads();
  WalkOn on;
  walk_whole<LMAX, LMAX * 4>(a, (int)blockIdx.x, 0, s_v, s_dump, on);
}

// Many windows: the walk of a class in pieces.  What a sequence cost long ago moves all totals of a window alike, so which sources can be
// the cheapest is mostly known from a walk that starts a few windows before (path_near_kernel, a block for every piece of every class, the
// step of path_chain_kernel): those whose sum is within 2^-30 of the least, a bit each.  path_walk_kernel then takes the totals: of the
// named source only, so a step is a lane exchange and two additions.  Where a piece begins it knows whether the piece's walk began from the
// same totals but for a constant (`alike`).  If not (overheads so large that a choice of 16 windows ago still matters), and where many windows
// of the piece have several sources named (ties), it walks the piece as path_chain_kernel does: what is lost then is path_near_kernel's time.
// Totals are those of the whole walk to the last bit.  With costs >= 0 (a piece with others is never alike), m the least total that a piece
// starts from, D the constant and e = 100 * 2^-53 * (D + sum) the rounding of both walks in 50 windows, a source whose sum is more than 2^-30 of the
// least beyond it in the piece is beyond it by more than 2^-30 m - 2 * 2^-33 m - 2 e > 0 in the whole walk, as D <= 2^13 m.
// Bounds: the issue of NL^2 sums and comparisons a window (the pieces, 51 us for the day of 25 classes and 48 layouts), then the latency of a
// lane exchange and two additions, 0.096 us a window (138) in place of 0.225 (324).  Measured (us of dyn_select_path; the whole walk, this):
// the day 450, 271; with ten times its overheads 450, 277, fifty times 450, 364, five times (joining and re-sharding then cost the same, and
// a fifth of the windows have ties) 450, 480; 95 680 cells of 38 layouts and 1196 windows 543, 416; 517 windows of 64 layouts, most without
// requests, 204, 140; 320 of 51 148, 116, with many ties 148, 171.
constexpr int kWalkGroup = 8, kWalkRing = 3, kWalkAhead = 4;
constexpr int kWalkThreads = 256;
static_assert(DYN_PATH_PIECE % kWalkGroup == 0 && DYN_PATH_PIECE % 16 == 0, "pieces begin where groups and the whole walk's passes do");

// What path_near_kernel leaves of a piece, in the space of the predecessors: the totals it starts from, then for every piece and class
constexpr int kPieceEmpty = 1;                               // a window where a destination has no source (a sequence starts), or is beyond the last
constexpr int kPieceBelow = 2;                               // a cost below zero: never alike
constexpr int kPieceTie = 4;                                 // times the windows where a destination has several sources
constexpr int kTies = 4;                                     // so many are taken one by one, a microsecond each; a piece of more is walked as a whole, 7 us more
__device__ __forceinline__ double* piece_start(const PathArgs& a, int piece, int g) { return (double*)a.pred + ((size_t)piece * a.G + g) * a.n_layout; }
__device__ __forceinline__ int* piece_flags(const PathArgs& a, int piece, int g) {
  const int n_piece = (a.n_window + DYN_PATH_PIECE - 1) / DYN_PATH_PIECE;
  return (int*)piece_start(a, n_piece, 0) + (size_t)piece * a.G + g;
}
static_assert(((DYN_PATH_NEAR_LEAST + DYN_PATH_PIECE - 1) / DYN_PATH_PIECE) * (sizeof(double) + sizeof(int)) <= DYN_PATH_NEAR_LEAST * sizeof(int32_t), "they fit");

template <int LMAX>
__global__ __launch_bounds__(LMAX * 4) void path_near_kernel(PathArgs a) {
  constexpr int SPL = LMAX / 4, kBefore = DYN_PATH_BEFORE;
  static_assert(SPL <= 16, "a row's bits");
  static_assert(kBefore % 8 == 0 && DYN_PATH_PIECE % 8 == 0, "the passes below");
  __shared__ double s_v[2][LMAX];
  __shared__ int s_flag;
  const int NL = a.n_layout, NW = a.n_window, G = a.G, g = blockIdx.y;
  const double inf = __builtin_inf();
  if (threadIdx.x < LMAX) s_v[0][threadIdx.x] = inf;
  if (threadIdx.x == 0) s_flag = 0;
  __syncthreads();
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int r = lane >> 4, p = lane & 15, d = (int)(threadIdx.x / DYN_WAVE) * 16 + p;
  const int src = r * SPL + min(p, SPL - 1);
  const bool on = d < NL;
  double t[SPL];
#pragma unroll
  for (int q = 0; q < SPL; ++q) {
    const int ls = r * SPL + q;
    const double over = a.transition[(size_t)min(ls, NL - 1) * NL + (on ? d : 0)];
    t[q] = on && ls < NL ? over : inf;
  }
  const int piece = (int)blockIdx.x;
  const int w0 = piece * DYN_PATH_PIECE, w1 = min(NW, w0 + DYN_PATH_PIECE), wb = max(0, w0 - kBefore);
  const double* col = a.min_cost + (size_t)g * NL + (on ? d : 0);
  const size_t step = (size_t)G * NL;
  uint16_t* bits = (uint16_t*)(a.near + (size_t)g * NL + (on ? d : 0)) + r;   // of this row in window w: bits[w * step * 4]
  constexpr int kAhead = 8;                                  // costs in flight, in registers of their own
  double c[kAhead];
#pragma unroll
  for (int u = 0; u < kAhead; ++u) c[u] = col[(size_t)min(wb + u, NW - 1) * step];
  uint32_t signs = 0;                                        // the upper bit: a cost below zero
  uint32_t several = 0, empty = w1 < w0 + DYN_PATH_PIECE ? 1u : 0u;   // wave-uniform
  double start = inf;
#pragma unroll 1
  for (int wa = wb; wa < w1; wa += kAhead) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int w = wa + u;
      const double cw = on && w < NW ? c[u] : inf;
      signs |= (uint32_t)((uint64_t)__double_as_longlong(cw) >> 32);
      c[u] = col[(size_t)min(w + kAhead, NW - 1) * step];
      const double v = s_v[u & 1][src];
      const bool alive = __ballot((int)(__double_as_longlong(v) >> 32) < 0x7FF00000) != 0;
      double m[SPL], x[SPL];
      add_sources<0, SPL>(v, t, m);
#pragma unroll
      for (int q = 0; q < SPL; ++q) x[q] = m[q];
#pragma unroll
      for (int k = 1; k < SPL; k *= 2)
#pragma unroll
        for (int q = 0; q + k < SPL; q += 2 * k) x[q] = __builtin_fmin(x[q], x[q + k]);
      const double arrive = rows_min_f64(x[0]);
      const double now = (!alive || !(cw < inf)) ? cw : arrive + cw;
      if (r == 0) s_v[(u & 1) ^ 1][d] = now;
      if (wa >= w0 && w < w1) {                              // block-uniform
        const double near = arrive + __builtin_fabs(arrive) * 0x1p-30;
        uint32_t b = 0;
#pragma unroll
        for (int q = 0; q < SPL; ++q) b |= m[q] <= near ? 1u << q : 0u;
        if (!(arrive < inf)) b = alive ? (1u << SPL) - 1u : 0u;   // the sums overflow: all are asked for; or no sequence arrives
        if (on) bits[(size_t)w * step * 4] = (uint16_t)b;
        // of the wave's destinations (a bit each, the same in all rows): with several sources, and with none
        const uint64_t who = __ballot(b != 0), twice = __ballot((b & (b - 1)) != 0);
        const uint32_t lo = (uint32_t)who, hi = (uint32_t)(who >> 32), any = lo | hi, rows = (uint32_t)twice | (uint32_t)(twice >> 32) | (lo & hi);
        const uint32_t has = (uint32_t)__ballot(cw < inf) & 0xFFFFu;
        several += ((rows | (rows >> 16) | (any & (any >> 16))) & has) != 0 ? 1u : 0u;
        empty |= has & ~(any | (any >> 16));
      }
      if (u == kAhead - 1 && wa + kAhead == w0) start = now;
      lds_barrier();
    }
  }
  const int flags = (empty ? kPieceEmpty : 0) | (__ballot((signs >> 31) != 0) != 0 ? kPieceBelow : 0);
  if (lane == 0 && flags) atomicOr(&s_flag, flags);
  if (lane == 0 && several) atomicAdd(&s_flag, (int)several * kPieceTie);   // of all waves: a window may count more than once
  __syncthreads();
  if (r == 0 && on) piece_start(a, piece, g)[d] = start;
  if (threadIdx.x == 0) *piece_flags(a, piece, g) = s_flag;
}

// Source layout of a bit of `near`: a row's 16 bits hold the SPL sources of the row.
__device__ __forceinline__ int near_source(uint64_t bits, int SPL, int NL) {
  const int b = __builtin_ctzll(bits | (1ull << 63));
  return min((b >> 4) * SPL + (b & 15), NL - 1);
}
__device__ __forceinline__ double exchange_f64(double v, int lane4) {  // of the lane lane4 / 4, which must be active
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(lane4, (int)(uint32_t)u);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(lane4, (int)(uint32_t)(u >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  return __longlong_as_double((long long)(((uint64_t)(uint32_t)dpp_mov<CTRL>((int)(uint32_t)(u >> 32)) << 32) | (uint32_t)dpp_mov<CTRL>((int)(uint32_t)u)));
}
__device__ __forceinline__ double wave_min_f64(double v) {   // least of a full wave, in every lane
  v = __builtin_fmin(v, dpp_f64<0x121>(v));                  // row_ror 1, 2, 4, 8
  v = __builtin_fmin(v, dpp_f64<0x122>(v));
  v = __builtin_fmin(v, dpp_f64<0x124>(v));
  v = __builtin_fmin(v, dpp_f64<0x128>(v));
  return rows_min_f64(v);
}

// Whether a piece's walk started from the totals v but for a constant (a lane per layout, +inf on lanes beyond them; a full wave).
__device__ __forceinline__ bool alike(double v, double start) {
  const double inf = __builtin_inf();
  const bool has = v < inf;
  if (__ballot(has != (start < inf)) != 0) return false;     // a NaN start too
  const uint64_t who = __ballot(has);
  if (who == 0) return true;                                 // a new sequence starts with the piece
  const double least = wave_min_f64(has ? start : inf);
  const double by = has ? v - start : 0.0, first = readlane_f64(by, __builtin_ctzll(who));
  return __ballot(has && !(__builtin_fabs(by - first) <= least * 0x1p-33)) == 0 && __builtin_fabs(first) <= least * 0x1p13;
}

// Where a piece begins, the first wave says how it is walked: lane = layout, v = the totals of the window before.
struct PieceStart {
  const PathArgs& a;
  int g, next;                                               // the next piece to say it of
  int* s_how;                                                // [2], pieces in turn: all waves have read a word long before it is written again
  double start;
  int flags;
  static __device__ __forceinline__ int own_lane() {         // opaque: no addresses of these rare steps in registers during the walk
    int lane = threadIdx.x & (DYN_WAVE - 1);
    asm volatile("" : "+v"(lane));
    return lane;
  }
  __device__ __forceinline__ void fetch() {
    const int lane = own_lane();
    const bool in = next * DYN_PATH_PIECE < a.n_window;
    start = in && lane < a.n_layout ? piece_start(a, next, g)[lane] : __builtin_inf();
    flags = in ? *piece_flags(a, next, g) : 0;
  }
  // Where the sources are not right path_pred_kernel is told to look at all.
  __device__ __forceinline__ void say(double v) {
    const int lane = own_lane();
    const bool same = next == 0 || (alike(v, start) && (flags & kPieceBelow) == 0);
    if (!same && lane < DYN_PATH_PIECE && next * DYN_PATH_PIECE + lane < a.n_window)
      a.near[((size_t)(next * DYN_PATH_PIECE + lane) * a.G + g) * a.n_layout] = ~0ull;
    if (lane == 0) s_how[next & 1] = !same || flags >= (kTies + 1) * kPieceTie ? kWhole : flags >= kPieceTie ? kSeveral : flags != 0 ? kEmpty : kPlain;
    ++next;
    fetch();
  }
  __device__ __forceinline__ int how(int w) const { return __builtin_amdgcn_readfirstlane(s_how[(w / DYN_PATH_PIECE) & 1]); }   // of the piece of window w
  static constexpr int kPlain = 0, kEmpty = 1, kSeveral = 2, kWhole = 3;   // one source everywhere; or none; or in few windows several; all sums
};
static_assert(DYN_PATH_PIECE <= DYN_WAVE, "a lane marks a window");
template <int LMAX>
struct WalkWholePieces {                                     // until a piece that need not be walked as a whole
  PieceStart& at;
  double (*s_v)[LMAX];
  __device__ __forceinline__ bool more(int w) {
    if (w % DYN_PATH_PIECE != 0 || w >= at.a.n_window) return true;   // block-uniform
    if (threadIdx.x < DYN_WAVE) at.say(threadIdx.x < LMAX ? s_v[0][threadIdx.x] : __builtin_inf());
    lds_barrier();
    return at.how(w) == PieceStart::kWhole;
  }
};

// A block per class.  Of pieces with one source everywhere (or none) the first wave adds, lane = destination layout; the others fetch the costs,
// sources and overheads of the group of eight windows after the next, which need no totals: three groups in LDS, so that the block finds
// room beside another stream's kernel (20 KB with 48 layouts; 90 KB were held by rows of 64 lanes, the overhead table and the further sources).
template <int LMAX>
__global__ __launch_bounds__(kWalkThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void path_walk_kernel(PathArgs a) {
  constexpr int SPL = LMAX / 4, kHelpers = kWalkThreads / DYN_WAVE - 1, kEach = (kWalkGroup + kHelpers - 1) / kHelpers;
  constexpr int kRows = kWalkRing * kWalkGroup;
  constexpr uint32_t kNone = 255u;                           // others are four times the source, and one more where there are several
  __shared__ double2 s_c[kRows][LMAX];                       // cost, overhead from the source
  __shared__ uint8_t s_l[kRows][LMAX];
  __shared__ double s_v[2][LMAX];
  __shared__ int s_how[2];
  const int NL = a.n_layout, NW = a.n_window, G = a.G, g = blockIdx.x;
  double* s_dump = (double*)s_c;                             // the whole walk needs no rows
  static_assert(kRows * LMAX * sizeof(double2) >= kWalkThreads * sizeof(double), "a word for every thread");
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE);
  const double inf = __builtin_inf();
  const size_t step = (size_t)G * NL;
  const bool lay = lane < NL;
  PieceStart at{a, g, 0, s_how, inf, 0};
  double v = inf;                                            // of the first wave: before the first window as after one without a feasible candidate
  if (wave == 0) {
    at.fetch();
    at.say(v);
  }
  __syncthreads();

  int w = 0, n_whole = 0;
#pragma unroll 1
  while (w < NW) {
    int how = at.how(w);                                     // block-uniform
    if (how == PieceStart::kWhole) {
      if (wave == 0 && lane < LMAX) s_v[0][lane] = v;
      lds_barrier();
      WalkWholePieces<LMAX> more{at, s_v};
      const int from = w;
      w = walk_whole<LMAX, kWalkThreads>(a, g, w, s_v, s_dump, more);
      n_whole += w - from;
      if (wave == 0) v = lane < LMAX ? s_v[0][lane] : inf;
      continue;
    }
    int ld = lay ? lane : 0;
    asm volatile("" : "+v"(ld));                             // no addresses of this part in registers during the other one
    int buf = 0;
    auto after = [&]() {                                     // the group is done; false: the last one of this kind
      w += kWalkGroup;
      buf = buf + 1 == kWalkRing ? 0 : buf + 1;
      lds_barrier();
      if (w % DYN_PATH_PIECE == 0 && w < NW) how = at.how(w);
      return w < NW && how != PieceStart::kWhole;
    };
    // Both kinds of waves in loops of their own: registers of loads in flight would make the other kind wait.
    if (wave > 0) {                                          // a helper's windows of a group: wave - 1, + kHelpers, ...
      double c[kEach], over[kEach];
      uint64_t b[kEach];
      auto load = [&](int w) {
#pragma unroll
        for (int u = 0; u < kEach; ++u) {
          const size_t at_w = (size_t)min(w + wave - 1 + u * kHelpers, NW - 1) * step + (size_t)g * NL + ld;
          c[u] = a.min_cost[at_w];
          b[u] = a.near[at_w];
        }
      };
      auto look_up = [&](int w, int buf) {                   // of the windows loaded before
#pragma unroll
        for (int u = 0; u < kEach; ++u) {
          const int i = wave - 1 + u * kHelpers;
          const bool has = w + i < NW && c[u] < inf;
          const int l = near_source(b[u], SPL, NL);
          over[u] = a.transition[(size_t)l * NL + ld];
          if (i < kWalkGroup && lay) {
            s_c[buf * kWalkGroup + i][ld].x = has ? c[u] : inf;
            s_l[buf * kWalkGroup + i][ld] = (uint8_t)(b[u] == 0 ? kNone : 4u * (uint32_t)l + (has && (b[u] & (b[u] - 1)) != 0 ? 1u : 0u));
          }
        }
        __builtin_amdgcn_sched_barrier(0);                   // the next loads go to the same registers: nothing to hand on
      };
      auto put = [&](int buf) {                              // the overheads, which took a while
#pragma unroll
        for (int u = 0; u < kEach; ++u) {
          const int i = wave - 1 + u * kHelpers;
          if (i < kWalkGroup && lay) s_c[buf * kWalkGroup + i][ld].y = over[u];
        }
      };
      load(w); look_up(w, 0); put(0);
      load(w + kWalkGroup); look_up(w + kWalkGroup, 1); put(1);
      load(w + 2 * kWalkGroup);
      lds_barrier();
      do {
        const int b2 = buf + 2 < kWalkRing ? buf + 2 : buf + 2 - kWalkRing;   // nobody reads that buffer now
        look_up(w + 2 * kWalkGroup, b2);
        load(w + 3 * kWalkGroup);
        put(b2);
      } while (after());
    } else {                                                 // a lane's source is a layout
      double* tot_l = a.totals + (size_t)g * NL + ld;
      double2 rc[kWalkAhead];
      uint32_t rl[kWalkAhead];
      lds_barrier();
#pragma unroll
      for (int u = 0; u < kWalkAhead; ++u) { rc[u] = s_c[u][ld]; rl[u] = s_l[u][ld]; }
      do {
        const int b1 = buf + 1 == kWalkRing ? 0 : buf + 1;
        auto next = [&](int u) {                             // window u + kWalkAhead of this group, or of the next one
          const int row = u + kWalkAhead < kWalkGroup ? buf * kWalkGroup + u + kWalkAhead : b1 * kWalkGroup + u + kWalkAhead - kWalkGroup;
          rc[u % kWalkAhead] = s_c[row][ld];
          rl[u % kWalkAhead] = s_l[row][ld];
        };
        double* tot = tot_l + (size_t)w * step;
        if (how == PieceStart::kPlain) {                     // block-uniform
#pragma unroll
          for (int u = 0; u < kWalkGroup; ++u) {
            const int i = u % kWalkAhead;
            const double x = (exchange_f64(v, (int)rl[i]) + rc[i].y) + rc[i].x;
            v = lay ? x : inf;
            if (lay) *tot = v;
            tot += step;
            next(u);
          }
        } else if (how == PieceStart::kEmpty) {
#pragma unroll
          for (int u = 0; u < kWalkGroup; ++u) {
            const int i = u % kWalkAhead;
            const bool none = rl[i] == kNone;                // the first window of a sequence
            const double arrive = exchange_f64(v, none ? 0 : (int)rl[i]) + rc[i].y;
            v = lay ? (none ? rc[i].x : arrive + rc[i].x) : inf;
            if (lay && w + u < NW) *tot = v;
            tot += step;
            next(u);
          }
        } else {
#pragma unroll
          for (int u = 0; u < kWalkGroup; ++u) {
            const int i = u % kWalkAhead;
            const bool none = rl[i] == kNone, more = lay && (rl[i] & 3u) == 1u;
            double arrive = exchange_f64(v, none ? 0 : (int)(rl[i] & ~3u)) + rc[i].y;
            if (__ballot(more) != 0) {                       // wave-uniform
              const uint64_t b = a.near[(size_t)(w + u) * step + (size_t)g * NL + ld];
              for (uint64_t rest = more ? b & (b - 1) : 0ull; __ballot(rest != 0) != 0; rest &= rest - 1) {
                const int q = near_source(rest, SPL, NL);
                const double x = exchange_f64(v, 4 * q) + a.transition[(size_t)q * NL + ld];
                if (rest != 0) arrive = __builtin_fmin(arrive, x);
              }
            }
            v = lay ? (none ? rc[i].x : arrive + rc[i].x) : inf;
            if (lay && w + u < NW) *tot = v;
            tot += step;
            next(u);
          }
        }
        if ((w + kWalkGroup) % DYN_PATH_PIECE == 0 && w + kWalkGroup < NW) at.say(v);
      } while (after());
    }
  }
  if (threadIdx.x == 0) a.whole[g] = (uint32_t)n_whole;
}

// One wave per (window, class), lane = destination layout: where
// the cheapest arrival in every layout of the next window comes from (least total + overhead, then the lowest
// candidate among the sources that reach it), as (candidate << 6) | its layout, -1: none; and the best end and the total
// of a sequence that ends in this window.  The sums are those of the walk, from the same operands.
// NEAR: of the named sources only, which hold every source that reaches the least sum; of all where more than four are named (also
// where path_walk_kernel found that they are not right).
template <int LMAX, bool NEAR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(LMAX <= 32 ? 4 : 3, 8))) void path_pred_kernel(PathArgs a) {
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int NL = a.n_layout, NW = a.n_window, G = a.G;
  const double inf = __builtin_inf();
  const bool on = lane < NL;
  const int ld = on ? lane : 0;
  double t[NEAR ? 1 : LMAX];                                 // the lane's column of the table
  if constexpr (!NEAR) {
#pragma unroll
    for (int l = 0; l < LMAX; ++l) t[l] = (on && l < NL) ? a.transition[(size_t)l * NL + lane] : inf;
  }
  const int64_t cells = (int64_t)NW * G;
  const int64_t n_wave = (int64_t)gridDim.x * (blockDim.x / DYN_WAVE);
  for (int64_t cell = (int64_t)blockIdx.x * (blockDim.x / DYN_WAVE) + threadIdx.x / DYN_WAVE; cell < cells; cell += n_wave) {
    const int w = (int)(cell / G), g = (int)(cell % G);
    const double v = on ? a.totals[(size_t)cell * NL + lane] : inf;
    const int k = on ? a.min_k[(size_t)cell * NL + lane] : 0;
    const uint32_t pk = (v < inf) ? (((uint32_t)k << 6) | (uint32_t)lane) : 0xFFFFFFFFu;
    const double nv = (on && w + 1 < NW) ? a.totals[((size_t)cell + G) * NL + lane] : inf;
    uint64_t named = (NEAR && on && w + 1 < NW) ? a.near[((size_t)cell + G) * NL + lane] : 0ull;
    const bool gap = __ballot(v < inf) == 0;                 // no feasible candidate in this window
    const bool ends = !gap && __ballot(nv < inf) == 0;       // the next window has none, or does not exist
    double ev = inf;
    uint32_t ep = gap ? 0xFFFFFFFFu : 0u;
    if (ends) {                                              // wave-uniform
      ev = v;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) ev = fmin(ev, __shfl_xor(ev, d, DYN_WAVE));
      ep = (v == ev) ? pk : 0xFFFFFFFFu;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) ep = min(ep, (uint32_t)__shfl_xor((int)ep, d, DYN_WAVE));
    }
    if (lane == 0) {
      a.kend[(size_t)g * NW + w] = (int32_t)ep;              // -1 gap, the best end where a sequence ends, 0 otherwise
      a.end_total[(size_t)g * NW + w] = ev;                  // +inf where none ends
    }
    if (w + 1 >= NW) continue;
    double m = inf;
    uint32_t p = 0xFFFFFFFFu;                                // all ones: nothing arrives (then m is +inf)
    if (NEAR && __ballot(__popcll(named) > 4) == 0) {        // wave-uniform
      if (__ballot((named & (named - 1)) != 0) == 0) {
        const uint32_t sp = (uint32_t)__builtin_amdgcn_ds_bpermute(near_source(named, LMAX / 4, NL) * 4, (int)pk);
        if (named != 0) p = sp;
      } else {
        while (__ballot(named != 0) != 0) {
          const int q = near_source(named, LMAX / 4, NL);
          const double arr = exchange_f64(v, 4 * q) + a.transition[(size_t)q * NL + ld];
          const uint32_t sp = (uint32_t)__builtin_amdgcn_ds_bpermute(q * 4, (int)pk);
          const bool better = named != 0 && (arr < m || (arr == m && sp < p));
          m = better ? arr : m;
          p = better ? sp : p;
          named &= named - 1;
        }
      }
    } else if constexpr (NEAR) {                             // rare: the column stays in the cache
#pragma unroll 1
      for (int l0 = 0; l0 < LMAX; l0 += 8) {                 // lanes beyond the layouts hold +inf
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = a.transition[(size_t)min(l0 + u, NL - 1) * NL + ld];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const double arr = readlane_f64(v, l0 + u) + x[u];
          const uint32_t sp = (uint32_t)__builtin_amdgcn_readlane((int)pk, l0 + u);
          const bool better = arr < m || (arr == m && sp < p);
          m = better ? arr : m;
          p = better ? sp : p;
        }
      }
    } else {
#pragma unroll
      for (int l = 0; l < LMAX; ++l) {
        const double arr = readlane_f64(v, l) + t[l];
        const uint32_t sp = (uint32_t)__builtin_amdgcn_readlane((int)pk, l);
        const bool better = arr < m || (arr == m && sp < p);
        m = better ? arr : m;
        p = better ? sp : p;
      }
    }
    if (on) a.pred[((size_t)g * NW + w + 1) * NL + lane] = (int32_t)p;
  }
}

// Trace-back.  A window's choice depends on the next window's only through a small state: the layout chosen there,
// or "none" (the next window has no feasible candidate, starts a sequence, or does not exist).  Runs of
// DYN_PATH_RUN windows are therefore followed back for every possible entry state at once (one thread per state;
// path_trace_runs_kernel records the state each run is left with), a block then finds the state its run is really
// entered with by chaining those records from the last run down to its own, follows its run once more from that
// state and writes the selection (path_trace_write_kernel).  Both kernels stage a run's records in LDS.
__device__ __forceinline__ int trace_step(int ke, int state, const int32_t* s_bp, int i, int NL) {
  // record of window i of the run: -1 none, else (candidate << 6) | layout
  if (ke < 0) return -1;                                     // no feasible candidate in this window
  if (state == DYN_PATH_STATES - 1) return ke;               // last window of a sequence: its best end
  return s_bp[i * NL + state];                               // predecessor of the next window's choice
}

__device__ __forceinline__ void trace_stage(const PathArgs& a, int g, int lo, int hi, int32_t* s_bp, int32_t* s_ke) {
  const int NL = a.n_layout, NW = a.n_window;
  const int32_t* bp = a.pred + (size_t)g * NW * NL;          // [NW][NL]: where the cheapest arrival in layout l at window w comes from
  const int32_t* kend = a.kend + (size_t)g * NW;             // [NW]: -1 gap, best end where a sequence ends, 0 otherwise
  const int n_row = (hi < NW ? hi : NW - 1) - lo;            // predecessor records of the windows lo+1 .. hi
  constexpr int U = 16;                                      // records in flight per thread: a load at a time took 12 us of a run's 25
  const int32_t* from = bp + (size_t)(lo + 1) * NL;
  for (int i0 = threadIdx.x; i0 < n_row * NL; i0 += U * (int)blockDim.x) {
    int32_t x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = from[min(i0 + u * (int)blockDim.x, n_row * NL - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * (int)blockDim.x < n_row * NL) s_bp[i0 + u * (int)blockDim.x] = x[u];
  }
  for (int i = n_row * NL + threadIdx.x; i < (hi - lo) * NL; i += blockDim.x) s_bp[i] = -1;   // nothing follows the last window
  for (int i = threadIdx.x; i < hi - lo; i += blockDim.x) s_ke[i] = kend[lo + i];
  __syncthreads();
}

// A class's total: its sequences' totals added in time order (one wave; the loads of a chunk of windows are in flight together: a day is one round).
__device__ __forceinline__ void class_total(const PathArgs& a, int g) {
  const int NW = a.n_window, lane = threadIdx.x;
  const double inf = __builtin_inf();
  const double* end_total = a.end_total + (size_t)g * NW;
  constexpr int kAhead = 24;
  double total = 0.0;
  for (int w0 = 0; w0 < NW; w0 += kAhead * DYN_WAVE) {
    double v[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int w = w0 + j * DYN_WAVE + lane;
      v[j] = w < NW ? end_total[w] : inf;
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
      for (uint64_t at = __ballot(v[j] < inf); at != 0; at &= at - 1) total += readlane_f64(v[j], __builtin_ctzll(at));
  }
  if (lane == 0) a.path_cost[g] = total;
}

// grid (runs + 1, classes), 128 threads: thread s < DYN_PATH_STATES follows the run back from entry state s; the blocks
// beyond the runs add up the classes' totals.
__global__ __launch_bounds__(128) void path_trace_runs_kernel(PathArgs a) {
  __shared__ int32_t s_bp[DYN_PATH_RUN * DYN_WAVE];
  __shared__ int32_t s_ke[DYN_PATH_RUN];
  const int r = blockIdx.x, g = blockIdx.y, n_run = gridDim.x - 1;
  if (r == n_run) {                                          // block-uniform
    if (threadIdx.x < DYN_WAVE) class_total(a, g);
    return;
  }
  const int lo = r * DYN_PATH_RUN, hi = min(a.n_window, lo + DYN_PATH_RUN);
  trace_stage(a, g, lo, hi, s_bp, s_ke);
  int state = threadIdx.x;
  if (state >= DYN_PATH_STATES) return;
  if (state < DYN_PATH_STATES - 1 && state >= a.n_layout) state = DYN_PATH_STATES - 1;   // not a layout: never entered with
  for (int i = hi - lo - 1; i >= 0; --i) {
    const int rec = trace_step(s_ke[i], state, s_bp, i, a.n_layout);
    state = rec < 0 ? DYN_PATH_STATES - 1 : (rec & 63);
  }
  a.exits[((size_t)g * n_run + r) * DYN_PATH_STATES + threadIdx.x] = state;
}

// grid (runs, classes), 64 threads.
__global__ __launch_bounds__(DYN_WAVE) void path_trace_write_kernel(PathArgs a) {
  __shared__ int32_t s_bp[DYN_PATH_RUN * DYN_WAVE];
  __shared__ int32_t s_ke[DYN_PATH_RUN];
  __shared__ int32_t s_sel[DYN_PATH_RUN];
  const int r = blockIdx.x, g = blockIdx.y, n_run = gridDim.x;
  const int G = a.G, K = a.K;
  const int lo = r * DYN_PATH_RUN, hi = min(a.n_window, lo + DYN_PATH_RUN);
  trace_stage(a, g, lo, hi, s_bp, s_ke);
  // the state this run is entered with: the later runs' records chained from the end.  The records of kHop runs
  // are fetched together (lane s holds the record for entry state s), so a hop is a lane read, not a load.
  constexpr int kHop = 16;
  int state = DYN_PATH_STATES - 1;                           // nothing follows the last window; wave-uniform
  for (int top = n_run - 1; top > r; top -= kHop) {
    int by_layout[kHop], by_none[kHop];
#pragma unroll
    for (int j = 0; j < kHop; ++j) {
      const int q = max(top - j, r + 1);                     // runs at or below r are not used
      const int32_t* row = a.exits + ((size_t)g * n_run + q) * DYN_PATH_STATES;
      by_layout[j] = row[threadIdx.x];
      by_none[j] = row[DYN_PATH_STATES - 1];
    }
#pragma unroll
    for (int j = 0; j < kHop; ++j)
      if (top - j > r)
        state = state == DYN_PATH_STATES - 1 ? by_none[j] : __builtin_amdgcn_readlane(by_layout[j], __builtin_amdgcn_readfirstlane(state));
  }
  if (threadIdx.x == 0) {
    for (int i = hi - lo - 1; i >= 0; --i) {
      const int rec = trace_step(s_ke[i], state, s_bp, i, a.n_layout);
      state = rec < 0 ? DYN_PATH_STATES - 1 : (rec & 63);
      s_sel[i] = rec < 0 ? -1 : (rec >> 6);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < hi - lo; i += blockDim.x) {
    const int k = s_sel[i];
    const size_t cell = (size_t)(lo + i) * G + g;
    a.sel[cell] = k;
    a.sel_energy[cell] = k >= 0 ? a.energy[cell * K + k] : __builtin_inf();
  }
}

template <int LMAX>
void launch_layout_route(const PathArgs& a, hipStream_t s) {
  const int64_t cells = (int64_t)a.n_window * a.G;
  const int64_t n = cells * a.n_layout;
  hipLaunchKernelGGL(path_min_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  const dim3 pred((unsigned)std::min<int64_t>((cells + 3) / 4, 2048));
  if (a.near) {
    hipLaunchKernelGGL(path_near_kernel<LMAX>, dim3((unsigned)((a.n_window + DYN_PATH_PIECE - 1) / DYN_PATH_PIECE), (unsigned)a.G), dim3(LMAX * 4), 0, s, a);
    hipLaunchKernelGGL(path_walk_kernel<LMAX>, dim3((unsigned)a.G), dim3(kWalkThreads), 0, s, a);
    hipLaunchKernelGGL((path_pred_kernel<LMAX, true>), pred, dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL(path_chain_kernel<LMAX>, dim3((unsigned)a.G), dim3(LMAX * 4), 0, s, a);
    hipLaunchKernelGGL((path_pred_kernel<LMAX, false>), pred, dim3(256), 0, s, a);
  }
  const dim3 runs((unsigned)dyn_path_runs(a.n_window), (unsigned)a.G);
  hipLaunchKernelGGL(path_trace_runs_kernel, dim3(runs.x + 1, runs.y), dim3(128), 0, s, a);
  hipLaunchKernelGGL(path_trace_write_kernel, runs, dim3(DYN_WAVE), 0, s, a);
}

}  // namespace

size_t dyn_path_lds(int32_t K, int32_t n_layout) {
  return ((size_t)K + ((size_t)n_layout + 1) * n_layout + (2 + kParts) * ((size_t)n_layout + 1)) * sizeof(double) +
         ((size_t)(2 + kParts) * (n_layout + 1) + (size_t)kRun * n_layout + kRun) * sizeof(int32_t) +
         2 * (size_t)K * sizeof(uint16_t) + 16;
}

bool dyn_path_fits(int32_t K, int32_t n_layout) {
  if (K < 1 || n_layout < 1) return false;
  if (n_layout <= DYN_WAVE) return K <= (1 << 24);           // wave-per-class route: candidates are packed into 24 bits
  return K <= DYN_PATH_MAX_CONFIGS && n_layout < kThreads && dyn_path_lds(K, n_layout) <= DYN_LDS_BUDGET;
}

hipError_t dyn_launch_path(const PathArgs& a, hipStream_t s) {
  if (!dyn_path_fits(a.K, a.n_layout)) return hipErrorInvalidValue;
  DynTimed timed(DYN_K_PATH, s);
  if (a.n_layout <= DYN_WAVE) {
    if (a.n_layout <= 16) launch_layout_route<16>(a, s);
    else if (a.n_layout <= 32) launch_layout_route<32>(a, s);
    else if (a.n_layout <= 48) launch_layout_route<48>(a, s);
    else launch_layout_route<64>(a, s);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(path_kernel, dim3((unsigned)a.G), dim3(kThreads), dyn_path_lds(a.K, a.n_layout), s, a);
  return hipGetLastError();
}
