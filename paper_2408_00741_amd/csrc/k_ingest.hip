// Trace ingestion: every request goes to its cell (window from the timestamp,
// class from the input/output length bins of Table IV's convention): (input tokens, output tokens)
// in cell order, stably, and the cell offsets.  In general that is a least-significant-digit radix sort.
//
// A trace that is already in window order (a request log is in time order) does not need the
// general sort: the order kernel notices it (a word in the workspace header stays 0; it also
// writes where every window starts), and one block per window then moves its requests, stably,
// to their cells (window_sort_kernel).  So does a trace of a few such runs, while no window of it is too long.  Any other
// trace takes the radix sort.  The host does not read the word: all routes are enqueued and the kernels of a
// route not taken return at their first instruction.  Runs, the long windows that window_sort_kernel leaves and the general sort
// are one launch: a route that is not taken costs one empty launch (4 to 5 us), of unordered_kernel or of window_sort_kernel.
#include <string.h>

#include <algorithm>
#include <atomic>

#include "dyn_internal.h"
#include "dyn_device.h"

namespace {

// Window of a timestamp: floor(t / window_s), the quotient formed from RN(1 / window_s) by div_by (correctly rounded
// for timestamps whose quotient is a normal number; a handful of multiply-adds instead of a division).  Quotients that are
// not finite, and tiny ones (below 2^-900, where a residual could underflow), take the IEEE division; clamped, out-of-range flagged.
__device__ __forceinline__ double window_of(double t, double window_s, double r_window, int32_t n_window, uint32_t* bad) {
  double q = div_by(t, window_s, r_window);
  if (!(fabs(q) >= 0x1p-900 && fabs(q) <= 0x1p900)) q = t / window_s;   // also NaN: a residual step on an infinite product
  double wq = floor(q);
  if (!(wq >= 0.0)) { *bad = DYN_WS_BAD_REQUEST; wq = 0.0; }                      // negative or NaN
  if (!(wq < (double)n_window)) { *bad = DYN_WS_BAD_REQUEST; wq = (double)(n_window - 1); }
  return wq;
}

// The classes' edges in LDS where they fit (`room` ints), else where they are.  A barrier is due before they are read.
struct ClassEdges { const int32_t* in; const int32_t* out; };
__device__ __forceinline__ ClassEdges stage_edges(const IngestArgs& a, int32_t* lds, int room) {
  const int n_in = a.n_model * (a.n_in_bin - 1), n_out = a.n_model * (a.n_out_bin - 1);
  if (n_in + n_out > room) return {a.d_in_edge, a.d_out_edge};
  for (int q = threadIdx.x; q < n_in; q += blockDim.x) lds[q] = a.d_in_edge[q];
  for (int q = threadIdx.x; q < n_out; q += blockDim.x) lds[n_in + q] = a.d_out_edge[q];
  return {lds, lds + n_in};
}

// Classes of N requests (input and output tokens, model; a bad model index is clamped and flagged).  One model: an edge is
// read once for all of them.
template <int N>
__device__ __forceinline__ void classes_of(const IngestArgs& a, const ClassEdges& e, const int32_t* x, const int32_t* y, const int32_t* mdl, uint32_t* cls, uint32_t* bad) {
  const int n_ie = a.n_in_bin - 1, n_oe = a.n_out_bin - 1;
  int m[N], bi[N], bo[N];
#pragma unroll
  for (int r = 0; r < N; ++r) {
    m[r] = 0; bi[r] = 0; bo[r] = 0;
    if (a.model) {
      m[r] = mdl[r];
      if (m[r] < 0 || m[r] >= a.n_model) { *bad = DYN_WS_BAD_REQUEST; m[r] = 0; }
    }
  }
  if (a.model) {
    for (int q = 0; q < n_ie; ++q) {
#pragma unroll
      for (int r = 0; r < N; ++r) bi[r] += x[r] >= e.in[m[r] * n_ie + q] ? 1 : 0;
    }
    for (int q = 0; q < n_oe; ++q) {
#pragma unroll
      for (int r = 0; r < N; ++r) bo[r] += y[r] >= e.out[m[r] * n_oe + q] ? 1 : 0;
    }
  } else {
    for (int q = 0; q < n_ie; ++q) {
      const int32_t edge = e.in[q];
#pragma unroll
      for (int r = 0; r < N; ++r) bi[r] += x[r] >= edge ? 1 : 0;
    }
    for (int q = 0; q < n_oe; ++q) {
      const int32_t edge = e.out[q];
#pragma unroll
      for (int r = 0; r < N; ++r) bo[r] += y[r] >= edge ? 1 : 0;
    }
  }
#pragma unroll
  for (int r = 0; r < N; ++r) cls[r] = (uint32_t)((m[r] * a.n_in_bin + bi[r]) * a.n_out_bin + bo[r]);
}

// dst[from .. to) = value, a run of every lane (empty: from >= to): the lane writes a few, its wave the others.  All lanes call it.
__device__ __forceinline__ void fill_runs(int64_t* dst, uint32_t from, uint32_t to, int64_t value) {
  constexpr int kOwn = 16;
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  if (from < to) dst[from++] = value;              // as a rule the only one
  if (__ballot(from < to) == 0) return;
#pragma unroll 1
  for (int q = 1; q < kOwn && from < to; ++q) dst[from++] = value;
#pragma unroll 1
  for (uint64_t more = __ballot(from < to); more != 0; more &= more - 1) {
    const int who = __builtin_ctzll(more);
    const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)to, who);
    const int64_t v = readlane_i64(value, who);
    for (uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)from, who) + lane; at < end; at += DYN_WAVE) dst[at] = v;
  }
}

// Is the trace in window order, and where does every window start?  Only the timestamps are read (8 bytes a request): the
// routes compute classes from the tokens that they move anyway.  A wave takes kOrderRows rows of 64 consecutive
// requests, all loads in flight together.  Windows without requests are filled by whole waves (a thread per request with 2000
// of them before the log's first one took 50 us).
// A log's requests can also lie in a few windows of its grid.  A window is one block's work on both window routes, so a log
// with a window that alone takes longer than the sort of all is sorted (a.many).  One wave in 16 counts for
// this: one sample of its window if all its requests lie in one.  Neighbouring windows have counters of their own, and a mean
// window that long never comes here (dyn_ingest_always_sorts), so windows that share one matter little.
constexpr int kOrderRows = 8;
constexpr int kSampleStep = 4 * kOrderRows * DYN_WAVE;   // requests a sample stands for: those of a block, of a large log those of four
__global__ __launch_bounds__(256) void order_kernel(IngestArgs a, double r_window, uint32_t sparse) {
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  if (a.n_req == 0) {
    for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w <= a.n_window; w += (int64_t)gridDim.x * blockDim.x) a.win_off[w] = 0;
    return;
  }
  const int64_t base = ((int64_t)blockIdx.x * blockDim.x + (threadIdx.x - lane)) * kOrderRows;   // the wave's first request
  if (base >= a.n_req) return;
  double t[kOrderRows];
#pragma unroll
  for (int r = 0; r < kOrderRows; ++r) t[r] = a.t_s[std::min<int64_t>(base + r * DYN_WAVE + lane, a.n_req - 1)];
  uint32_t bad = 0, ignore = 0;
  // the window of the request before the wave's first
  double left = base > 0 ? window_of(a.t_s[base - 1], a.window_s, r_window, a.n_window, &ignore) : -1.0;
  double first = 0.0;                              // the wave's first window, in its first lane
#pragma unroll
  for (int r = 0; r < kOrderRows; ++r) {
    const int64_t i = base + r * DYN_WAVE + lane;
    const bool in = i < a.n_req;                       // past the end: the last request again
    const double wq = window_of(t[r], a.window_s, r_window, a.n_window, &bad);
    // Window order: compare with the request before.  Where the window changes the boundaries are written: in a trace in
    // window order win_off[w] = number of requests in windows before w (the values are not used otherwise).
    if (r == 0) first = wq;
    double wp = __shfl_up(wq, 1, DYN_WAVE);
    if (lane == 0) wp = left;
    left = __shfl(wq, DYN_WAVE - 1, DYN_WAVE);
    // The boundaries only matter to the window route: a wave that sees a request out of order, or finds the flag
    // raised already, writes none (on a shuffled trace every request would otherwise fill hundreds of them).
    const bool back = in && wp > wq;
    if (__ballot(in && (wp != wq || i == a.n_req - 1)) == 0) continue;
    const uint64_t any = __ballot(back);
    if (any != 0) {                                    // a request out of order: a run starts here
      if (__hip_atomic_load(a.unsorted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= DYN_WS_MAX_BREAKS) {
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(a.unsorted, (uint32_t)__popcll(any));
        at = __shfl(at, 0, DYN_WAVE) + (uint32_t)__popcll(any & ((1ull << lane) - 1ull));
        if (back && at < DYN_WS_MAX_BREAKS) a.unsorted[DYN_WS_HEADER_BREAK_WORD - DYN_WS_HEADER_ORDER_WORD + at] = (uint32_t)i;
      }
      continue;
    }
    if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(a.unsorted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0u) {
      fill_runs(a.win_off, (uint32_t)((int)wp + 1), in ? (uint32_t)((int)wq + 1) : 0u, i);
      if (__ballot(i == a.n_req - 1) != 0) fill_runs(a.win_off, (uint32_t)((int)wq + 1), i == a.n_req - 1 ? (uint32_t)a.n_window + 1u : 0u, a.n_req);
    }
  }
  if (a.many != 0 && (blockIdx.x & sparse) == 0 && threadIdx.x == 0 && base + kOrderRows * DYN_WAVE <= a.n_req && first == left)
    if (atomicAdd(&a.block_hist[(uint32_t)first % DYN_INGEST_COUNTERS], 1u) + 1u == a.many) atomicAdd(a.unsorted, DYN_WS_MAX_BREAKS + 1u);
  if (bad) atomicOr(a.status, bad);
}

// The route is chosen on the device: the kernels of all routes are launched and those of a route that is not taken return
// at once.  The order word is the number of requests whose window is before that of the request before them, as the order
// kernel left it (counted no further than past DYN_WS_MAX_BREAKS):
//   0      the trace is moved window by window;
//   a few  it is a few runs, each in window order (the logs of several front ends, one after the other): moved window by
//          window too, a window being a piece of every run, which its block finds by bisection;
//   more   the general sort.
// Where the line lies: a window of runs costs its block 8 us and 0.3 us a run (finding the pieces, the barriers of a tile)
// and 4 us a million requests, the sort 50 us and 30 us a million (two passes).  Measured (us by runs, sorted): 6 M requests in
// 1440 windows and 6 runs 89, 252; 1 M in 1000 and 6: 44, 78; 50 000 in 100 and 6: 13, 50; 9 M in 6000 and 6: 243, 371;
// 9 M in 2016 and 48: 228, 344; 300 000 in 2016 and 40: 171, 63; 9 M in 20 000 and 9: 836, 414.
enum Route { kByWindow, kByRuns, kSort };
__device__ __forceinline__ Route route_of(const IngestArgs& a) {
  const uint32_t breaks = *a.unsorted;
  if (breaks == 0) return kByWindow;
  if (breaks > DYN_WS_MAX_BREAKS) return kSort;
  const int64_t rounds = (a.n_window + (int64_t)gridDim.x - 1) / gridDim.x;   // of the unordered kernel (the other only asks for kByWindow)
  return rounds * (80 + 3 * (int64_t)breaks) < 500 + a.n_req * 26 / 100000 ? kByRuns : kSort;
}

// Class edges from the kernel's arguments into the workspace (a few hundred values at most per launch): the host
// arrays are free when the call returns and nothing waits for the stream.  The first launch also writes the
// workspace header: status 0, the order word (past DYN_WS_MAX_BREAKS when the general sort is forced).
struct EdgePack { int32_t v[DYN_EDGE_PACK]; };
__global__ void edge_store_kernel(EdgePack p, int n_a, int32_t* __restrict__ dst_a, int n_b, int32_t* __restrict__ dst_b,
                                  WsHeader* header, uint32_t order_word, uint32_t* counters) {
  for (int i = threadIdx.x; i < n_a; i += blockDim.x) dst_a[i] = p.v[i];
  for (int i = threadIdx.x; i < n_b; i += blockDim.x) dst_b[i] = p.v[n_a + i];
  if (header && threadIdx.x == 0) {
    header->status = 0u;
    header->kind = DYN_WS_KIND_WORD;
    header->cells = 0;
    ((uint32_t*)header)[DYN_WS_HEADER_ORDER_WORD] = order_word;
    for (int q = 0; q < 3; ++q) ((uint32_t*)header)[DYN_WS_HEADER_BARRIER_WORD + q] = 0u;
    ((uint32_t*)header)[DYN_WS_HEADER_LEFT_WORD] = 0u;
  }
  if (header && counters)
    for (int q = threadIdx.x; q < DYN_INGEST_COUNTERS; q += blockDim.x) counters[q] = 0u;
}

// exclusive sum over the block's threads; `wave_sum`: a word of LDS per wave
template <int WAVES>
__device__ __forceinline__ uint32_t block_exclusive_sum(uint32_t v, uint32_t* wave_sum) {
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = threadIdx.x / DYN_WAVE;
  uint32_t incl = v;
#pragma unroll
  for (int k = 1; k < DYN_WAVE; k <<= 1) {
    const uint32_t up = __shfl_up(incl, k, DYN_WAVE);
    if (lane >= k) incl += up;
  }
  if (WAVES == 1) return incl - v;
  if (lane == DYN_WAVE - 1) wave_sum[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) before += w < wave ? wave_sum[w] : 0u;
  __syncthreads();
  return before + incl - v;
}

// ---- the general sort ----------------------------------------------------------------------
// All radix passes and the offsets in one launch, with barriers between the phases that all its blocks pass: a trace in
// window order costs this one launch, which returns at its first instruction.  Every block owns a contiguous run of tiles.  A
// pass is: digit counts of every block's run -> barrier -> one wave per digit turns the blocks' counts into
// inclusive sums -> barrier -> every block moves its run, a tile at a time -> barrier.
//
// What bounds it: bytes through the last-level cache (a request is read and written once a pass, its key once more)
// and the barriers.  Measured at 6 M requests and 51 840 cells (two passes of 8 bits):
// - A cache write-back or invalidation is done once per block, by the thread that waits, not by every wave of it: an acquiring
//   fence by all 8 waves of 256 blocks costs 17 us a barrier, by one wave 2.  Data for other blocks is stored
//   through the L2 (put), so the write-back finds it clean; scattered runs cost the same either way.
// - A tile is ordered by digit in LDS before it is written, so that a digit's requests leave as one run: 8 M single words
//   scattered cost 93 us, runs of 16 words 13 us, of 32 words 9.5 us.  So the tile of the large
//   blocks is 8192 requests: 32 to a digit.
// - All loads of a thread's eight requests are in flight together, also where only keys are counted or compared.
// 523 us with separate scan phases, all waves fencing and single words scattered; 225 us so.
//
// The barrier: an arrival counter in the workspace header, zeroed with the header; barrier number k is passed when
// the counter reaches k * blocks.  The block that arrives last says so in a word of its own, which the others watch: watching the
// counter they held up the arrivals (six million requests 335 us, 280 so).  Only blocks that run take part (join_team), so other work on the device can
// delay a barrier but not stop it; if it takes seconds all the same, the wait is given up (every block leaves,
// DYN_WS_SORT_ABANDONED is raised).
struct RadixArgs {
  IngestArgs t;
  double r_window;
  uint32_t* barrier; uint32_t* join; uint32_t* members; uint32_t* passed;
  int64_t cells;
  int32_t passes, bits;
  int32_t blocks;                                // that sort (the grid may have more, for the runs)
};

constexpr uint32_t kBarrierSpins = 1u << 22;     // x about a microsecond per look: seconds
// The blocks that sort together: those that run when the first one has waited for them.
struct RadixTeam { int blocks, block; };
constexpr uint32_t kTeamClosed = 1u << 31;
constexpr uint32_t kTeamSpins = 256, kTeamMaxSpins = 1u << 15;   // x a third of a microsecond: the leader's wait for blocks that do not run yet
constexpr int kRadixItems = 8;                   // requests per thread and tile
constexpr int kLargeWaves = 16, kSmallWaves = 4; // of a block: dyn_launch_ingest says where the line lies

// a store that other blocks read after the next barrier
template <typename T>
__device__ __forceinline__ void put(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// false: given up (block-uniform).  All writes of the block before the call are visible to every block after it: every
// wave waits for its own stores, and the waiting thread releases before it arrives and acquires after it has seen
// the others (the block's other waves share its caches and follow it through the block barrier).
__device__ __forceinline__ bool grid_barrier(uint32_t* counter, uint32_t* passed, uint32_t number, uint32_t blocks, uint32_t* s_flag) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    uint32_t spins = 0;
    bool ok = true;
    if (__hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == number * blocks) {
      put(passed, number);
    } else {
      while (__hip_atomic_load(passed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < number) {
        if (++spins > kBarrierSpins) { ok = false; break; }
        __builtin_amdgcn_s_sleep(8);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *s_flag = ok ? 1u : 0u;
  }
  __syncthreads();
  return *s_flag != 0u;
}

// LDS of a block: the wave counters of a tile are done with when its requests' places are known, and are then the
// second buffer of the move.
template <int WAVES>
struct RadixLds {
  static constexpr int kThreads = WAVES * DYN_WAVE, kTile = kThreads * kRadixItems;
  static constexpr int kOwn = DYN_INGEST_MAX_BINS / kThreads;   // digits a thread owns in the scans
  static constexpr int kCopies = WAVES >= 8 ? 4 : 2;
  static_assert(kTile * sizeof(uint32_t) == WAVES * DYN_INGEST_MAX_BINS * sizeof(uint16_t), "the wave counters become the second move buffer");
  uint32_t move[kTile];
  union {
    uint16_t wcnt[WAVES][DYN_INGEST_MAX_BINS];
    uint32_t cnt[kCopies][DYN_INGEST_MAX_BINS];  // digit counts of the block's run, a few copies
    uint32_t move2[kTile];
  };
  uint32_t to[DYN_INGEST_MAX_BINS];              // output position of a digit's first request of the tile, less its place in the tile
  uint32_t wave_sum[WAVES];
  uint32_t flag;
};

// Which of the sorting blocks this one is, and how many there are ({0, 0}: it came too late, or the wait was given up).  The
// first block to arrive waits for the rest of `all` and then closes the team; a block that arrives later leaves.  So every
// block that the barriers wait for is running, whatever else the device is busy with.  It waits as long as the sort would take
// longer with the blocks that are there than with all (`work`: looks that one block alone takes for the sort), but at
// least a moment and at most some milliseconds.  After a moment only, 20 M requests beside an evaluation were at times left to a few
// blocks for 23 ms.
__device__ __forceinline__ RadixTeam join_team(uint32_t* join, uint32_t* members, uint32_t* passed, uint32_t all, float work, uint32_t* status, uint32_t* s_ticket, uint32_t* s_members) {
  if (threadIdx.x == 0) {
    const uint32_t ticket = atomicAdd(join, 1u);
    uint32_t n = 0;
    if (ticket == 0) {
      for (uint32_t spins = 0; spins < kTeamMaxSpins; ++spins) {
        const uint32_t here = __hip_atomic_load(join, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (here >= all || (spins >= kTeamSpins && (float)spins > work / (float)here - work / (float)all)) break;
        __builtin_amdgcn_s_sleep(4);
      }
      n = atomicOr(join, kTeamClosed);
      put(passed, 0u);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      put(members, n);
    } else if (ticket < kTeamClosed) {
      for (uint32_t spins = 0; n == 0 && spins < kBarrierSpins; ++spins) {
        n = __hip_atomic_load(members, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (n == 0) __builtin_amdgcn_s_sleep(4);
      }
      if (n == 0) atomicOr(status, DYN_WS_SORT_ABANDONED);
    }
    *s_members = n;
    *s_ticket = ticket;
  }
  __syncthreads();
  const RadixTeam m = {__builtin_amdgcn_readfirstlane((int)*s_members), __builtin_amdgcn_readfirstlane((int)*s_ticket)};
  __syncthreads();
  return m;
}

// Keys of the requests [beg, end): cell = window * classes + class.
template <int WAVES>
__device__ __forceinline__ void radix_keys(const IngestArgs& a, double r_window, int64_t beg, int64_t end, RadixLds<WAVES>& s) {
  constexpr int kThreads = RadixLds<WAVES>::kThreads;
  const ClassEdges edges = stage_edges(a, (int32_t*)s.move, RadixLds<WAVES>::kTile);
  __syncthreads();
  const uint32_t G = (uint32_t)(a.n_model * a.n_in_bin * a.n_out_bin);
  uint32_t bad = 0;
  constexpr int N = 4;
  for (int64_t at = beg; at < end; at += N * kThreads) {
    double t[N];
    int32_t x[N], y[N], mdl[N];
    uint32_t cls[N];
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const int64_t i = std::min<int64_t>(at + r * kThreads + threadIdx.x, end - 1);
      t[r] = a.t_s[i];
      x[r] = a.in_tok[i];
      y[r] = a.out_tok[i];
      mdl[r] = a.model ? a.model[i] : 0;
    }
    classes_of<N>(a, edges, x, y, mdl, cls, &bad);
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const int64_t i = at + r * kThreads + threadIdx.x;
      const uint32_t w = (uint32_t)window_of(t[r], a.window_s, r_window, a.n_window, &bad);
      if (i < end) put(a.key_a + i, w * G + cls[r]);
    }
  }
  if (bad) atomicOr(a.status, bad);
  __syncthreads();
}

// Digit counts of the keys [beg, end) -> hist[digit][block].  In runs of equal digits (the keys of a later pass) a wave
// adds once for all its lanes; else lanes add to one of four copies, which shortens the queues of equal digits.
template <int WAVES>
__device__ __forceinline__ void radix_count(const uint32_t* keys, int64_t beg, int64_t end, int shift, int bits, uint32_t* hist, RadixTeam m, RadixLds<WAVES>& s) {
  constexpr int kThreads = RadixLds<WAVES>::kThreads, kTile = RadixLds<WAVES>::kTile, kCopies = RadixLds<WAVES>::kCopies;
  const int nbins = 1 << bits;
  const uint32_t mask = (uint32_t)nbins - 1u;
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  for (int b = threadIdx.x; b < kCopies * DYN_INGEST_MAX_BINS; b += kThreads) (&s.cnt[0][0])[b] = 0;
  __syncthreads();
  uint32_t* mine = s.cnt[lane & (kCopies - 1)];
  for (int64_t at = beg; at < end; at += kTile) {
    uint32_t key[kRadixItems];
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
      const int64_t i = at + r * kThreads + threadIdx.x;
      key[r] = keys[i < end ? i : end - 1];
    }
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
      const bool in = at + r * kThreads + threadIdx.x < end;
      const uint32_t d = (key[r] >> shift) & mask;
      const uint64_t there = __ballot(in);
      if (there == 0) continue;
      const uint32_t first = __builtin_amdgcn_readfirstlane(d);   // lanes that are in are a prefix of the wave
      if (__ballot(in && d != first) == 0) {
        if (lane == 0) atomicAdd(&mine[first], (uint32_t)__popcll(there));
      } else if (in) {
        atomicAdd(&mine[d], 1u);
      }
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nbins; b += kThreads) {
    uint32_t n = 0;
#pragma unroll
    for (int q = 0; q < kCopies; ++q) n += s.cnt[q][b];
    put(&hist[(size_t)b * m.blocks + m.block], n);
  }
}

// hist[d][0 .. blocks) -> inclusive sums, one wave per digit where the blocks are many
template <int WAVES>
__device__ __forceinline__ void radix_scan(uint32_t* hist, int bits, RadixTeam m) {
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int n = m.blocks;
  if (n <= 8) {                                  // a few counts: a thread per digit
    for (int d = m.block * WAVES * DYN_WAVE + threadIdx.x; d < (1 << bits); d += n * WAVES * DYN_WAVE) {
      uint32_t sum = 0;
      for (int q = 0; q < n; ++q) put(&hist[(size_t)d * n + q], sum += hist[(size_t)d * n + q]);
    }
    return;
  }
  for (int d = (int)(threadIdx.x / DYN_WAVE) * n + m.block; d < (1 << bits); d += WAVES * n) {
    uint32_t* row = hist + (size_t)d * n;
    uint32_t carry = 0;
    for (int base = 0; base < n; base += 4 * DYN_WAVE) {
      uint32_t v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = row[min(base + q * DYN_WAVE + lane, n - 1)];   // past the end: not written
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int k = 1; k < DYN_WAVE; k <<= 1) {
          const uint32_t up = __shfl_up(v[q], k, DYN_WAVE);
          if (lane >= k) v[q] += up;
        }
        v[q] += carry;
        carry = __shfl(v[q], DYN_WAVE - 1, DYN_WAVE);
        if (base + q * DYN_WAVE + lane < n) put(&row[base + q * DYN_WAVE + lane], v[q]);
      }
    }
  }
}

// Stable move of one tile of `count` requests (FULL: a whole one).  What is missing to a whole one takes part as requests of
// the last digit, behind all others, and is not written.  Every wave owns a contiguous run of rows of 64 requests and
// walks them in order; a request's rank among the row's requests with its digit comes from wave ballots.  `next`: output
// position of the next request of each digit that the thread owns (threadIdx.x * kOwn ...), moved on.
template <int WAVES, bool FULL>
__device__ __forceinline__ void radix_tile(const uint32_t* keys_in, const int32_t* in_in, const int32_t* out_in, uint32_t* keys_out,
                                           int32_t* in_out, int32_t* out_out, int count, int shift, int bits, uint32_t* next, RadixLds<WAVES>& s) {
  constexpr int kThreads = RadixLds<WAVES>::kThreads, kOwn = RadixLds<WAVES>::kOwn;
  const int nbins = 1 << bits;
  const uint32_t mask = (uint32_t)nbins - 1u;
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = threadIdx.x / DYN_WAVE;
  const int at = wave * (kRadixItems * DYN_WAVE) + lane;
  uint32_t key[kRadixItems], pos[kRadixItems];
  int32_t vin[kRadixItems], vout[kRadixItems];
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const int i = FULL ? at + r * DYN_WAVE : min(at + r * DYN_WAVE, count - 1);
    key[r] = keys_in[i];
    vin[r] = in_in[i];
    vout[r] = out_in[i];
    if (!FULL && at + r * DYN_WAVE >= count) key[r] = ~0u;
  }
#pragma unroll
  for (int q = 0; q < kRadixItems; ++q) s.move2[q * kThreads + threadIdx.x] = 0;   // the wave counters
  __syncthreads();
  uint16_t* my = s.wcnt[wave];
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const uint32_t d = (key[r] >> shift) & mask;
    uint64_t peers = ~0ull;
    for (int b = 0; b < bits; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const uint32_t before = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull)), group = (uint32_t)__popcll(peers);
    pos[r] = my[d] + before;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (before == group - 1) my[d] = (uint16_t)(pos[r] + 1);   // one lane per digit advances it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // per digit: where its requests start in the tile, and where each wave's among them do
  uint32_t total[kOwn], sum = 0;
#pragma unroll
  for (int q = 0; q < kOwn; ++q) {
    total[q] = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) total[q] += s.wcnt[w][threadIdx.x * kOwn + q];
    sum += total[q];
  }
  uint32_t start = block_exclusive_sum<WAVES>(sum, s.wave_sum);
#pragma unroll
  for (int q = 0; q < kOwn; ++q) {
    const int d = threadIdx.x * kOwn + q;
    s.to[d] = next[q] - start;
    next[q] += total[q];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const uint32_t c = s.wcnt[w][d];
      s.wcnt[w][d] = (uint16_t)start;
      start += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) pos[r] += my[(key[r] >> shift) & mask];
  __syncthreads();                               // the wave counters are done with
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    s.move[pos[r]] = key[r];
    s.move2[pos[r]] = (uint32_t)vin[r];
  }
  __syncthreads();
  uint32_t dst[kRadixItems];
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const int i = r * kThreads + threadIdx.x;
    const uint32_t k = s.move[i];
    dst[r] = s.to[(k >> shift) & mask] + (uint32_t)i;
    if (FULL || i < count) {
      put(keys_out + dst[r], k);
      put(in_out + dst[r], (int32_t)s.move2[i]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) s.move[pos[r]] = (uint32_t)vout[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRadixItems; ++r) {
    const int i = r * kThreads + threadIdx.x;
    if (FULL || i < count) put(out_out + dst[r], (int32_t)s.move[i]);
  }
}

// Stable move of the requests [beg, end).
template <int WAVES>
__device__ __forceinline__ void radix_move(const uint32_t* keys_in, const int32_t* in_in, const int32_t* out_in, uint32_t* keys_out,
                                           int32_t* in_out, int32_t* out_out, int64_t beg, int64_t end, int shift, int bits,
                                           const uint32_t* hist, RadixTeam m, RadixLds<WAVES>& s) {
  constexpr int kTile = RadixLds<WAVES>::kTile, kOwn = RadixLds<WAVES>::kOwn;
  const int nbins = 1 << bits;
  uint32_t next[kOwn];                             // output position of the next request of each owned digit
  {
    uint32_t total[kOwn], sum = 0;
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      const int d = threadIdx.x * kOwn + q;
      const uint32_t* row = hist + (size_t)d * m.blocks;
      total[q] = d < nbins ? row[m.blocks - 1] : 0u;
      next[q] = d < nbins && m.block > 0 ? row[m.block - 1] : 0u;
      sum += total[q];
    }
    uint32_t base = block_exclusive_sum<WAVES>(sum, s.wave_sum);
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      next[q] += base;
      base += total[q];
    }
  }
  int64_t at = beg;
  for (; at + kTile <= end; at += kTile)
    radix_tile<WAVES, true>(keys_in + at, in_in + at, out_in + at, keys_out, in_out, out_out, kTile, shift, bits, next, s);
  if (at < end) radix_tile<WAVES, false>(keys_in + at, in_in + at, out_in + at, keys_out, in_out, out_out, (int)(end - at), shift, bits, next, s);
}

// ---- a trace in window order ----------------------------------------------------------------
// One block per window.  The requests are ranked by class as in the general sort (a wave walks rows of 64 in order, ranks
// inside a row from ballots), put in class order in LDS and written from there: the window's part of the output is one
// run.  A window of more than a tile counts its classes first and then goes tile by tile.
// What bounds it: vector instructions (ranking and classes, 100 a row of 64 requests: 26 us of ten million requests) and
// bytes (16 a request: 30 us).  The tile is the largest that lets two blocks share a compute unit (76 KB of LDS, 24 requests
// a thread): a window of one tile needs no counting and no look-up of where a class goes.  Ten million requests in 1440
// windows: 47 us; 62 with 16 requests a thread, 75 with 8; 72 with keys read twice and single words scattered (and
// 53 us for the kernel that wrote the keys, where order_kernel takes 19).
// Of the variants the compiler spills <8, 24, 4> 24 vector registers (72 bytes of scratch a thread) and <4, 8, 6> 40; the
// others none.  With fewer requests a thread nothing is spilled and the day's log takes longer (above).
constexpr size_t kWinEdges = 2048;               // class edges that a block stages in LDS

template <int WAVES, int ITEMS>
struct WinLds {
  static constexpr int kThreads = WAVES * DYN_WAVE;
  static constexpr int kTile = kThreads * ITEMS;   // ITEMS requests per thread and tile
  static constexpr int kOwn = DYN_INGEST_MAX_BINS / kThreads;   // classes a thread owns at most
  uint32_t move[kTile];
  union {
    uint16_t wcnt[WAVES][DYN_INGEST_MAX_BINS];
    uint32_t cnt[DYN_INGEST_MAX_BINS];           // class totals of a long window
    uint16_t cls[kTile];                         // of a long window's tile in class order
  };
  uint32_t to[DYN_INGEST_MAX_BINS];              // place in a long window of a class's first request of the tile, less its place in the tile
  uint32_t wave_sum[WAVES];
};

// The window's pieces in a trace of several runs: where the run starts, the piece's bounds; then the piece's end in the
// window, what to add to a place in the window to have the request's index, and the window's first output position and length.
struct RunLds {
  uint32_t run_start[DYN_WS_MAX_BREAKS + 2], bound[2 * (DYN_WS_MAX_BREAKS + 1)];
  int32_t piece_end[DYN_WS_MAX_BREAKS + 1];
  uint32_t piece_add[DYN_WS_MAX_BREAKS + 1];
  uint32_t out[2];
};

// Element i of a run of 4-byte values, i * 4 < 2^32: one 32-bit offset instead of a 64-bit address.
template <typename T>
__device__ __forceinline__ T& at32(T* p, uint32_t i) { return *(T*)((char*)p + (i << 2)); }

// Index of the request at place j of the window; `piece`: that of a place before it.
__device__ __forceinline__ uint32_t window_request(const RunLds& s, uint32_t j, int& piece) {
  while ((int)j >= s.piece_end[piece]) ++piece;
  return s.piece_add[piece] + j;
}

// The pieces of window w in a trace of several runs (the breaks come in any order).
template <int THREADS>
__device__ __forceinline__ void find_pieces(const IngestArgs& a, double r_window, int w, RunLds& s) {
  const uint32_t* breaks = a.unsorted + (DYN_WS_HEADER_BREAK_WORD - DYN_WS_HEADER_ORDER_WORD);
  const int n_break = (int)*a.unsorted, n_run = n_break + 1, lane = threadIdx.x;
  if (lane < n_break) {
    const uint32_t mine = breaks[lane];
    int rank = 1;
    for (int q = 0; q < n_break; ++q) rank += breaks[q] < mine ? 1 : 0;
    s.run_start[rank] = mine;
  }
  if (lane == 0) {
    s.run_start[0] = 0;
    s.run_start[n_run] = (uint32_t)a.n_req;
  }
  __syncthreads();
  // first request of the run in window w (q even) or after it: a wave per question, 64 probes a step
  for (int q = threadIdx.x / DYN_WAVE; q < 2 * n_run; q += THREADS / DYN_WAVE) {
    uint32_t lo = s.run_start[q >> 1], hi = s.run_start[(q >> 1) + 1], ignore = 0;
    const double at = (double)(w + (q & 1));
    while (lo < hi) {                              // requests before lo lie in earlier windows, those from hi on do not
      const uint32_t step = (hi - lo + DYN_WAVE - 1) / DYN_WAVE;
      const uint64_t mine = (uint64_t)lo + (uint64_t)(threadIdx.x & (DYN_WAVE - 1)) * step + (step - 1);   // the last of the lane's share
      const bool early = mine < hi && window_of(a.t_s[mine < hi ? mine : hi - 1], a.window_s, r_window, a.n_window, &ignore) < at;
      const uint32_t shares = (uint32_t)__popcll(__ballot(early));
      const uint64_t next = (uint64_t)lo + (uint64_t)shares * step;
      lo = next < hi ? (uint32_t)next : hi;
      if (next + step - 1 < hi) hi = (uint32_t)(next + step - 1);
    }
    if ((threadIdx.x & (DYN_WAVE - 1)) == 0) s.bound[q] = lo;
  }
  __syncthreads();
  if (lane < DYN_WAVE) {
    const uint32_t from = lane < n_run ? s.bound[2 * lane] : 0u, len = lane < n_run ? s.bound[2 * lane + 1] - from : 0u;
    uint32_t end = len, before = lane < n_run ? from - s.run_start[lane] : 0u;
#pragma unroll
    for (int k = 1; k < DYN_WAVE; k <<= 1) {
      const uint32_t up = __shfl_up(end, k, DYN_WAVE);
      before += __shfl_xor(before, k, DYN_WAVE);
      if (lane >= k) end += up;
    }
    if (lane < n_run) {
      s.piece_end[lane] = (int32_t)end;
      s.piece_add[lane] = from - (end - len);
    }
    if (lane == DYN_WAVE - 1) {
      s.out[0] = before;
      s.out[1] = end;
    }
  }
  __syncthreads();
}

// One tile of `count` requests; LONG: of a window of several tiles.  `next`: place in the window of the next request of each
// class that the thread owns (set here for a window of one tile).  `off`: the window's cell offsets, written by its first tile.
template <int WAVES, int ITEMS, bool LONG, bool RUNS>
__device__ __forceinline__ void window_tile(const IngestArgs& a, const ClassEdges& edges, const int32_t* in_in, const int32_t* out_in, const int32_t* model,
                                            int32_t* in_out, int32_t* out_out, int tile, int count, int bits, int G, int64_t beg, int64_t* off, uint32_t* next, uint32_t* bad, WinLds<WAVES, ITEMS>& s, const RunLds* p) {
  constexpr int kThreads = WAVES * DYN_WAVE, kOwn = WinLds<WAVES, ITEMS>::kOwn;
  constexpr int N = 8;                             // rows whose classes are computed together
  const int nbins = 1 << bits, own = (nbins + kThreads - 1) / kThreads;   // classes, and those a thread owns: threadIdx.x * own ...
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = threadIdx.x / DYN_WAVE;
  const int rows = (count + kThreads - 1) / kThreads;   // rows per wave: a short tile is shared by all waves
  const int at = wave * rows * DYN_WAVE + lane;
  uint32_t place[ITEMS];                       // class << 16 | rank in the wave, later the place in the tile
  int32_t vin[ITEMS], vout[ITEMS];
  int piece = 0;                                   // the lane's places only grow
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (r / N * N < rows) {
      const uint32_t i = (uint32_t)min(at + r * DYN_WAVE, count - 1);
      if (RUNS) {
        const uint32_t j = window_request(*p, (uint32_t)tile + i, piece);
        vin[r] = in_in[j];
        vout[r] = out_in[j];
      } else {
        vin[r] = at32(in_in, i);
        vout[r] = at32(out_in, i);
      }
    }
  piece = 0;
#pragma unroll
  for (int v = 0; v < WAVES; ++v)
    for (int b = threadIdx.x; b < nbins; b += kThreads) s.wcnt[v][b] = 0;
  __syncthreads();
  uint16_t* my = s.wcnt[wave];
  // what is missing to the rows takes part as requests of the last class, behind all others, and is not written
  const uint32_t last = (1u << bits) - 1u;
#pragma unroll
  for (int g = 0; g < ITEMS; g += N) {
    if (g >= rows) continue;                       // the same for the whole block
    int32_t mdl[N];
    uint32_t cls[N];
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const uint32_t i = (uint32_t)min(at + (g + r) * DYN_WAVE, count - 1);
      mdl[r] = 0;
      if (model) mdl[r] = RUNS ? model[window_request(*p, (uint32_t)tile + i, piece)] : at32(model, i);
    }
    classes_of<N>(a, edges, vin + g, vout + g, mdl, cls, bad);
#pragma unroll
    for (int r = 0; r < N; ++r) {
      if (g + r >= rows) continue;
      const uint32_t c = at + (g + r) * DYN_WAVE < count ? cls[r] : last;
      uint32_t lo = ~0u, hi = ~0u;
      for (int b = 0; b < bits; ++b) {
        const int bit = __builtin_amdgcn_sbfe((int)c, b, 1);   // 0 or -1
        const uint64_t bal = __ballot(bit != 0);
        lo &= ~((uint32_t)bal ^ (uint32_t)bit);
        hi &= ~((uint32_t)(bal >> 32) ^ (uint32_t)bit);
      }
      const uint32_t before = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
      const uint32_t group = (uint32_t)__popc(lo) + (uint32_t)__popc(hi);
      const uint32_t rank = my[c] + before;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (before == group - 1) my[c] = (uint16_t)(rank + 1);   // one lane per class advances it
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      place[g + r] = c << 16 | rank;
    }
  }
  __syncthreads();
  // per class: where its requests start in the tile, and where each wave's among them do
  uint32_t total[kOwn], sum = 0;
#pragma unroll
  for (int q = 0; q < kOwn; ++q) {
    total[q] = 0;
    const int d = threadIdx.x * own + q;
    if (q < own && d < nbins) {
#pragma unroll
      for (int v = 0; v < WAVES; ++v) total[q] += s.wcnt[v][d];
      sum += total[q];
    }
  }
  uint32_t start = block_exclusive_sum<WAVES>(sum, s.wave_sum);
#pragma unroll
  for (int q = 0; q < kOwn; ++q) {
    const int d = threadIdx.x * own + q;
    if (q >= own || d >= nbins) continue;
    if (!LONG) next[q] = start;
    if (off && d < G) off[d] = beg + next[q];
    if (LONG) {
      s.to[d] = next[q] - start;
      next[q] += total[q];
    }
#pragma unroll
    for (int v = 0; v < WAVES; ++v) {
      const uint32_t c = s.wcnt[v][d];
      s.wcnt[v][d] = (uint16_t)start;
      start += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (r < rows) place[r] += my[place[r] >> 16];
  if (LONG) {
    __syncthreads();                               // the wave counters are done with
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
      if (r < rows) s.cls[place[r] & 0xFFFFu] = (uint16_t)(place[r] >> 16);
  }
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (r < rows) s.move[place[r] & 0xFFFFu] = (uint32_t)vin[r];
  __syncthreads();
  auto write = [&](int32_t* out) {
    auto one = [&](uint32_t i) {
      if (LONG) out[s.to[s.cls[i]] + i] = (int32_t)s.move[i];
      else at32(out, i) = (int32_t)s.move[i];
    };
    int i = threadIdx.x;
    for (; i + 3 * kThreads < count; i += 4 * kThreads) {
#pragma unroll
      for (int q = 0; q < 4; ++q) one((uint32_t)(i + q * kThreads));
    }
    for (; i < count; i += kThreads) one((uint32_t)i);
  };
  write(in_out);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (r < rows) s.move[place[r] & 0xFFFFu] = (uint32_t)vout[r];
  __syncthreads();
  write(out_out);
}

// A window: `len` requests whose output starts at `beg`.
template <int WAVES, int ITEMS, bool RUNS>
__device__ __forceinline__ void window_move(const IngestArgs& a, int w, int64_t beg, int len, const ClassEdges& edges, WinLds<WAVES, ITEMS>& s, const RunLds* p = nullptr) {
  constexpr int kThreads = WAVES * DYN_WAVE, kTile = kThreads * ITEMS, kOwn = WinLds<WAVES, ITEMS>::kOwn;
  const int32_t G = a.n_model * a.n_in_bin * a.n_out_bin;
  int64_t* off = a.cell_off + (int64_t)w * G;
  if (len <= 0) {
    for (int d = threadIdx.x; d < G; d += kThreads) off[d] = beg;
    return;
  }
  const int64_t from = RUNS ? 0 : beg;             // what the requests are counted from
  const int32_t* in_in = a.in_tok + from;
  const int32_t* out_in = a.out_tok + from;
  const int32_t* model = a.model ? a.model + from : nullptr;
  int32_t* in_out = a.in_sorted + beg;
  int32_t* out_out = a.out_sorted + beg;
  uint32_t bad = 0;
  int bits = 0;
  while ((1 << bits) < G) ++bits;
  uint32_t next[kOwn];
  if (len <= kTile) {
    window_tile<WAVES, ITEMS, false, RUNS>(a, edges, in_in, out_in, model, in_out, out_out, 0, len, bits, G, beg, off, next, &bad, s, p);
  } else {
    for (int d = threadIdx.x; d < DYN_INGEST_MAX_BINS; d += kThreads) s.cnt[d] = 0;
    __syncthreads();
    int piece = 0;
    for (int at = 0; at < len; at += 4 * kThreads) {
      int32_t x[4], y[4], mdl[4];
      uint32_t d[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        uint32_t i = (uint32_t)min(at + r * kThreads + (int)threadIdx.x, len - 1);
        if (RUNS) i = window_request(*p, i, piece);
        x[r] = in_in[i];
        y[r] = out_in[i];
        mdl[r] = model ? model[i] : 0;
      }
      classes_of<4>(a, edges, x, y, mdl, d, &bad);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (at + r * kThreads + (int)threadIdx.x < len) atomicAdd(&s.cnt[d[r]], 1u);
    }
    __syncthreads();
    const int own = ((1 << bits) + kThreads - 1) / kThreads;
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < kOwn; ++q)
      if (q < own && (int)threadIdx.x * own + q < DYN_INGEST_MAX_BINS) sum += s.cnt[threadIdx.x * own + q];
    uint32_t base = block_exclusive_sum<WAVES>(sum, s.wave_sum);
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      next[q] = base;
      if (q < own && (int)threadIdx.x * own + q < DYN_INGEST_MAX_BINS) base += s.cnt[threadIdx.x * own + q];
    }
    for (int tile = 0; tile < len; tile += kTile) {
      __syncthreads();                             // what the counts or the last tile left in LDS has been read
      const int skip = RUNS ? 0 : tile;
      window_tile<WAVES, ITEMS, true, RUNS>(a, edges, in_in + skip, out_in + skip, model ? model + skip : nullptr, in_out, out_out, tile, min(kTile, len - tile), bits, G,
                                            beg, tile == 0 ? off : nullptr, next, &bad, s, p);
    }
  }
  if (bad) atomicOr(a.status, bad);
}

template <int WAVES, int ITEMS, int PER_SIMD>
__global__ __launch_bounds__(WAVES* DYN_WAVE) __attribute__((amdgpu_waves_per_eu(PER_SIMD, PER_SIMD))) void window_sort_kernel(IngestArgs a, int edge_room, int longest) {
  if (route_of(a) != kByWindow) return;
  __shared__ WinLds<WAVES, ITEMS> s;
  extern __shared__ int32_t s_edge[];
  const int w = blockIdx.x;
  const int64_t beg = a.win_off[w];
  const int len = (int)(a.win_off[w + 1] - beg);
  if (w == a.n_window - 1 && threadIdx.x == 0) a.cell_off[(int64_t)a.n_window * a.n_model * a.n_in_bin * a.n_out_bin] = a.n_req;
  if (len > longest) {                             // for the larger blocks of the kernel after this one
    if (threadIdx.x == 0) a.key_a[atomicAdd(a.unsorted + (DYN_WS_HEADER_LEFT_WORD - DYN_WS_HEADER_ORDER_WORD), 1u)] = (uint32_t)w;
    return;
  }
  const ClassEdges edges = stage_edges(a, s_edge, edge_room);
  window_move<WAVES, ITEMS, false>(a, w, beg, len, edges, s);
}

// The windows of a trace of a few runs (RUNS), or the `n` windows that window_sort_kernel left: a list, each of them one
// piece.  The blocks share them.
template <int WAVES, bool RUNS>
__device__ __forceinline__ void shared_windows(const IngestArgs& a, double r_window, int n, WinLds<WAVES, kRadixItems>& s, RunLds& p, int32_t* s_edge, int edge_room) {
  const ClassEdges edges = stage_edges(a, s_edge, edge_room);
  if (RUNS && blockIdx.x == 0 && threadIdx.x == 0) a.cell_off[(int64_t)a.n_window * a.n_model * a.n_in_bin * a.n_out_bin] = a.n_req;
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    if (RUNS) {
      find_pieces<WAVES * DYN_WAVE>(a, r_window, i, p);
      window_move<WAVES, kRadixItems, true>(a, i, p.out[0], (int)p.out[1], edges, s, &p);
    } else {
      const int w = (int)a.key_a[i];
      const int64_t beg = a.win_off[w];
      window_move<WAVES, kRadixItems, false>(a, w, beg, (int)(a.win_off[w + 1] - beg), edges, s);
    }
    __syncthreads();
  }
}

// A trace that is not in window order, and the long windows of one that is.
template <int WAVES>
__global__ __launch_bounds__(WAVES* DYN_WAVE) __attribute__((amdgpu_waves_per_eu(4, 4))) void unordered_kernel(RadixArgs g) {
  constexpr int kThreads = RadixLds<WAVES>::kThreads, kTile = RadixLds<WAVES>::kTile;
  constexpr int kRunEdges = WAVES >= 8 ? 2048 : 256;
  const IngestArgs& a = g.t;
  const Route route = route_of(a);               // the same for every block
  const int n_left = route == kByWindow ? (int)a.unsorted[DYN_WS_HEADER_LEFT_WORD - DYN_WS_HEADER_ORDER_WORD] : 0;
  if (route == kByWindow && (int)blockIdx.x >= n_left) return;
  __shared__ union {
    RadixLds<WAVES> radix;
    struct {
      WinLds<WAVES, kRadixItems> win;
      RunLds run;
      int32_t edge[kRunEdges];
    } runs;
  } lds;
  if (route == kByWindow) {
    shared_windows<WAVES, false>(a, g.r_window, n_left, lds.runs.win, lds.runs.run, lds.runs.edge, kRunEdges);
    return;
  }
  if (route == kByRuns) {
    shared_windows<WAVES, true>(a, g.r_window, a.n_window, lds.runs.win, lds.runs.run, lds.runs.edge, kRunEdges);
    return;
  }
  if ((int)blockIdx.x >= g.blocks) return;
  RadixLds<WAVES>& s = lds.radix;
  const RadixTeam m = join_team(g.join, g.members, g.passed, (uint32_t)g.blocks, (float)a.n_req * 0.012f * (float)g.passes, a.status, &s.wave_sum[0], &s.flag);
  if (m.blocks == 0) return;
  uint32_t passed = 0;                           // barriers behind this block
  auto sync = [&]() {
    ++passed;
    const bool ok = grid_barrier(g.barrier, g.passed, passed, (uint32_t)m.blocks, &s.flag);
    if (!ok && threadIdx.x == 0) atomicOr(a.status, DYN_WS_SORT_ABANDONED);
    return ok;
  };
  const int n_tile = (int)((a.n_req + kTile - 1) / kTile);
  const int tiles = n_tile / m.blocks, more = n_tile % m.blocks;   // the first `more` blocks take one tile more
  const int64_t beg = (int64_t)(m.block * tiles + min(m.block, more)) * kTile;
  const int64_t end = std::min<int64_t>(a.n_req, beg + (int64_t)(tiles + (m.block < more ? 1 : 0)) * kTile);
  radix_keys(a, g.r_window, beg, end, s);
  const uint32_t* k_src = a.key_a;
  uint32_t* k_dst = a.key_b;
  const int32_t *i_src = a.in_tok, *o_src = a.out_tok;
  for (int p = 0; p < g.passes; ++p) {
    const bool to_final = ((g.passes - 1 - p) % 2) == 0;   // ping-pong so that the last pass lands in the caller's arrays
    int32_t* i_dst = to_final ? a.in_sorted : a.in_tmp;
    int32_t* o_dst = to_final ? a.out_sorted : a.out_tmp;
    const int shift = p * g.bits;
    radix_count(k_src, beg, end, shift, g.bits, a.block_hist, m, s);
    if (!sync()) return;
    radix_scan<WAVES>(a.block_hist, g.bits, m);
    if (!sync()) return;
    radix_move(k_src, i_src, o_src, k_dst, i_dst, o_dst, beg, end, shift, g.bits, a.block_hist, m, s);
    if (!sync()) return;
    i_src = i_dst;
    o_src = o_dst;
    uint32_t* old_src = const_cast<uint32_t*>(k_src);      // both key buffers live in the workspace
    k_src = k_dst;
    k_dst = old_src;
  }
  if (a.n_req == 0)
    for (int64_t c = threadIdx.x; c <= g.cells; c += kThreads) a.cell_off[c] = 0;
  // The offsets (cell_off[c] = number of requests with key < c), a tile of sorted keys in LDS at a time: a request fills
  // the cells from the key before it on (by one thread the 35 000 empty cells before the log of a grid's last minutes took 1.1 ms).
  // What is left behind the last request is its block's.
  uint32_t left = 0;                             // one more than the key before the tile
  for (int64_t at = beg; at < end; at += kTile) {
    const int count = (int)std::min<int64_t>(kTile, end - at);
    left = at > 0 ? __hip_atomic_load(k_src + at - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u : 0u;
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) s.move[r * kThreads + threadIdx.x] = k_src[std::min<int64_t>(at + r * kThreads + threadIdx.x, end - 1)];
    __syncthreads();
#pragma unroll 1
    for (int i = threadIdx.x; i - (int)threadIdx.x < count; i += kThreads) {
      const uint32_t from = i > 0 ? s.move[min(i, count) - 1] + 1u : left, to = s.move[min(i, count - 1)] + 1u;   // beyond the tile: equal
      fill_runs(a.cell_off, from, to, at + i);
    }
    left = s.move[count - 1] + 1u;
    __syncthreads();
  }
  if (end == a.n_req && beg < end)
    for (int64_t c = (int64_t)left + threadIdx.x; c <= g.cells; c += kThreads) a.cell_off[c] = a.n_req;
}

}  // namespace

// Which logs are sorted, and have their runs and long windows moved, by small blocks: four waves, 128 registers and 22 KB of LDS.
// A kernel's blocks have to fit beside what runs on other streams, also where they return at once: beside an evaluation,
// which fills every compute unit, blocks of more than 28 KB, or of more registers than four waves of 128, wait until it is
// through (empty kernels, us: 4 waves of 128 registers and 20 KB 9, 28 KB 35, 40 KB 830; 8 waves of 64 registers and
// 16 KB 9, of 128 840; 16 waves 830).  Ingests beside an evaluation, large blocks and small (us): 20 000 requests 780, 45;
// 1 M 840, 81; 1 M in six runs 907, 142; 300 000 unordered 947, 168.  Alone: 20 000 16, 16; 1 M in six runs 74, 48;
// unordered 20 000 86, 75, 300 000 78, 81, 600 000 93, 122, 1 M 102, 128.  Larger logs take large blocks all the same,
// whose tiles write longer runs (six million unordered 280), and so do logs of long windows: theirs move as quickly
// only there (500 000 in nine runs and 60 windows 38, 63).  Two small blocks to a unit: four are quicker alone (1 M in six
// runs 48, 38) and wait longer for their places (700 000 in time order beside a kernel that fills the device 79, 96).
constexpr int64_t kSmallLog = 1 << 20;
bool small_blocks(int64_t n_req, int32_t n_window) { return n_req <= kSmallLog && 1.75 * (double)n_req / n_window <= 4096.0; }
constexpr int64_t kSmallTile = RadixLds<kSmallWaves>::kTile, kLargeTile = RadixLds<kLargeWaves>::kTile;

// Blocks that the digit counts have room for at ten bits a digit (grows with n_req).
int64_t dyn_ingest_blocks(int64_t n_req) {
  const int64_t n = std::max<int64_t>(n_req, 1);
  return std::max((n + kLargeTile - 1) / kLargeTile, (std::min(n, kSmallLog) + kSmallTile - 1) / kSmallTile);
}

hipError_t dyn_launch_edges(const int32_t* in_edge, size_t n_in, const int32_t* out_edge, size_t n_out, int32_t* d_in,
                            int32_t* d_out, WsHeader* header, uint32_t order_word, uint32_t* counters, hipStream_t s) {
  EdgePack p;
  if (n_in + n_out <= DYN_EDGE_PACK) {          // the usual case: header and both lists in one launch
    if (n_in) memcpy(p.v, in_edge, n_in * sizeof(int32_t));
    if (n_out) memcpy(p.v + n_in, out_edge, n_out * sizeof(int32_t));
    hipLaunchKernelGGL(edge_store_kernel, dim3(1), dim3(256), 0, s, p, (int)n_in, d_in, (int)n_out, d_out, header, order_word, counters);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(edge_store_kernel, dim3(1), dim3(64), 0, s, p, 0, d_in, 0, d_out, header, order_word, counters);
  const struct { const int32_t* src; size_t n; int32_t* dst; } parts[2] = {{in_edge, n_in, d_in}, {out_edge, n_out, d_out}};
  for (const auto& part : parts)
    for (size_t at = 0; at < part.n; at += DYN_EDGE_PACK) {
      const int n = (int)std::min<size_t>(DYN_EDGE_PACK, part.n - at);
      memcpy(p.v, part.src + at, (size_t)n * sizeof(int32_t));
      hipLaunchKernelGGL(edge_store_kernel, dim3(1), dim3(256), 0, s, p, n, part.dst + at, 0, part.dst, (WsHeader*)nullptr, 0u, (uint32_t*)nullptr);
    }
  return hipGetLastError();
}

static int sort_passes(int32_t key_bits) { return key_bits <= 0 ? 1 : (key_bits + 9) / 10; }

// Whether to sort whatever the order: more classes than the window route counts, or windows so long that one block each
// takes longer than the whole sort.  Measured: the window route 2 us per thousand requests of a window, the sort
// 30 us and 12 to 16 us a pass and million.  10 M requests in 20, 60, 120 windows: 1041, 384, 225 us by window, 216, 333,
// 334 sorted; 1 M in 5, 20, 60: 405, 120, 55 and 50, 56, 81; one window of 10 000, 30 000: 26, 76 and 34, 35.
bool dyn_ingest_always_sorts(int64_t n_req, int32_t n_window, int64_t n_class, int32_t key_bits) {
  if (n_class > DYN_INGEST_MAX_BINS) return true;
  return 2e-3 * (double)n_req / n_window > 30.0 + 15e-6 * sort_passes(key_bits) * (double)n_req;
}

// Samples of one window (order_kernel) after which the log is sorted: those of the longest window that one block moves while
// the device sorts everything.  The block 8 us and 1.5 us a thousand requests, the sort 50 us and 16 us a pass and million; in a
// small log 8 and 4, and 70 and 45.
// Measured (us; the window routes and the sort): ordered, 10 M requests in 3 of 2016 windows 6750, 378; 6 M in 10 of
// 1440 1266, 276; 500 000 in 5 of 2016 (by 64 threads) 1575, 102; six runs, 10 M in 3 of 2016 5100, 373.
uint32_t dyn_ingest_many(int64_t n_req, int32_t n_window, int32_t key_bits) {
  const bool small = small_blocks(n_req, n_window);
  const double passes = sort_passes(key_bits) * (double)n_req;
  const double longest = small ? (62.0 + 45e-6 * passes) / 4e-3 : (42.0 + 16e-6 * passes) / 1.5e-3;
  return (double)n_req > longest ? (uint32_t)(longest / (small ? kSampleStep : 4 * kSampleStep)) + 1u : 0u;
}

hipError_t dyn_launch_ingest(const IngestArgs& a, hipStream_t s) {
  const int64_t n = a.n_req;
  const int32_t G = a.n_model * a.n_in_bin * a.n_out_bin;
  const int64_t cells = (int64_t)a.n_window * G;
  hipError_t e;
  const double r_window = 1.0 / a.window_s;
  if (!a.force_sort) {        // in window order: one block per window moves its requests to their cells
    // the order kernel ORs into the flag word, which the header kernel before it set to 0
    const int64_t per_block = 256 * kOrderRows;
    hipLaunchKernelGGL(order_kernel, dim3((unsigned)std::max<int64_t>(1, (n + per_block - 1) / per_block)), dim3(256), 0, s, a, r_window, small_blocks(n, a.n_window) ? 0u : 3u);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const size_t n_edge = (size_t)a.n_model * ((a.n_in_bin - 1) + (a.n_out_bin - 1));
    const size_t room = n_edge <= kWinEdges ? n_edge : 0;
    // The smallest tile that holds a window of 1.75 times the mean (traffic is not even).  Measured (us, by mean requests per
    // window; 1440 to 2016 windows, 17 280 for 579), tiles of 512, 2048, 4096 and 12 288: 10: 7, 12, 13, 27; 198: 9, 13, 15, 28;
    // 579: 78, 69, 102, 207; 694: 27, 11, 16, 23; 1389: 45, 22, 15, 26; 2778: 81, 33, 31, 29; 6944: 189, 65, 61, 45.
    // A longer window than the tile goes to the 16-wave blocks of the next kernel, which ran empty before: 1.5 us a thousand
    // requests, where these take 15, 4.1, 3.1 and 2.0.  Of the largest tile only what is far longer than four tiles
    // and than the others: where all are long these blocks, twice as many, are as quick.  Measured (us; all here, and left):
    // 500 000 requests in 50 of 2016 windows 221, 36; 200 000 in 20 of 1440 207, 35; 1000 in 1 of 60 31, 16; 580 000 in 1000 of
    // 2016 54, 53; 20 M in 100 of 2016 519, 365; evenly, 580 000 and 2.3 M in 2016 28, 26 and 32, 32.
    const dim3 grid((unsigned)a.n_window);
    const size_t lds = room * sizeof(int32_t);
    const double peak = 1.75 * (double)n / a.n_window;
    if (peak <= 512) hipLaunchKernelGGL((window_sort_kernel<1, 8, 4>), grid, dim3(DYN_WAVE), lds, s, a, (int)room, 512);
    else if (peak <= 2048) hipLaunchKernelGGL((window_sort_kernel<4, 8, 6>), grid, dim3(4 * DYN_WAVE), lds, s, a, (int)room, 2048);
    else if (peak <= 4096) hipLaunchKernelGGL((window_sort_kernel<4, 16, 4>), grid, dim3(4 * DYN_WAVE), lds, s, a, (int)room, 4096);
    else hipLaunchKernelGGL((window_sort_kernel<8, 24, 4>), grid, dim3(8 * DYN_WAVE), lds, s, a, (int)room, std::max(4 * 12288, (int)(4 * n / a.n_window)));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (n == 0) return hipSuccess;   // nothing to sort: the flag word stays 0
  }
  const int passes = sort_passes(a.key_bits);
  const int bits = a.key_bits <= 0 ? 1 : (a.key_bits + passes - 1) / passes;
  // one block per compute unit (asked once per device)
  static std::atomic<int> units[64];
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64) {
    n_cu = units[dev].load(std::memory_order_relaxed);
    if (n_cu == 0) {
      if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1) n_cu = 1;
      units[dev].store(n_cu, std::memory_order_relaxed);
    }
  }
  (void)hipGetLastError();
  RadixArgs r;
  r.t = a; r.r_window = r_window; r.cells = cells; r.passes = passes; r.bits = bits;
  r.barrier = a.unsorted + (DYN_WS_HEADER_BARRIER_WORD - DYN_WS_HEADER_ORDER_WORD); r.join = r.barrier + 1; r.members = r.barrier + 2;
  r.passed = a.unsorted + (DYN_WS_HEADER_BREAK_WORD + DYN_WS_MAX_BREAKS - 1 - DYN_WS_HEADER_ORDER_WORD);   // the last break's word: a log that is sorted needs no breaks
  // a block for every tile, as far as they fit the device and the digit counts (a word per digit and block) the workspace
  const int64_t room = ((int64_t)DYN_INGEST_MAX_BINS * a.n_block) >> bits;
  const bool small = small_blocks(n, a.n_window);
  const int64_t n_tile = small ? (n + kSmallTile - 1) / kSmallTile : (n + kLargeTile - 1) / kLargeTile, at_once = (int64_t)n_cu * (small ? 2 : 1);
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>({(int64_t)n_cu, n_tile, room}));
  r.blocks = (int32_t)blocks;
  const int64_t grid = a.force_sort ? blocks : std::max<int64_t>(blocks, std::min<int64_t>(at_once, a.n_window));
  if (small) hipLaunchKernelGGL(unordered_kernel<kSmallWaves>, dim3((unsigned)grid), dim3(kSmallWaves * DYN_WAVE), 0, s, r);
  else hipLaunchKernelGGL(unordered_kernel<kLargeWaves>, dim3((unsigned)grid), dim3(kLargeWaves * DYN_WAVE), 0, s, r);
  return hipGetLastError();
}
