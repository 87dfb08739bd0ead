// Trace ingestion: every request gets the key of its cell (window from the timestamp,
// class from the input/output length bins of Table IV's convention), then a stable
// least-significant-digit radix sort by key moves (input tokens, output tokens) into cell
// order, and the cell offsets are read off the sorted keys.
//
// A trace that is already in window order (a request log is in time order) does not need the
// general sort: the key kernel notices it (a flag word in the workspace header stays 0; it also
// writes where every window starts), and one block per window then counts its requests by class
// and moves them, stably, to their cells (window_sort_kernel).  Any other trace takes the radix
// sort.  The host does not read the flag: both routes are enqueued and the kernels of the route
// not taken return at their first instruction.  The general sort is one launch with grid-wide
// barriers between the phases, so the route not taken costs one empty launch.
#include <string.h>

#include <algorithm>
#include <atomic>

#include "dyn_internal.h"
#include "dyn_device.h"

namespace {

constexpr int kWaves = 4;
constexpr int kRows = 32;                              // rows of 64 requests per wave
constexpr int kTile = kWaves * kRows * DYN_WAVE;       // 8192 requests per block

constexpr int kKeyRows = 4;                            // requests per thread of the key kernel (rows of 256)

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

// A block takes kKeyRows rows of 256 consecutive requests (all loads of a thread in flight together); the class
// edges sit in LDS when they fit (lds_edges != 0).
__global__ __launch_bounds__(256) void key_kernel(IngestArgs a, double r_window, int lds_edges) {
  extern __shared__ int32_t s_edge[];                  // [n_model][n_in_bin - 1] then [n_model][n_out_bin - 1]
  const int n_ie = a.n_in_bin - 1, n_oe = a.n_out_bin - 1;
  const int32_t* in_edge = a.d_in_edge;
  const int32_t* out_edge = a.d_out_edge;
  if (lds_edges) {
    for (int q = threadIdx.x; q < a.n_model * n_ie; q += blockDim.x) s_edge[q] = a.d_in_edge[q];
    for (int q = threadIdx.x; q < a.n_model * n_oe; q += blockDim.x) s_edge[a.n_model * n_ie + q] = a.d_out_edge[q];
    __syncthreads();
    in_edge = s_edge;
    out_edge = s_edge + a.n_model * n_ie;
  }
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int64_t base = (int64_t)blockIdx.x * (kKeyRows * 256) + threadIdx.x;
  double t[kKeyRows], tp[kKeyRows];
  int32_t x[kKeyRows], y[kKeyRows], md[kKeyRows];
#pragma unroll
  for (int r = 0; r < kKeyRows; ++r) {
    const int64_t i = base + r * 256;
    const bool in = i < a.n_req;
    t[r] = in ? a.t_s[i] : 0.0;
    tp[r] = (in && lane == 0 && i > 0) ? a.t_s[i - 1] : 0.0;   // the request before a wave's first
    x[r] = in ? a.in_tok[i] : 0;
    y[r] = in ? a.out_tok[i] : 0;
    md[r] = (in && a.model) ? a.model[i] : 0;
  }
  const int64_t G = (int64_t)a.n_model * a.n_in_bin * a.n_out_bin;
  uint32_t bad = 0;
  bool dis = false;
#pragma unroll
  for (int r = 0; r < kKeyRows; ++r) {
    const int64_t i = base + r * 256;
    const bool in = i < a.n_req;                       // the lanes that are in are a prefix of the wave: lane - 1 is among them
    uint32_t bad_r = 0;
    const double wq = window_of(t[r], a.window_s, r_window, a.n_window, &bad_r);
    int32_t mdl = md[r];
    if (mdl < 0 || mdl >= a.n_model) { bad_r = DYN_WS_BAD_REQUEST; mdl = 0; }
    const int32_t* ie = in_edge + (size_t)mdl * n_ie;
    const int32_t* oe = out_edge + (size_t)mdl * n_oe;
    int bi = 0, bo = 0;
    for (int e = 0; e < n_ie; ++e) bi += (x[r] >= ie[e]) ? 1 : 0;
    for (int e = 0; e < n_oe; ++e) bo += (y[r] >= oe[e]) ? 1 : 0;
    const int64_t g = ((int64_t)mdl * a.n_in_bin + bi) * a.n_out_bin + bo;
    // Window order: compare with the request before (the neighbouring lane; the first lane of a wave recomputes it).
    // Where the window changes the boundaries are written: in a trace in window order win_off[w] = number of
    // requests in windows before w (the values are not used otherwise).
    double wp = __shfl_up(wq, 1, DYN_WAVE);
    if (lane == 0) {
      uint32_t ignore = 0;
      wp = window_of(tp[r], a.window_s, r_window, a.n_window, &ignore);
    }
    if (i == 0) wp = -1.0;
    // The boundaries only matter to the window route: a wave that sees a request out of order, or finds the flag
    // raised already, writes none (on a shuffled trace every request would otherwise fill hundreds of them).
    const bool back = in && wp > wq;
    const bool fill = __ballot(back) == 0 && __hip_atomic_load(a.unsorted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u;
    if (in) {
      a.key_a[i] = (uint32_t)((int64_t)wq * G + g);
      bad |= bad_r;
      dis = dis || back;
      if (fill) {
        for (int64_t w = (int64_t)wp + 1; w <= (int64_t)wq; ++w) a.win_off[w] = i;
        if (i == a.n_req - 1)
          for (int64_t w = (int64_t)wq + 1; w <= a.n_window; ++w) a.win_off[w] = a.n_req;
      }
    }
  }
  if (bad) atomicOr(a.status, bad);
  const uint64_t any = __ballot(dis);
  if (any && lane == __builtin_ctzll(any) && __hip_atomic_load(a.unsorted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u)
    atomicOr(a.unsorted, 1u);
}

// The route is chosen on the device: every kernel of the two routes is launched and the kernels of the route that
// is not taken return at once.  `order` is the flag word the key kernel leaves: 0 = every request's window is at
// or after the window of the request before it (the trace is moved window by window), else the general sort runs.
__device__ __forceinline__ bool sort_route(const uint32_t* order) { return *order != 0u; }

// Class edges from the kernel's arguments into the workspace (a few hundred values at most per launch): the host
// arrays are free when the call returns and nothing waits for the stream.  The first launch also writes the
// workspace header: status 0, the order word (1 when the general sort is forced).
struct EdgePack { int32_t v[DYN_EDGE_PACK]; };
__global__ void edge_store_kernel(EdgePack p, int n_a, int32_t* __restrict__ dst_a, int n_b, int32_t* __restrict__ dst_b,
                                  WsHeader* header, uint32_t order_word) {
  for (int i = threadIdx.x; i < n_a; i += blockDim.x) dst_a[i] = p.v[i];
  for (int i = threadIdx.x; i < n_b; i += blockDim.x) dst_b[i] = p.v[n_a + i];
  if (header && threadIdx.x == 0) {
    header->status = 0u;
    header->kind = DYN_WS_KIND_WORD;
    header->cells = 0;
    ((uint32_t*)header)[DYN_WS_HEADER_ORDER_WORD] = order_word;
    for (int q = 0; q < 3; ++q) ((uint32_t*)header)[DYN_WS_HEADER_BARRIER_WORD + q] = 0u;
  }
}

// cell_off[c] = number of requests with key < c, read off the sorted keys
__device__ __forceinline__ void offsets_at(int64_t i, int64_t prev, int64_t cur, int64_t n, int64_t cells, int64_t* cell_off) {
  if (i == n || cur > cells) cur = cells;
  for (int64_t c = prev + 1; c <= cur; ++c) cell_off[c] = i;
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
//   scattered cost 93 us, runs of 16 words 13 us, of 32 words 9.5 us.  So the tile is 8192 requests: 32 to a digit.
// - All loads of a thread's eight requests are in flight together, also where only keys are counted or compared.
// 523 us with separate scan phases, all waves fencing and single words scattered; 225 us so.
//
// The barrier: an arrival counter in the workspace header, zeroed with the header; barrier number k is passed when
// the counter reaches k * blocks.  Only blocks that run take part (join_team), so other work on the device can
// delay a barrier but not stop it; if it takes seconds all the same, the wait is given up (every block leaves,
// DYN_WS_SORT_ABANDONED is raised).
struct RadixArgs {
  const uint32_t* order;
  uint32_t* barrier; uint32_t* join; uint32_t* members; uint32_t* status;
  uint32_t* key_a; uint32_t* key_b;
  const int32_t* in_tok; const int32_t* out_tok;
  int32_t* in_sorted; int32_t* out_sorted; int32_t* in_tmp; int32_t* out_tmp;
  uint32_t* hist;                                // [digit][block]
  int64_t n, cells; int64_t* cell_off;
  int32_t passes, bits;
};

constexpr uint32_t kBarrierSpins = 1u << 22;     // x about a microsecond per look: seconds
// The blocks that sort together: those that run when the first one has waited for them.
struct RadixTeam { int blocks, block; };
constexpr uint32_t kTeamClosed = 1u << 31;
constexpr uint32_t kTeamSpins = 256;             // x a third of a microsecond: the leader's wait for blocks that do not run yet
constexpr int kRadixWaves = 16;
constexpr int kRadixThreads = kRadixWaves * DYN_WAVE;
constexpr int kRadixItems = 8;                   // requests per thread and tile
constexpr int kRadixTile = kRadixThreads * kRadixItems;
constexpr int kRadixOwn = DYN_INGEST_MAX_BINS / kRadixThreads;   // digits a thread owns in the scans
static_assert(kRadixTile * sizeof(uint32_t) == kRadixWaves * DYN_INGEST_MAX_BINS * sizeof(uint16_t), "the wave counters become the second move buffer");

// a store that other blocks read after the next barrier
template <typename T>
__device__ __forceinline__ void put(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// false: given up (block-uniform).  All writes of the block before the call are visible to every block after it: every
// wave waits for its own stores, and the waiting thread releases before it arrives and acquires after it has seen
// the others (the block's other waves share its caches and follow it through the block barrier).
__device__ __forceinline__ bool grid_barrier(uint32_t* counter, uint32_t target, uint32_t* s_flag) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t spins = 0;
    bool ok = true;
    while (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (++spins > kBarrierSpins) { ok = false; break; }
      __builtin_amdgcn_s_sleep(8);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *s_flag = ok ? 1u : 0u;
  }
  __syncthreads();
  return *s_flag != 0u;
}

// LDS of a block: the wave counters of a tile are done with when its requests' places are known, and are then the
// second buffer of the move.
struct RadixLds {
  uint32_t move[kRadixTile];
  union {
    uint16_t wcnt[kRadixWaves][DYN_INGEST_MAX_BINS];
    uint32_t cnt[4][DYN_INGEST_MAX_BINS];        // digit counts of the block's run, four copies
    uint32_t move2[kRadixTile];
  };
  uint32_t to[DYN_INGEST_MAX_BINS];              // output position of a digit's first request of the tile, less its place in the tile
  uint32_t wave_sum[kRadixWaves];
  uint32_t flag;
};

// Which of the sorting blocks this one is, and how many there are ({0, 0}: it came too late, or the wait was given up).  The
// first block to arrive waits a moment for the rest of the grid and then closes the team; a block that arrives later leaves.
// So every block that the barriers wait for is running, whatever else the device is busy with.
__device__ __forceinline__ RadixTeam join_team(uint32_t* join, uint32_t* members, uint32_t* status, RadixLds& s) {
  if (threadIdx.x == 0) {
    const uint32_t ticket = atomicAdd(join, 1u);
    uint32_t n = 0;
    if (ticket == 0) {
      for (uint32_t spins = 0; spins < kTeamSpins && __hip_atomic_load(join, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < gridDim.x; ++spins) __builtin_amdgcn_s_sleep(4);
      n = atomicOr(join, kTeamClosed);
      put(members, n);
    } else if (ticket < kTeamClosed) {
      for (uint32_t spins = 0; n == 0 && spins < kBarrierSpins; ++spins) {
        n = __hip_atomic_load(members, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (n == 0) __builtin_amdgcn_s_sleep(4);
      }
      if (n == 0) atomicOr(status, DYN_WS_SORT_ABANDONED);
    }
    s.flag = n;
    s.wave_sum[0] = ticket;
  }
  __syncthreads();
  const RadixTeam m = {__builtin_amdgcn_readfirstlane((int)s.flag), __builtin_amdgcn_readfirstlane((int)s.wave_sum[0])};
  __syncthreads();
  return m;
}

// Digit counts of the keys [beg, end) -> hist[digit][block].  In runs of equal digits (the keys of a later pass) a wave
// adds once for all its lanes; else lanes add to one of four copies, which shortens the queues of equal digits.
__device__ __forceinline__ void radix_count(const uint32_t* keys, int64_t beg, int64_t end, int shift, int bits, uint32_t* hist, RadixTeam m, RadixLds& s) {
  const int nbins = 1 << bits;
  const uint32_t mask = (uint32_t)nbins - 1u;
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  for (int b = threadIdx.x; b < 4 * DYN_INGEST_MAX_BINS; b += kRadixThreads) (&s.cnt[0][0])[b] = 0;
  __syncthreads();
  uint32_t* mine = s.cnt[lane & 3];
  for (int64_t at = beg; at < end; at += kRadixTile) {
    uint32_t key[kRadixItems];
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
      const int64_t i = at + r * kRadixThreads + threadIdx.x;
      key[r] = keys[i < end ? i : end - 1];
    }
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
      const bool in = at + r * kRadixThreads + threadIdx.x < end;
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
  for (int b = threadIdx.x; b < nbins; b += kRadixThreads)
    put(&hist[(size_t)b * m.blocks + m.block], s.cnt[0][b] + s.cnt[1][b] + s.cnt[2][b] + s.cnt[3][b]);
}

// hist[d][0 .. blocks) -> inclusive sums, one wave per digit
__device__ __forceinline__ void radix_scan(uint32_t* hist, int bits, RadixTeam m) {
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int n = m.blocks;
  for (int d = (int)(threadIdx.x / DYN_WAVE) * n + m.block; d < (1 << bits); d += kRadixWaves * n) {
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

// exclusive sum over the block's threads
__device__ __forceinline__ uint32_t radix_block_scan(uint32_t v, RadixLds& s) {
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = threadIdx.x / DYN_WAVE;
  uint32_t incl = v;
#pragma unroll
  for (int k = 1; k < DYN_WAVE; k <<= 1) {
    const uint32_t up = __shfl_up(incl, k, DYN_WAVE);
    if (lane >= k) incl += up;
  }
  if (lane == DYN_WAVE - 1) s.wave_sum[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave; ++w) before += s.wave_sum[w];
  __syncthreads();
  return before + incl - v;
}

// Stable move of one tile of `count` requests (FULL: kRadixTile).  What is missing to kRadixTile takes part as requests of
// the last digit, behind all others, and is not written.  Every wave owns a contiguous run of rows of 64 requests and
// walks them in order; a request's rank among the row's requests with its digit comes from wave ballots.  `next`: output
// position of the next request of each digit that the thread owns (threadIdx.x * kRadixOwn ...), moved on.
template <bool FULL>
__device__ __forceinline__ void radix_tile(const uint32_t* keys_in, const int32_t* in_in, const int32_t* out_in, uint32_t* keys_out,
                                           int32_t* in_out, int32_t* out_out, int count, int shift, int bits, uint32_t* next, RadixLds& s) {
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
  for (int q = 0; q < kRadixItems; ++q) s.move2[q * kRadixThreads + threadIdx.x] = 0;   // the wave counters
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
  uint32_t total[kRadixOwn], sum = 0;
#pragma unroll
  for (int q = 0; q < kRadixOwn; ++q) {
    total[q] = 0;
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) total[q] += s.wcnt[w][threadIdx.x * kRadixOwn + q];
    sum += total[q];
  }
  uint32_t start = radix_block_scan(sum, s);
#pragma unroll
  for (int q = 0; q < kRadixOwn; ++q) {
    const int d = threadIdx.x * kRadixOwn + q;
    s.to[d] = next[q] - start;
    next[q] += total[q];
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) {
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
    const int i = r * kRadixThreads + threadIdx.x;
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
    const int i = r * kRadixThreads + threadIdx.x;
    if (FULL || i < count) put(out_out + dst[r], (int32_t)s.move[i]);
  }
}

// Stable move of the requests [beg, end).
__device__ __forceinline__ void radix_move(const uint32_t* keys_in, const int32_t* in_in, const int32_t* out_in, uint32_t* keys_out,
                                           int32_t* in_out, int32_t* out_out, int64_t beg, int64_t end, int shift, int bits,
                                           const uint32_t* hist, RadixTeam m, RadixLds& s) {
  const int nbins = 1 << bits;
  uint32_t next[kRadixOwn];                             // output position of the next request of each owned digit
  {
    uint32_t total[kRadixOwn], sum = 0;
#pragma unroll
    for (int q = 0; q < kRadixOwn; ++q) {
      const int d = threadIdx.x * kRadixOwn + q;
      const uint32_t* row = hist + (size_t)d * m.blocks;
      total[q] = d < nbins ? row[m.blocks - 1] : 0u;
      next[q] = d < nbins && m.block > 0 ? row[m.block - 1] : 0u;
      sum += total[q];
    }
    uint32_t base = radix_block_scan(sum, s);
#pragma unroll
    for (int q = 0; q < kRadixOwn; ++q) {
      next[q] += base;
      base += total[q];
    }
  }
  int64_t at = beg;
  for (; at + kRadixTile <= end; at += kRadixTile)
    radix_tile<true>(keys_in + at, in_in + at, out_in + at, keys_out, in_out, out_out, kRadixTile, shift, bits, next, s);
  if (at < end) radix_tile<false>(keys_in + at, in_in + at, out_in + at, keys_out, in_out, out_out, (int)(end - at), shift, bits, next, s);
}

__global__ __launch_bounds__(kRadixThreads) void radix_route_kernel(RadixArgs a) {
  if (!sort_route(a.order)) return;              // the same word for every block: all leave, or none
  __shared__ RadixLds s;
  const RadixTeam m = join_team(a.join, a.members, a.status, s);
  if (m.blocks == 0) return;
  uint32_t passed = 0;                           // barriers behind this block
  auto sync = [&]() {
    ++passed;
    const bool ok = grid_barrier(a.barrier, passed * (uint32_t)m.blocks, &s.flag);
    if (!ok && threadIdx.x == 0) atomicOr(a.status, DYN_WS_SORT_ABANDONED);
    return ok;
  };
  const int n_tile = (int)((a.n + kRadixTile - 1) / kRadixTile);
  const int tiles = n_tile / m.blocks, more = n_tile % m.blocks;   // the first `more` blocks take one tile more
  const int64_t beg = (int64_t)(m.block * tiles + min(m.block, more)) * kRadixTile;
  const int64_t end = std::min<int64_t>(a.n, beg + (int64_t)(tiles + (m.block < more ? 1 : 0)) * kRadixTile);
  const uint32_t* k_src = a.key_a;
  uint32_t* k_dst = a.key_b;
  const int32_t *i_src = a.in_tok, *o_src = a.out_tok;
  for (int p = 0; p < a.passes; ++p) {
    const bool to_final = ((a.passes - 1 - p) % 2) == 0;   // ping-pong so that the last pass lands in the caller's arrays
    int32_t* i_dst = to_final ? a.in_sorted : a.in_tmp;
    int32_t* o_dst = to_final ? a.out_sorted : a.out_tmp;
    const int shift = p * a.bits;
    radix_count(k_src, beg, end, shift, a.bits, a.hist, m, s);
    if (!sync()) return;
    radix_scan(a.hist, a.bits, m);
    if (!sync()) return;
    radix_move(k_src, i_src, o_src, k_dst, i_dst, o_dst, beg, end, shift, a.bits, a.hist, m, s);
    if (!sync()) return;
    i_src = i_dst;
    o_src = o_dst;
    uint32_t* old_src = const_cast<uint32_t*>(k_src);      // both key buffers live in the workspace
    k_src = k_dst;
    k_dst = old_src;
  }
  if (a.n == 0)
    for (int64_t c = threadIdx.x; c <= a.cells; c += kRadixThreads) a.cell_off[c] = 0;
  // the offsets: a block goes over its run of the sorted keys, every key beside the one before it
  for (int64_t at = beg; at < end; at += kRadixTile) {
    uint32_t key[kRadixItems], left[kRadixItems];
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
      const int64_t i = std::min<int64_t>(at + r * kRadixThreads + threadIdx.x, end - 1);
      key[r] = k_src[i];
      left[r] = k_src[i > 0 ? i - 1 : 0];
    }
#pragma unroll 1
    for (int r = 0; r < kRadixItems; ++r) {
      const int64_t i = at + r * kRadixThreads + threadIdx.x;
      uint32_t k = key[0], l = left[0];
#pragma unroll
      for (int q = 1; q < kRadixItems; ++q) {
        k = r == q ? key[q] : k;
        l = r == q ? left[q] : l;
      }
      if (i < end && (k != l || i == 0)) offsets_at(i, i == 0 ? -1 : (int64_t)l, k, a.n, a.cells, a.cell_off);
      if (i == a.n - 1) offsets_at(a.n, k, a.cells, a.n, a.cells, a.cell_off);
    }
  }
}

// ---- a trace in window order ----------------------------------------------------------------
// win_off[w] = number of requests in windows before w, read off the keys (window = key / G)
__global__ __launch_bounds__(256) void window_offsets_kernel(const uint32_t* __restrict__ keys, int64_t n, uint32_t G,
                                                             int32_t n_window, int64_t* __restrict__ win_off) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i > n) return;
  const int64_t prev = i == 0 ? -1 : (int64_t)(keys[i - 1] / G);
  int64_t cur = i == n ? n_window : (int64_t)(keys[i] / G);
  if (cur > n_window) cur = n_window;
  for (int64_t w = prev + 1; w <= cur; ++w) win_off[w] = i;
}

// One block per window: class totals of the window, their exclusive prefix (the window's cell offsets),
// then a stable move tile by tile: every wave owns a contiguous run of rows of a tile and walks them in
// order, a request's position = start of its class + requests of the class in earlier tiles and earlier
// waves' runs + its rank among the lanes of its row with the same class (wave ballots).
__global__ __launch_bounds__(kWaves* DYN_WAVE) void window_sort_kernel(
    const uint32_t* __restrict__ keys, const int32_t* __restrict__ in_in, const int32_t* __restrict__ out_in,
    int32_t* __restrict__ in_out, int32_t* __restrict__ out_out, const int64_t* __restrict__ win_off, int32_t G,
    int32_t n_window, int64_t n, int64_t* __restrict__ cell_off, const uint32_t* __restrict__ order) {
  if (sort_route(order)) return;
  __shared__ uint32_t wcnt[kWaves][DYN_INGEST_MAX_BINS];
  __shared__ uint32_t run[DYN_INGEST_MAX_BINS];          // next output position of every class, relative to the window's start
  const int w = blockIdx.x;
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = threadIdx.x / DYN_WAVE;
  const int64_t beg = win_off[w], end = win_off[w + 1];
  const uint32_t key0 = (uint32_t)w * (uint32_t)G;
  int bits = 0;
  while ((1 << bits) < G) ++bits;
  for (int d = threadIdx.x; d < G; d += blockDim.x) run[d] = 0;
  __syncthreads();
  {                                                      // class totals of the window, four loads per thread in flight
    int64_t i = beg + threadIdx.x;
    for (; i + 3 * (int64_t)blockDim.x < end; i += 4 * (int64_t)blockDim.x) {
      const uint32_t k0 = keys[i], k1 = keys[i + blockDim.x], k2 = keys[i + 2 * blockDim.x], k3 = keys[i + 3 * blockDim.x];
      atomicAdd(&run[k0 - key0], 1u); atomicAdd(&run[k1 - key0], 1u); atomicAdd(&run[k2 - key0], 1u); atomicAdd(&run[k3 - key0], 1u);
    }
    for (; i < end; i += blockDim.x) atomicAdd(&run[keys[i] - key0], 1u);
  }
  __syncthreads();
  if (threadIdx.x == 0) {                                // exclusive prefix over the classes
    uint32_t acc = 0;
    for (int d = 0; d < G; ++d) {
      const uint32_t c = run[d];
      run[d] = acc;
      acc += c;
    }
  }
  __syncthreads();
  for (int d = threadIdx.x; d < G; d += blockDim.x) cell_off[(int64_t)w * G + d] = beg + run[d];
  if (w == n_window - 1 && threadIdx.x == 0) cell_off[(int64_t)n_window * G] = n;

  for (int64_t tile = beg; tile < end; tile += kTile) {
    for (int b = threadIdx.x; b < kWaves * G; b += blockDim.x) wcnt[b / G][b % G] = 0;
    __syncthreads();
    // phase 1: class counts of each wave's run of rows
    const int64_t wbase = tile + (int64_t)wave * (kRows * DYN_WAVE);
    uint32_t cls[kRows];
    int32_t vin[kRows], vout[kRows];                     // the payload, loaded with the keys: not one row at a time later
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const int64_t idx = wbase + r * DYN_WAVE + lane;
      cls[r] = idx < end ? keys[idx] - key0 : 0u;
      vin[r] = idx < end ? in_in[idx] : 0;
      vout[r] = idx < end ? out_in[idx] : 0;
      if (idx < end) atomicAdd(&wcnt[wave][cls[r]], 1u);
    }
    __syncthreads();
    // phase 2: per class, the first output position of each wave's requests
    for (int d = threadIdx.x; d < G; d += blockDim.x) {
      uint32_t pos = run[d];
      for (int q = 0; q < kWaves; ++q) {
        const uint32_t c = wcnt[q][d];
        wcnt[q][d] = pos;
        pos += c;
      }
      run[d] = pos;
    }
    __syncthreads();
    // phase 3: rows in order; inside a row, rank among the lanes with the same class
    uint32_t* my = wcnt[wave];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const int64_t idx = wbase + r * DYN_WAVE + lane;
      const bool valid = idx < end;
      if (__ballot(valid) == 0) break;                   // wave-uniform: nothing left in this run
      const uint32_t d = cls[r];
      uint64_t peers = __ballot(valid);
      for (int b = 0; b < bits; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bal = __ballot(bit);
        peers &= bit ? bal : ~bal;
      }
      const int before = __popcll(peers & ((1ull << lane) - 1ull));
      const int group = __popcll(peers);
      uint32_t pos = 0;
      if (valid) pos = my[d] + (uint32_t)before;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (valid && before == group - 1) my[d] += (uint32_t)group;   // one lane per class advances it
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (valid) {
        in_out[beg + pos] = vin[r];
        out_out[beg + pos] = vout[r];
      }
    }
    __syncthreads();
  }
}

}  // namespace

int64_t dyn_ingest_blocks(int64_t n_req) { return n_req > 0 ? (n_req + kTile - 1) / kTile : 1; }

hipError_t dyn_launch_edges(const int32_t* in_edge, size_t n_in, const int32_t* out_edge, size_t n_out, int32_t* d_in,
                            int32_t* d_out, WsHeader* header, uint32_t order_word, hipStream_t s) {
  EdgePack p;
  if (n_in + n_out <= DYN_EDGE_PACK) {          // the usual case: header and both lists in one launch
    if (n_in) memcpy(p.v, in_edge, n_in * sizeof(int32_t));
    if (n_out) memcpy(p.v + n_in, out_edge, n_out * sizeof(int32_t));
    hipLaunchKernelGGL(edge_store_kernel, dim3(1), dim3(256), 0, s, p, (int)n_in, d_in, (int)n_out, d_out, header, order_word);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(edge_store_kernel, dim3(1), dim3(64), 0, s, p, 0, d_in, 0, d_out, header, order_word);
  const struct { const int32_t* src; size_t n; int32_t* dst; } parts[2] = {{in_edge, n_in, d_in}, {out_edge, n_out, d_out}};
  for (const auto& part : parts)
    for (size_t at = 0; at < part.n; at += DYN_EDGE_PACK) {
      const int n = (int)std::min<size_t>(DYN_EDGE_PACK, part.n - at);
      memcpy(p.v, part.src + at, (size_t)n * sizeof(int32_t));
      hipLaunchKernelGGL(edge_store_kernel, dim3(1), dim3(256), 0, s, p, n, part.dst + at, 0, part.dst, (WsHeader*)nullptr, 0u);
    }
  return hipGetLastError();
}

hipError_t dyn_launch_ingest(const IngestArgs& a, hipStream_t s) {
  const int64_t n = a.n_req;
  const int32_t G = a.n_model * a.n_in_bin * a.n_out_bin;
  const int64_t cells = (int64_t)a.n_window * G;
  hipError_t e;
  // Keys, and whether the trace is in window order already: the key kernel ORs into the flag word, which the header
  // kernel before it set to 0, or to 1 when the general sort is forced (more classes than the window route counts).
  if (n > 0) {
    const size_t edge_bytes = (size_t)a.n_model * ((a.n_in_bin - 1) + (a.n_out_bin - 1)) * sizeof(int32_t);
    const int lds_edges = edge_bytes <= 32 * 1024 ? 1 : 0;
    hipLaunchKernelGGL(key_kernel, dim3((unsigned)((n + kKeyRows * 256 - 1) / (kKeyRows * 256))), dim3(256), lds_edges ? edge_bytes : 0, s, a,
                       1.0 / a.window_s, lds_edges);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  } else {
    hipLaunchKernelGGL(window_offsets_kernel, dim3(1), dim3(256), 0, s, a.key_a, n, (uint32_t)G, a.n_window, a.win_off);
  }
  if (!a.force_sort) {        // in window order: one block per window moves its requests to their cells
    hipLaunchKernelGGL(window_sort_kernel, dim3((unsigned)a.n_window), dim3(kWaves * DYN_WAVE), 0, s, a.key_a, a.in_tok,
                       a.out_tok, a.in_sorted, a.out_sorted, a.win_off, G, a.n_window, n, a.cell_off, a.unsorted);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (n == 0) return hipSuccess;   // nothing to sort: the flag word stays 0
  }
  const int passes = a.key_bits <= 0 ? 1 : (a.key_bits + 9) / 10;
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
  r.order = a.unsorted; r.barrier = a.unsorted + (DYN_WS_HEADER_BARRIER_WORD - DYN_WS_HEADER_ORDER_WORD); r.status = a.status;
  r.join = r.barrier + 1; r.members = r.barrier + 2;
  r.key_a = a.key_a; r.key_b = a.key_b; r.in_tok = a.in_tok; r.out_tok = a.out_tok;
  r.in_sorted = a.in_sorted; r.out_sorted = a.out_sorted; r.in_tmp = a.in_tmp; r.out_tmp = a.out_tmp;
  r.hist = a.block_hist; r.n = n; r.cells = cells; r.cell_off = a.cell_off;
  r.passes = passes; r.bits = bits;
  // a block for every tile, as far as they fit the device and the digit counts (a word per digit and block) the workspace
  const int64_t room = ((int64_t)DYN_INGEST_MAX_BINS * a.n_block) >> bits;
  const int64_t n_tile = (n + kRadixTile - 1) / kRadixTile;
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>({(int64_t)n_cu, n_tile, room}));
  hipLaunchKernelGGL(radix_route_kernel, dim3((unsigned)blocks), dim3(kRadixThreads), 0, s, r);
  return hipGetLastError();
}
