// Tick-level load inside a window: every window is split into n_tick ticks (sub-windows of
// the sorted trace), each request is served under the load of its own tick (the instance
// manager re-tunes the frequency every few seconds under the current load, Section IV-B
// "Scale-up/down").  Per (window, class) cell and candidate configuration the profile is
// looked up once per tick; the window's energy is the sum over its ticks.
//
// The per-request percentile still collapses, tick by tick: inside one tick TTFT is
// input length x a non-negative constant, so the cell's j-th largest TTFT (j = m - rank + 1)
// is among the j largest input lengths of each tick scaled by that tick's prefill time.
// The request stream is read once, independent of the configurations:
//   tick_tight_kernel, tick_tight_block_kernel  the cells whose percentile is settled without lists (below), and the lists
//                      of long cells and of few ones;
//   long_count, long_rank   cells of more than 4096 requests, a block for every piece of a tick (at the head of tick_cell_kernel
//                      and of tick_deep_kernel, so that a trace without such cells pays for no launch)
//   tick_cell_kernel   of the cells left, per cell every tick's load, its min(j, count) largest input lengths in
//                      descending order (j <= 64: kept sorted in a wave's lanes) and the cell's
//                      j-th largest input length x_j; what the later kernels do with the cell;
//   tick_deep_kernel   the same lists and x_j for the cells with j > 64 (a block per cell:
//                      bitonic sort of a tick in LDS); beyond j = 8192 the lists are whole ticks, and a
//                      tick of more than 8192 requests is then sorted in pieces of 8192 (marked: the
//                      general kernel searches every piece);
//   tick_space_kernel  the cells with j <= 16: per (cell, configuration) a walk over the ticks, energy in time
//                      order, the TBT percentile (largest tick TBT when every non-empty tick holds j
//                      requests, else from the four largest tick TBTs), the TTFT percentile through a
//                      sorted register list of the scaled candidates;
//   tick_general_kernel every other cell, (cell, tile) by (cell, tile): the ticks' prefill times (TBTs)
//                      kept in an LDS strip, the TBT percentile by taking ticks in descending TBT
//                      order, the TTFT percentile from the bracket [x_j * least, x_j * largest prefill
//                      time of the ticks]: a single value, or settled by ranking the ticks that hold
//                      lengths equal to x_j, or bisected on the ticks' sorted lists.
#include <algorithm>
#include <type_traits>

#include "dyn_ticks.h"
#include "dyn_device.h"

namespace {

constexpr int kWavesPerBlock = 4;
constexpr int kFastDepth = DYN_TICK_FAST;
constexpr int kDeepCap = DYN_TICK_DEPTH;     // largest j, and the largest tick the deep-cell kernel sorts in one go
constexpr int kDeepBlocks = 512;
constexpr int kListBlocks = 2048;            // of the cell kernel: eight to a compute unit; with a wave for every cell of a day the empty ones took 10 us
constexpr int kGeneralBlocks = 1024;          // grid of the general kernel when the device cannot be asked what fits
constexpr int kListCap = 2048;               // list entries of one cell the general kernel stages in LDS
constexpr int kStripBytes = 32 * 1024;       // per-tick values of a block's configurations in the general kernel
static_assert(kDeepCap == 8192, "the deep-cell kernel's LDS buffer");
// LDS stride of a staged table row in doubles: odd, so that lanes reading the same load bracket of
// different rows do not all fall into one bank
#define DYN_SLOT_STRIDE(n_rho) ((3 * (n_rho)) | 1)

__global__ void tick_init_kernel(uint32_t* counters) {
  counters[0] = 0u;
  counters[1] = 0u;
  counters[2] = 0u;
  counters[3] = 0u;
  counters[4] = 0u;
  counters[5] = 0u;
}

// How the TBT percentile of a cell can be found (lane q holds tick q's request count, 0 beyond the ticks): from the
// largest tick TBT when every non-empty tick holds j requests (DENSE); from the four largest tick TBTs when any four
// non-empty ticks hold j between them: the four smallest counts do, or there are no more than four (SMALL).
__device__ __forceinline__ uint32_t tbt_route(int32_t cnt_l, int64_t j64, int lane) {
  uint32_t flags = 0;
  uint32_t cpos = cnt_l > 0 ? (uint32_t)cnt_l : 0xFFFFFFFFu;
  if ((int64_t)wave_min_u32(cpos) >= j64) flags |= DYN_TP_DENSE;
  int64_t s4 = 0;
  bool all_in = false;
  for (int r = 0; r < 4; ++r) {
    const uint32_t mn = wave_min_u32(cpos);
    if (mn == 0xFFFFFFFFu) { all_in = true; break; }
    s4 += mn;
    const uint64_t who = __ballot(cpos == mn);
    if (lane == (int)__builtin_ctzll(who)) cpos = 0xFFFFFFFFu;
  }
  if (all_in || s4 >= j64) flags |= DYN_TP_SMALL;
  return flags;
}

// The walk kernel keeps a register list of 16 candidates beside the largest tick TBT, of 8 beside the four largest.
__device__ __forceinline__ bool walks_with_lists(uint32_t flags, int64_t j64) {
  return ((flags & DYN_TP_DENSE) && j64 <= kFastDepth) || ((flags & DYN_TP_SMALL) && j64 <= kFastDepth / 2);
}

// ---- cells settled by their ties at x_j ----------------------------------------------------------
// With theta_g = the least ratio (smallest / largest prefill time of a table row) over the rows of class g, every
// configuration of the class has per-tick prefill times within a factor theta_g of each other.  If theta_g * (x_j + 1) > x_j
// (flat prefill tables: always), a request longer than x_j has a larger TTFT than any request of length x_j, whatever
// their ticks, and a shorter one a smaller TTFT: the cell's j-th largest TTFT belongs to a request of length x_j, and
// it is x_j times the prefill time that ranks (j - number of longer requests) from the top among the ticks, each tick
// counted as often as it holds requests of length x_j.  All the evaluation needs of such a cell is x_j, that rank and
// the per-tick counts.  A wave takes a cell whose ticks fit its registers (rows of 64 requests, the same number of
// rows for every tick, two 16-bit lengths to a register), finds x_j by the bit-wise search of the window-level
// aggregation and counts.  The evaluation keeps four ticks: the rank must be within their reach from the top or from
// the bottom (tight_place), else the cell is ranked over all ticks by the general kernel, like a cell whose TBT
// percentile needs all ticks.  Cells it cannot take (the bound does not hold, ticks too uneven for the registers,
// token counts of 2^16 or more) are listed for the kernel that builds per-tick lists.
struct TightCell {
  uint32_t tok_l;     // lane q: token sum of tick q
  uint32_t eq_l;      // lane q: requests of length x_j in tick q
  uint32_t xj, place; // place: the rank among the ticks, from the top, or from the bottom with DYN_TIGHT_FROM_BELOW set
  uint32_t need;      // the rank from the top
  bool walk;          // the rank is within reach of the walk's four ticks from one end
};
enum Settled { kNotTaken, kSettled, kBoundFails, kListed };   // kBoundFails: token sums and x_j are known, the ticks' lists are needed; kListed: those are written too
constexpr int kListedDepth = 4;                // largest j whose lists tight_cell takes out of its registers
constexpr int kListedRegs = 16;                // and how many of those at most: more would spill

// The bound of a cell: of its class, except that a cell whose requests are all of one tick has one prefill time.
__device__ __forceinline__ float cell_theta(float theta, int32_t cnt_l) { return __popcll(__ballot(cnt_l > 0)) <= 1 ? 1.0f : theta; }
#define DYN_TIGHT_FROM_BELOW 0x80000000u

// The up to four smallest positive per-tick counts of a wave (e_l: lane q holds tick q's count, 0 elsewhere), ascending,
// 0xFFFFFFFF where there are fewer; returns the number of positive counts.  Wave-uniform results.
__device__ __forceinline__ int smallest_four(uint32_t e_l, int lane, uint32_t (&m4)[4]) {
  const int npos = __popcll(__ballot(e_l > 0u));
  uint32_t cur = e_l > 0u ? e_l : 0xFFFFFFFFu;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    m4[i] = wave_min_u32(cur);
    const uint64_t at = __ballot(cur == m4[i] && cur != 0xFFFFFFFFu);
    if (at != 0 && lane == __builtin_ctzll(at)) cur = 0xFFFFFFFFu;   // one lane leaves per round
  }
  return npos;
}

// Where the walk finds the rank `need` (1 .. n_eq) among the ticks weighted by their counts of lengths equal to x_j,
// with its list of four ticks: from the top if the four ticks of largest prefill time are sure to weigh `need`
// together (need <= 4, or at most four ticks have such lengths, or the four smallest positive counts add up to it),
// else from the bottom by the same test on n_eq - need + 1, else not at all (returns false; `place` = need).
__device__ __forceinline__ bool tight_place(int need, int n_eq, int npos, uint32_t s4, uint32_t* place) {
  const int below = n_eq - need + 1;
  *place = (uint32_t)need;
  if (need <= 4 || npos <= 4 || (uint32_t)need <= s4) return true;
  if (below <= 4 || (uint32_t)below <= s4) {
    *place = (uint32_t)below | DYN_TIGHT_FROM_BELOW;
    return true;
  }
  return false;
}

template <int P, bool LISTS>   // P registers = 2P rows; LISTS: cells with short lists are listed here
__device__ __forceinline__ Settled tight_cell(const int32_t* __restrict__ in, const int32_t* __restrict__ out, int64_t beg_l,
                                              int32_t cnt_l, int T, int rpt, int m, int rank, float theta, int lane,
                                              int32_t* __restrict__ list, TightCell* res) {
  uint32_t v[P];
  uint32_t orv = 0, lmax = 0, lmax2 = 0, tok_acc = 0, tok_l = 0;
  constexpr int CH = P < 4 ? P : 4;      // registers per round: up to 8 + 8 loads in flight
  int q = 0, r = 0;                      // tick and row of the slot being filled (wave-uniform)
#pragma unroll
  for (int p0 = 0; p0 < P; p0 += CH) {
    uint32_t a[2 * CH], b[2 * CH];
    int qs[2 * CH], rs[2 * CH];
#pragma unroll
    for (int u = 0; u < 2 * CH; ++u) {
      qs[u] = q; rs[u] = r;
      // lane reads without a branch around them: beyond the last tick the lane index is clamped and the count zeroed
      const int qc = q < DYN_WAVE - 1 ? q : DYN_WAVE - 1;
      const int64_t beg_q = readlane_i64(beg_l, qc);
      const int cnt_q = __builtin_amdgcn_readlane(cnt_l, qc);
      const int left = (q < T ? cnt_q : 0) - r * DYN_WAVE;
      const bool ok = lane < left;
      // the padding of a slot without a request goes into its half of the register now; the length is ORed in below
      // (a lane without a request loads 0), so no mask has to live across the loads
      if (u % 2 == 0) v[p0 + u / 2] = ok ? 0u : 0xFFFFu;
      else v[p0 + u / 2] |= ok ? 0u : 0xFFFF0000u;
      const int64_t row_q = beg_q + (int64_t)(r * DYN_WAVE);   // one scalar offset for both arrays
      a[u] = ok ? (uint32_t)in[row_q + lane] : 0u;
      b[u] = ok ? (uint32_t)out[row_q + lane] : 0u;
      if (++r == rpt) { r = 0; ++q; }
    }
#pragma unroll
    for (int u = 0; u < 2 * CH; ++u) {
      tok_acc += a[u] + b[u];
      orv |= a[u] | b[u];
      if (u % 2 == 0) lmax = max(lmax, a[u]); else lmax2 = max(lmax2, a[u]);
      if (rs[u] == rpt - 1) {            // the tick's last row: its token sum goes to lane q (below 2^30 when the cell qualifies)
        const uint32_t tok = wave_sum_u32(tok_acc);
        if (lane == qs[u]) tok_l = tok;
        tok_acc = 0;
      }
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      v[p0 + u] |= (a[2 * u] & 0xFFFFu) | (a[2 * u + 1] << 16);   // lengths of 2^16 and more: the cell is given up below
    }
    // keep the rounds apart: with all loads hoisted to the top 4P loaded values would be live at once
    if (CH == 4)
      asm volatile("" : "+v"(tok_acc), "+v"(tok_l), "+v"(orv), "+v"(lmax), "+v"(lmax2), "+v"(v[p0]), "+v"(v[p0 + 1]),
                   "+v"(v[p0 + 2]), "+v"(v[p0 + 3])::"memory");
  }
  orv = wave_or_u32(orv);
  if (orv >= (1u << 16)) return kNotTaken;   // wave-uniform
  const uint32_t top = wave_max_u32(max(lmax, lmax2));
  if (top == 0xFFFFu) return kNotTaken;  // the padding value itself; the search's candidates (up to top + 1) must fit 16 bits
  uint32_t xj = top;
  const int j = m - rank + 1;
  if (rank != m) {
    uint32_t lo = 0;
    if (j <= 2 * DYN_WAVE) {
      const int nb = 32 - __builtin_clz(top | 1u);
      for (int b = nb - 1; b >= 0; --b) {   // largest c with #{the 128 half-lane maxima >= c} >= j (all elements of the cell)
        const uint32_t cand = lo | (1u << b);
        if (__popcll(__ballot(lmax >= cand)) + __popcll(__ballot(lmax2 >= cand)) >= j) lo = cand;
      }
    }
    uint32_t d = 0;
    const int nb = 32 - __builtin_clz((top - lo) | 1u);
    for (int b = nb - 1; b >= 0; --b) {
      const uint32_t cand = lo + (d | (1u << b));
      const uint16_t cand_lo = (uint16_t)cand;   // low half by a 16-bit compare; high half: hi < cand exactly when the
      const uint32_t cand_hi = cand << 16;       // whole register < cand << 16
      int below = 0;
#pragma unroll
      for (int i = 0; i < P; ++i)
        below += __popcll(__ballot((uint16_t)v[i] < cand_lo)) + __popcll(__ballot(v[i] < cand_hi));
      if (below < rank) d |= 1u << b;
    }
    xj = lo + d;
  }
  // the bound: theta * (x_j + 1) > x_j, with theta below the true ratio by 2^-21 at least (so that no rounding of the
  // scaled lengths can turn the order around)
  res->tok_l = tok_l;
  res->xj = xj;
  if (!((double)theta * ((double)xj + 1.0) > (double)xj)) {
    if (!LISTS || P > kListedRegs || j > kListedDepth) return kBoundFails;
    // The lists of a cell with few places in them, from the registers: a lane keeps the largest lengths of its tick in
    // order, and at the tick's end the wave takes the largest of all lanes j times.  As a launch of their own these lists cost
    // as much as this kernel, which had read the same requests (11 000 cells of 9 and 24 requests: 107 and 122 us).
    if constexpr (LISTS && P <= kListedRegs) {
    int32_t best[kListedDepth], take[kListedDepth];
#pragma unroll
    for (int p = 0; p < kListedDepth; ++p) { best[p] = -1; take[p] = -1; }
    q = 0; r = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        int32_t x = (int32_t)(h ? v[i] >> 16 : v[i] & 0xFFFFu);
        x = x == 0xFFFF ? -1 : x;        // padding
        if (j == 1) best[0] = max(best[0], x);   // wave-uniform
        else {
#pragma unroll
          for (int p = 0; p < kListedDepth; ++p) {
            const int32_t hi = max(best[p], x);
            x = min(best[p], x);
            best[p] = hi;
          }
        }
        if (++r == rpt) {
#pragma unroll
          for (int p = 0; p < kListedDepth; ++p) {
            if (p < j && q < T) {        // wave-uniform
              const int32_t mx = wave_max_i32(best[0]);
              if (lane == q) take[p] = mx;
              if (j > 1) {
                const uint64_t who = __ballot(best[0] == mx);
                if (lane == __builtin_ctzll(who)) {
#pragma unroll
                  for (int u = 0; u + 1 < kListedDepth; ++u) best[u] = best[u + 1];
                  best[kListedDepth - 1] = -1;
                }
              }
            }
          }
#pragma unroll
          for (int p = 0; p < kListedDepth; ++p) best[p] = -1;
          r = 0; ++q;
        }
      }
    }
#pragma unroll
    for (int p = 0; p < kListedDepth; ++p)
      if (p < j && p < cnt_l) list[beg_l + p] = take[p];
    }
    return kListed;
  }
  // longer requests, and per tick the requests of length x_j.  The padding (0xFFFF in every slot beyond a tick's
  // requests) counts as longer: it is taken off afterwards.
  int n_gt = -(2 * P * DYN_WAVE - m), n_eq = 0, eq_acc = 0;
  uint32_t eq_l = 0;
  q = 0; r = 0;
  const uint32_t xj_hi = xj << 16;
#pragma unroll
  for (int i = 0; i < P; ++i) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // low half by 16-bit compares; high half on the whole register (hi > x_j exactly when v >= (x_j + 1) << 16)
      n_gt += h ? __popcll(__ballot(v[i] >= xj_hi + 0x10000u)) : __popcll(__ballot((uint16_t)v[i] > (uint16_t)xj));
      eq_acc += h ? __popcll(__ballot((v[i] >> 16) == xj)) : __popcll(__ballot((uint16_t)v[i] == (uint16_t)xj));
      if (++r == rpt) {
        if (lane == q) eq_l = (uint32_t)eq_acc;
        n_eq += eq_acc;
        eq_acc = 0;
        r = 0; ++q;
      }
    }
  }
  const int need = j - n_gt;             // 1 .. n_eq
  uint32_t place = (uint32_t)need;       // out of the list's reach from both ends: for the general kernel, from the top
  res->walk = true;
  if (need > 4 && n_eq - need + 1 > 4) {
    uint32_t m4[4];
    const int npos = smallest_four(eq_l, lane, m4);
    const uint32_t s4 = npos >= 4 ? m4[0] + m4[1] + m4[2] + m4[3] : 0u;   // counts stay below 2^24
    res->walk = tight_place(need, n_eq, npos, s4, &place);
  } else if (need > 4) {
    place = (uint32_t)(n_eq - need + 1) | DYN_TIGHT_FROM_BELOW;
  }
  res->need = (uint32_t)need;
  res->eq_l = eq_l;
  res->place = place;
  return kSettled;
}

// A long cell goes to the blocks that share it without being read first where its bound fails for any x_j of 50 or more, or where a
// wave of its block would hold more than 64 rows.  Measured (us of the call; a block per cell, shared): 60 cells of 65 000 requests and
// 12 ticks 140, 117; 288 of 13 900 and 30 ticks 254, 209; 12 of 4700 and 30 ticks (at most 24 rows) 96, 117.
constexpr int kLongRows = 64;
__device__ __forceinline__ bool long_at_once(const TickCellArgs& a, int64_t m, int g, int32_t cnt_l, int rows) {
  if (!a.sure || m <= DYN_TICK_LONG) return false;   // most cells, before the class's bound is there
  return rows > kLongRows || (m >= a.table_from && cell_theta(a.theta[g], cnt_l) < 0.98f);
}

// An entry of list_cells: the cell, with DYN_LIST_SKIP set for one that the block kernel leaves to tick_cell_kernel unseen (fewer than 2^30 cells).
#define DYN_LIST_DONE 0xFFFFFFFFu
#define DYN_LIST_SKIP 0x80000000u

// LISTS: for profiles whose prefill times depend on the load; the other form is smaller (ticks of a day 79 against 87 us, 8000 cells of
// 11 requests 8.8 against 12.7).
template <bool LISTS>
__global__ __launch_bounds__(kWavesPerBlock* DYN_WAVE) __attribute__((amdgpu_waves_per_eu(6, 8))) void tick_tight_kernel(TickCellArgs a) {
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE);
  const int T = a.n_tick, G = a.G;
  const int64_t cells = (int64_t)a.n_window * G;
  const int64_t c = (int64_t)blockIdx.x * kWavesPerBlock + wave;
  if (c >= cells) return;
  if (c == 0 && lane == 0) {                     // single writer of the header
    a.header->status = 0u;
    a.header->kind = DYN_WS_KIND_CELLS;
    a.header->cells = cells * T;
  }
  const int64_t w = c / G;
  const int g = (int)(c % G);
  const int64_t f0 = (w * T) * G + g;           // fine cell of tick 0; tick q is q*G further
  int64_t beg_l = 0;
  int32_t cnt_l = 0;
  uint32_t bad_l = 0;
  if (lane < T) {
    const int64_t f = f0 + (int64_t)lane * G;
    const int64_t b = a.fine_off[f], e = a.fine_off[f + 1];
    if (b < 0 || e < b || e > a.n_req) bad_l = DYN_WS_BAD_OFFSETS;   // such a tick is treated as empty
    else { beg_l = b; cnt_l = (int32_t)(e - b); }
  }
  const int64_t m_cell = (int64_t)wave_sum_u64((uint64_t)(uint32_t)cnt_l);
  const int64_t rank = (a.pct_num * m_cell + a.pct_den - 1) / a.pct_den;
  const int64_t j64 = m_cell > 0 ? m_cell - rank + 1 : 0;
  TightCell tc;
  tc.tok_l = 0; tc.eq_l = 0; tc.xj = 0; tc.place = 0; tc.need = 0; tc.walk = true;
  uint32_t flags = 0;
  Settled done = m_cell == 0 ? kSettled : kNotTaken;   // an empty cell: loads 0, nothing else
  if (m_cell > 0) {
    flags = tbt_route(cnt_l, j64, lane);
    const int rpt = ((int)wave_max_u32((uint32_t)cnt_l) + DYN_WAVE - 1) / DYN_WAVE;   // rows per tick
    const int rows = T * rpt;
    // with few cells on the whole device a cell of many rows is quicker with a block's waves: it goes on the list
    if (rows <= 128 && !(a.few_cells && rows > 8) && !long_at_once(a, m_cell, g, cnt_l, 0)) {
      const float theta = cell_theta(a.theta[g], cnt_l);
      const int m = (int)m_cell, rk = (int)rank;
      if (rows <= 4) done = tight_cell<2, LISTS>(a.in, a.out, beg_l, cnt_l, T, rpt, m, rk, theta, lane, a.top, &tc);
      else if (rows <= 8) done = tight_cell<4, LISTS>(a.in, a.out, beg_l, cnt_l, T, rpt, m, rk, theta, lane, a.top, &tc);
      else if (rows <= 16) done = tight_cell<8, LISTS>(a.in, a.out, beg_l, cnt_l, T, rpt, m, rk, theta, lane, a.top, &tc);
      else if (rows <= 32) done = tight_cell<16, LISTS>(a.in, a.out, beg_l, cnt_l, T, rpt, m, rk, theta, lane, a.top, &tc);
      else if (rows <= 64) done = tight_cell<32, LISTS>(a.in, a.out, beg_l, cnt_l, T, rpt, m, rk, theta, lane, a.top, &tc);
      else done = tight_cell<64, LISTS>(a.in, a.out, beg_l, cnt_l, T, rpt, m, rk, theta, lane, a.top, &tc);
      if (done == kListed) {                     // j <= 4: any four non-empty ticks hold as many requests, so the walk takes it
        tc.eq_l = (uint32_t)beg_l;               // where the tick's list is (n_req < 2^31)
        if (lane == 0) atomicAdd(&a.counters[3], 1u);
      }
      if (done == kSettled) {
        flags |= DYN_TP_TIGHT;
        // the walk keeps four ticks and finds the TBT percentile from the largest tick TBT or the four largest
        if (!tc.walk || !(flags & (DYN_TP_DENSE | DYN_TP_SMALL))) {
          flags |= DYN_TP_GENERAL;
          tc.place = tc.need;
        }
      }
    }
  }
  if (done != kSettled && done != kListed) {     // the kernel that builds per-tick lists writes everything about this cell
    const bool skip = done == kBoundFails && !a.few_cells && j64 <= DYN_TICK_WAVE;   // the next kernel would find out the same and leave it
    if (lane == 0) a.list_cells[atomicAdd(&a.counters[2], 1u)] = (uint32_t)c | (skip ? DYN_LIST_SKIP : 0u);
    return;
  }
  if (lane < T) {
    TickRec r;
    r.load = div_by((double)tc.tok_l, a.tick_s, a.r_tick);
    r.off = tc.eq_l;                             // no list: the tick's requests of length x_j
    r.cnt = cnt_l;
    a.rec[c * T + lane] = r;
    a.cstat[f0 + (int64_t)lane * G] = (uint8_t)bad_l;   // every fine cell writes its own status byte
  }
  if (lane == 0) {
    TickPlan p;
    p.j = (int32_t)j64;
    p.xj = (int32_t)tc.xj;
    p.flags = flags;
    p.place = tc.place;
    a.plan[c] = p;
    if (flags & DYN_TP_GENERAL) a.slow_list[atomicAdd(&a.counters[1], 1u)] = (uint32_t)c;
  }
}

// ---- long cells: many blocks share a cell --------------------------------------------------------
// A block streams a cell at about 16 GB/s, and sorts a tick's lengths in hundreds of barriers; few cells of many requests left the
// device idle for milliseconds.  Here a cell's ticks are cut into pieces, a block each, and nothing is sorted:
//   long_count  token sums per tick, and the cell's lengths counted by exponent and six bits (coarse_bin).  The cell's last block
//               finds the bin that holds x_j, how far apart the prefill times of its ticks lie under any configuration (theta, from
//               the least and the largest tick load), and so which lengths can decide: those of the bin where
//               theta * (x + 1) > x (as above, the ties at x_j settle the cell), else those from theta * bin to bin / theta and no longer than the
//               cell's longest (540 cells of 12 ticks, an hour's load, 246 us without that, 238 with it; 63 of 14 ticks and 4200 requests, whose
//               tables to bin / theta were too wide, so that one block made the lists, 859, 223);
//   long_rank   every such length counted per tick.  The cell's last block turns the counts into "how many are at least so
//               long", reads x_j off them, and the ties or the tables are the general kernel's and the walk's.
// Cells it cannot take (lengths of 2^16 and more at the rank, negative token counts, a theta that leaves more than kLongRange lengths, no
// room in the pool: 4 M words, sixteen cells of 64 ticks at the widest) go to the lists as before; which of many get room is the order of an atomic.  Bound: two reads of the lengths and the two launches.
constexpr int kLongBlocks = 1024;              // at most: four to a compute unit
constexpr int64_t kLongPiece = 4096;           // requests of a piece, about
constexpr int kLongRange = 4096;               // lengths of a table
// words of a slot: the coarse counts, per tick the token sum (64 bits) and the OR of the token counts, then
constexpr int kSlotSum = kCoarseBins, kSlotOr = kSlotSum + 2 * DYN_TICK_MAX, kSlotCell = kSlotOr + DYN_TICK_MAX, kSlotDone = kSlotCell + 1,
              kSlotDone2 = kSlotCell + 2, kSlotFrom = kSlotCell + 3, kSlotN = kSlotCell + 4, kSlotLow = kSlotCell + 5, kSlotBits = kSlotCell + 6,
              kSlotTheta = kSlotCell + 7, kSlotPool = kSlotCell + 8;   // kSlotN: lengths counted, 0: the cell went to the lists
static_assert(kSlotPool < DYN_TICK_SLOT_WORDS && kSlotSum % 2 == 0 && kSlotCell % 4 == 0, "the slot");
constexpr int kLongPer = (kCoarseBins + 255) / 256;
constexpr int kLongWords = kLongPer * 256 + 64;   // LDS of long_count
static_assert(kLongWords >= kWavesPerBlock * DYN_WAVE && kLongRange + 1 + 520 + 64 <= kDeepCap, "LDS");
static_assert(kWavesPerBlock * DYN_WAVE == 256, "blocks of 256 threads");

// Pieces of a tick, so that the cells' pieces keep the device busy and are not too small.
__device__ __forceinline__ int long_split(const TickCellArgs& a, int n_long) {
  const int64_t units = (int64_t)n_long * a.n_tick;
  const int64_t want = a.n_req / (units * kLongPiece) + 1, most = 2 * kLongBlocks / units;
  return (int)max((int64_t)1, min(want, most));
}
__host__ __device__ __forceinline__ int long_blocks(const TickCellArgs& a) {   // no more than there can be pieces
  const int64_t most = a.n_req / kLongPiece + (int64_t)a.n_slot * a.n_tick;
  return a.n_slot > 0 ? (int)(most < kLongBlocks ? most : kLongBlocks) : 0;
}
struct LongUnit {
  int slot, q;
  int64_t c, beg;    // the cell; first request of the piece
  int n;             // its requests
};
__device__ __forceinline__ LongUnit long_unit(const TickCellArgs& a, uint32_t unit, int split) {
  LongUnit u;
  const uint32_t per = (uint32_t)(a.n_tick * split);
  u.slot = (int)(unit / per);
  const uint32_t in_cell = unit - (uint32_t)u.slot * per, s = in_cell % (uint32_t)split;
  u.q = (int)(in_cell / (uint32_t)split);
  u.c = a.slots[(size_t)u.slot * DYN_TICK_SLOT_WORDS + kSlotCell];
  const int64_t f = ((u.c / a.G) * a.n_tick + u.q) * a.G + u.c % a.G;
  const int64_t b = a.fine_off[f], e = a.fine_off[f + 1];
  const int64_t cnt = (b < 0 || e < b || e > a.n_req) ? 0 : e - b;   // such a tick is treated as empty
  u.beg = b + cnt * s / split;
  u.n = (int)(cnt * (s + 1) / split - cnt * s / split);
  return u;
}
__device__ __forceinline__ uint32_t seen(const uint32_t* at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Adds at the device's coherence point; the old value comes back, so a block that has waited for it knows that the sum is there.
__device__ __forceinline__ uint32_t add_seen(uint32_t* at, uint32_t v) { return __hip_atomic_fetch_add(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// A cell's ticks in a wave's lanes, as in the kernels above.
struct CellTicks {
  int64_t beg_l, m, j, rank;
  int32_t cnt_l;
  uint32_t bad_l;
};
__device__ __forceinline__ CellTicks cell_ticks(const TickCellArgs& a, int64_t c, int lane) {
  CellTicks t;
  t.beg_l = 0; t.cnt_l = 0; t.bad_l = 0;
  if (lane < a.n_tick) {
    const int64_t f = ((c / a.G) * a.n_tick + lane) * a.G + c % a.G;
    const int64_t b = a.fine_off[f], e = a.fine_off[f + 1];
    if (b < 0 || e < b || e > a.n_req) t.bad_l = DYN_WS_BAD_OFFSETS;
    else { t.beg_l = b; t.cnt_l = (int32_t)(e - b); }
  }
  t.m = (int64_t)wave_sum_u64((uint64_t)(uint32_t)t.cnt_l);
  t.rank = (a.pct_num * t.m + a.pct_den - 1) / a.pct_den;
  t.j = t.m > 0 ? t.m - t.rank + 1 : 0;
  return t;
}

// This thread's part of: the least ratio (smallest / largest) of a configuration's prefill times at loads from lmin to lmax.  A row is
// linear between its load points, so its extremes are at the ends or at the points between them.
__device__ __forceinline__ float theta_between(const TickCellArgs& a, int g, double lmin, double lmax) {
  const double* rg = a.gridpack + 1;             // the load points
  const double top = rg[a.n_rho - 1];
  const int R = a.n_rho;
  float theta = 1.0f;
#pragma unroll 1
  for (int k = threadIdx.x; k < a.K; k += 256) {
    const DevCfg cf = a.cfg[k];
    const size_t row = (size_t)g * a.n_tp_f;
    const bool two = cf.u != 0.0;
    const double ml = two ? (1.0 - cf.u) * a.ml[row + cf.row_lo] + cf.u * a.ml[row + cf.row_hi] : a.ml[row + cf.row_lo];
    const double *lo = a.tab + (row + cf.row_lo) * 3 * R, *hi = a.tab + (row + cf.row_hi) * 3 * R;
    auto point = [&](int i) { return two ? (1.0 - cf.u) * lo[3 * i] + cf.u * hi[3 * i] : lo[3 * i]; };
    const double den = cf.nd * ml;
    double mn = __builtin_inf(), mx = -__builtin_inf();
    int from = 0;
#pragma unroll 1
    for (int e = 0; e < 2; ++e) {                // the lower end, the upper end and the points between them
      const double rho = fmin((e ? lmax : lmin) / den, top);
      int jj = a.jstart[(int)(fmax(rho, 0.0) * a.bucket_scale)];
      while (jj > 0 && rg[jj] > rho) --jj;
      while (jj < R - 2 && rg[jj + 1] <= rho) ++jj;
      const double t = (rho - rg[jj]) / (rg[jj + 1] - rg[jj]);
      double v = (1.0 - t) * point(jj) + t * point(jj + 1);
      mn = fmin(mn, v);
      mx = fmax(mx, v);
#pragma unroll 1
      for (int i = e ? from + 1 : jj + 1; i <= jj; ++i) {
        v = point(i);
        mn = fmin(mn, v);
        mx = fmax(mx, v);
      }
      from = jj;
    }
    theta = fminf(theta, (mx > 0.0 && mn > 0.0) ? (float)(mn / mx) * 0.999999f : 0.0f);   // below mn / mx by 2^-21 at least
  }
  return theta;
}

// First pass, and what the cell's last block decides.  `s`: kLongWords words of LDS.
__device__ __forceinline__ void long_count(const TickCellArgs& a, int n_share, uint32_t* s) {
  const int n_long = (int)min(a.counters[4], (uint32_t)a.n_slot);   // complete: written by the kernel before this one
  if (n_long == 0) return;
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE), tid = threadIdx.x;
  const int T = a.n_tick, split = long_split(a, n_long);
  const uint32_t n_unit = (uint32_t)(n_long * T * split);
  uint32_t* s_x = s + kLongPer * 256;            // [64]
  for (uint32_t unit = blockIdx.x; unit < n_unit; unit += n_share) {
    const LongUnit u = long_unit(a, unit, split);
    uint32_t* at = a.slots + (size_t)u.slot * DYN_TICK_SLOT_WORDS;
    uint32_t old = 0;
    if (u.n > 0) {                               // block-uniform
#pragma unroll
      for (int b = 0; b < kLongPer; ++b) s[b * 256 + tid] = 0u;
      __syncthreads();
      const int32_t *pi = a.in + u.beg, *po = a.out + u.beg;
      uint64_t acc = 0;
      uint32_t orv = 0;
      constexpr int U = 8;
      for (int i0 = 0; i0 < u.n; i0 += U * 256) {
        int32_t x[U], y[U];
#pragma unroll
        for (int v = 0; v < U; ++v) {
          const uint32_t i = (uint32_t)min(i0 + v * 256 + tid, u.n - 1);
          x[v] = pi[i];
          y[v] = po[i];
        }
#pragma unroll
        for (int v = 0; v < U; ++v) {
          const bool ok = i0 + v * 256 + tid < u.n;
          acc += ok ? (uint64_t)((int64_t)x[v] + (int64_t)y[v]) : 0;
          orv |= (uint32_t)(x[v] | y[v]);        // beyond the piece: its last request again
          if (ok) atomicAdd(&s[coarse_bin((uint32_t)x[v])], 1u);
        }
      }
      acc = wave_sum_u64(acc);
      orv = wave_or_u32(orv);
      if (lane == 0) {
        old += (uint32_t)__hip_atomic_fetch_add((unsigned long long*)(at + kSlotSum) + u.q, (unsigned long long)acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        old += __hip_atomic_fetch_or(&at[kSlotOr + u.q], orv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
#pragma unroll
      for (int b = 0; b < kLongPer; ++b) {
        const uint32_t k = b * 256 + tid < kCoarseBins ? s[b * 256 + tid] : 0u;
        if (k) old += add_seen(&at[b * 256 + tid], k);
      }
    }
    asm volatile("" ::"v"(old) : "memory");
    __syncthreads();
    if (tid == 0) s_x[0] = add_seen(&at[kSlotDone], 1u) + 1u == (uint32_t)(T * split) ? 1u : 0u;
    __syncthreads();
    const bool last = s_x[0] != 0u;
    __syncthreads();
    if (!last) continue;                         // block-uniform
    // the cell's last block
    const int64_t c = u.c;
    const int g = (int)(c % a.G);
    const CellTicks ct = cell_ticks(a, c, lane);
#pragma unroll
    for (int b = 0; b < kLongPer; ++b) s[b * 256 + tid] = b * 256 + tid < kCoarseBins ? seen(&at[b * 256 + tid]) : 0u;
    uint64_t tok = 0;
    uint32_t or_l = 0;
    if (lane < T) {
      tok = (uint64_t)seen(&at[kSlotSum + 2 * lane]) | ((uint64_t)seen(&at[kSlotSum + 2 * lane + 1]) << 32);
      or_l = seen(&at[kSlotOr + lane]);
    }
    const double load = div_by((double)tok, a.tick_s, a.r_tick);
    __syncthreads();
    uint32_t k[kLongPer];
#pragma unroll
    for (int b = 0; b < kLongPer; ++b) k[b] = s[tid * kLongPer + b];
    uint32_t longest = 0;                        // the last bin that holds a request
#pragma unroll
    for (int b = 0; b < kLongPer; ++b) longest = k[b] ? (uint32_t)(tid * kLongPer + b) : longest;
    longest = wave_max_u32(longest);
    if (lane == 0) s_x[8 + wave] = longest;      // find_bin's barriers are between this and its use
    int64_t below;
    int bits;
    const uint32_t low = coarse_low(find_bin<kWavesPerBlock>(k, ct.rank, s_x, &below), &bits);
    const uint32_t high = low + ((1u << bits) - 1u);
    bool ok = low < 65536u && (wave_or_u32(or_l) >> 31) == 0u;   // wave-uniform, the same in every wave
    float theta = cell_theta(a.theta[g], ct.cnt_l);
    const bool by_class = (double)theta * ((double)high + 1.0) > (double)high;
    if (!by_class) {                             // block-uniform: the loads of this cell
      double lmin = ct.cnt_l > 0 ? load : __builtin_inf(), lmax = ct.cnt_l > 0 ? load : 0.0;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        lmin = fmin(lmin, __shfl_xor(lmin, d, DYN_WAVE));
        lmax = fmax(lmax, __shfl_xor(lmax, d, DYN_WAVE));
      }
      const uint32_t th = wave_min_u32(__float_as_uint(ok ? theta_between(a, g, lmin, lmax) : 0.0f));   // floats >= 0 order like their bits
      if (lane == 0) s_x[wave] = th;
      __syncthreads();
      theta = __uint_as_float(min(min(s_x[0], s_x[1]), min(s_x[2], s_x[3])));
      __syncthreads();
    }
    const bool tight = (double)theta * ((double)high + 1.0) > (double)high;
    int from = (int)low, n = (int)(high - low) + 1;
    if (ok && !tight) {
      ok = theta > 0.25f;
      if (ok) {
        from = max(0, (int)((double)low * (double)theta) - 1);
        n = (int)((double)high / (double)theta) + 3 - from;
        int bits_l;
        const uint32_t low_l = coarse_low((int)max(max(s_x[8], s_x[9]), max(s_x[10], s_x[11])), &bits_l);
        if (low_l < 65536u) n = min(n, (int)(low_l + (1u << bits_l)) - from);   // beyond the longest request there is nothing to count
        ok = n <= kLongRange;
      }
    }
    const uint32_t words = (uint32_t)(DYN_TICK_TABLE_HEAD + T * (n + 1) + 3) & ~3u;
    uint32_t pool = 0;
    if (ok) {                                    // block-uniform
      if (tid == 0) s_x[4] = atomicAdd(&a.counters[5], words);
      __syncthreads();
      pool = s_x[4];
      __syncthreads();
      ok = pool <= a.pool_words && words <= a.pool_words - pool;
    }
    if (ok)
      for (uint32_t i = tid; i < words / 4; i += 256) ((uint4*)(a.pool + pool))[i] = make_uint4(0u, 0u, 0u, 0u);
    const bool raw = ct.j > DYN_TICK_DEPTH;
    if (wave == 0 && lane < T) {
      TickRec r;
      r.load = load;
      r.off = (uint32_t)ct.beg_l;
      r.cnt = ct.cnt_l;
      a.rec[c * T + lane] = r;
      a.cstat[((c / a.G) * T + lane) * a.G + g] = (uint8_t)(ct.bad_l | (or_l >> 31 ? DYN_WS_BAD_REQUEST : 0u));
    }
    const uint32_t route = tbt_route(ct.cnt_l, ct.j, lane);
    if (tid == 0) {
      at[kSlotFrom] = (uint32_t)from;
      at[kSlotN] = ok ? (uint32_t)n : 0u;
      at[kSlotLow] = low;
      at[kSlotBits] = (uint32_t)bits | (tight ? 0x100u : 0u);
      at[kSlotTheta] = __float_as_uint(theta);
      at[kSlotPool] = pool;
      if (!ok) {                                 // lists, by one block
        TickPlan p;
        p.j = (int32_t)ct.j;
        p.xj = 0;
        p.flags = route | (raw ? DYN_TP_RAW : ct.j > DYN_TICK_WAVE ? DYN_TP_DEEP : 0u);
        p.place = 0;
        if (raw || !walks_with_lists(route, ct.j)) {
          p.flags |= DYN_TP_GENERAL;
          a.slow_list[atomicAdd(&a.counters[1], 1u)] = (uint32_t)c;
        } else {
          atomicAdd(&a.counters[3], 1u);
        }
        a.plan[c] = p;
        a.deep_list[atomicAdd(&a.counters[0], 1u)] = (uint32_t)c;
      }
    }
    __syncthreads();                             // LDS is reused by the next unit
  }
}

// Second pass: the lengths from `from` on, counted per tick, and the plan from the cell's last block.  `s`: kDeepCap words of LDS.
__device__ __forceinline__ void long_rank(const TickCellArgs& a, uint32_t* s) {
  const int n_long = (int)min(a.counters[4], (uint32_t)a.n_slot);
  if (n_long == 0) return;
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE), tid = threadIdx.x;
  const int T = a.n_tick, split = long_split(a, n_long);
  const uint32_t n_unit = (uint32_t)(n_long * T * split);
  uint32_t* s_all = s + kLongRange + 1;          // [513] the cell's requests of at least every length of the bin
  uint32_t* s_x = s_all + 520;
  for (uint32_t unit = blockIdx.x; unit < n_unit; unit += gridDim.x) {
    const LongUnit u = long_unit(a, unit, split);
    uint32_t* at = a.slots + (size_t)u.slot * DYN_TICK_SLOT_WORDS;
    const int from = (int)at[kSlotFrom], n = (int)at[kSlotN];
    if (n == 0) continue;                        // block-uniform
    const int stride = n + 1;
    uint32_t* table = a.pool + at[kSlotPool] + DYN_TICK_TABLE_HEAD;
    uint32_t old = 0;
    if (u.n > 0) {
      for (int i = tid; i <= n; i += 256) s[i] = 0u;
      __syncthreads();
      const int32_t* pi = a.in + u.beg;
      constexpr int U = 8;
      uint32_t above = 0;
      for (int i0 = 0; i0 < u.n; i0 += U * 256) {
        int32_t x[U];
#pragma unroll
        for (int v = 0; v < U; ++v) x[v] = pi[(uint32_t)min(i0 + v * 256 + tid, u.n - 1)];
#pragma unroll
        for (int v = 0; v < U; ++v) {
          if (i0 + v * 256 + tid < u.n && x[v] >= from) {
            if (x[v] - from < n) atomicAdd(&s[x[v] - from], 1u);
            else ++above;
          }
        }
      }
      above = wave_sum_u32(above);
      if (lane == 0 && above) atomicAdd(&s[n], above);
      __syncthreads();
      for (int i = tid; i <= n; i += 256)
        if (s[i]) old += add_seen(&table[(size_t)u.q * stride + i], s[i]);
    }
    asm volatile("" ::"v"(old) : "memory");
    __syncthreads();
    if (tid == 0) s_x[0] = add_seen(&at[kSlotDone2], 1u) + 1u == (uint32_t)(T * split) ? 1u : 0u;
    __syncthreads();
    const bool last = s_x[0] != 0u;
    __syncthreads();
    if (!last) continue;                         // block-uniform
    // the cell's last block: how many are at least so long, per tick (a wave each) and for the lengths of the bin in all
    const int64_t c = u.c;
    const int low = (int)at[kSlotLow], bits = (int)(at[kSlotBits] & 0xFFu), in_bin = 1 << bits;
    const bool tight = (at[kSlotBits] & 0x100u) != 0u;
    const CellTicks ct = cell_ticks(a, c, lane);
    for (int i = tid; i <= in_bin; i += 256) s_all[i] = 0u;
    __syncthreads();
    for (int q = wave; q < T; q += kWavesPerBlock) {
      uint32_t* row = table + (size_t)q * stride;
      uint32_t more = 0;                         // of at least the length after the chunk
      for (int top = (n / 512) * 512; top >= 0; top -= 512) {   // the last entry counts what is longer than the table's lengths
        uint32_t x[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) x[v] = top + lane * 8 + v <= n ? seen(&row[top + lane * 8 + v]) : 0u;
#pragma unroll
        for (int v = 6; v >= 0; --v) x[v] += x[v + 1];
        uint32_t after = x[0];                   // of this lane's entries and all after them
#pragma unroll
        for (int d = 1; d < DYN_WAVE; d <<= 1) {
          const uint32_t o = __shfl_down(after, d, DYN_WAVE);
          if (lane + d < DYN_WAVE) after += o;
        }
        const uint32_t rest = more + after - x[0];
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          const int i = top + lane * 8 + v, b = from + i - low;
          if (i <= n) {
            row[i] = x[v] + rest;
            if (b >= 0 && b <= in_bin) atomicAdd(&s_all[b], x[v] + rest);
          }
        }
        more += (uint32_t)__builtin_amdgcn_readlane((int)after, 0);
      }
    }
    __threadfence_block();
    __syncthreads();
    if (tid == 0) s_x[0] = 0u;
    __syncthreads();
    for (int b = tid; b < in_bin; b += 256)      // the largest length that j requests reach: exactly one, the counts descend
      if (s_all[b] >= (uint32_t)ct.j && (b + 1 == in_bin || s_all[b + 1] < (uint32_t)ct.j)) s_x[0] = (uint32_t)b;
    __syncthreads();
    const int b = (int)s_x[0], xj = low + b;
    const int n_gt = (int)s_all[b + 1], n_eq = (int)s_all[b] - n_gt, need = (int)ct.j - n_gt;
    const uint32_t* row = table + (size_t)min(lane, T - 1) * stride + (xj - from);
    const uint32_t eq_l = lane < T && ct.cnt_l > 0 ? row[0] - row[1] : 0u;
    uint32_t flags = tbt_route(ct.cnt_l, ct.j, lane), place;
    if (tight) {
      uint32_t m4[4];
      const int npos = smallest_four(eq_l, lane, m4);
      const uint64_t s4 = npos >= 4 ? (uint64_t)m4[0] + m4[1] + m4[2] + m4[3] : 0u;
      flags |= DYN_TP_TIGHT;
      if (!tight_place(need, n_eq, npos, (uint32_t)min(s4, (uint64_t)0xFFFFFFFFu), &place) || !(flags & (DYN_TP_DENSE | DYN_TP_SMALL))) {
        flags |= DYN_TP_GENERAL;
        place = (uint32_t)need;
      }
    } else {
      flags |= DYN_TP_TABLE | DYN_TP_GENERAL;
      place = at[kSlotPool];
    }
    if (wave == 0 && tight && lane < T) a.rec[c * T + lane].off = eq_l;
    if (tid == 0) {
      if (!tight) {                              // with x_j known fewer lengths can decide
        const double theta = (double)__uint_as_float(at[kSlotTheta]);
        const int lo = max(from, (int)((double)xj * theta) - 1), hi = min(from + n - 1, (int)((double)xj / theta) + 2);
        table[-DYN_TICK_TABLE_HEAD] = (uint32_t)lo;
        table[-DYN_TICK_TABLE_HEAD + 1] = (uint32_t)(hi - lo + 1);
        table[-DYN_TICK_TABLE_HEAD + 2] = (uint32_t)stride;
        table[-DYN_TICK_TABLE_HEAD + 3] = (uint32_t)(lo - from);
      }
      TickPlan p;
      p.j = (int32_t)ct.j;
      p.xj = xj;
      p.flags = flags;
      p.place = place;
      a.plan[c] = p;
      if (flags & DYN_TP_GENERAL) a.slow_list[atomicAdd(&a.counters[1], 1u)] = (uint32_t)c;
    }
    __syncthreads();                             // LDS is reused by the next unit
  }
}


// The same for the listed cells whose ticks do not fit one wave's registers: a block per cell, wave w takes the ticks
// w, w + WAVES, ...; x_j by the bit-wise search with the waves' counts added up through LDS (one barrier per bit).  A cell
// it settles is taken off the list (its entry becomes DYN_LIST_DONE).
constexpr int kTightWaves = 4, kTightManyWaves = 8;   // of a block: dyn_launch_tick_cell says where the line lies
constexpr int kTightUnits = 4096;              // waves that the device holds at once (registers)

template <int WAVES, int P>   // P registers = 2P rows per wave
__device__ __forceinline__ Settled tight_cell_block(const int32_t* __restrict__ in, const int32_t* __restrict__ out,
                                                 int64_t beg_l, int32_t cnt_l, int T, int rpt, int m, int rank, float theta,
                                                 int lane, int wave, uint32_t* s_x /* [2][WAVES] */,
                                                 uint32_t* s_m /* [4 * WAVES] */, TightCell* res) {
  uint32_t v[P];
  uint32_t orv = 0, vmax = 0, tok_acc = 0, tok_l = 0;
  constexpr int CH = 4;
  int q = wave, r = 0;                   // tick and row of the slot being filled (wave-uniform)
#pragma unroll
  for (int p0 = 0; p0 < P; p0 += CH) {
    uint32_t a[2 * CH], b[2 * CH];
    int qs[2 * CH], rs[2 * CH];
#pragma unroll
    for (int u = 0; u < 2 * CH; ++u) {
      qs[u] = q; rs[u] = r;
      // lane reads without a branch around them: beyond the last tick the lane index is clamped and the count zeroed
      const int qc = q < DYN_WAVE - 1 ? q : DYN_WAVE - 1;
      const int64_t beg_q = readlane_i64(beg_l, qc);
      const int cnt_q = __builtin_amdgcn_readlane(cnt_l, qc);
      const int left = (q < T ? cnt_q : 0) - r * DYN_WAVE;
      const bool ok = lane < left;
      // the padding of a slot without a request goes into its half of the register now; the length is ORed in below
      // (a lane without a request loads 0), so no mask has to live across the loads
      if (u % 2 == 0) v[p0 + u / 2] = ok ? 0u : 0xFFFFu;
      else v[p0 + u / 2] |= ok ? 0u : 0xFFFF0000u;
      const int64_t row_q = beg_q + (int64_t)(r * DYN_WAVE);   // one scalar offset for both arrays
      a[u] = ok ? (uint32_t)in[row_q + lane] : 0u;
      b[u] = ok ? (uint32_t)out[row_q + lane] : 0u;
      if (++r == rpt) { r = 0; q += WAVES; }
    }
#pragma unroll
    for (int u = 0; u < 2 * CH; ++u) {
      tok_acc += a[u] + b[u];
      orv |= a[u] | b[u];
      vmax = max(vmax, a[u]);
      if (rs[u] == rpt - 1) {
        const uint32_t tok = wave_sum_u32(tok_acc);
        if (lane == qs[u]) tok_l = tok;
        tok_acc = 0;
      }
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      v[p0 + u] |= (a[2 * u] & 0xFFFFu) | (a[2 * u + 1] << 16);   // lengths of 2^16 and more: the cell is given up below
    }
    asm volatile("" : "+v"(tok_acc), "+v"(tok_l), "+v"(orv), "+v"(vmax), "+v"(v[p0]), "+v"(v[p0 + 1]), "+v"(v[p0 + 2]),
                 "+v"(v[p0 + 3])::"memory");
  }
  // sums over the block: every wave writes its word, a barrier, every wave reads all of them (two buffers in turn)
  int turn = 0;
  auto block_or = [&](uint32_t x) {
    if (lane == 0) s_x[turn * WAVES + wave] = x;
    __syncthreads();
    uint32_t all = 0;
    for (int w = 0; w < WAVES; ++w) all |= s_x[turn * WAVES + w];
    turn ^= 1;
    return all;
  };
  auto block_max = [&](uint32_t x) {
    if (lane == 0) s_x[turn * WAVES + wave] = x;
    __syncthreads();
    uint32_t all = 0;
    for (int w = 0; w < WAVES; ++w) all = max(all, s_x[turn * WAVES + w]);
    turn ^= 1;
    return all;
  };
  auto block_sum = [&](uint32_t x) {
    if (lane == 0) s_x[turn * WAVES + wave] = x;
    __syncthreads();
    uint32_t all = 0;
    for (int w = 0; w < WAVES; ++w) all += s_x[turn * WAVES + w];
    turn ^= 1;
    return all;
  };
  const uint32_t all_or = block_or(wave_or_u32(orv));
  const uint32_t top = block_max(wave_max_u32(vmax));
  if (all_or >= (1u << 16) || top == 0xFFFFu) return kNotTaken;   // block-uniform; 0xFFFF is the padding value
  uint32_t xj = top;
  const int j = m - rank + 1;
  if (rank != m) {
    uint32_t d = 0;
    const int nb = 32 - __builtin_clz(top | 1u);
    for (int b = nb - 1; b >= 0; --b) {
      const uint32_t cand = d | (1u << b);
      const uint16_t cand_lo = (uint16_t)cand;
      const uint32_t cand_hi = cand << 16;
      int below = 0;
#pragma unroll
      for (int i = 0; i < P; ++i)
        below += __popcll(__ballot((uint16_t)v[i] < cand_lo)) + __popcll(__ballot(v[i] < cand_hi));
      if ((int)block_sum((uint32_t)below) < rank) d |= 1u << b;
    }
    xj = d;
  }
  res->tok_l = tok_l;                    // lanes q with q % 8 == wave
  res->xj = xj;
  if (!((double)theta * ((double)xj + 1.0) > (double)xj)) return kBoundFails;
  int n_gt = 0, n_eq = 0, eq_acc = 0;      // the padding (0xFFFF) counts as longer: taken off after the block's sum
  uint32_t eq_l = 0;
  q = wave; r = 0;
  const uint32_t xj_hi = xj << 16;
#pragma unroll
  for (int i = 0; i < P; ++i) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      n_gt += h ? __popcll(__ballot(v[i] >= xj_hi + 0x10000u)) : __popcll(__ballot((uint16_t)v[i] > (uint16_t)xj));
      eq_acc += h ? __popcll(__ballot((v[i] >> 16) == xj)) : __popcll(__ballot((uint16_t)v[i] == (uint16_t)xj));
      if (++r == rpt) {
        if (lane == q) eq_l = (uint32_t)eq_acc;
        n_eq += eq_acc;
        eq_acc = 0;
        r = 0; q += WAVES;
      }
    }
  }
  n_gt = (int)block_sum((uint32_t)n_gt) - (2 * P * DYN_WAVE * WAVES - m);
  n_eq = (int)block_sum((uint32_t)n_eq);
  const int need = j - n_gt;
  uint32_t place = (uint32_t)need;
  res->walk = true;
  if (need > 4 && n_eq - need + 1 > 4) {   // block-uniform
    // every wave's four smallest positive counts meet in LDS; the four smallest of them are the block's
    uint32_t m4[4];
    const int npos_w = smallest_four(eq_l, lane, m4);
    const int npos = (int)block_sum((uint32_t)npos_w);
    if (lane < 4) s_m[wave * 4 + lane] = lane == 0 ? m4[0] : lane == 1 ? m4[1] : lane == 2 ? m4[2] : m4[3];
    __syncthreads();
    uint32_t best[4] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
    for (int i = 0; i < 4 * WAVES; ++i) {
      uint32_t x = s_m[i];
#pragma unroll
      for (int k = 0; k < 4; ++k) {        // insertion into the ascending four
        const uint32_t lo = min(best[k], x);
        x = max(best[k], x);
        best[k] = lo;
      }
    }
    __syncthreads();                       // s_m is free again
    const uint32_t s4 = npos >= 4 ? best[0] + best[1] + best[2] + best[3] : 0u;
    res->walk = tight_place(need, n_eq, npos, s4, &place);
  } else if (need > 4) {
    place = (uint32_t)(n_eq - need + 1) | DYN_TIGHT_FROM_BELOW;
  }
  res->need = (uint32_t)need;
  res->eq_l = eq_l;
  res->place = place;
  return kSettled;
}

// The n_top largest of a tick's `cnt` input lengths (all below 2^16, cnt <= kListTick) in descending order to dst, by one
// wave in LDS: the n_top-th largest by a bit-wise search, what is above it gathered in place, the rest of the places
// filled with it, a bitonic sort of that many.
constexpr int kListTick = 2048;
__device__ __forceinline__ void tick_list(const int32_t* __restrict__ src, int cnt, int n_top, int32_t* dst, uint16_t* buf, int lane) {
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  int32_t mx = 0;
  for (int i0 = 0; i0 < cnt; i0 += 8 * DYN_WAVE) {
    int32_t x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = src[min(i0 + u * DYN_WAVE + lane, cnt - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      mx = max(mx, x[u]);
      if (i0 + u * DYN_WAVE + lane < cnt) buf[i0 + u * DYN_WAVE + lane] = (uint16_t)x[u];
    }
  }
  wave_sync();
  if (n_top < cnt) {
    int32_t thr = 0;
    for (int b = 31 - __builtin_clz((uint32_t)wave_max_i32(mx) | 1u); b >= 0; --b) {
      const int32_t cand = thr | (1 << b);
      int above = 0;
      for (int i0 = 0; i0 < cnt; i0 += 4 * DYN_WAVE) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = i0 + u * DYN_WAVE + lane;
          above += __popcll(__ballot(i < cnt && buf[min(i, cnt - 1)] >= cand));
        }
      }
      if (above >= n_top) thr = cand;
    }
    int got = 0;                                   // fewer than n_top values are above thr
    for (int i0 = 0; i0 < cnt; i0 += DYN_WAVE) {
      const int32_t x = i0 + lane < cnt ? buf[i0 + lane] : 0;
      const bool take = i0 + lane < cnt && x > thr;
      const uint64_t who = __ballot(take);
      wave_sync();                                 // the row is read before places in it are written
      if (take) buf[got + __popcll(who & ((1ull << lane) - 1ull))] = (uint16_t)x;
      got += __popcll(who);
    }
    wave_sync();
    for (int i = got + lane; i < n_top; i += DYN_WAVE) buf[i] = (uint16_t)thr;
  }
  int n2 = 2;
  while (n2 < n_top) n2 <<= 1;                     // at most kListTick
  for (int i = n_top + lane; i < n2; i += DYN_WAVE) buf[i] = 0;   // as short as any: behind the n_top
  wave_sync();
  for (int k = 2; k <= n2; k <<= 1)
    for (int d = k >> 1; d > 0; d >>= 1) {
      for (int p = lane; p < n2 / 2; p += DYN_WAVE) {
        const int i = ((p & ~(d - 1)) << 1) | (p & (d - 1)), o = i | d;   // the pair's places
        const int32_t u = buf[i], v = buf[o];
        const bool down = (i & k) == 0;            // descending runs first: the whole ends descending
        if (down ? u < v : u > v) { buf[i] = (uint16_t)v; buf[o] = (uint16_t)u; }
      }
      wave_sync();
    }
  for (int i = lane; i < n_top; i += DYN_WAVE) dst[i] = buf[i];
  wave_sync();                                     // buf is reused
}

template <int WAVES>
__global__ __launch_bounds__(WAVES* DYN_WAVE) __attribute__((amdgpu_waves_per_eu(4, 4))) void tick_tight_block_kernel(TickCellArgs a) {
  __shared__ uint32_t s_x[2 * WAVES];
  __shared__ uint32_t s_m[4 * WAVES];
  __shared__ uint16_t s_list[WAVES][kListTick];
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE);
  const int T = a.n_tick, G = a.G;
  const uint32_t n_item = a.counters[2];         // complete: written by the kernel before this one
  for (uint32_t item = blockIdx.x; item < n_item; item += gridDim.x) {
    const uint32_t entry = a.list_cells[item];
    if (entry & DYN_LIST_SKIP) continue;         // block-uniform
    const int64_t c = entry;
    const int64_t w = c / G;
    const int g = (int)(c % G);
    const int64_t f0 = (w * T) * G + g;
    int64_t beg_l = 0;
    int32_t cnt_l = 0;
    uint32_t bad_l = 0;
    if (lane < T) {
      const int64_t f = f0 + (int64_t)lane * G;
      const int64_t b = a.fine_off[f], e = a.fine_off[f + 1];
      if (b < 0 || e < b || e > a.n_req) bad_l = DYN_WS_BAD_OFFSETS;
      else { beg_l = b; cnt_l = (int32_t)(e - b); }
    }
    const int64_t m_cell = (int64_t)wave_sum_u64((uint64_t)(uint32_t)cnt_l);
    const int64_t rank = (a.pct_num * m_cell + a.pct_den - 1) / a.pct_den;
    const int64_t j64 = m_cell > 0 ? m_cell - rank + 1 : 0;
    const int rpt = ((int)wave_max_u32((uint32_t)cnt_l) + DYN_WAVE - 1) / DYN_WAVE;
    const int rows = ((T + WAVES - 1) / WAVES) * rpt;   // rows of the wave with most ticks
    TightCell tc;
    tc.tok_l = 0; tc.eq_l = 0; tc.xj = 0; tc.place = 0; tc.need = 0; tc.walk = true;
    Settled done = kNotTaken;                    // block-uniform from here on
    if (m_cell > 0 && m_cell < (1 << 24) && rows <= 128 && !long_at_once(a, m_cell, g, cnt_l, rows)) {
      const float theta = cell_theta(a.theta[g], cnt_l);
      const int m = (int)m_cell, rk = (int)rank;
      if (rows <= 16) done = tight_cell_block<WAVES, 8>(a.in, a.out, beg_l, cnt_l, T, rpt, m, rk, theta, lane, wave, s_x, s_m, &tc);
      else if (rows <= 32) done = tight_cell_block<WAVES, 16>(a.in, a.out, beg_l, cnt_l, T, rpt, m, rk, theta, lane, wave, s_x, s_m, &tc);
      else if (rows <= 64) done = tight_cell_block<WAVES, 32>(a.in, a.out, beg_l, cnt_l, T, rpt, m, rk, theta, lane, wave, s_x, s_m, &tc);
      else done = tight_cell_block<WAVES, 64>(a.in, a.out, beg_l, cnt_l, T, rpt, m, rk, theta, lane, wave, s_x, s_m, &tc);
    }
    __syncthreads();                             // s_x is reused by the next item
    const bool lists = T >= 2 && (a.few_cells || j64 > DYN_TICK_WAVE) && j64 <= DYN_TICK_DEPTH && wave_max_u32((uint32_t)cnt_l) <= kListTick;   // can be made here
    if (done != kSettled && m_cell > DYN_TICK_LONG && a.n_slot > 0 && !(done == kBoundFails && lists && m_cell < a.table_from)) {   // block-uniform: to the blocks that share it, if a slot is left
      if (threadIdx.x == 0) s_x[0] = atomicAdd(&a.counters[4], 1u);
      __syncthreads();
      const uint32_t slot = s_x[0];
      __syncthreads();
      if (slot < (uint32_t)a.n_slot) {
        uint4* at = (uint4*)(a.slots + (size_t)slot * DYN_TICK_SLOT_WORDS);
        for (int i = threadIdx.x; i < DYN_TICK_SLOT_WORDS / 4; i += WAVES * DYN_WAVE)
          at[i] = make_uint4(i == kSlotCell / 4 ? (uint32_t)c : 0u, 0u, 0u, 0u);
        if (threadIdx.x == 0) a.list_cells[item] = DYN_LIST_DONE;
        continue;
      }
    }
    if (done == kNotTaken) continue;
    uint32_t flags = tbt_route(cnt_l, j64, lane);
    if (done == kSettled) {
      flags |= DYN_TP_TIGHT;
      if (!tc.walk || !(flags & (DYN_TP_DENSE | DYN_TP_SMALL))) {
        flags |= DYN_TP_GENERAL;
        tc.place = tc.need;
      }
    } else {
      // Its lists, a tick per wave at a time, where that is better than what follows: few cells on the whole device, or a
      // list beyond the 64 entries that one wave keeps sorted (a block per cell, tick after tick).  540 cells of up to
      // 6800 requests and 12 ticks: 83 us in this kernel (74 with eight waves a block); 26, then 227 in tick_cell_kernel and 462 in
      // tick_deep_kernel without.  A single tick is one wave's work here, and all four of the deep kernel's there.
      if (!lists) continue;
      for (int q = wave; q < T; q += WAVES) {
        const int64_t beg_q = readlane_i64(beg_l, q);
        const int cnt_q = __builtin_amdgcn_readlane(cnt_l, q);
        if (cnt_q > 0) tick_list(a.in + beg_q, cnt_q, j64 < cnt_q ? (int)j64 : cnt_q, a.top + beg_q, s_list[wave], lane);
      }
      if (j64 > DYN_TICK_WAVE) flags |= DYN_TP_DEEP;
      flags |= walks_with_lists(flags, j64) ? 0u : DYN_TP_GENERAL;
      tc.eq_l = (uint32_t)beg_l;                 // where the tick's list is (n_req < 2^31)
    }
    if (lane < T && (lane % WAVES) == wave) {   // the wave that walked the tick
      TickRec r;
      r.load = div_by((double)tc.tok_l, a.tick_s, a.r_tick);
      r.off = tc.eq_l;
      r.cnt = cnt_l;
      a.rec[c * T + lane] = r;
      a.cstat[f0 + (int64_t)lane * G] = (uint8_t)bad_l;
    }
    if (threadIdx.x == 0) {
      TickPlan p;
      p.j = (int32_t)j64;
      p.xj = (int32_t)tc.xj;
      p.flags = flags;
      p.place = tc.place;
      a.plan[c] = p;
      if (flags & DYN_TP_GENERAL) a.slow_list[atomicAdd(&a.counters[1], 1u)] = (uint32_t)c;
      else if (done == kBoundFails) atomicAdd(&a.counters[3], 1u);   // a cell the walk takes with its lists
      a.list_cells[item] = DYN_LIST_DONE;
    }
  }
}

// ---- per-tick loads and candidate lists ------------------------------------------------------
// One wave per (window, class) cell walks the cell's ticks.  Lane q holds tick q's offsets;
// the cell's request count gives j.  Per tick the wave streams the tick's requests once:
// token sum (the tick's load) and, for 0 < j <= 64, the j largest input lengths, kept sorted
// (descending) in the wave's lanes.  A row of 64 new values is merged either by j rounds of
// "take the maximum of kept and new values" or, when few new values can still enter the
// first j positions, by ranking: a value's position is the number of values that beat it
// (kept values win ties against new ones, lower lanes against higher ones), and the merged
// order is written through a 64-word LDS buffer.  A second list, merged with every finished
// tick's list, holds the j largest lengths of the whole cell: its last entry is x_j.
// The first blocks take the long cells (long_count), in the registers and LDS of this kernel: spills are long_count's, the loop over listed cells has
// none.  What sharing the launch costs that loop (us of the kernel without, with it; thousands of listed cells): 316 322, 124 126, 241 250; a launch of its
// own would cost every call 2 to 4.5.  With eight waves a SIMD for the loop 296, but long_count on long cells 22.7 and 26.1.
__global__ __launch_bounds__(kWavesPerBlock* DYN_WAVE) __attribute__((amdgpu_waves_per_eu(6, 8))) void tick_cell_kernel(TickCellArgs a) {
  __shared__ uint32_t s_long[kLongWords];
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE);
  const int T = a.n_tick, G = a.G;
  const int n_share = long_blocks(a);
  if ((int)blockIdx.x < n_share) {              // block-uniform: the first blocks share the long cells
    long_count(a, n_share, s_long);
    return;
  }
  int32_t (*s_buf)[DYN_WAVE] = (int32_t (*)[DYN_WAVE])s_long;
  const uint32_t n_item = a.counters[2];        // complete: written by the kernel before this one
  for (uint32_t item = (blockIdx.x - n_share) * kWavesPerBlock + wave; item < n_item; item += (gridDim.x - n_share) * kWavesPerBlock) {
  if (a.list_cells[item] == DYN_LIST_DONE) continue;   // settled by the kernel before this one
  const int64_t c = a.list_cells[item] & ~DYN_LIST_SKIP;
  const int64_t w = c / G;
  const int g = (int)(c % G);
  const int64_t f0 = (w * T) * G + g;           // fine cell of tick 0; tick q is q*G further

  int64_t beg_l = 0;
  int32_t cnt_l = 0;
  uint32_t bad_l = 0;
  if (lane < T) {
    const int64_t f = f0 + (int64_t)lane * G;
    const int64_t b = a.fine_off[f], e = a.fine_off[f + 1];
    if (b < 0 || e < b || e > a.n_req) bad_l = DYN_WS_BAD_OFFSETS;   // such a tick is treated as empty
    else { beg_l = b; cnt_l = (int32_t)(e - b); }
  }
  const int64_t m_cell = (int64_t)wave_sum_u64((uint64_t)(uint32_t)cnt_l);
  const int64_t rank = (a.pct_num * m_cell + a.pct_den - 1) / a.pct_den;
  const int64_t j64 = m_cell > 0 ? m_cell - rank + 1 : 0;
  const bool raw = j64 > DYN_TICK_DEPTH;         // deeper than a cut-down list: whole ticks are sorted, or scanned unsorted
  const bool deep = !raw && j64 > DYN_TICK_WAVE;
  const int keep = (raw || deep) ? 0 : (int)j64;                // wave-uniform, 0 .. 64

  // How the TBT percentile can be found: from the largest tick TBT when every non-empty tick holds
  // j requests; from the four largest tick TBTs when any four non-empty ticks hold j between them
  // (the four smallest counts do, or there are no more than four).
  uint32_t flags = raw ? DYN_TP_RAW : (deep ? DYN_TP_DEEP : 0u);
  if (m_cell > 0) {
    flags |= tbt_route(cnt_l, j64, lane);
    if (raw || !walks_with_lists(flags, j64)) flags |= DYN_TP_GENERAL;
  }

  int32_t* buf = s_buf[wave];
  // Merges the values `cx` of the lanes with `mine` set into the descending list `best` (one entry per lane,
  // -1 = none); the first `keep` positions of the result are exact.
  auto merge = [&](int32_t best, int32_t cx, bool mine) -> int32_t {
    uint64_t mask = __ballot(mine);
    if (mask == 0) return best;
    if (__popcll(mask) * 10 > keep * 16) {
      // rounds of maximum extraction over kept and new values; a taken value leaves its lane
      int32_t bv = best, cv = mine ? cx : -1, nb = -1;
      for (int i = 0; i < keep; ++i) {
        const int32_t mx = wave_max_i32(max(bv, cv));
        if (mx < 0) break;
        const uint64_t ub = __ballot(bv == mx);
        if (ub) {
          if (lane == (int)__builtin_ctzll(ub)) bv = -1;
        } else {
          const uint64_t uc = __ballot(cv == mx);
          if (lane == (int)__builtin_ctzll(uc)) cv = -1;
        }
        if (lane == i) nb = mx;
      }
      return nb;
    }
    int rb = lane;      // position of my kept value: the kept values before it + new values above it
    int rc = 0;         // position of my new value: kept values >= it + new values that beat it
    while (mask) {
      const int u = __builtin_ctzll(mask);
      mask &= mask - 1;
      const int32_t v = __builtin_amdgcn_readlane(cx, u);
      const int n_ge = __popcll(__ballot(best >= v));
      rb += (v > best) ? 1 : 0;
      rc += (v > cx || (v == cx && u < lane)) ? 1 : 0;
      if (lane == u) rc += n_ge;
    }
    // the positions are a permutation of 0 .. 63 + (new values): every slot below 64 is written once
    if (rb < DYN_WAVE) buf[rb] = best;
    if (mine && rc < DYN_WAVE) buf[rc] = cx;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int32_t merged = buf[lane];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return merged;
  };

  double load_l = 0.0;
  uint32_t neg_mask_lo = 0, neg_mask_hi = 0;    // ticks holding a negative token count
  int32_t gbest = -1;                           // the j largest input lengths of the cell so far
  bool g_empty = true;
  // (x, y) always hold the row after the one being processed: the next row of the same tick,
  // else the first row of the next tick
  int32_t x, y;
  auto fetch = [&](int64_t at, int32_t left) {   // `left` requests from `at` on, one per lane
    x = lane < left ? a.in[at + lane] : -1;
    y = lane < left ? a.out[at + lane] : 0;
  };
  fetch(readlane_i64(beg_l, 0), __builtin_amdgcn_readlane(cnt_l, 0));
  for (int q = 0; q < T; ++q) {
    const int64_t beg_q = readlane_i64(beg_l, q);
    const int32_t n_q = __builtin_amdgcn_readlane(cnt_l, q);
    int64_t beg_n = 0;
    int32_t n_n = 0;
    if (q + 1 < T) {
      beg_n = readlane_i64(beg_l, q + 1);
      n_n = __builtin_amdgcn_readlane(cnt_l, q + 1);
    }
    if (n_q == 0) fetch(beg_n, n_n);              // nothing was fetched for an empty tick
    uint64_t acc = 0;
    uint32_t orv = 0;
    int32_t best = -1;                            // input lengths are >= 0
    for (int32_t r0 = 0; r0 < n_q; r0 += DYN_WAVE) {
      const int nrow = n_q - r0 < DYN_WAVE ? n_q - r0 : DYN_WAVE;
      const bool have = lane < nrow;
      const int32_t cx = x, cy = y;
      if (r0 + DYN_WAVE < n_q) fetch(beg_q + r0 + DYN_WAVE, n_q - r0 - DYN_WAVE);
      else fetch(beg_n, n_n);
      acc += have ? (uint64_t)((int64_t)cx + (int64_t)cy) : 0;
      orv |= have ? (uint32_t)(cx | cy) : 0u;
      if (keep == 0) continue;
      const int32_t thr = __builtin_amdgcn_readlane(best, keep - 1);
      best = merge(best, cx, have && cx > thr);    // a value <= thr has `keep` kept values ahead of it
    }
    // the tick's token sum: 32-bit lanes when every lane's sum is small enough for it
    uint64_t tok;
    if (__ballot((acc >> 25) != 0) == 0) tok = wave_sum_u32((uint32_t)acc);
    else tok = wave_sum_u64(acc);
    if (__ballot((int32_t)orv < 0)) {
      if (q < 32) neg_mask_lo |= 1u << q; else neg_mask_hi |= 1u << (q - 32);
    }
    if (lane == q) load_l = div_by((double)tok, a.tick_s, a.r_tick);
    const int n_top = keep < n_q ? keep : n_q;
    if (lane < n_top) a.top[beg_q + lane] = best;           // the tick's list sits where its requests start
    if (n_top > 0) {                             // towards x_j: the walk prunes its lists with it, the general kernel brackets with it
      const int32_t mine_v = lane < n_top ? best : -1;
      if (g_empty) {
        gbest = mine_v;
        g_empty = false;
      } else {
        const int32_t thr = __builtin_amdgcn_readlane(gbest, keep - 1);
        gbest = merge(gbest, mine_v, mine_v > thr);
      }
    }
  }
  if (lane < T) {
    const int64_t f = f0 + (int64_t)lane * G;
    TickRec r;
    r.load = load_l;
    r.off = (uint32_t)beg_l;                     // n_req < 2^31
    r.cnt = cnt_l;
    a.rec[c * T + lane] = r;
    const uint32_t neg = lane < 32 ? (neg_mask_lo >> lane) & 1u : (neg_mask_hi >> (lane - 32)) & 1u;
    // every fine cell writes its own status byte: nothing to clear beforehand
    a.cstat[f] = (uint8_t)(bad_l | (neg ? DYN_WS_BAD_REQUEST : 0u));
  }
  const int32_t xj = keep > 0 ? __builtin_amdgcn_readlane(gbest, keep - 1) : 0;
  if (lane == 0) {
    TickPlan p;
    p.j = (int32_t)j64;                          // below 2^31 like the number of requests
    p.xj = xj < 0 ? 0 : xj;
    p.flags = flags;
    p.place = 0;
    a.plan[c] = p;
    if (deep || raw) a.deep_list[atomicAdd(&a.counters[0], 1u)] = (uint32_t)c;   // x_j and the sorted ticks come from there
    if (flags & DYN_TP_GENERAL) a.slow_list[atomicAdd(&a.counters[1], 1u)] = (uint32_t)c;
    else if (j64 > 0) atomicAdd(&a.counters[3], 1u);   // a cell the walk takes with its lists
  }
  }
}

// ---- cells whose percentile lies more than 64 deep ------------------------------------------------
// A block per listed cell.  x_j by a most-significant-bit-first search on the value, every step a
// count over the cell's requests; then every tick's min(j, count) largest input lengths in descending
// order: a tick of up to 8192 requests is sorted whole in LDS (bitonic), a larger one is first cut
// down to its j largest (threshold by the same bit search, the values above it gathered, the rest of
// the j places filled with the threshold itself).
__global__ __launch_bounds__(256) void tick_deep_kernel(TickCellArgs a) {
  __shared__ int32_t s_val[kDeepCap];
  __shared__ uint32_t s_part[4];
  __shared__ uint32_t s_fill;
  const int tid = threadIdx.x, lane = tid & (DYN_WAVE - 1), wave = tid / DYN_WAVE;
  const int T = a.n_tick;
  const uint32_t n_deep = a.counters[0];         // complete: written by the kernel before this one
  long_rank(a, (uint32_t*)s_val);
  auto block_sum = [&](uint32_t v) -> uint32_t {
    const uint32_t ws = wave_sum_u32(v);
    __syncthreads();
    if (lane == 0) s_part[wave] = ws;
    __syncthreads();
    return s_part[0] + s_part[1] + s_part[2] + s_part[3];
  };
  auto block_max = [&](int32_t v) -> int32_t {
    const int32_t wm = wave_max_i32(v);
    __syncthreads();
    if (lane == 0) s_part[wave] = (uint32_t)wm;
    __syncthreads();
    return max(max((int32_t)s_part[0], (int32_t)s_part[1]), max((int32_t)s_part[2], (int32_t)s_part[3]));
  };
  // j-th largest value of the ticks q0 .. q1-1 of the cell (at least j values, all bits above `bits` clear)
  auto jth_largest = [&](const TickRec* rec, int q0, int q1, int bits, int32_t j) -> int32_t {
    int32_t v = 0;
    for (int b = bits - 1; b >= 0; --b) {
      const int32_t cand = v | (int32_t)(1u << b);
      uint32_t n = 0;
      for (int q = q0; q < q1; ++q) {
        const TickRec r = rec[q];
        const int32_t* src = a.in + r.off;
        for (int i = tid; i < r.cnt; i += 256) n += src[i] >= cand ? 1u : 0u;
      }
      if (block_sum(n) >= (uint32_t)j) v = cand;
    }
    return v;
  };
  for (uint32_t it = blockIdx.x; it < n_deep; it += gridDim.x) {
    const int64_t c = a.deep_list[it];
    const int32_t j = a.plan[c].j;               // beyond 64; beyond 8192 for DYN_TP_RAW cells
    const TickRec* rec = a.rec + c * T;
    int32_t mx = 0;
    for (int q = 0; q < T; ++q) {
      const TickRec r = rec[q];
      const int32_t* src = a.in + r.off;
      for (int i = tid; i < r.cnt; i += 256) mx = max(mx, src[i]);
    }
    mx = block_max(mx);
    const int bits = 32 - __builtin_clz((uint32_t)mx | 1u);   // mx >= 0: at most 31
    const int32_t xj = jth_largest(rec, 0, T, bits, j);
    if (tid == 0) a.plan[c].xj = xj;
    // sorts s_val[0 .. n_sort) descending (bitonic, padded to a power of two) and writes its first n_out entries to dst
    auto sort_and_store = [&](int n_sort, int n_out, int32_t* dst) {
      int n2 = 2;
      while (n2 < n_sort) n2 <<= 1;              // at most 8192
      for (int i = n_sort + tid; i < n2; i += 256) s_val[i] = (int32_t)0x80000000;
      __syncthreads();
      for (int k = 2; k <= n2; k <<= 1)
        for (int d = k >> 1; d > 0; d >>= 1) {
          for (int i = tid; i < n2; i += 256) {
            const int o = i ^ d;
            if (o > i) {
              const int32_t u = s_val[i], v = s_val[o];
              const bool down = (i & k) == 0;    // descending runs first: the whole array ends descending
              if (down ? u < v : u > v) { s_val[i] = v; s_val[o] = u; }
            }
          }
          __syncthreads();
        }
      for (int i = tid; i < n_out; i += 256) dst[i] = s_val[i];
      __syncthreads();                           // s_val is reused
    };
    for (int q = 0; q < T; ++q) {
      const TickRec r = rec[q];
      if (r.cnt == 0) continue;                  // block-uniform
      const int32_t* src = a.in + r.off;
      int32_t* dst = a.top + r.off;
      if (r.cnt <= kDeepCap) {
        for (int i = tid; i < r.cnt; i += 256) s_val[i] = src[i];
        sort_and_store(r.cnt, r.cnt < j ? r.cnt : j, dst);
      } else if (j > kDeepCap) {                 // block-uniform: neither the tick nor its j largest fit: sorted piece by piece
        for (int base = 0; base < r.cnt; base += kDeepCap) {
          const int n = r.cnt - base < kDeepCap ? r.cnt - base : kDeepCap;
          for (int i = tid; i < n; i += 256) s_val[i] = src[base + i];
          sort_and_store(n, n, dst + base);
        }
        if (tid == 0) a.rec[c * T + q].off = r.off | DYN_TICK_PIECES;
      } else {                                   // more than 8192 requests, of which the j <= 8192 largest are wanted
        const int32_t thr = jth_largest(rec, q, q + 1, bits, j);
        if (tid == 0) s_fill = 0u;
        __syncthreads();
        for (int i = tid; i < r.cnt; i += 256) {
          const int32_t v = src[i];
          if (v > thr) {                         // fewer than j of them
            const uint32_t at = atomicAdd(&s_fill, 1u);
            if (at < (uint32_t)kDeepCap) s_val[at] = v;
          }
        }
        __syncthreads();
        const int got = (int)min(s_fill, (uint32_t)j);
        for (int i = got + tid; i < j; i += 256) s_val[i] = thr;
        sort_and_store(j, j, dst);
      }
    }
  }
}

// ---- evaluation of the (cell, configuration) space -----------------------------------------------
// A tick's candidates (descending input lengths x its prefill time) against the sorted list
// s[0] >= ... >= s[JF-1]: once one of them cannot enter the list in any lane, the rest of
// that tick cannot either.
// Lengths below `xmin` (block-uniform) cannot reach the cell's percentile under any configuration of the block.
template <int JF>
__device__ __forceinline__ void offer_tick(double (&s)[JF], const int32_t* s_top, int T, int q, int nc, int xmin, double pf) {
  for (int x = 0; x < nc; ++x) {
    const int len = __builtin_amdgcn_readfirstlane(s_top[x * T + q]);
    if (len < xmin) break;
    double v = (double)len * pf;
    if (__ballot(v > s[JF - 1]) == 0) break;
#pragma unroll
    for (int i = 0; i < JF; ++i) {
      const double hi = max_num(s[i], v);
      v = min_num(s[i], v);
      s[i] = hi;
    }
  }
}

// Power of the configuration at load 0: what table_lookup returns for it (bracket 0, weight 0 on the second load point).
template <bool TWO>
__device__ __forceinline__ double idle_power(const Lookup& L) {
  const double a = L.lo[2];
  return TWO ? L.omu * a + L.u * L.hi[2] : a;
}

// The four largest tick TBTs with their request counts (descending; ties keep the earlier tick first).
struct TbtTop {
  double tb[4];
  int32_t cnt[4];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < 4; ++i) { tb[i] = -__builtin_inf(); cnt[i] = 0; }
  }
  __device__ __forceinline__ void offer(double v, int32_t c) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool gt = v > tb[i];
      const double tv = tb[i];
      const int32_t tc = cnt[i];
      tb[i] = gt ? v : tv;
      cnt[i] = gt ? c : tc;
      v = gt ? tv : v;
      c = gt ? tc : c;
    }
  }
  __device__ __forceinline__ double jth(int32_t j) const {    // the kept ticks hold at least j requests
    double r = tb[3];
    int32_t cum = 0;
    bool found = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      cum += cnt[i];
      const bool hit = !found && cum >= j;
      r = hit ? tb[i] : r;
      found = found || hit;
    }
    return r;
  }
};

struct WalkOut {
  double e, ttft, tbt;
  bool ov;
};

// One walk over the ticks of a cell with lists, in time order, two look-ups in flight.  The cell's j <= JF largest scaled
// candidates go through a sorted list that starts with JF - j copies of +inf, so that its last entry is the j-th
// largest of what was inserted.  SPARSE: the TBT percentile from the four largest tick TBTs, else the largest tick TBT.
template <int JF, bool SPARSE, int AXIS, bool TWO>
__device__ __forceinline__ WalkOut walk_ticks(const Lookup& L, int T, int j, const double* s_load, const int32_t* s_cnt,
                                              const int32_t* s_top, int xmin, double nd, double tick_s) {
  double s[JF];
#pragma unroll
  for (int i = 0; i < JF; ++i) s[i] = i < JF - j ? __builtin_inf() : -__builtin_inf();
  double e = 0.0, tbmax = -__builtin_inf();
  TbtTop tt;
  if (SPARSE) tt.clear();
  bool ov = false;
  auto one = [&](int q, int c, const Looked& r) {
    if (SPARSE) tt.offer(r.v[1], c); else tbmax = max_num(tbmax, r.v[1]);
    offer_tick<JF>(s, s_top, T, q, c < j ? c : j, xmin, r.v[0]);
  };
  // a tick without requests has load 0: the tables at their first load point, no look-up
  const double e_idle = (nd * idle_power<TWO>(L)) * tick_s;
  int q = 0;
  for (; q + 2 <= T; q += 2) {
    const int c0 = s_cnt[q], c1 = s_cnt[q + 1];                 // block-uniform
    if (c0 > 0 && c1 > 0) {
      const double load[2] = {s_load[q], s_load[q + 1]};
      Looked r[2];
      table_lookups<AXIS, TWO, kAllColumns, 2>(L, load, r);
      ov = ov | r[0].ov | r[1].ov;
      e += (nd * r[0].v[2]) * tick_s;                // ticks in time order
      e += (nd * r[1].v[2]) * tick_s;
      one(q, c0, r[0]);
      one(q + 1, c1, r[1]);
    } else {
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const int cd = d ? c1 : c0;
        if (cd > 0) {
          const Looked r = table_lookup<AXIS, TWO>(L, s_load[q + d]);
          ov = ov | r.ov;
          e += (nd * r.v[2]) * tick_s;
          one(q + d, cd, r);
        } else {
          e += e_idle;
        }
      }
    }
  }
  if (q < T) {
    const int c = s_cnt[q];
    if (c > 0) {
      const Looked r = table_lookup<AXIS, TWO>(L, s_load[q]);
      ov = ov | r.ov;
      e += (nd * r.v[2]) * tick_s;
      one(q, c, r);
    } else {
      e += e_idle;
    }
  }
  WalkOut r;
  r.e = e; r.ov = ov; r.ttft = s[JF - 1];
  r.tbt = SPARSE ? tt.jth(j) : tbmax;
  return r;
}

// A plan read by scalar loads: it is the same for the wave, and written by an earlier kernel.
typedef __attribute__((address_space(4))) TickPlan ScalarPlan;
__device__ __forceinline__ TickPlan load_plan(const TickPlan* at) {
  const ScalarPlan* p = (const ScalarPlan*)at;
  TickPlan r;
  r.j = p->j; r.xj = p->xj; r.flags = p->flags; r.place = p->place;
  return r;
}

typedef const __attribute__((address_space(4))) TickRec ScalarRec;   // the same of its ticks

// Of a cell that needs no lists, as bits: which ticks hold requests, which hold requests of length x_j and whose loads come near the
// largest; the largest load, 0 if no tick holds requests.
struct TickMask {
  uint64_t some, eq, top;
  double top_load;
};
// A tick per lane.  Loads are compared by their high words (loads >= 0 order like their bits): a step is 2^-20 of the load or less, and
// half of that at least, so a load within DYN_TICK_NEAR of the largest is two steps away at most.
__device__ __forceinline__ TickMask tick_mask(const TickRec& r, bool asks, int T, int lane) {
  static_assert(DYN_TICK_NEAR == 0x1p-20, "a step of the high word");
  TickMask m;
  if (T <= 2) {                                  // not worth the exchange between the lanes: 7500 cells of one tick and 2048 candidates 148 us, 142
    m.some = m.eq = 0;
    m.top_load = 0.0;
    for (int q = 0; q < T; ++q) {
      if (__builtin_amdgcn_readlane(r.cnt, q) <= 0) continue;
      m.some |= 1u << q;
      if (asks && __builtin_amdgcn_readlane((int)r.off, q) > 0) m.eq |= 1u << q;
      m.top_load = fmax(m.top_load, lane_f64(r.load, q));
    }
    m.top = m.some;
    return m;
  }
  const bool some = lane < T && r.cnt > 0;
  m.some = __ballot(some);
  m.eq = __ballot(some && asks && (int32_t)r.off > 0);
  const int32_t hi = some ? (int32_t)((uint64_t)__double_as_longlong(r.load) >> 32) : -0x7FFFFFFF;
  const int32_t most = wave_max_i32(hi);
  m.top = __ballot(some && hi >= most - 2);
  m.top_load = 0.0;
  uint64_t left = __ballot(some && hi == most);
  if (left) m.top_load = lane_f64(r.load, __builtin_ctzll(left));
  for (left &= left - 1; left; left &= left - 1) m.top_load = fmax(m.top_load, lane_f64(r.load, __builtin_ctzll(left)));
  return m;
}

// The walk without lists, in time order.  The TBT percentile is the largest tick TBT, which only ticks whose loads come near the
// largest can have (dyn_profile.d_steep; where a candidate's row does not say so, and with rows between two frequencies, all are
// asked); SPARSE: it comes from the four largest tick TBTs.  The TTFT percentile is x_j times the prefill time of rank `place` (bit
// 31: from below) among the ticks, each counted as often as it holds requests of length x_j (`off`): where that is one tick its
// own, else the four largest (smallest) are kept with their counts.  So most ticks are asked for their power only: they go through a loop
// of their own that touches nothing but the energy.  What a tick is asked about itself is a bit of a mask in scalar registers, and
// whether any is overloaded is asked of the largest load (a rounded quotient is monotone).
template <bool SPARSE, int AXIS, bool TWO>
__device__ __forceinline__ WalkOut walk_masked(const Lookup& L, int T, const TickPlan& pl, const TickRec& rec, ScalarRec* at,
                                               double nd, double tick_s, double e_idle, double steep, int lane) {
  const TickMask m = tick_mask(rec, pl.j > 0, T, lane);
  constexpr int JF = 4;
  double s[JF];
  int wt[JF];
  const double sign = (pl.place & DYN_TIGHT_FROM_BELOW) ? -1.0 : 1.0;
#pragma unroll
  for (int i = 0; i < JF; ++i) { s[i] = -__builtin_inf(); wt[i] = 0; }
  double e = 0.0, tbmax = -__builtin_inf();
  TbtTop tt;
  if (SPARSE) tt.clear();
  const double top_rho = div_by(m.top_load, L.den, L.rden);
  const bool one_eq = (m.eq & (m.eq - 1)) == 0;  // of the cell's j-th largest length there is one, or several in one tick
  uint64_t asked = m.eq | (SPARSE || TWO || __ballot(top_rho < steep) != 0 ? m.some : m.top);
  uint64_t some = m.some;
  double next = at[0].load;
  for (int q = 0;;) {
    const int stop = asked ? __builtin_ctzll(asked) : T;
    for (; q < stop; ++q, some >>= 1) {
      const double load = next;
      next = at[min(q + 1, T - 1)].load;
      if (some & 1) e += (nd * table_lookup<AXIS, TWO, kPower>(L, load).v[2]) * tick_s;
      else e += e_idle;                          // load 0: the tables at their first load point, no look-up
    }
    if (!asked) break;
    const Looked r = table_lookup<AXIS, TWO, kAllColumns>(L, next);
    next = at[min(q + 1, T - 1)].load;
    e += (nd * r.v[2]) * tick_s;
    if (SPARSE) tt.offer(r.v[1], __builtin_amdgcn_readlane(rec.cnt, q)); else tbmax = max_num(tbmax, r.v[1]);
    if (m.eq >> q & 1) {
      double key = r.v[0] * sign;
      if (one_eq) {
        s[0] = key;
      } else if (__ballot(key > s[JF - 1]) != 0) {
        int w_in = __builtin_amdgcn_readlane((int)rec.off, q);
#pragma unroll
        for (int i = 0; i < JF; ++i) {
          const bool gt = key > s[i];
          const double tk = s[i];
          const int tw = wt[i];
          s[i] = gt ? key : tk;
          wt[i] = gt ? w_in : tw;
          key = gt ? tk : key;
          w_in = gt ? tw : w_in;
        }
      }
    }
    ++q; some >>= 1;
    asked &= asked - 1;
  }
  WalkOut o;
  o.e = e;
  o.ov = top_rho > L.rho_max;
  double pick = s[0];
  if (!one_eq) {
    const int want = (int)(pl.place & ~DYN_TIGHT_FROM_BELOW);
    pick = s[JF - 1];
    int cum = 0;
    bool found = false;
#pragma unroll
    for (int i = 0; i < JF; ++i) {
      cum += wt[i];
      const bool hit = !found && cum >= want;
      pick = hit ? s[i] : pick;
      found = found || hit;
    }
  }
  o.ttft = (double)pl.xj * (pick * sign);
  o.tbt = SPARSE ? tt.jth(pl.j) : tbmax;
  return o;
}

// Per-thread state of one configuration inside a (class, tile) block.
struct CfgState {
  Lookup L;
  double nd, slo_ttft, slo_tbt, idle_term;
  uint32_t fl_budget, koff;
  int row_lo, k0;                // k0: the wave's first configuration
  bool live;
};

// The constants of configuration k_raw (>= K: a copy of the last one that stores nothing): `g` is
// block-uniform; the table rows are either the block's LDS copy (LDS) or global memory.
template <bool LDS, int AXIS>
__device__ __forceinline__ void load_config(const TickArgs& a, int g, int k_raw, const double* s_tab, const Axis& axis,
                                            const uint16_t* s_js, CfgState* st) {
  const SpaceArgs& sa = a.s;
  const int n_rho = sa.n_rho;
  st->live = k_raw < sa.K;                // every lane stays alive for the wave reduction
  const DevCfg c = sa.cfg[st->live ? k_raw : sa.K - 1];
  st->row_lo = c.row_lo;
  const size_t grow = (size_t)g * sa.n_tp_f;
  const double ml_lo = sa.ml[grow + c.row_lo], ml_hi = sa.ml[grow + c.row_hi];
  const double p0_lo = sa.pw0[grow + c.row_lo], p0_hi = sa.pw0[grow + c.row_hi];
  const bool two_rows = c.u != 0.0;
  Lookup& L = st->L;
  L.u = c.u;
  L.omu = 1.0 - c.u;
  const double ml = two_rows ? L.omu * ml_lo + c.u * ml_hi : ml_lo;
  L.den = c.nd * ml;
  L.rden = 1.0 / L.den;
  use_axis<AXIS>(sa.axis, axis, s_js, &L);
  if (LDS) {      // kept apart so that the address space of the rows is known at compile time
    L.lo = s_tab + (size_t)c.slot_lo * DYN_SLOT_STRIDE(n_rho);
    L.hi = s_tab + (size_t)c.slot_hi * DYN_SLOT_STRIDE(n_rho);
  } else {
    L.lo = sa.tab + (grow + c.row_lo) * 3 * n_rho;
    L.hi = sa.tab + (grow + c.row_hi) * 3 * n_rho;
  }
  st->nd = c.nd;
  st->slo_ttft = sa.slo_ttft[g];
  st->slo_tbt = sa.slo_tbt[g];
  const int32_t bud = sa.budget[g];
  st->fl_budget = (bud > 0 && c.gpus > bud) ? DYN_F_BUDGET : 0u;
  const double pw0 = two_rows ? L.omu * p0_lo + c.u * p0_hi : p0_lo;
  st->idle_term = sa.idle_w * ((c.nd * pw0) * a.window_s);
  st->k0 = __builtin_amdgcn_readfirstlane(k_raw);   // tiles are multiples of 64 configurations wide
  st->koff = (uint32_t)k_raw * 8u;        // where it is live
}

// The rows a tile needs, a wave a row: which row it is comes by a scalar load, and the loads of several are in flight together.
__device__ __forceinline__ void stage_rows(const SpaceArgs& sa, int g, int tile, double* s_tab) {
  const int per_slot = 3 * sa.n_rho, lane = threadIdx.x & (DYN_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE), waves = blockDim.x / DYN_WAVE;
  const int32_t* rows = sa.tile_rows + tile * sa.n_slot;
  const double* base = sa.tab + (size_t)g * sa.n_tp_f * per_slot;
#pragma unroll 2
  for (int slot = wave; slot < sa.n_slot; slot += waves) {
    const double* src = base + (size_t)max(rows[slot], 0) * per_slot;
    double* dst = s_tab + slot * DYN_SLOT_STRIDE(sa.n_rho);
    double v[4];
    for (int i0 = 0; i0 < per_slot; i0 += 4 * DYN_WAVE) {
#pragma unroll
      for (int q = 0; q < 4; ++q) if (i0 + q * DYN_WAVE + lane < per_slot) v[q] = src[i0 + q * DYN_WAVE + lane];
#pragma unroll
      for (int q = 0; q < 4; ++q) if (i0 + q * DYN_WAVE + lane < per_slot) dst[i0 + q * DYN_WAVE + lane] = v[q];
    }
  }
}

// A wave-uniform address that stays in scalar registers: the compiler otherwise adds the lane's offset to the array's start once, outside
// the loop over the cells, and keeps a 64-bit address per array in vector registers it does not have (the reloads then wait for the
// stores before them).
template <typename T>
__device__ __forceinline__ auto row_start(T* p) {
  uint64_t at = uniform_u64((uint64_t)(uintptr_t)p);
  asm("" : "+s"(at));
  return (__attribute__((address_space(1))) char*)at;
}

// Flags, streaming stores of the four outputs and the wave's partial selection for one cell.
__device__ __forceinline__ void emit_cell(const SpaceArgs& sa, const CfgState& st, size_t cell, bool empty, bool ov, double e,
                                          double p_ttft, double p_tbt) {
  uint32_t fl = st.fl_budget;
  if (ov) fl |= DYN_F_OVERLOAD;
  if (p_ttft > st.slo_ttft) fl |= DYN_F_TTFT;
  if (p_tbt > st.slo_tbt) fl |= DYN_F_TBT;
  if (!fl) fl = DYN_F_FEASIBLE;
  if (empty) fl |= DYN_F_EMPTY;
  const double cost = e + st.idle_term;
  if (st.live) {
    const size_t row = cell * (size_t)sa.K;
    uint32_t koff = st.koff;
    asm("" : "+v"(koff));                    // 32 bits up to the store, which widens it itself
    __builtin_nontemporal_store(e, (__attribute__((address_space(1))) double*)(row_start(sa.energy + row) + koff));
    __builtin_nontemporal_store(p_ttft, (__attribute__((address_space(1))) double*)(row_start(sa.p99_ttft + row) + koff));
    __builtin_nontemporal_store(p_tbt, (__attribute__((address_space(1))) double*)(row_start(sa.p99_tbt + row) + koff));
    __builtin_nontemporal_store((uint8_t)fl, (__attribute__((address_space(1))) uint8_t*)(row_start(sa.flags + row) + (koff >> 3)));
  }
  // least cost among this wave's feasible configurations (costs >= +0 order like their bits)
  const bool feas = st.live && (fl & DYN_F_FEASIBLE);
  const uint64_t bits = (uint64_t)__double_as_longlong(cost);
  const uint32_t hi = feas ? (uint32_t)(bits >> 32) : 0xFFFFFFFFu;
  const uint32_t lo = feas ? (uint32_t)bits : 0xFFFFFFFFu;
  const uint32_t mh = wave_min_u32(hi);
  uint64_t win = __ballot(feas && hi == mh);
  if (__popcll(win) > 1) {
    const uint32_t mlo = wave_min_u32(hi == mh ? lo : 0xFFFFFFFFu);
    win = __ballot(feas && hi == mh && lo == mlo);
  }
  const int wl = win ? __builtin_ctzll(win) : 0;
  if ((int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) == wl) {
    auto* p = (__attribute__((address_space(1))) SelPart*)row_start(sa.part + (cell * (size_t)sa.n_wslot + st.k0 / DYN_WAVE));
    p->cost = win ? cost : __builtin_inf();
    p->energy = win ? e : __builtin_inf();
    p->k = win ? st.k0 + wl : -1;
    p->pad = 0;
  }
}

// A block walks a run of windows of one (class, tile): the empty cells, the cells that are not evaluated and
// the cells the cell kernel left to this kernel (the others are the general kernel's).  The next cell's
// candidate lists are kept in flight (NPRE registers per thread) while the current one is evaluated.
// LDS: [table rows n_slot*3*n_rho] [load axis]
//      [per window of the block, per tick: load] [the same: request count] [the same: list offset]
//      [per window: plan] [two buffers of candidate lists, [position][tick]] [bucket index (16-bit)]
template <int TB, bool LDS, int AXIS, bool TWO>
__global__ __launch_bounds__(DYN_MAX_TILE) __attribute__((amdgpu_waves_per_eu(4, 4))) void tick_space_kernel(TickArgs a) {
  constexpr int NPRE = kFastDepth * TB / DYN_WAVE;   // blocks have at least 64 threads; n_tick <= TB
  extern __shared__ double smem[];
  const SpaceArgs& sa = a.s;
  const int tile = blockIdx.x % sa.n_tile;
  const int g = (blockIdx.x / sa.n_tile) % sa.G;
  const int chunk = blockIdx.x / (sa.n_tile * sa.G);
  const int n_rho = sa.n_rho, T = a.n_tick;
  const int w0 = chunk * sa.win_per_block;
  const int w1 = min(w0 + sa.win_per_block, sa.n_window);

  double* s_tab = smem;
  const Axis axis = place_axis<AXIS>(smem + (LDS ? (size_t)sa.n_slot * DYN_SLOT_STRIDE(n_rho) : 0), n_rho, sa.axis.n_bucket);
  uint32_t* s_ratio = (uint32_t*)axis.end;                      // [4] per wave (two doubles' room)
  double* s_load = (double*)s_ratio + 2;                        // [win_per_block][T]
  TickPlan* s_plan = (TickPlan*)(s_load + sa.win_per_block * T);   // [win_per_block]
  int32_t* s_cnt = (int32_t*)(s_plan + sa.win_per_block);       // [win_per_block][T] requests per tick
  uint32_t* s_off = (uint32_t*)(s_cnt + sa.win_per_block * T);  // [win_per_block][T] start of the tick's list
  int32_t* s_top = (int32_t*)(s_off + sa.win_per_block * T);    // [2][kFastDepth][T]
  uint16_t* s_js = (uint16_t*)(s_top + 2 * T * kFastDepth);     // [n_bucket + 1]

  // a block without a cell that is walked with lists has nothing to stage; most traces have no such cell at all
  if (a.counters[3] == 0u) return;
  bool any = false;
  for (int w = w0; w < w1; ++w) {
    const TickPlan p = a.plan[(size_t)w * sa.G + g];
    any = any || (p.j > 0 && !(p.flags & (DYN_TP_GENERAL | DYN_TP_TIGHT)));
  }
  if (!any) return;                                             // block-uniform

  if (LDS) stage_rows(sa, g, tile, s_tab);
  stage_axis<AXIS>(sa.axis, axis, s_js);
  for (int i = threadIdx.x; i < (w1 - w0) * T; i += blockDim.x) {   // the ticks of this block's cells
    const int dw = i / T, q = i - dw * T;
    const TickRec r = a.rec[((size_t)(w0 + dw) * sa.G + g) * T + q];
    s_load[i] = r.load;
    s_cnt[i] = r.cnt;
    s_off[i] = r.off;
  }
  for (int i = threadIdx.x; i < w1 - w0; i += blockDim.x) s_plan[i] = a.plan[(size_t)(w0 + i) * sa.G + g];
  {
    // How far apart a configuration's per-tick prefill times can lie: theta = least / largest entry of its table
    // row(s), as a float rounded down; the block uses the smallest theta of its configurations.
    const int k_mine = min(tile * sa.tile + (int)threadIdx.x, sa.K - 1);
    const DevCfg c = sa.cfg[k_mine];
    const double* span = a.pfspan + 2 * ((size_t)g * sa.n_tp_f);
    double mn = span[2 * c.row_lo], mx = span[2 * c.row_lo + 1];
    if (c.u != 0.0) {
      mn = min_num(mn, span[2 * c.row_hi]);
      mx = max_num(mx, span[2 * c.row_hi + 1]);
    }
    const float th = (mx > 0.0 && mn > 0.0) ? (float)(mn / mx) * 0.999999f : 0.0f;   // below mn / mx by 2^-21 at least
    const uint32_t bits = wave_min_u32(__float_as_uint(th));                          // floats >= 0 order like their bits
    if ((threadIdx.x & (DYN_WAVE - 1)) == 0) s_ratio[threadIdx.x / DYN_WAVE] = bits;
  }
  __syncthreads();
  CfgState st;
  load_config<LDS, AXIS>(a, g, tile * sa.tile + (int)threadIdx.x, s_tab, axis, s_js, &st);
  uint32_t ratio_bits = s_ratio[0];
  for (int i = 1; i < (int)blockDim.x / DYN_WAVE; ++i) ratio_bits = min(ratio_bits, s_ratio[i]);
  const double theta = (double)__uint_as_float(ratio_bits);

  // the cells this kernel walks with candidates: their lists are staged [position][tick]
  auto listed = [&](const TickPlan& p) { return p.j > 0 && !(p.flags & (DYN_TP_GENERAL | DYN_TP_TIGHT)); };
  int32_t pre[NPRE];
  auto prefetch = [&](int w) {
    if (w >= w1) return;
    const TickPlan p = s_plan[w - w0];
    if (!listed(p)) return;
    const int n = p.j * T;                     // at most kFastDepth * TB
    const int32_t* cnt_w = s_cnt + (w - w0) * T;
    const uint32_t* off_w = s_off + (w - w0) * T;
#pragma unroll
    for (int r = 0; r < NPRE; ++r) {
      const int i = threadIdx.x + r * blockDim.x;
      if (i < n) {
        const int pos = i / T, q = i - pos * T;
        pre[r] = pos < cnt_w[q] ? a.top[(size_t)off_w[q] + pos] : 0;   // a tick's list has min(j, count) entries
      }
    }
  };
  prefetch(w0);
  int buf = 0;
  for (int w = w0; w < w1; ++w) {
    const size_t cell = (size_t)w * sa.G + g;
    const int32_t* cnt_w = s_cnt + (w - w0) * T;
    const double* load_w = s_load + (w - w0) * T;
    const TickPlan pl = s_plan[w - w0];
    if (!listed(pl)) {                           // block-uniform: another kernel's cell
      prefetch(w + 1);
      continue;
    }
    const int j = pl.j;
    // two buffers: the lists of the cell before this one may still be read by slower waves
    int32_t* top_w = s_top + buf * (T * kFastDepth);
    {
      buf ^= 1;
      const int n = j * T;
#pragma unroll
      for (int r = 0; r < NPRE; ++r) {
        const int i = threadIdx.x + r * blockDim.x;
        if (i < n) top_w[i] = pre[r];
      }
      __syncthreads();
    }
    prefetch(w + 1);

    // Pruning: a request of length a < x_j * theta has, under every configuration of the block, TTFT = a * pf <
    // x_j * (least pf of that configuration) <= the TTFT of each of the j requests of length >= x_j: it lies below the
    // percentile, which is the j-th largest of what is left all the same.  With flat prefill tables what is left are
    // the cell's j largest lengths, whichever ticks hold them.
    const int xmin = (int)((double)pl.xj * theta);
    WalkOut o;
    if (pl.flags & DYN_TP_DENSE) {
      if (j == 1) o = walk_ticks<1, false, AXIS, TWO>(st.L, T, j, load_w, cnt_w, top_w, xmin, st.nd, a.tick_s);
      else if (j <= 4) o = walk_ticks<4, false, AXIS, TWO>(st.L, T, j, load_w, cnt_w, top_w, xmin, st.nd, a.tick_s);
      else if (j <= 8) o = walk_ticks<8, false, AXIS, TWO>(st.L, T, j, load_w, cnt_w, top_w, xmin, st.nd, a.tick_s);
      else o = walk_ticks<kFastDepth, false, AXIS, TWO>(st.L, T, j, load_w, cnt_w, top_w, xmin, st.nd, a.tick_s);
    } else {
      if (j <= 4) o = walk_ticks<4, true, AXIS, TWO>(st.L, T, j, load_w, cnt_w, top_w, xmin, st.nd, a.tick_s);
      else o = walk_ticks<kFastDepth / 2, true, AXIS, TWO>(st.L, T, j, load_w, cnt_w, top_w, xmin, st.nd, a.tick_s);
    }
    emit_cell(sa, st, cell, false, o.ov, o.e, o.ttft, o.tbt);
  }
}

// The same block mapping for the cells that need no lists: empty cells, cells that are not evaluated, and the cells
// settled by their ticks' requests of length x_j (DYN_TP_TIGHT).  A wave takes a cell's ticks from global memory into its lanes, the
// next cell's while it walks this one; nothing is staged per cell and the block has no barrier after its set-up.
// LDS: [load axis] [table rows] [bucket index (16-bit)]
// Waves a SIMD: six leave 80 registers, which do for the even form; the others lack five there, and their reloads wait for the stores before them (36 000 cells of 576
// candidates on uneven points, 12 ticks 920 us, with five waves 870; one tick 445, 394).
constexpr int tight_waves(int axis, bool two) { return axis == DYN_AXIS_EVEN && !two ? 6 : 5; }
template <bool LDS, int AXIS, bool TWO>
__global__ __launch_bounds__(DYN_MAX_TILE) __attribute__((amdgpu_waves_per_eu(tight_waves(AXIS, TWO), tight_waves(AXIS, TWO)))) void tick_tight_walk_kernel(TickArgs a) {
  extern __shared__ double smem[];
  const SpaceArgs& sa = a.s;
  const int tile = blockIdx.x % sa.n_tile;
  const int g = (blockIdx.x / sa.n_tile) % sa.G;
  const int chunk = blockIdx.x / (sa.n_tile * sa.G);
  const int n_rho = sa.n_rho, T = a.n_tick;
  // the first n_long chunks are of win_long windows, the rest of win_per_block
  const int w0 = min(chunk, a.n_long) * a.win_long + max(chunk - a.n_long, 0) * sa.win_per_block;
  const int w1 = min(w0 + (chunk < a.n_long ? a.win_long : sa.win_per_block), sa.n_window);
  const int lane = threadIdx.x & (DYN_WAVE - 1);

  const Axis axis = place_axis<AXIS>(smem, n_rho, sa.axis.n_bucket);   // at the start: its place is an offset in the instruction
  double* s_tab = axis.end;
  uint16_t* s_js = (uint16_t*)(s_tab + (LDS ? (size_t)sa.n_slot * DYN_SLOT_STRIDE(n_rho) : 0));   // [n_bucket + 1]

  auto mine = [](const TickPlan& p) {
    return p.j == 0 || ((p.flags & DYN_TP_TIGHT) && !(p.flags & DYN_TP_GENERAL));
  };
  bool any = false;
  for (int w = w0; w < w1 && !any; ++w) any = mine(load_plan(a.plan + (size_t)w * sa.G + g));
  if (!any) return;                                             // block-uniform

  if (LDS) stage_rows(sa, g, tile, s_tab);
  stage_axis<AXIS>(sa.axis, axis, s_js);
  CfgState st;
  load_config<LDS, AXIS>(a, g, tile * sa.tile + (int)threadIdx.x, s_tab, axis, s_js, &st);
  // the least utilization from which a tick's TBT is above every other's when its load is, over the wave's candidates
  // (by the high word, one up: infinity stays)
  const uint32_t steep_hi = wave_max_u32((uint32_t)((uint64_t)__double_as_longlong(a.steep[(size_t)g * sa.n_tp_f + st.row_lo]) >> 32));
  const double steep = __longlong_as_double((long long)((uint64_t)min(steep_hi + 1u, 0x7FF00000u) << 32));
  const size_t cell0 = (size_t)w0 * sa.G + g;
  const TickRec* rec = a.rec + cell0 * T + min(lane, T - 1);
  const TickPlan* plan = a.plan + cell0;
  TickRec next = *rec;
  TickPlan next_plan = load_plan(plan);
  __syncthreads();
  const double e_idle = (st.nd * idle_power<TWO>(st.L)) * a.tick_s;
  for (int w = w0; w < w1; ++w) {
    const TickRec r = next;
    const TickPlan pl = next_plan;
    if (w + 1 < w1) {
      rec += (size_t)sa.G * T;
      plan += sa.G;
      next = *rec;
      next_plan = load_plan(plan);
    }
    if (!mine(pl)) continue;                     // block-uniform
    const bool empty = pl.j == 0;
    const size_t cell = (size_t)w * sa.G + g;
    WalkOut o;
    if (empty || (pl.flags & DYN_TP_DENSE)) {
      o = walk_masked<false, AXIS, TWO>(st.L, T, pl, r, (ScalarRec*)(a.rec + cell * T), st.nd, a.tick_s, e_idle, steep, lane);
      if (empty) o.ttft = o.tbt = 0.0;           // its ticks' power at load 0 remains
    } else {
      o = walk_masked<true, AXIS, TWO>(st.L, T, pl, r, (ScalarRec*)(a.rec + cell * T), st.nd, a.tick_s, e_idle, steep, lane);
    }
    emit_cell(sa, st, cell, empty, o.ov, o.e, o.ttft, o.tbt);
  }
}

// Weighted order statistic over the ticks: the largest value v among those of the ticks with weight > 0 such that the
// ticks with a value >= v weigh at least `need` together (ticks are taken in descending order of value, equal
// values together).  strip[q * NT + tid] is this thread's value of tick q.
__device__ __forceinline__ double weighted_from_top(const double* strip, const int32_t* weight, int T, int NT, int need, int tid) {
  double prev = __builtin_inf(), val = 0.0;
  while (need > 0) {
    double best = -__builtin_inf();
    int c = 0;
    for (int q = 0; q < T; ++q) {
      const int wq = weight[q];
      if (wq == 0) continue;
      const double v = strip[q * NT + tid];
      const bool lt = v < prev;
      const bool gt = lt && v > best;
      const bool eq = lt && v == best;
      c = gt ? wq : (eq ? c + wq : c);
      best = gt ? v : best;
    }
    if (c == 0) break;                       // cannot happen while the weights add up to at least `need`
    need -= c;
    prev = best;
    val = best;
  }
  return val;
}

// The cells the cell kernel left to this kernel, (cell, tile) by (cell, tile), the items dealt round-robin to a
// fixed grid so that runs of heavy cells spread over the chip.  A block of NT threads takes the tile's
// configurations NT at a time.  One strip in LDS holds a value per (tick, configuration).  Cells whose
// non-empty ticks all hold j requests: one pass over the ticks (energy, largest TBT = the TBT percentile,
// prefill times into the strip).  Other cells: a first pass with the TBTs in the strip, the TBT percentile
// by taking ticks in descending TBT order until j requests are covered, then the look-ups again for the
// prefill times.  The TTFT percentile lies in the bracket [x_j * least, x_j * largest prefill time].  If
// its ends differ but the prefill times are so close that (x_j + 1) * least > x_j * largest, the scaled
// lengths above x_j lie above the bracket and those below it below: the percentile is x_j times the
// prefill time that ranks (j - number of lengths above x_j) among the ticks weighted by their number of
// lengths equal to x_j.  Otherwise the bracket is bisected: a probe value v is ranked in every tick's list
// (binary search on the scaled entries), and either at least j scaled entries are >= v, then the least
// of them is a new lower end, or fewer, then the largest one below v is a new upper end.  Both ends are
// values of the lists from then on, so the search ends with the percentile itself.  A cell with tables (DYN_TP_TABLE) is searched the same way
// over all lengths, a probe ranked by one entry of every tick's table.
// LDS: [load axis] [strip NT x n_tick]
//      [per tick: load] [per tick: count] [per tick: entries listed] [per tick: entries equal to x_j]
//      [per tick: start of its list, then two words] [the cell's lists when they fit] [bucket index]
template <int AXIS, bool TWO>
__global__ __launch_bounds__(DYN_MAX_TILE) void tick_general_kernel(TickArgs a) {
  extern __shared__ double smem[];
  const SpaceArgs& sa = a.s;
  const int n_rho = sa.n_rho, T = a.n_tick;
  const int tid = threadIdx.x, NT = blockDim.x;
  // The table rows stay in global memory (they are read through the caches): consecutive items of a block belong to
  // different classes, and staging a class's rows per item cost more than the look-ups of the item.
  const Axis axis = place_axis<AXIS>(smem, n_rho, sa.axis.n_bucket);
  double* s_strip = axis.end;                                   // [T][NT]
  double* s_load = s_strip + (size_t)T * NT;                    // [T]
  int32_t* s_cnt = (int32_t*)(s_load + T);                      // [T]
  int32_t* s_len = s_cnt + T;                                   // [T] min(j, count)
  int32_t* s_neq = s_len + T;                                   // [T] listed lengths equal to x_j
  uint32_t* s_lbase = (uint32_t*)(s_neq + T);                   // [T] start of the tick's list; [T]: entries staged in LDS + 1, or 0; [T+1]: lengths above x_j
  uint32_t* s_goff = s_lbase + T + 2;                           // [T] start of the tick's list in global memory
  int32_t* s_lists = (int32_t*)(s_goff + T);                    // [kListCap]
  uint16_t* s_js = (uint16_t*)(s_lists + kListCap);             // [n_bucket + 1]

  const uint64_t n_item = (uint64_t)a.counters[1] * (uint64_t)sa.n_tile;   // complete: written by the cell kernel
  if (blockIdx.x >= n_item) return;                              // block-uniform
  stage_axis<AXIS>(sa.axis, axis, s_js);
  for (uint64_t item = blockIdx.x; item < n_item; item += gridDim.x) {
    const size_t cell = a.slow_list[item / (uint64_t)sa.n_tile];
    const int tile = (int)(item % (uint64_t)sa.n_tile);
    const int g = (int)(cell % sa.G);
    __syncthreads();                           // the previous item's LDS data has been consumed
    const TickPlan pl = a.plan[cell];
    const int j = pl.j;
    const bool dense = (pl.flags & DYN_TP_DENSE) != 0;
    const bool tight = (pl.flags & DYN_TP_TIGHT) != 0;   // no lists: per tick the number of requests of length x_j, and the rank among them
    const bool tabled = (pl.flags & DYN_TP_TABLE) != 0;  // no lists: how many requests are at least so long, per tick
    const bool raw = (pl.flags & DYN_TP_RAW) != 0;       // the lists are whole ticks; a tick marked DYN_TICK_PIECES is sorted in pieces of DYN_TICK_DEPTH
    const TickRec* rec = a.rec + cell * T;
    if (tid < DYN_WAVE) {                      // the first wave, a tick per lane: where each tick's list is read from
      TickRec r;
      r.load = 0.0; r.off = 0u; r.cnt = 0;
      if (tid < T) r = rec[tid];
      const bool pieces = raw && (r.off & DYN_TICK_PIECES) != 0u;
      const uint32_t off = raw ? (r.off & ~DYN_TICK_PIECES) : r.off;
      const int len = (tid < T && !tight && !tabled) ? (raw ? r.cnt : min(r.cnt, j)) : 0;
      int incl = len;                          // inclusive prefix over the ticks
#pragma unroll
      for (int d = 1; d < DYN_WAVE; d <<= 1) {
        const int up = __shfl_up(incl, d, DYN_WAVE);
        if (tid >= d) incl += up;
      }
      const uint32_t total = (uint32_t)__builtin_amdgcn_readlane(incl, DYN_WAVE - 1);
      const bool fits = !raw && total <= (uint32_t)kListCap;
      if (tid < T) {
        s_load[tid] = r.load;
        s_cnt[tid] = r.cnt;
        s_len[tid] = pieces ? -len : len;        // negative: a long tick whose list is sorted piece by piece
        s_goff[tid] = off;
        s_lbase[tid] = fits ? (uint32_t)(incl - len) : off;
        if (tight) s_neq[tid] = (int32_t)r.off;
      }
      if (tid == 0) {
        s_lbase[T] = fits ? total + 1u : 0u;   // 0: the lists stay in global memory
        s_lbase[T + 1] = 0u;
      }
    }
    __syncthreads();
    const bool staged = s_lbase[T] != 0u;
    if (staged) {                              // one flat copy: the loads of all ticks are in flight together
      const int total = (int)s_lbase[T] - 1;
#pragma unroll 4
      for (int i = tid; i < total; i += NT) {
        int l = 0, h = T - 1;                  // the tick whose list holds entry i: the last q with s_lbase[q] <= i
        while (l < h) {
          const int mid = (l + h + 1) >> 1;
          if ((int)s_lbase[mid] <= i) l = mid; else h = mid - 1;
        }
        s_lists[i] = a.top[(size_t)s_goff[l] + (uint32_t)(i - (int)s_lbase[l])];
      }
      __syncthreads();
    }
    const int32_t* lists = staged ? s_lists : a.top;
    // the table of a tick: entry i counts its requests of at least t_from + i, 0 <= i <= t_n
    const uint32_t* t_at = a.pool + (tabled ? pl.place : 0u);
    int t_from = 0, t_n = 0, t_stride = 0;
    if (tabled) {                              // block-uniform
      t_from = (int)t_at[0];
      t_n = (int)t_at[1];
      t_stride = (int)t_at[2];
      t_at += DYN_TICK_TABLE_HEAD + t_at[3];
      if (T * (t_n + 1) <= kListCap) {
        for (int i = tid; i < T * (t_n + 1); i += NT) s_lists[i] = (int32_t)t_at[(size_t)(i / (t_n + 1)) * t_stride + i % (t_n + 1)];
        __syncthreads();
        t_at = (const uint32_t*)s_lists;
        t_stride = t_n + 1;
      }
      if (tid < T) {
        const uint32_t* row = t_at + (size_t)tid * t_stride + (pl.xj - t_from);
        s_neq[tid] = (int32_t)(row[0] - row[1]);
        if (row[1]) atomicAdd(&s_lbase[T + 1], row[1]);
      }
    }
    if (tid < T && !tight && !tabled && s_len[tid] < 0) s_neq[tid] = 0;
    if (tid < T && !tight && !tabled && s_len[tid] >= 0) {        // per tick: listed lengths above x_j and equal to it (the list is descending)
      const int len = s_len[tid];
      const int32_t* lq = lists + s_lbase[tid];
      int l = 0, h = len;                      // first entry <= x_j
      while (l < h) {
        const int mid = (l + h) >> 1;
        if (lq[mid] > pl.xj) l = mid + 1; else h = mid;
      }
      const int n_gt = l;
      h = len;                                 // first entry < x_j
      while (l < h) {
        const int mid = (l + h) >> 1;
        if (lq[mid] >= pl.xj) l = mid + 1; else h = mid;
      }
      s_neq[tid] = l - n_gt;
      if (n_gt) atomicAdd(&s_lbase[T + 1], (uint32_t)n_gt);
    }
    if (raw) {                                 // block-uniform: the same two counts of the ticks sorted in pieces, by the whole block (from the trace)
      __syncthreads();
      for (int q = 0; q < T; ++q) {
        const int len = -s_len[q];
        if (len <= 0) continue;
        const int32_t* lq = a.in + s_lbase[q];
        uint32_t n_gt = 0;
        int32_t n_eq = 0;
        for (int i = tid; i < len; i += NT) {
          const int32_t x = lq[i];
          n_gt += x > pl.xj ? 1u : 0u;
          n_eq += x == pl.xj ? 1 : 0;
        }
        if (n_gt) atomicAdd(&s_lbase[T + 1], n_gt);
        if (n_eq) atomicAdd(&s_neq[q], n_eq);
      }
    }
    __syncthreads();
    const double xj = (double)pl.xj;
    const int need_eq = tight ? (int)pl.place : j - (int)s_lbase[T + 1];   // >= 1: fewer than j lengths lie above the j-th largest

    for (int sub = 0; sub < sa.tile; sub += NT) {
      const bool in_tile = sub + (tid & ~(DYN_WAVE - 1)) < sa.tile;   // wave-uniform: a wave past the tile's end stores nothing
      CfgState st;
      load_config<false, AXIS>(a, g, tile * sa.tile + (in_tile ? sub + tid : 0), nullptr, axis, s_js, &st);
      double e = 0.0, pf_min = __builtin_inf(), pf_max = -__builtin_inf(), tb_max = -__builtin_inf();
      bool ov = false;
      const double e_idle = (st.nd * idle_power<TWO>(st.L)) * a.tick_s;
      for (int q = 0; q < T; ++q) {            // energy in time order; the strip takes the prefill times, or first the TBTs
        if (s_cnt[q] == 0) {                   // block-uniform: load 0, and nothing of this tick enters a percentile
          e += e_idle;
          continue;
        }
        const Looked r = table_lookup<AXIS, TWO>(st.L, s_load[q]);
        const double pf = r.v[0];
        ov = r.ov | ov;
        e += (st.nd * r.v[2]) * a.tick_s;
        s_strip[q * NT + tid] = dense ? pf : r.v[1];
        pf_min = min_num(pf_min, pf);
        pf_max = max_num(pf_max, pf);
        tb_max = max_num(tb_max, r.v[1]);
      }
      double p_tbt = tb_max;
      if (!dense) {                            // block-uniform
        p_tbt = weighted_from_top(s_strip, s_cnt, T, NT, j, tid);
        for (int q = 0; q < T; ++q) {
          if (s_cnt[q] == 0) continue;
          s_strip[q * NT + tid] = table_lookup<AXIS, TWO, kPrefill>(st.L, s_load[q]).v[0];
        }
      }
      // TTFT percentile
      double lo = xj * pf_min, hi = xj * pf_max;
      bool open = lo != hi;
      if (tight || (open && xj * pf_max < (xj + 0.5) * pf_min)) {
        // only lengths equal to x_j scale into the bracket: rank the ticks' prefill times by those
        lo = hi = xj * weighted_from_top(s_strip, s_neq, T, NT, need_eq, tid);
        open = false;
      }
      while (open) {
        double v = lo + (hi - lo) * 0.5;
        if (!(v > lo)) v = hi;
        int n_ge = 0;
        double a_min = __builtin_inf(), b_max = -__builtin_inf();
        if (tabled) {                          // the ends are lengths, held by a request or not: the last one standing is
          for (int q = 0; q < T; ++q) {
            if (s_cnt[q] == 0) continue;
            const double pf = s_strip[q * NT + tid];   // above 0, like theta
            int x = (int)(v / pf);             // the least length with x * pf >= v
            while ((double)x * pf < v) ++x;
            while (x > 0 && (double)(x - 1) * pf >= v) --x;
            n_ge += (int)t_at[(size_t)q * t_stride + min(max(x - t_from, 0), t_n)];
            a_min = min_num(a_min, (double)x * pf);
            b_max = max_num(b_max, (double)(x - 1) * pf);
          }
        } else for (int q = 0; q < T; ++q) {
          int len = s_len[q];
          if (len == 0) continue;
          const double pf = s_strip[q * NT + tid];
          const int32_t* lq = lists + s_lbase[q];
          if (len < 0) {                       // block-uniform: a long tick, sorted piece by piece
            len = -len;
            for (int base = 0; base < len; base += DYN_TICK_DEPTH) {
              const int n = len - base < DYN_TICK_DEPTH ? len - base : DYN_TICK_DEPTH;
              const int32_t* lp = lq + base;
              int l = 0, h = n;                // entries [0, l) of the piece are >= v scaled, entries [h, n) are below
              while (l < h) {
                const int mid = (l + h) >> 1;
                const bool ge = (double)lp[mid] * pf >= v;
                l = ge ? mid + 1 : l;
                h = ge ? h : mid;
              }
              n_ge += l;
              if (l > 0) a_min = min_num(a_min, (double)lp[l - 1] * pf);
              if (l < n) b_max = max_num(b_max, (double)lp[l] * pf);
            }
            continue;
          }
          int l = 0, h = len;                  // entries [0, l) are >= v scaled, entries [h, len) are below
          while (l < h) {
            const int mid = (l + h) >> 1;
            const bool ge = (double)lq[mid] * pf >= v;
            l = ge ? mid + 1 : l;
            h = ge ? h : mid;
          }
          n_ge += l;
          if (l > 0) a_min = min_num(a_min, (double)lq[l - 1] * pf);
          if (l < len) b_max = max_num(b_max, (double)lq[l] * pf);
        }
        if (n_ge >= j) lo = a_min; else hi = b_max;
        open = lo < hi;                        // also ends a search that lost its bracket (never with consistent lists)
      }
      if (in_tile) emit_cell(sa, st, cell, false, ov, e, lo, p_tbt);
      __syncthreads();                         // the strip is rewritten by the next group of configurations
    }
  }
}

size_t tick_lds_tail(const TickArgs& a, int32_t n_tick, int32_t win_per_block, int axis) {
  return dyn_axis_lds(a.s.axis, axis) + 2 * sizeof(double) + (size_t)win_per_block * (n_tick * (sizeof(double) + 2 * sizeof(int32_t)) + sizeof(TickPlan)) +
         (size_t)2 * n_tick * kFastDepth * sizeof(int32_t);
}
size_t general_lds_tail(const TickArgs& a, int32_t n_tick, int nt, int axis) {
  return dyn_axis_lds(a.s.axis, axis) + (size_t)n_tick * nt * sizeof(double) + (size_t)n_tick * (sizeof(double) + 5 * sizeof(int32_t)) +
         2 * sizeof(uint32_t) + (size_t)kListCap * sizeof(int32_t);
}
// Threads of a block of the general kernel: the tile's width, less where the strip (one double per tick and
// thread) would pass 32 KB.
int general_threads(const TickArgs& a) {
  const int cap = a.n_tick <= 16 ? 256 : (a.n_tick <= 32 ? 128 : 64);
  return a.s.tile < cap ? a.s.tile : cap;
}
static_assert(256 * 16 * sizeof(double) <= kStripBytes && 128 * 32 * sizeof(double) <= kStripBytes &&
                  64 * DYN_TICK_MAX * sizeof(double) <= kStripBytes,
              "the strip of the general kernel");

template <bool LDS, int AXIS, bool TWO>
void launch_tight_walk(const TickArgs& a, dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  hipLaunchKernelGGL((tick_tight_walk_kernel<LDS, AXIS, TWO>), grid, block, lds, s, a);
}
template <bool LDS, int AXIS, bool TWO>
void launch_space(const TickArgs& a, dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  if (a.n_tick <= 16) hipLaunchKernelGGL((tick_space_kernel<16, LDS, AXIS, TWO>), grid, block, lds, s, a);
  else hipLaunchKernelGGL((tick_space_kernel<DYN_TICK_MAX, LDS, AXIS, TWO>), grid, block, lds, s, a);
}
template <int AXIS, bool TWO>
void launch_general(const TickArgs& a, size_t lds, hipStream_t s) {
  DynTimed timed(DYN_K_TICK_MERGE, s);
  // The items are dealt round-robin to the grid: as many blocks as the device holds at once, so that none starts late.
  const int nt = general_threads(a);
  int per_cu = 0, blocks = kGeneralBlocks;
  if (a.n_cu > 0 && hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, tick_general_kernel<AXIS, TWO>, nt, lds) == hipSuccess &&
      per_cu > 0)
    blocks = per_cu * a.n_cu;
  blocks = (int)std::min<int64_t>(blocks, (int64_t)a.s.n_window * a.s.G * a.s.n_tile);
  hipLaunchKernelGGL((tick_general_kernel<AXIS, TWO>), dim3(blocks), dim3(nt), lds, s, a);
}

template <int V> using Int = std::integral_constant<int, V>;
template <typename L, typename F>
void dispatch_axis(L lds, int axis, bool two, F&& f) {
  auto with = [&](auto x) { if (two) f(lds, x, std::true_type()); else f(lds, x, std::false_type()); };
  if (axis == DYN_AXIS_EVEN) with(Int<DYN_AXIS_EVEN>());
  else if (axis == DYN_AXIS_SINGLE) with(Int<DYN_AXIS_SINGLE>());
  else with(Int<DYN_AXIS_SEARCH>());
}
template <typename F>
void dispatch(bool lds, int axis, bool two, F&& f) {
  if (lds) dispatch_axis(std::true_type(), axis, two, f); else dispatch_axis(std::false_type(), axis, two, f);
}
// Preferences when LDS is short: keep the table rows in LDS first, the quicker form of the load axis second (without it the bracket is
// searched; without the rows the tables are read from global memory).
template <typename Tail>
int axis_that_fits(const TickArgs& a, size_t tab, Tail&& tail) {
  const int axis = dyn_axis(a.s.axis);
  return tail(axis) + tab <= DYN_LDS_BUDGET ? axis : DYN_AXIS_SEARCH;
}

}  // namespace

hipError_t dyn_launch_tick_cell(const TickCellArgs& a, hipStream_t s) {
  const int64_t cells = (int64_t)a.n_window * a.G;
  const int64_t blocks = (cells + kWavesPerBlock - 1) / kWavesPerBlock;
  DynTimed timed(DYN_K_TICK_TOP, s);
  hipLaunchKernelGGL(tick_init_kernel, dim3(1), dim3(1), 0, s, a.counters);
  if (a.flat) hipLaunchKernelGGL(tick_tight_kernel<false>, dim3((unsigned)blocks), dim3(kWavesPerBlock * DYN_WAVE), 0, s, a);
  else hipLaunchKernelGGL(tick_tight_kernel<true>, dim3((unsigned)blocks), dim3(kWavesPerBlock * DYN_WAVE), 0, s, a);
  // Eight waves where that halves the rows a wave holds and the cells are long enough to share, or where cells are too long for
  // four; such a block (33 KB of LDS) waits beside kernels of other streams that fill the device, one of four finds its place.
  // Measured (us of the call; four waves, eight): 4 M requests, 12 500 cells of 30 ticks, prefill by load 988, 1113; 1500 cells of 1
  // tick 630, 684, of 3 819, 852, of 5 flat 142, 114; 1000 of 10 360, 366; 540 cells of 1 M and 12 ticks 266, 256; long cells: 500 of
  // 8000 and 30 ticks flat 2649, 162; 240 of 16 700 and 6 ticks 2758, 126; 100 of 20 000 and 10 ticks 102, 119.
  const int T = a.n_tick;
  const int64_t mean = a.n_req / cells;
  const int64_t rows = (T + 3) / 4 * (mean * 5 / 4 / T / DYN_WAVE + 1);   // of a wave of four in a cell somewhat longer than the mean
  const bool many = T > 4 && ((mean > 1000 && 2 * ((T + 7) / 8) <= (T + 3) / 4) || rows > 128);
  if (many) hipLaunchKernelGGL(tick_tight_block_kernel<kTightManyWaves>, dim3((unsigned)std::min<int64_t>(cells, kTightUnits / kTightManyWaves)), dim3(kTightManyWaves * DYN_WAVE), 0, s, a);
  else hipLaunchKernelGGL(tick_tight_block_kernel<kTightWaves>, dim3((unsigned)std::min<int64_t>(cells, kTightUnits / kTightWaves)), dim3(kTightWaves * DYN_WAVE), 0, s, a);
  hipLaunchKernelGGL(tick_cell_kernel, dim3((unsigned)std::min<int64_t>(blocks, kListBlocks) + long_blocks(a)), dim3(kWavesPerBlock * DYN_WAVE), 0, s, a);
  hipLaunchKernelGGL(tick_deep_kernel, dim3(kDeepBlocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Windows over which the staging (3 us, and 0.12 for every value a thread stages) is 15 % of a block's life, at 0.6 us a tick.
static int64_t stage_windows(const TickArgs& a) {
  const double stage = 3.0 + 0.12 * (double)a.s.n_slot * (3 * a.s.n_rho) / a.s.tile;
  return (int64_t)(stage / (0.15 * 0.6 * a.n_tick)) + 1;
}

// Windows a block of the evaluation kernels walks.  About 8192 blocks keep cells that differ apart from each other; beyond 16
// windows a block gains nothing more from its staged rows (a day of 12 ticks: 10 .. 20 alike).  With few ticks a window is soon
// walked (0.6 us a tick, the chain of one look-up) and the staging would be most of a block's life: such blocks walk until it is 15 % of it, as long as the blocks fill three quarters of the device.  Measured (us of
// the call; 8192 blocks, this): 8000 cells of 1 tick and 252 candidates 68, 47; 2800 of 5 ticks 55, 43; 2300 of 6 and 60 candidates 72,
// 56; 10 800 of 6 and lists 259, 238.  Less again where the per-tick records would not fit beside the table rows.
int32_t dyn_tick_win_per_block(const TickArgs& a) {
  const SpaceArgs& sa = a.s;
  const size_t tab = (size_t)sa.n_slot * DYN_SLOT_STRIDE(sa.n_rho) * sizeof(double);
  const int64_t cell_tiles = (int64_t)sa.n_window * sa.G * sa.n_tile;
  const int64_t for_stage = stage_windows(a);
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(20 * DYN_WAVE / sa.tile, (160 * 1024) / (int64_t)(tab + 8192)));
  const int64_t for_device = cell_tiles / std::max<int64_t>(1, per_cu * a.n_cu * 3 / 4);
  int32_t wpb = (int32_t)std::max<int64_t>(1, std::min<int64_t>(16, std::max((cell_tiles + 8191) / 8192, std::min(for_stage, for_device))));
  while (wpb > 1 && tab + tick_lds_tail(a, a.n_tick, wpb, dyn_axis(sa.axis)) > DYN_LDS_BUDGET) wpb /= 2;
  return wpb;
}

// How the walk without lists cuts a (class, tile)'s windows.  A block spends 7 us on its set-up where the device is full, 0.43 on a tick:
// long blocks lose the least by it, but one that begins last runs alone to its end, and the classes differ (22 to 48 us for the same
// windows, by how many ticks hold requests of the percentile's length).  So where every place on the device has windows enough, blocks of
// many windows come first and leave four rounds of blocks of few.  36 000 cells of 576 candidates and 12 ticks, us of the call: 14
// windows a block 441, 10 436, 20 first and then 7 417, 20 and 5 410, 16 and 5 410, 24 and 8 424.  Other shapes, blocks of one size and of two: 30 ticks 772, 685; 40 ticks
// and 256 candidates 603, 566; 6 ticks and 100 classes 898, 869; 5 ticks and 2048 candidates 697, 672; 12 ticks and 1152 630, 602, and 320 651, 629, and 192 515, 489; 200 load
// points 1019, 868; mostly cells with lists 905, 902.  A block's LDS is its rows and its axis (uneven points 956 without the axis, 918).
static void tight_chunks(TickArgs& a, size_t tab, int axis) {
  SpaceArgs& sa = a.s;
  const int64_t few = std::max<int64_t>(2, std::min<int64_t>(16, stage_windows(a))), many = 4 * few;
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(4 * tight_waves(axis, sa.two_rows) * DYN_WAVE / sa.tile, (160 * 1024) / (int64_t)(tab + dyn_axis_lds(sa.axis, axis))));
  const int64_t places = per_cu * std::max(1, a.n_cu), columns = (int64_t)sa.G * sa.n_tile;
  const int64_t kept = (4 * few * places + columns - 1) / columns;   // windows left to the blocks of few
  a.win_long = (int32_t)many;
  a.n_long = 0;
  if (columns * sa.n_window < 2 * many * places || sa.n_window - kept < many) return;
  a.n_long = (int32_t)((sa.n_window - kept) / many);
  sa.win_per_block = (int32_t)few;
}

hipError_t dyn_launch_tick_space(const TickArgs& a_in, hipStream_t s) {
  TickArgs a = a_in;
  SpaceArgs& sa = a.s;
  sa.win_per_block = dyn_tick_win_per_block(a);
  const int n_chunk = (sa.n_window + sa.win_per_block - 1) / sa.win_per_block;
  const dim3 grid((unsigned)((size_t)n_chunk * sa.G * sa.n_tile)), block(sa.tile);
  const size_t tab = (size_t)sa.n_slot * DYN_SLOT_STRIDE(sa.n_rho) * sizeof(double);
  {
    DynTimed timed(DYN_K_TICK_SPACE, s);         // both walks
    {
    const int32_t wpb_list = sa.win_per_block;
    const int axis = axis_that_fits(a, tab, [&](int x) { return dyn_axis_lds(sa.axis, x); });
    tight_chunks(a, tab, axis);
    const int64_t chunks = a.n_long + (sa.n_window - (int64_t)a.n_long * a.win_long + sa.win_per_block - 1) / sa.win_per_block;
    const dim3 grid_t((unsigned)(chunks * sa.G * sa.n_tile));
    const size_t tail = dyn_axis_lds(sa.axis, axis);
    const bool lds = sa.n_slot > 0 && tab + tail <= DYN_LDS_BUDGET;
    if (!lds && tail > DYN_LDS_BUDGET) return hipErrorInvalidValue;
    const size_t bytes = (lds ? tab : 0) + tail;
    dispatch(lds, axis, a.s.two_rows, [&](auto L, auto S, auto W) {
      launch_tight_walk<decltype(L)::value, decltype(S)::value, decltype(W)::value>(a, grid_t, block, bytes, s);
    });
    sa.win_per_block = wpb_list;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  {
    // With more than a few places a cell the lists are long where the walk takes them, and only some of the cells are the walk's: blocks of
    // few windows keep those apart.  Measured (us of the call; the windows above, about 8192 blocks): 8000 cells of 500 requests, 50 places
    // 924, 889, 25 places 782, 743; 2760 of 1350, 13 places 753, 728; one place: 10 800 of 9 requests 234, 252, 11 300 of 24 290, 295.
    dim3 grid_l = grid;
    if (a.mean_depth > kListedDepth) {
      const int64_t cell_tiles = (int64_t)sa.n_window * sa.G * sa.n_tile;
      sa.win_per_block = std::min(sa.win_per_block, (int32_t)std::max<int64_t>(1, std::min<int64_t>(16, (cell_tiles + 8191) / 8192)));
      grid_l.x = (unsigned)((size_t)((sa.n_window + sa.win_per_block - 1) / sa.win_per_block) * sa.G * sa.n_tile);
    }
    const int axis = axis_that_fits(a, tab, [&](int x) { return tick_lds_tail(a, a.n_tick, sa.win_per_block, x); });
    const size_t tail = tick_lds_tail(a, a.n_tick, sa.win_per_block, axis);
    const bool lds = sa.n_slot > 0 && tab + tail <= DYN_LDS_BUDGET;
    if (!lds && tail > DYN_LDS_BUDGET) return hipErrorInvalidValue;
    const size_t bytes = (lds ? tab : 0) + tail;
    dispatch(lds, axis, a.s.two_rows, [&](auto L, auto S, auto W) {
      launch_space<decltype(L)::value, decltype(S)::value, decltype(W)::value>(a, grid_l, block, bytes, s);
    });
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  }
  {
    const int nt = general_threads(a);
    const int axis = axis_that_fits(a, 0, [&](int x) { return general_lds_tail(a, a.n_tick, nt, x); });
    const size_t tail = general_lds_tail(a, a.n_tick, nt, axis);
    if (tail > DYN_LDS_BUDGET) return hipErrorInvalidValue;
    dispatch(false, axis, a.s.two_rows, [&](auto, auto S, auto W) {
      launch_general<decltype(S)::value, decltype(W)::value>(a, tail, s);
    });
  }
  return hipGetLastError();
}
