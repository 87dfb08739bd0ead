// Per-cell aggregation and rank selection: one wavefront per (window, class) cell streams
// the cell's requests once and produces the exact token sums (the class's load in the
// window, Section III-A "Request loads") and the input length of nearest rank
// ceil(pct*m) (the request whose TTFT is the cell's P99 under every configuration, since
// per-request TTFT = input tokens x a non-negative per-(cell, configuration) factor and
// IEEE multiplication by a non-negative constant is monotone).
//
// Cells of up to 2048 requests are held in registers (32 values per lane at most) and the
// selection is a most-significant-bit-first search on the value: for every bit one
// compare per register row and a scalar population count of the wave mask, no LDS and no
// cross-lane traffic.  The search interval is first narrowed to [lo, max], where lo is the
// j-th largest of the 64 per-lane maxima (j = m - rank + 1; those maxima are elements of
// the cell, so the j-th largest element cannot be below it): for a high percentile only a
// few bits are left.  Larger cells are streamed from global memory by the whole block,
// once for the sums and once per 10-bit digit, through an LDS histogram (radix select).
#include <algorithm>
#include <type_traits>

#include "dyn_device.h"

namespace {

constexpr int kWavesPerBlock = 4;
constexpr int kHistBits = 10;
constexpr int kHistBins = 1 << kHistBits;
constexpr int kRegRowsMax = 32;  // register path handles m <= 64 * kRegRowsMax

struct CellOut {
  int64_t tin, tout;
  uint32_t p99;
  uint32_t orv;
};

// Exact token sums of a register-sized cell the slow way (16-bit halves keep every partial
// sum inside 32 bits: at most 32 values per lane, 2048 per wave); only needed when a token
// count of 2^20 or more makes plain 32-bit sums unsafe.
__device__ __forceinline__ void cell_sums_wide(const int32_t* __restrict__ in, const int32_t* __restrict__ out,
                                               int64_t beg, int m, int lane, int64_t* tin, int64_t* tout) {
  int lo_in = 0, hi_in = 0, lo_out = 0, hi_out = 0;
#pragma unroll 1
  for (int idx = lane; idx < m; idx += DYN_WAVE) {
    const int a = in[beg + idx];
    const int b = out[beg + idx];
    lo_in += a & 0xFFFF;
    hi_in += a >> 16;
    lo_out += b & 0xFFFF;
    hi_out += b >> 16;
  }
  *tin = ((int64_t)wave_sum_i32(hi_in) << 16) + (int64_t)wave_sum_i32(lo_in);
  *tout = ((int64_t)wave_sum_i32(hi_out) << 16) + (int64_t)wave_sum_i32(lo_out);
}

// Reduction of a register-resident cell of m <= 64*R requests: v[i] = input tokens of request
// i*64 + lane (0xFFFFFFFF beyond m); s_in / s_out / or_all / lmax = the lane's sums, OR and
// largest input over its requests.
template <int R>
__device__ __forceinline__ CellOut cell_reduce(const uint32_t (&v)[R], uint32_t s_in, uint32_t s_out, uint32_t or_all,
                                               uint32_t lmax, const int32_t* __restrict__ in,
                                               const int32_t* __restrict__ out, int64_t beg, int m, int rank, int lane) {
  CellOut r;
  r.orv = wave_or_u32(or_all);
  // at most 2048 values: if all are below 2^20 the 32-bit sums are exact (else redone below)
  r.tin = (int64_t)(uint32_t)wave_sum_i32((int)s_in);
  r.tout = (int64_t)(uint32_t)wave_sum_i32((int)s_out);
  // Answer = largest a with #{v < a} < rank.  It lies in [lo, top]: top = largest element,
  // lo = 0, or for cells of several rows the j-th largest per-lane maximum, j = m - rank + 1.
  const uint32_t top = wave_max_u32(lmax);
  if (rank == m) {                          // the nearest rank of a small cell is its last: the maximum
    r.p99 = top;
  } else {
    uint32_t lo = 0;
    if (R >= 4) {
      const int j = m - rank + 1;
      if (j <= DYN_WAVE) {
        const int nb = 32 - __builtin_clz(top | 1u);
        for (int b = nb - 1; b >= 0; --b) {   // largest c with #{lane maxima >= c} >= j
          const uint32_t cand = lo | (1u << b);
          if (__popcll(__ballot(lmax >= cand)) >= j) lo = cand;
        }
      }
    }
    uint32_t d = 0;
    const int nb = 32 - __builtin_clz((top - lo) | 1u);
    for (int b = nb - 1; b >= 0; --b) {
      const uint32_t cand = lo + (d | (1u << b));
      int below = 0;
#pragma unroll
      for (int i = 0; i < R; ++i) below += __popcll(__ballot(v[i] < cand));
      if (below < rank) d |= 1u << b;
    }
    r.p99 = lo + d;
  }
  if (r.orv >= (1u << 20)) cell_sums_wide(in, out, beg, m, lane, &r.tin, &r.tout);
  return r;
}

// Register-resident cell: m <= 64*R requests.
template <int R>
__device__ __forceinline__ CellOut cell_in_registers(const int32_t* __restrict__ in,
                                                     const int32_t* __restrict__ out, int64_t beg,
                                                     int m, int rank, int lane) {
  uint32_t v[R];
  uint32_t s_in = 0, s_out = 0, or_all = 0, lmax = 0;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int idx = i * DYN_WAVE + lane;
    const bool ok = idx < m;
    const uint32_t a = ok ? (uint32_t)in[beg + idx] : 0u;
    const uint32_t b = ok ? (uint32_t)out[beg + idx] : 0u;
    v[i] = ok ? a : 0xFFFFFFFFu;  // padding is never below a candidate value
    or_all |= a | b;
    lmax = max(lmax, a);
    s_in += a;
    s_out += b;
  }
  return cell_reduce<R>(v, s_in, s_out, or_all, lmax, in, out, beg, m, rank, lane);
}

// Any register-sized cell (0 < mi <= 64 * kRegRowsMax) by one wave.
__device__ __forceinline__ CellOut cell_by_wave(const int32_t* __restrict__ in, const int32_t* __restrict__ out,
                                                int64_t beg, int mi, int rk, int lane) {
  if (mi <= 64 * 1) return cell_in_registers<1>(in, out, beg, mi, rk, lane);
  if (mi <= 64 * 2) return cell_in_registers<2>(in, out, beg, mi, rk, lane);
  if (mi <= 64 * 3) return cell_in_registers<3>(in, out, beg, mi, rk, lane);
  if (mi <= 64 * 4) return cell_in_registers<4>(in, out, beg, mi, rk, lane);
  if (mi <= 64 * 6) return cell_in_registers<6>(in, out, beg, mi, rk, lane);
  if (mi <= 64 * 8) return cell_in_registers<8>(in, out, beg, mi, rk, lane);
  if (mi <= 64 * 12) return cell_in_registers<12>(in, out, beg, mi, rk, lane);
  if (mi <= 64 * 16) return cell_in_registers<16>(in, out, beg, mi, rk, lane);
  if (mi <= 64 * 24) return cell_in_registers<24>(in, out, beg, mi, rk, lane);
  return cell_in_registers<32>(in, out, beg, mi, rk, lane);
}

// The threads of a group wait for each other: the whole block at a barrier; a single wave runs in lockstep and its LDS
// operations complete in program order, so only the compiler has to be kept from moving them across this point.
template <int WAVES>
__device__ __forceinline__ void group_sync() {
  if (WAVES == 1) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  } else {
    __syncthreads();
  }
}

// The value of rank `need` (counted from the bottom) among those of the cell's values whose bits from hi_bit on are `prefix`, 10 bits a
// pass over the cell.  `hist` and `xch` as below.
constexpr int kXchWords = 16;
template <int U, int WAVES>   // U independent loads in flight
__device__ __forceinline__ uint32_t rank_by_group(const int32_t* __restrict__ in, int64_t beg, int64_t m, int hi_bit, uint32_t prefix,
                                                  int64_t need, uint32_t* hist, int64_t* xch) {
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int tid = WAVES == 1 ? lane : (int)threadIdx.x, wave = tid / DYN_WAVE;
  constexpr int nthr = WAVES * DYN_WAVE;
  while (hi_bit > 0) {
    const int w = hi_bit < kHistBits ? hi_bit : kHistBits;
    const int shift = hi_bit - w;
    const uint32_t dmask = (1u << w) - 1u;
    group_sync<WAVES>();
    for (int b = tid; b < kHistBins; b += nthr) hist[b] = 0;
    group_sync<WAVES>();
    for (int64_t i0 = 0; i0 < m; i0 += U * nthr) {
      uint32_t a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = i0 + u * nthr + tid;
        a[u] = i < m ? (uint32_t)in[beg + i] : 0u;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = i0 + u * nthr + tid;
        const bool match = i < m && (hi_bit >= 32 ? true : ((a[u] >> hi_bit) == prefix));
        if (match) atomicAdd(&hist[(a[u] >> shift) & dmask], 1u);
      }
    }
    group_sync<WAVES>();
    if (wave == 0) {
      // lane l owns bins [16 l, 16 l + 16); find the bin where the running count reaches `need`
      constexpr int per = kHistBins / DYN_WAVE;
      uint32_t cnt[per];
      int64_t mine = 0;
#pragma unroll
      for (int q = 0; q < per; ++q) {
        cnt[q] = hist[lane * per + q];
        mine += cnt[q];
      }
      int64_t incl = mine;  // inclusive scan over lanes
#pragma unroll
      for (int d = 1; d < DYN_WAVE; d <<= 1) {
        const int64_t up = __shfl_up(incl, d, DYN_WAVE);
        if (lane >= d) incl += up;
      }
      const uint64_t reach = __ballot(incl >= need);
      const int owner = reach ? __builtin_ctzll(reach) : DYN_WAVE - 1;  // reach != 0: need <= matches
      int64_t run = incl - mine;
      bool found = false;
      uint32_t digit = (uint32_t)(lane * per + per - 1);
      int64_t below = 0;
#pragma unroll
      for (int q = 0; q < per; ++q) {
        const bool hit = !found && (run + cnt[q] >= need || q == per - 1);
        if (hit) {
          digit = (uint32_t)(lane * per + q);
          below = run;
          found = true;
        }
        run += cnt[q];
      }
      if (lane == owner) { xch[12] = (int64_t)digit; xch[13] = below; }
    }
    group_sync<WAVES>();
    const uint32_t digit = (uint32_t)xch[12];
    need -= xch[13];
    prefix = (prefix << w) | digit;
    hi_bit = shift;
  }
  group_sync<WAVES>();
  return prefix;
}

// Large cell, by a group of WAVES waves (the whole block, or one wave on its own): the group streams the cell from
// global memory once for the sums and once per 10-bit digit of the selection (radix select through one LDS histogram).
// Every thread returns the same result.  `hist` (kHistBins counters) and `xch` (kXchWords) are LDS scratch of the
// group; the caller guarantees nobody else uses them.
template <int U, int WAVES>   // U independent loads per array in flight
__device__ __forceinline__ CellOut cell_by_group(const int32_t* __restrict__ in, const int32_t* __restrict__ out, int64_t beg,
                                 int64_t m, int64_t rank, uint32_t* hist, int64_t* xch) {
  static_assert(WAVES * 3 <= 12, "words 12 and 13 pass the digit on");
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int tid = WAVES == 1 ? lane : (int)threadIdx.x, wave = tid / DYN_WAVE;
  constexpr int nthr = WAVES * DYN_WAVE;
  int64_t sin = 0, sout = 0;
  uint32_t orv = 0;
  for (int64_t i0 = 0; i0 < m; i0 += U * nthr) {
    int a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * nthr + tid;
      a[u] = i < m ? in[beg + i] : 0;
      b[u] = i < m ? out[beg + i] : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sin += a[u];
      sout += b[u];
      orv |= (uint32_t)(a[u] | b[u]);
    }
  }
  sin = wave_sum_i64(sin);
  sout = wave_sum_i64(sout);
  orv = wave_or_u32(orv);
  group_sync<WAVES>();
  if (lane == 0) { xch[wave * 3 + 0] = sin; xch[wave * 3 + 1] = sout; xch[wave * 3 + 2] = (int64_t)orv; }
  group_sync<WAVES>();
  CellOut r;
  r.tin = r.tout = 0;
  r.orv = 0;
  for (int w = 0; w < WAVES; ++w) {
    r.tin += xch[w * 3 + 0];
    r.tout += xch[w * 3 + 1];
    r.orv |= (uint32_t)xch[w * 3 + 2];
  }

  // bits >= 32 - clz of the answer are zero
  r.p99 = rank_by_group<U, WAVES>(in, beg, m, 32 - __builtin_clz(r.orv | 1u), 0u, rank, hist, xch);
  return r;
}

// Register-resident cell of 2048 < m <= 128*P requests by one wave: two 16-bit input lengths to a register (request
// i*64 + lane in half i%2 of register i/2; 0xFFFF beyond m).  Same sums and the same search as above.  Returns false,
// and nothing else, when a token count of 2^16 or more (a negative one included) rules the packing out: the caller
// streams the cell instead.
constexpr int kPackedRowsMax = 128;  // the packed path handles m <= 64 * kPackedRowsMax
template <int P>
__device__ __forceinline__ bool cell_in_registers_packed(const int32_t* __restrict__ in, const int32_t* __restrict__ out,
                                                         int m, int rank, int lane, CellOut* res) {
  uint32_t v[P];
  uint32_t s_in = 0, s_out = 0, orv = 0, lmax = 0, lmax2 = 0;   // lmax / lmax2: largest input of the even / odd rows
  constexpr int CH = 4;                  // registers per round: 8 + 8 loads in flight
  static_assert(P % CH == 0, "whole rounds");
#pragma unroll
  for (int p0 = 0; p0 < P; p0 += CH) {
    uint32_t a[2 * CH], b[2 * CH];
#pragma unroll
    for (int u = 0; u < 2 * CH; ++u) {
      const int idx = (2 * p0 + u) * DYN_WAVE + lane;
      a[u] = idx < m ? (uint32_t)in[idx] : 0u;
      b[u] = idx < m ? (uint32_t)out[idx] : 0u;
    }
#pragma unroll
    for (int u = 0; u < 2 * CH; ++u) {
      s_in += a[u];
      s_out += b[u];
      orv |= a[u] | b[u];
      if (u % 2 == 0) lmax = max(lmax, a[u]);
      else lmax2 = max(lmax2, a[u]);
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int idx = (2 * (p0 + u)) * DYN_WAVE + lane;
      const uint32_t x0 = idx < m ? a[2 * u] & 0xFFFFu : 0xFFFFu;
      const uint32_t x1 = idx + DYN_WAVE < m ? a[2 * u + 1] & 0xFFFFu : 0xFFFFu;
      v[p0 + u] = x0 | (x1 << 16);
    }
    // keep the rounds apart (the next round's loads after this round's arithmetic): with all loads hoisted to the
    // top, or the arithmetic sunk to the end, 4P loaded values would be live at once
    asm volatile("" : "+v"(s_in), "+v"(s_out), "+v"(orv), "+v"(lmax), "+v"(lmax2), "+v"(v[p0]), "+v"(v[p0 + 1]),
                 "+v"(v[p0 + 2]), "+v"(v[p0 + 3])::"memory");
  }
  orv = wave_or_u32(orv);
  if (orv >= (1u << 16)) return false;   // uniform over the wave
  // all values below 2^16: a lane's sum stays below 2^23, the wave's below 2^29
  res->orv = orv;
  res->tin = (int64_t)wave_sum_u32(s_in);
  res->tout = (int64_t)wave_sum_u32(s_out);
  const uint32_t top = wave_max_u32(max(lmax, lmax2));
  if (top == 0xFFFFu) return false;      // the padding value; and the search's candidates (up to top + 1) must fit 16 bits
  if (rank == m) {
    res->p99 = top;
    return true;
  }
  uint32_t lo = 0;
  const int j = m - rank + 1;
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
    // low half by a 16-bit compare; high half: hi < cand exactly when the whole register < cand << 16 (no unpacking,
    // which the compiler would otherwise hoist out of this loop into 2P registers)
    const uint16_t cand_lo = (uint16_t)cand;
    const uint32_t cand_hi = cand << 16;
    int below = 0;
#pragma unroll
    for (int i = 0; i < P; ++i)
      below += __popcll(__ballot((uint16_t)v[i] < cand_lo)) + __popcll(__ballot(v[i] < cand_hi));
    if (below < rank) d |= 1u << b;
  }
  res->p99 = lo + d;
  return true;
}

__device__ __forceinline__ bool cell_by_wave_packed(const int32_t* __restrict__ in, const int32_t* __restrict__ out,
                                                    int mi, int rk, int lane, CellOut* res) {
  if (mi <= 128 * 24) return cell_in_registers_packed<24>(in, out, mi, rk, lane, res);
  if (mi <= 128 * 32) return cell_in_registers_packed<32>(in, out, mi, rk, lane, res);
  if (mi <= 128 * 48) return cell_in_registers_packed<48>(in, out, mi, rk, lane, res);
  return cell_in_registers_packed<64>(in, out, mi, rk, lane, res);
}

__device__ __forceinline__ void write_cell(int64_t c, const CellOut& r, int64_t m, uint32_t bad, double window_s,
                                           double r_window,
                                           int64_t cells, int64_t* __restrict__ tin, int64_t* __restrict__ tout,
                                           int32_t* __restrict__ in_p99, CellRec* __restrict__ rec,
                                           uint8_t* __restrict__ cstat, WsHeader* __restrict__ header) {
  tin[c] = r.tin;
  tout[c] = r.tout;
  in_p99[c] = (int32_t)r.p99;
  CellRec cr;
  cr.load = div_by((double)(r.tin + r.tout), window_s, r_window);   // tokens / window_s, r_window = RN(1 / window_s)
  cr.xp99 = (double)(int32_t)r.p99;
  cr.nonempty = m > 0 ? 1.0 : 0.0;
  cr.pad = 0.0;
  rec[c] = cr;
  cstat[c] = (uint8_t)bad;       // every cell writes its own byte: nothing to clear beforehand
  if (c == 0) {                  // single writer of the header
    header->status = 0u;
    header->kind = DYN_WS_KIND_CELLS;
    header->cells = cells;
  }
}

// Four consecutive cells per block, one wave each; cells beyond the register tiers are then
// taken one after the other by the whole block.
__global__ __launch_bounds__(kWavesPerBlock* DYN_WAVE) __attribute__((amdgpu_waves_per_eu(6, 8))) void cell_aggregate_kernel(
    const int32_t* __restrict__ in, const int32_t* __restrict__ out,
    const int64_t* __restrict__ cell_off, int64_t n_req, int64_t cells, double window_s, double r_window,
    int32_t pct_num, int32_t pct_den, int64_t* __restrict__ tin, int64_t* __restrict__ tout,
    int32_t* __restrict__ in_p99, CellRec* __restrict__ rec, uint8_t* __restrict__ cstat,
    WsHeader* __restrict__ header) {
  __shared__ uint32_t s_hist[kWavesPerBlock][kHistBins];
  __shared__ int64_t s_xch[kWavesPerBlock][kXchWords];
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE);
  const int64_t c0 = (int64_t)blockIdx.x * kWavesPerBlock;
  // lane q of every wave holds offset q of the block's cells (kWavesPerBlock + 1 of them)
  const int nc = (int)(cells - c0 < kWavesPerBlock ? cells - c0 : kWavesPerBlock);
  const int64_t myoff = lane <= nc ? cell_off[c0 + lane] : 0;
  const int64_t nxoff = __shfl_down(myoff, 1, DYN_WAVE);
  const bool sound = lane < nc && myoff >= 0 && nxoff >= myoff && nxoff <= n_req;
  // cells of this block left to the whole block, and cells beyond the plain register tiers that a wave takes with
  // packed registers (both uniform over the block)
  const uint32_t big_mask = (uint32_t)__ballot(sound && nxoff - myoff > DYN_WAVE * kPackedRowsMax);
  const uint32_t packed_mask = (uint32_t)__ballot(sound && nxoff - myoff > DYN_WAVE * kRegRowsMax &&
                                                  nxoff - myoff <= DYN_WAVE * kPackedRowsMax);
  if (wave < nc && !((big_mask >> wave) & 1u)) {
    const int64_t c = c0 + wave;
    int64_t beg = readlane_i64(myoff, wave), end = readlane_i64(nxoff, wave);
    // the status lives in a scalar register while the cell is reduced (a vector register would be spilled)
    uint32_t bad = __builtin_amdgcn_readfirstlane((beg < 0 || end < beg || end > n_req) ? DYN_WS_BAD_OFFSETS : 0u);
    asm volatile("" : "+s"(bad));
    if (bad) beg = end = 0;   // never read outside the trace
    const int mi = (int)(end - beg);
    CellOut r;
    r.tin = r.tout = 0;
    r.p99 = 0;
    r.orv = 0;
    if (mi > 0) {
      const int rk = (int)(((int64_t)pct_num * mi + pct_den - 1) / pct_den);
      if ((packed_mask >> wave) & 1u) {
        // values the packing cannot hold: the wave streams its cell on its own (its own histogram; no other wave waits)
        if (!cell_by_wave_packed(in + beg, out + beg, mi, rk, lane, &r))
          r = cell_by_group<8, 1>(in, out, beg, mi, rk, s_hist[wave], s_xch[wave]);
      } else {
        r = cell_by_wave(in, out, beg, mi, rk, lane);
      }
      asm volatile("" : "+s"(bad));
      if (r.orv >> 31) bad |= DYN_WS_BAD_REQUEST;  // a negative token count
    }
    if (lane == 0) write_cell(c, r, mi, bad, window_s, r_window, cells, tin, tout, in_p99, rec, cstat, header);
  }
  if (big_mask == 0) return;   // uniform over the block
  for (int q = 0; q < kWavesPerBlock; ++q) {
    if (!((big_mask >> q) & 1u)) continue;
    const int64_t beg = cell_off[c0 + q];          // read again (the mask vouches for them): nothing is kept in
    const int64_t m = cell_off[c0 + q + 1] - beg;  // registers across the waves' own cells
    const int64_t rank = ((int64_t)pct_num * m + pct_den - 1) / pct_den;
    const CellOut r = cell_by_group<8, kWavesPerBlock>(in, out, beg, m, rank, s_hist[0], s_xch[0]);
    const uint32_t bad = (r.orv >> 31) ? DYN_WS_BAD_REQUEST : 0u;
    if (threadIdx.x == 0) write_cell(c0 + q, r, m, bad, window_s, r_window, cells, tin, tout, in_p99, rec, cstat, header);
  }
}

// Traces cut into many small cells (a tick-level view: a few dozen requests per cell).  A wave
// per cell spends its life waiting for two dependent loads and its 64 lanes reduce a handful
// of values.  Here a wave takes kTinyCells consecutive cells.  Their requests are one contiguous
// run of the trace: if it has at most kTinyCap requests the wave copies it to LDS (coalesced,
// all loads in flight at once) and kTinyLanes lanes per cell walk the cell's requests, each
// keeping sums, the OR and the two largest inputs; a quad exchange combines them.  That
// settles every cell whose nearest rank is its largest or second-largest input (any cell of
// fewer than 200 requests at the 99th percentile); the others, cells with token counts of
// 2^20 or more, and groups whose run does not fit are taken one cell at a time by the wave
// (cells beyond 64 * kRegRowsMax requests by the whole block, after a block barrier).
constexpr int kTinyCells = 16;
constexpr int kTinyLanes = DYN_WAVE / kTinyCells;
constexpr int kTinyCap = 1024;
static_assert(kTinyLanes == 4, "the quad exchange below combines four lanes");

__global__ __launch_bounds__(kWavesPerBlock* DYN_WAVE) __attribute__((amdgpu_waves_per_eu(4, 4))) void cell_aggregate_tiny_kernel(
    const int32_t* __restrict__ in, const int32_t* __restrict__ out,
    const int64_t* __restrict__ cell_off, int64_t n_req, int64_t cells, double window_s, double r_window,
    int32_t pct_num, int32_t pct_den, int64_t* __restrict__ tin, int64_t* __restrict__ tout,
    int32_t* __restrict__ in_p99, CellRec* __restrict__ rec, uint8_t* __restrict__ cstat,
    WsHeader* __restrict__ header) {
  __shared__ uint2 s_run[kWavesPerBlock][kTinyCap];
  __shared__ int64_t s_off[kWavesPerBlock][kTinyCells + 1];
  __shared__ uint32_t s_big[kWavesPerBlock];
  __shared__ uint32_t s_hist[kHistBins];
  __shared__ int64_t s_xch[kXchWords];
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE);
  const int64_t c0 = ((int64_t)blockIdx.x * kWavesPerBlock + wave) * kTinyCells;
  const int nq = cells - c0 < kTinyCells ? (int)(cells - c0 > 0 ? cells - c0 : 0) : kTinyCells;   // cells of this wave
  const int64_t myoff = (nq > 0 && lane <= nq) ? cell_off[c0 + lane] : 0;
  const int64_t nxoff = __shfl_down(myoff, 1, DYN_WAVE);
  const bool good = lane < nq && myoff >= 0 && nxoff >= myoff && nxoff <= n_req;   // never read outside the trace
  const int64_t len = good ? nxoff - myoff : 0;
  const uint32_t good_mask = (uint32_t)__ballot(good);
  const uint32_t big_mask = (uint32_t)__ballot(len > DYN_WAVE * kRegRowsMax);
  const int len32 = (int)(len > 0x7FFFFFFF ? 0x7FFFFFFF : len);
  if (lane <= kTinyCells) s_off[wave][lane] = myoff;
  if (lane == 0) s_big[wave] = big_mask;

  const int u = lane / kTinyLanes, sub = lane % kTinyLanes;   // this lane's cell of the wave, and its share of it
  CellOut mine;                                  // lane kTinyLanes * u keeps the result of cell u
  mine.tin = mine.tout = 0;
  mine.p99 = 0;
  mine.orv = 0;
  int my_m = 0;
  uint32_t my_bad = 0;
  if (nq > 0) {
    const uint32_t grp = (1u << nq) - 1u;
    const int64_t sb = readlane_i64(myoff, 0), se = readlane_i64(myoff, nq);
    if ((good_mask & grp) == grp && se - sb <= kTinyCap) {
      // every offset of the group is in order: 0 <= sb <= each cell's bounds <= se <= n_req
      const int span = (int)(se - sb);
      uint2* run = s_run[wave];
#pragma unroll 4
      for (int pos = lane; pos < span; pos += DYN_WAVE) run[pos] = make_uint2((uint32_t)in[sb + pos], (uint32_t)out[sb + pos]);
      // the run is read back by other lanes of this wave only
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int64_t ob = __shfl(myoff, u, DYN_WAVE), oe = __shfl(myoff, u + 1, DYN_WAVE);
      const int m = u < nq ? (int)(oe - ob) : 0;
      const int rb = u < nq ? (int)(ob - sb) : 0;
      uint32_t s_in = 0, s_out = 0, orv = 0, t1 = 0, t2 = 0;   // t1 >= t2: the two largest inputs so far
      for (int i = rb + sub; i < rb + m; i += kTinyLanes) {
        const uint2 v = run[i];
        s_in += v.x;
        s_out += v.y;
        orv |= v.x | v.y;
        t2 = max(t2, min(t1, v.x));
        t1 = max(t1, v.x);
      }
#pragma unroll
      for (int step = 0; step < 2; ++step) {     // lanes sub ^ 1, then sub ^ 2
        const uint32_t o_in = step ? (uint32_t)dpp_mov<0x4E>((int)s_in) : (uint32_t)dpp_mov<0xB1>((int)s_in);
        const uint32_t o_out = step ? (uint32_t)dpp_mov<0x4E>((int)s_out) : (uint32_t)dpp_mov<0xB1>((int)s_out);
        const uint32_t o_or = step ? (uint32_t)dpp_mov<0x4E>((int)orv) : (uint32_t)dpp_mov<0xB1>((int)orv);
        const uint32_t o1 = step ? (uint32_t)dpp_mov<0x4E>((int)t1) : (uint32_t)dpp_mov<0xB1>((int)t1);
        const uint32_t o2 = step ? (uint32_t)dpp_mov<0x4E>((int)t2) : (uint32_t)dpp_mov<0xB1>((int)t2);
        s_in += o_in;
        s_out += o_out;
        orv |= o_or;
        t2 = max(max(t2, o2), min(t1, o1));
        t1 = max(t1, o1);
      }
      // nearest rank ceil(pct * m) counted from the top: j = 1 is the largest input
      const int rk = m > 0 ? (int)(((int64_t)pct_num * m + pct_den - 1) / pct_den) : 0;
      const int j = m - rk + 1;
      // at most 1024 values: 32-bit sums are exact if all are below 2^20
      const bool again = m > 0 && (orv >= (1u << 20) || j > 2);
      mine.tin = (int64_t)s_in;
      mine.tout = (int64_t)s_out;
      mine.p99 = j == 1 ? t1 : t2;
      mine.orv = orv;
      my_m = m;
      uint64_t todo = __ballot(sub == 0 && again);
      while (todo) {                             // uniform over the wave
        const int l = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int q = l / kTinyLanes;
        const int64_t beg = readlane_i64(myoff, q);
        const int mi = __builtin_amdgcn_readlane(len32, q);
        const int rk1 = (int)(((int64_t)pct_num * mi + pct_den - 1) / pct_den);
        const CellOut r = cell_by_wave(in, out, beg, mi, rk1, lane);
        if (lane == l) mine = r;
      }
      if (mine.orv >> 31) my_bad = DYN_WS_BAD_REQUEST;   // a negative token count
    } else {
#pragma unroll 1
      for (int q = 0; q < nq; ++q) {
        if ((big_mask >> q) & 1u) continue;      // uniform over the wave
        CellOut r;
        r.tin = r.tout = 0;
        r.p99 = 0;
        r.orv = 0;
        uint32_t bad = 0;
        int mi = 0;
        if (!((good_mask >> q) & 1u)) {
          bad = DYN_WS_BAD_OFFSETS;
        } else {
          const int64_t beg = readlane_i64(myoff, q);
          mi = __builtin_amdgcn_readlane(len32, q);
          if (mi > 0) {
            const int rk = (int)(((int64_t)pct_num * mi + pct_den - 1) / pct_den);
            r = cell_by_wave(in, out, beg, mi, rk, lane);
            if (r.orv >> 31) bad |= DYN_WS_BAD_REQUEST;
          }
        }
        if (lane == q * kTinyLanes) { mine = r; my_m = mi; my_bad = bad; }
      }
    }
  }
  if (sub == 0 && u < nq && !((big_mask >> u) & 1u))
    write_cell(c0 + u, mine, my_m, my_bad, window_s, r_window, cells, tin, tout, in_p99, rec, cstat, header);
  __syncthreads();             // every wave of the block arrives here: s_off and s_big are complete
  if ((s_big[0] | s_big[1] | s_big[2] | s_big[3]) == 0) return;   // uniform over the block
  static_assert(kWavesPerBlock == 4, "the line above names the block's four waves");
  for (int w = 0; w < kWavesPerBlock; ++w)
    for (int q = 0; q < kTinyCells; ++q) {
      if (!((s_big[w] >> q) & 1u)) continue;
      const int64_t beg = s_off[w][q];
      const int64_t m = s_off[w][q + 1] - beg;
      const int64_t rank = ((int64_t)pct_num * m + pct_den - 1) / pct_den;
      const CellOut r = cell_by_group<2, kWavesPerBlock>(in, out, beg, m, rank, s_hist, s_xch);
      const uint32_t bad = (r.orv >> 31) ? DYN_WS_BAD_REQUEST : 0u;
      const int64_t c = ((int64_t)blockIdx.x * kWavesPerBlock + w) * kTinyCells + q;
      if (threadIdx.x == 0) write_cell(c, r, m, bad, window_s, r_window, cells, tin, tout, in_p99, rec, cstat, header);
    }
}

// ---- long cells: many blocks share a cell --------------------------------------------------------
// A block streams a cell at about 16 GB/s (a memory latency for every 16 KB), so a few cells of many requests leave the device
// idle.  Here a cell beyond what a block holds in registers is cut into pieces, a block each.  The first pass takes the sums and counts
// the lengths by exponent and the six bits below it (exact below 64, otherwise a bin is at most 1/64 of its value wide) in LDS and adds
// the counts to the cell's counters in the workspace; in the second every block finds the bin that holds the rank, counts the lengths
// in it by its 256 parts, and the last block of the cell to be done finds the answer.  Lengths below 2^15 are exact then; what is left
// of a wider bin that block searches alone.  Bounds: the launches (3 us each), then reading 8 and 4 bytes a request.
// Measured (us of dyn_eval_select; a block per cell, this): 20 M requests in one cell 22 090, 71 (the first pass 28: 5.7 TB/s, the second 25);
// in 48 cells 1109, 72; in 500 174, 88; 3.8 M in 3 cells 2817, 39; 12.8 M in 8 cells of mixed pools 3194, 61.  The line: 9 cells of mean
// 4500 37, 40, of 8000 48, 40; 500 of 4500 45, 52, of 8000 57, 51; 1000 of 8000 67, 71, of 12 000 87, 78; one of 9000 30, 37, of 16 000 35, 37.
constexpr int64_t kLongCell = 8192;                // what a block still holds in registers
constexpr int kLongSlots = 1024;                   // slots of the workspace: several copies a cell where cells are few
constexpr int kLongCopies = 4;                     // at most: blocks that add to one counter hold each other up (28 us against 11 for 900 blocks and 3 cells)
constexpr int64_t kLongMean = 9000, kLongLeast = 20000;   // requests per cell, and in all, from which the two launches are worth it
constexpr int kLongBlocks = 512;                   // pieces of a whole trace, two blocks to a compute unit
constexpr int64_t kLongShare = 32;                  // pieces of a mean cell that one copy of its counters takes
constexpr int64_t kLongPiece = 4096;               // least requests of a piece: 16 a thread
constexpr int kFineBins = 256;
constexpr int kSlotsPerBlock = 8;                  // cleared by one block of long_prepare
// words of the workspace: long cells, pieces; the cells [kBlockCells at most]; every slot's first piece and the end; the slots
constexpr int kLongCellsAt = 64, kLongFirstAt = kLongCellsAt + 1024, kLongHeadWords = kLongFirstAt + 1088;
// words of a slot: the counts, the two sums (64 bits), the OR of all token counts, blocks done
constexpr int kFineAt = kCoarseBins, kSumsAt = kFineAt + kFineBins, kOrAt = kSumsAt + 4, kDoneAt = kOrAt + 1;
constexpr int kLongSlotWords = 2048;
static_assert((kLongHeadWords + (size_t)kLongSlots * kLongSlotWords) * sizeof(uint32_t) <= DYN_CELL_MANY_MAX && kLongSlots + 1 <= 1088 && kLongHeadWords % 64 == 0, "the workspace");
static_assert(kDoneAt < kLongSlotWords && kSumsAt % 2 == 0, "the slot");

struct LongArgs {
  int64_t from;      // cells of more requests are long
  int64_t piece;     // requests of a piece
  int32_t n_cell, copies;  // cells (each may be long); slots of a cell, a power of two
  uint32_t* work;
};

// Block 0 of these lists the long cells and their pieces, the others clear the slots.  `s` is LDS scratch of kHistBins words.
__device__ __forceinline__ void long_prepare(const LongArgs& a, const int64_t* __restrict__ cell_off, int64_t n_req, int64_t cells, int part, uint32_t* s) {
  if (part > 0) {
    const int s0 = (part - 1) * kSlotsPerBlock, s1 = min(s0 + kSlotsPerBlock, a.n_cell * a.copies);
    uint4* at = (uint4*)(a.work + kLongHeadWords + (size_t)s0 * kLongSlotWords);
    for (int i = threadIdx.x; i < (s1 - s0) * (kLongSlotWords / 4); i += blockDim.x) at[i] = make_uint4(0u, 0u, 0u, 0u);
    return;
  }
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = threadIdx.x / DYN_WAVE;
  int n = 0;                                         // long cells so far, block-uniform
  uint32_t pieces = 0;
  for (int64_t c0 = 0; c0 < cells; c0 += blockDim.x) {
    const int64_t c = c0 + threadIdx.x;
    const int64_t beg = c < cells ? cell_off[c] : 0, end = c < cells ? cell_off[c + 1] : 0;
    const bool is = beg >= 0 && end <= n_req && end - beg > a.from;
    const uint32_t mine = is ? (uint32_t)((end - beg + a.piece - 1) / a.piece) : 0u;
    const uint64_t who = __ballot(is);
    uint32_t incl = mine;
#pragma unroll
    for (int d = 1; d < DYN_WAVE; d <<= 1) {
      const uint32_t up = __shfl_up(incl, d, DYN_WAVE);
      if (lane >= d) incl += up;
    }
    if (lane == DYN_WAVE - 1) { s[2 * wave] = (uint32_t)__popcll(who); s[2 * wave + 1] = incl; }
    __syncthreads();
    int at = n + __popcll(who & ((1ull << lane) - 1ull));
    uint32_t first = pieces + incl - mine;
    for (int w = 0; w < (int)blockDim.x / DYN_WAVE; ++w) {
      if (w < wave) { at += (int)s[2 * w]; first += s[2 * w + 1]; }
      n += (int)s[2 * w];
      pieces += s[2 * w + 1];
    }
    __syncthreads();                                 // s is written again
    if (is) {
      a.work[kLongCellsAt + at] = (uint32_t)c;
      a.work[kLongFirstAt + at] = first;
    }
  }
  if (threadIdx.x == 0) {
    a.work[0] = (uint32_t)n;
    a.work[kLongFirstAt + n] = pieces;
  }
}

// ---- few cells: a block per long cell -----------------------------------------------------------
// With no more cells than compute units hold blocks, a wave per cell leaves most of the device idle while the longest cell
// decides the time.  Here cells of up to kWaveCell requests have a wave each and four waves share a longer one: up to kBlockRows
// values in each thread's registers, the bit-wise search with the waves' counts added up through LDS (a barrier a bit); beyond
// that the cell is streamed.  What bounds it is latency: offsets, requests, the bits of the search.  Four waves and not eight: a
// block of eight does not find its place beside other streams' kernels until they are through (nine cells of a minute
// 844 us beside an evaluation, 79 so, 46 with a wave per cell).
// Measured (us; a wave per cell, a block of eight waves each, this): 9 cells of 10 000 requests together 12.4, 9.3, 10.5; 180 of 300 000
// 18.0, 9.3, 10.5; 540 of 1 M 22.1, 13.2, 15.6; 1000 of 10 M 106, 41, 52; even cells: 40 of 2500 7.2, 8.9, 6.2; 1000 of 1024 5.4,
// 12.0, 5.9; 1000 of 3072 11.0, 16.4, 9.5; 1000 of 6144 19.1, 24.0, 23.0; 256 of 8000 21.5, 9.3, 10.8.  Few requests a cell, or
// more cells than are resident at once, are better with a wave per cell: 2500 of 1 M 7.3, 21.6 with a block each.
constexpr int kBlockWaves = 4;
constexpr int kBlockRows = 32;                     // register path: m <= 256 * kBlockRows
constexpr int kWaveCell = 3072;                    // up to here a wave on its own: 24 packed registers
constexpr int64_t kBlockCells = 1024;              // cells that the device holds at once this way
constexpr int64_t kBlockMean = 1000;               // requests per cell
static_assert(kBlockCells <= kLongSlots, "a slot for every cell");
static_assert(kWaveCell <= 128 * 24, "the packed form below");

template <int R>
__device__ __forceinline__ CellOut cell_by_block(const int32_t* __restrict__ in, const int32_t* __restrict__ out, int m, int rank, int64_t* xch, uint32_t* s_n) {
  constexpr int kThreads = kBlockWaves * DYN_WAVE;
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = threadIdx.x / DYN_WAVE;
  uint32_t v[R], b[R], orv = 0, top = 0;
  int64_t sin = 0, sout = 0;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int at = min(i * kThreads + (int)threadIdx.x, m - 1);
    v[i] = (uint32_t)in[at];
    b[i] = (uint32_t)out[at];
  }
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const bool ok = i * kThreads + (int)threadIdx.x < m;
    sin += ok ? (int32_t)v[i] : 0;
    sout += ok ? (int32_t)b[i] : 0;
    orv |= v[i] | b[i];                            // beyond m: the last request again
    top = max(top, v[i]);
    v[i] = ok ? v[i] : 0xFFFFFFFFu;                // padding is never below a candidate value
  }
  sin = wave_sum_i64(sin);
  sout = wave_sum_i64(sout);
  orv = wave_or_u32(orv);
  top = wave_max_u32(top);
  if (lane == 0) {
    xch[wave * 3 + 0] = sin;
    xch[wave * 3 + 1] = sout;
    xch[wave * 3 + 2] = (int64_t)(((uint64_t)top << 32) | orv);
  }
  __syncthreads();
  CellOut r;
  r.tin = r.tout = 0;
  r.orv = top = 0;
#pragma unroll
  for (int w = 0; w < kBlockWaves; ++w) {
    r.tin += xch[w * 3 + 0];
    r.tout += xch[w * 3 + 1];
    r.orv |= (uint32_t)xch[w * 3 + 2];
    top = max(top, (uint32_t)((uint64_t)xch[w * 3 + 2] >> 32));
  }
  r.p99 = top;
  if (rank == m) return r;
  uint32_t d = 0;
  int turn = 0;                                    // two buffers: a wave may be a barrier ahead of the slowest reader
  for (int bit = 31 - __builtin_clz(top | 1u); bit >= 0; --bit) {
    const uint32_t cand = d | (1u << bit);
    int below = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) below += __popcll(__ballot(v[i] < cand));
    if (lane == 0) s_n[turn * kBlockWaves + wave] = (uint32_t)below;
    __syncthreads();
    uint32_t all = 0;
#pragma unroll
    for (int w = 0; w < kBlockWaves; ++w) all += s_n[turn * kBlockWaves + w];
    if ((int)all < rank) d = cand;
    turn ^= 1;
  }
  r.p99 = d;
  return r;
}

// LONG: cells beyond lg.from are left to the many blocks' kernels, which this one makes ready; the other form is what small calls were before those
// came in (a minute of 9 cells: 19.0 us a call against 19.15, of 25 cells 28.95, 29.3).
struct NoLong {};
template <bool LONG>
__global__ __launch_bounds__(kBlockWaves* DYN_WAVE) __attribute__((amdgpu_waves_per_eu(4, 8))) void cell_aggregate_block_kernel(
    const int32_t* __restrict__ in, const int32_t* __restrict__ out, const int64_t* __restrict__ cell_off, int64_t n_req, int64_t cells,
    double window_s, double r_window, int32_t pct_num, int32_t pct_den, int64_t* __restrict__ tin, int64_t* __restrict__ tout,
    int32_t* __restrict__ in_p99, CellRec* __restrict__ rec, uint8_t* __restrict__ cstat, WsHeader* __restrict__ header, std::conditional_t<LONG, LongArgs, NoLong> lg) {
  __shared__ uint32_t s_hist[kBlockWaves][kHistBins];
  __shared__ int64_t s_xch[kBlockWaves][kXchWords];
  __shared__ uint32_t s_n[2 * kBlockWaves];
  const int lane = threadIdx.x & (DYN_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE);
  // the first blocks take a cell per wave, one block for every cell follows
  const int64_t shared = (cells + kBlockWaves - 1) / kBlockWaves;
  if constexpr (LONG) {
    if ((int64_t)blockIdx.x >= cells + shared) {   // the blocks after those make the many blocks' kernels ready
      long_prepare(lg, cell_off, n_req, cells, (int)((int64_t)blockIdx.x - cells - shared), s_hist[0]);
      return;
    }
  }
  const bool alone = (int64_t)blockIdx.x < shared;
  const int64_t c = alone ? (int64_t)blockIdx.x * kBlockWaves + wave : (int64_t)blockIdx.x - shared;
  if (c >= cells) return;
  int64_t beg = cell_off[c], end = cell_off[c + 1];
  uint32_t bad = (beg < 0 || end < beg || end > n_req) ? DYN_WS_BAD_OFFSETS : 0u;
  if (bad) beg = end = 0;                          // never read outside the trace
  const int64_t m = end - beg;
  if constexpr (LONG) {
    if (m > lg.from) return;                       // the many blocks' (lg.from >= kWaveCell)
  }
  if (alone != (m <= kWaveCell)) return;           // uniform over the wave, and over a block that takes one cell
  CellOut r;
  r.tin = r.tout = 0;
  r.p99 = 0;
  r.orv = 0;
  if (m > 0) {
    const int64_t rank = ((int64_t)pct_num * m + pct_den - 1) / pct_den;
    constexpr int kThreads = kBlockWaves * DYN_WAVE;
    const int32_t *ci = in + beg, *co = out + beg;
    if (alone) {
      if (m <= DYN_WAVE * kRegRowsMax) r = cell_by_wave(in, out, beg, (int)m, (int)rank, lane);
      else if (!(m <= 128 * 24 && cell_in_registers_packed<24>(ci, co, (int)m, (int)rank, lane, &r)))   // the bound spares the search 3 of 11 us
        r = cell_by_group<8, 1>(in, out, beg, m, rank, s_hist[wave], s_xch[wave]);
    } else if (m <= kBlockRows / 2 * kThreads) r = cell_by_block<kBlockRows / 2>(ci, co, (int)m, (int)rank, s_xch[0], s_n);
    else if (m <= kBlockRows * kThreads) r = cell_by_block<kBlockRows>(ci, co, (int)m, (int)rank, s_xch[0], s_n);
    else r = cell_by_group<8, kBlockWaves>(in, out, beg, m, rank, s_hist[0], s_xch[0]);
    if (r.orv >> 31) bad |= DYN_WS_BAD_REQUEST;    // a negative token count
  }
  if (alone ? lane == 0 : threadIdx.x == 0) write_cell(c, r, m, bad, window_s, r_window, cells, tin, tout, in_p99, rec, cstat, header);
}

// The slots' first pieces into LDS (kLongSlots + 1 words); returns how many slots are used, *n_item the pieces.
__device__ __forceinline__ int long_table(const LongArgs& a, uint32_t* s_first, uint32_t* n_item) {
  const int n = (int)a.work[0];
  for (int i = threadIdx.x; i <= n; i += blockDim.x) s_first[i] = a.work[kLongFirstAt + i];
  __syncthreads();
  *n_item = n > 0 ? s_first[n] : 0u;
  return n;
}
__device__ __forceinline__ int long_slot(const uint32_t* s_first, int n, uint32_t item) {
  int l = 0, h = n - 1;                              // the last slot that starts at or before the item
  while (l < h) {
    const int mid = (l + h + 1) >> 1;
    if (s_first[mid] <= item) l = mid; else h = mid - 1;
  }
  return l;
}

// First pass: sums and coarse counts.
__global__ __launch_bounds__(kBlockWaves* DYN_WAVE) void cell_long_count_kernel(const int32_t* __restrict__ in, const int32_t* __restrict__ out,
                                                                                const int64_t* __restrict__ cell_off, LongArgs a) {
  __shared__ uint32_t s_first[kLongSlots + 1];
  __shared__ uint32_t s_bin[kCoarseBins];
  __shared__ int64_t s_sum[kBlockWaves][2];
  __shared__ uint32_t s_or[kBlockWaves];
  constexpr int kThreads = kBlockWaves * DYN_WAVE, U = 8;
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = threadIdx.x / DYN_WAVE;
  uint32_t n_item;
  const int n = long_table(a, s_first, &n_item);
  for (uint32_t item = blockIdx.x; item < n_item; item += gridDim.x) {
    const int slot = long_slot(s_first, n, item);
    const int64_t c = a.work[kLongCellsAt + slot];
    const int64_t end = cell_off[c + 1], beg = cell_off[c] + (int64_t)(item - s_first[slot]) * a.piece;
    const int m = (int)(end - beg < a.piece ? end - beg : a.piece);
    for (int b = threadIdx.x; b < kCoarseBins; b += kThreads) s_bin[b] = 0u;
    __syncthreads();
    const int32_t *pi = in + beg, *po = out + beg;
    int64_t sin = 0, sout = 0;
    uint32_t orv = 0;
    for (int i0 = 0; i0 < m; i0 += U * kThreads) {
      uint32_t x[U], y[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = min(i0 + u * kThreads + (int)threadIdx.x, m - 1);
        x[u] = (uint32_t)pi[i];
        y[u] = (uint32_t)po[i];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool ok = i0 + u * kThreads + (int)threadIdx.x < m;
        sin += ok ? (int32_t)x[u] : 0;
        sout += ok ? (int32_t)y[u] : 0;
        orv |= x[u] | y[u];                          // beyond the piece: its last request again
        if (ok) atomicAdd(&s_bin[coarse_bin(x[u])], 1u);
      }
    }
    sin = wave_sum_i64(sin);
    sout = wave_sum_i64(sout);
    orv = wave_or_u32(orv);
    if (lane == 0) { s_sum[wave][0] = sin; s_sum[wave][1] = sout; s_or[wave] = orv; }
    __syncthreads();
    uint32_t* at = a.work + kLongHeadWords + ((size_t)slot * a.copies + (item & (uint32_t)(a.copies - 1))) * kLongSlotWords;
    for (int b = threadIdx.x; b < kCoarseBins; b += kThreads) {
      const uint32_t k = s_bin[b];
      if (k) atomicAdd(&at[b], k);
    }
    if (threadIdx.x == 0) {
      int64_t t0 = 0, t1 = 0;
      uint32_t o = 0;
      for (int w = 0; w < kBlockWaves; ++w) { t0 += s_sum[w][0]; t1 += s_sum[w][1]; o |= s_or[w]; }
      atomicAdd((unsigned long long*)(at + kSumsAt), (unsigned long long)t0);
      atomicAdd((unsigned long long*)(at + kSumsAt) + 1, (unsigned long long)t1);
      atomicOr(&at[kOrAt], o);
    }
    __syncthreads();                                 // LDS is reused by the next item
  }
}

// Second pass: the bin that holds the rank, its parts counted, and the cell's outputs from the last block to be done with it.
__global__ __launch_bounds__(kBlockWaves* DYN_WAVE) void cell_long_rank_kernel(
    const int32_t* __restrict__ in, const int32_t* __restrict__ out, const int64_t* __restrict__ cell_off, int64_t cells, double window_s,
    double r_window, int32_t pct_num, int32_t pct_den, int64_t* __restrict__ tin, int64_t* __restrict__ tout, int32_t* __restrict__ in_p99,
    CellRec* __restrict__ rec, uint8_t* __restrict__ cstat, WsHeader* __restrict__ header, LongArgs a) {
  constexpr int kThreads = kBlockWaves * DYN_WAVE, U = 8, kPer = (kCoarseBins + kThreads - 1) / kThreads;
  __shared__ uint32_t s_first[kLongSlots + 1];
  __shared__ uint32_t s_bin[kPer * kThreads];
  __shared__ int64_t s_xch[kXchWords];
  __shared__ uint32_t s_find[kBlockWaves + 2];
  __shared__ uint32_t s_last;
  static_assert(kFineBins == kThreads && kHistBins <= kPer * kThreads, "a thread per part of a bin");
  uint32_t n_item;
  const int n = long_table(a, s_first, &n_item);
  for (uint32_t item = blockIdx.x; item < n_item; item += gridDim.x) {
    const int slot = long_slot(s_first, n, item);
    const int64_t c = a.work[kLongCellsAt + slot];
    const int64_t beg = cell_off[c], m = cell_off[c + 1] - beg;
    const int64_t rank = ((int64_t)pct_num * m + pct_den - 1) / pct_den;
    uint32_t* at = a.work + kLongHeadWords + (size_t)slot * a.copies * kLongSlotWords;   // the cell's first copy
    {                                                // the copies' counts, coalesced, then a thread's consecutive bins through LDS
      uint32_t t[kLongCopies][kPer];
#pragma unroll
      for (int y = 0; y < kLongCopies; ++y)          // all loads in flight: a copy that is not there is read as the first, then left out
#pragma unroll
        for (int q = 0; q < kPer; ++q)
          t[y][q] = at[(size_t)(y < a.copies ? y : 0) * kLongSlotWords + min(q * kThreads + (int)threadIdx.x, kCoarseBins)];
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        uint32_t all = 0;
#pragma unroll
        for (int y = 0; y < kLongCopies; ++y) all += y < a.copies ? t[y][q] : 0u;
        s_bin[q * kThreads + threadIdx.x] = q * kThreads + (int)threadIdx.x < kCoarseBins ? all : 0u;
      }
    }
    __syncthreads();
    uint32_t k[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) k[q] = s_bin[(int)threadIdx.x * kPer + q];
    int64_t below;
    int bits;
    const uint32_t low = coarse_low(find_bin<kBlockWaves>(k, rank, s_find, &below), &bits);
    const int shift = bits > 8 ? bits - 8 : 0;       // of a value in the bin to its part
    const uint32_t pieces = s_first[slot + 1] - s_first[slot];
    bool last = item == s_first[slot];
    if (bits > 0) {
      s_bin[threadIdx.x] = 0u;
      __syncthreads();
      const int64_t p0 = (int64_t)(item - s_first[slot]) * a.piece;
      const int32_t* pi = in + beg + p0;
      const int mp = (int)(m - p0 < a.piece ? m - p0 : a.piece);
      for (int i0 = 0; i0 < mp; i0 += U * kThreads) {
        uint32_t x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = (uint32_t)pi[min(i0 + u * kThreads + (int)threadIdx.x, mp - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (i0 + u * kThreads + (int)threadIdx.x < mp && (x[u] - low) >> bits == 0u) atomicAdd(&s_bin[(x[u] - low) >> shift], 1u);
      }
      __syncthreads();
      // The counts are added at the device's coherence point, and the block has every one of its old values back before it says that
      // it is done: whoever is last finds all counts there.
      uint32_t old = 0;
      const uint32_t mine = s_bin[threadIdx.x];
      if (mine) old = __hip_atomic_fetch_add(&at[(size_t)(item & (uint32_t)(a.copies - 1)) * kLongSlotWords + kFineAt + threadIdx.x], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("" ::"v"(old) : "memory");
      __syncthreads();
      if (threadIdx.x == 0) s_last = __hip_atomic_fetch_add(&at[kDoneAt], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == pieces ? 1u : 0u;
      __syncthreads();
      last = s_last != 0u;
    }
    if (last) {                                      // block-uniform
      CellOut r;
      r.p99 = low;
      if (bits > 0) {
        uint32_t f[1] = {0u};
#pragma unroll
        for (int y = 0; y < kLongCopies; ++y) {
          const uint32_t x = __hip_atomic_load(&at[(size_t)(y < a.copies ? y : 0) * kLongSlotWords + kFineAt + threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          f[0] += y < a.copies ? x : 0u;
        }
        int64_t less;
        const int part = find_bin<kBlockWaves>(f, rank - below, s_find, &less);
        r.p99 = low + ((uint32_t)part << shift);
        if (shift > 0) r.p99 = rank_by_group<U, kBlockWaves>(in, beg, m, shift, r.p99 >> shift, rank - below - less, s_bin, s_xch);
      }
      r.tin = r.tout = 0;
      r.orv = 0;
      for (int y = 0; y < a.copies; ++y) {
        const uint32_t* ay = at + (size_t)y * kLongSlotWords;
        r.tin += (int64_t)((const uint64_t*)(ay + kSumsAt))[0];
        r.tout += (int64_t)((const uint64_t*)(ay + kSumsAt))[1];
        r.orv |= ay[kOrAt];
      }
      const uint32_t bad = (r.orv >> 31) ? DYN_WS_BAD_REQUEST : 0u;   // a negative token count
      if (threadIdx.x == 0) write_cell(c, r, m, bad, window_s, r_window, cells, tin, tout, in_p99, rec, cstat, header);
    }
    __syncthreads();                                 // LDS is reused by the next item
  }
}

}  // namespace

hipError_t dyn_launch_cell_aggregate(const int32_t* in_tok, const int32_t* out_tok,
                                     const int64_t* cell_off, int64_t n_req, int64_t cells,
                                     double window_s, int32_t pct_num, int32_t pct_den,
                                     int64_t* tin, int64_t* tout, int32_t* in_p99, CellRec* rec,
                                     uint8_t* cstat, WsHeader* header, void* many, hipStream_t s) {
  DynTimed timed(DYN_K_CELL, s);
  if (cells <= kBlockCells && n_req > kBlockMean * cells) {
    const unsigned blocks = (unsigned)(cells + (cells + kBlockWaves - 1) / kBlockWaves);
    if (many && n_req > kLongMean * cells && n_req > kLongLeast) {
      LongArgs lg;
      lg.from = kLongCell;
      lg.n_cell = (int32_t)cells;
      lg.piece = std::max<int64_t>(kLongPiece, ((n_req + kLongBlocks - 1) / kLongBlocks + 255) / 256 * 256);
      lg.copies = 1;
      while (lg.copies < kLongCopies && 2 * lg.copies * cells <= kLongSlots && n_req > (kLongShare * lg.copies) * cells * lg.piece) lg.copies *= 2;
      lg.work = (uint32_t*)many;
      const unsigned prepare = 1 + (unsigned)(cells * lg.copies + kSlotsPerBlock - 1) / kSlotsPerBlock;
      const unsigned items = (unsigned)((n_req + lg.piece - 1) / lg.piece + std::min<int64_t>(cells, n_req / kLongCell));   // every long cell's last piece may be a short one
      hipLaunchKernelGGL(cell_aggregate_block_kernel<true>, dim3(blocks + prepare), dim3(kBlockWaves * DYN_WAVE), 0, s, in_tok, out_tok, cell_off, n_req, cells,
                         window_s, 1.0 / window_s, pct_num, pct_den, tin, tout, in_p99, rec, cstat, header, lg);
      hipLaunchKernelGGL(cell_long_count_kernel, dim3(items), dim3(kBlockWaves * DYN_WAVE), 0, s, in_tok, out_tok, cell_off, lg);
      hipLaunchKernelGGL(cell_long_rank_kernel, dim3(items), dim3(kBlockWaves * DYN_WAVE), 0, s, in_tok, out_tok, cell_off, cells, window_s, 1.0 / window_s,
                         pct_num, pct_den, tin, tout, in_p99, rec, cstat, header, lg);
    } else {
      hipLaunchKernelGGL(cell_aggregate_block_kernel<false>, dim3(blocks), dim3(kBlockWaves * DYN_WAVE), 0, s, in_tok, out_tok, cell_off, n_req, cells,
                         window_s, 1.0 / window_s, pct_num, pct_den, tin, tout, in_p99, rec, cstat, header, NoLong{});
    }
    return hipGetLastError();
  }
  if (n_req / 48 <= cells) {                     // a few dozen requests per cell on average
    const int64_t per = kWavesPerBlock * kTinyCells;
    hipLaunchKernelGGL(cell_aggregate_tiny_kernel, dim3((unsigned)((cells + per - 1) / per)),
                       dim3(kWavesPerBlock * DYN_WAVE), 0, s, in_tok, out_tok, cell_off, n_req, cells, window_s,
                       1.0 / window_s, pct_num, pct_den, tin, tout, in_p99, rec, cstat, header);
    return hipGetLastError();
  }
  const int64_t blocks = (cells + kWavesPerBlock - 1) / kWavesPerBlock;
  hipLaunchKernelGGL(cell_aggregate_kernel, dim3((unsigned)blocks), dim3(kWavesPerBlock * DYN_WAVE),
                     0, s, in_tok, out_tok, cell_off, n_req, cells, window_s, 1.0 / window_s, pct_num, pct_den, tin,
                     tout, in_p99, rec, cstat, header);
  return hipGetLastError();
}

size_t dyn_cell_many_bytes(int64_t cells) {
  return (kLongHeadWords + kLongSlotWords * (size_t)std::min<int64_t>(kLongSlots, kLongCopies * std::max<int64_t>(cells, 1))) * sizeof(uint32_t);
}
