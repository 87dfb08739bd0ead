// Pools that mix instance types (Eq. 1 in full): per (window, class) cell the number of
// instances of every tensor parallelism, their frequency and the part of the load each type
// takes, so that the energy is least within the GPU budget and the SLO.
//
// The load is split in n_share equal shares; type i takes a_i of them and its n_i instances
// share that part equally.  The frequency of a type does not depend on the other types, so
// the search has two steps:
//   mixed_type_*_kernel   E_i(n, a) = least energy of n instances of type i carrying a shares
//                         over the frequencies that meet the SLO (Section IV-B "Scale-up/down":
//                         filter, then least energy), for every (cell, i, n, a);
//   mixed_combine_kernel  per cell a dynamic programme over the types, state = (GPUs used,
//                         shares assigned): D_{i+1}[u + n tp_i][s + a] = min(D_i[u][s] + E_i(n, a)).
// Rounded addition is monotone, so the minimum over the partial sums of a prefix followed by
// one more addition is the minimum over the extended sums: the programme returns exactly the
// least of the sums 0 + E_0 + E_1 + ... taken in type order, which is how the total is defined.
#include <algorithm>

#include "dyn_mixed.h"
#include "dyn_device.h"

namespace {

// Minimum over each row of 16 lanes, left in every lane of the row.
__device__ __forceinline__ uint32_t row_min_u32(uint32_t x) {
  x = min(x, (uint32_t)dpp_mov<0x121>((int)x));
  x = min(x, (uint32_t)dpp_mov<0x122>((int)x));
  x = min(x, (uint32_t)dpp_mov<0x124>((int)x));
  x = min(x, (uint32_t)dpp_mov<0x128>((int)x));
  return x;
}

// Block = (run of windows, class, type).  A thread is (entry, frequency): 16 entries of 16
// frequency lanes per pass over the type's entries.  The type's table rows (all frequencies)
// sit in LDS.
// LDS: [rows n_f*3*n_rho] [load axis] [cell records win_per_block] [bucket index (16-bit)]
template <int AXIS>
__global__ __launch_bounds__(256) void mixed_type_kernel(MixedTypeArgs a) {
  extern __shared__ double smem[];
  const int n_rho = a.n_rho, n_f = a.n_f, S = a.n_share;
  const int i = blockIdx.x % a.n_tp;
  const int g = (blockIdx.x / a.n_tp) % a.G;
  const int chunk = blockIdx.x / (a.n_tp * a.G);
  const int n_ent = a.types.n_max[i] * S;          // entries of this type
  if (n_ent == 0) return;                          // block-uniform
  const int w0 = chunk * a.win_per_block;
  const int w1 = min(w0 + a.win_per_block, a.n_window);
  const int n_entry = a.types.off[a.n_tp];

  // rows one double apart from a multiple of the bank width: the 16 frequency lanes of an entry read
  // the same load bracket of 16 different rows, which would otherwise fall into one LDS bank
  const int row_stride = (3 * n_rho) | 1;
  double* s_tab = smem;                                        // [n_f][row_stride]: prefill, TBT, power of every load point
  const Axis axis = place_axis<AXIS>(s_tab + (size_t)n_f * row_stride, n_rho, a.axis.n_bucket);
  CellRec* s_rec = (CellRec*)axis.end;
  uint16_t* s_js = (uint16_t*)(s_rec + a.win_per_block);

  {
    const double* src = a.tab + ((size_t)g * a.n_tp + i) * n_f * 3 * n_rho;   // the type's rows are contiguous
    for (int q = threadIdx.x; q < n_f * 3 * n_rho; q += blockDim.x) {
      const int r = q / (3 * n_rho);
      s_tab[r * row_stride + (q - r * 3 * n_rho)] = src[q];
    }
  }
  stage_axis<AXIS>(a.axis, axis, s_js);
  for (int q = threadIdx.x; q < w1 - w0; q += blockDim.x) s_rec[q] = a.rec[(size_t)(w0 + q) * a.G + g];
  __syncthreads();

  const int f = threadIdx.x & (DYN_MIXED_FREQ_LANES - 1);
  const int row = threadIdx.x / DYN_MIXED_FREQ_LANES;         // 0 .. 15
  const bool f_ok = f < n_f;
  const int fc = f_ok ? f : 0;
  const double ml = a.ml[((size_t)g * a.n_tp + i) * n_f + fc];
  const double slo_ttft = a.slo_ttft[g], slo_tbt = a.slo_tbt[g];
  Lookup L;
  L.u = 0.0; L.omu = 1.0;
  use_axis<AXIS>(a.axis, axis, s_js, &L);
  L.lo = s_tab + (size_t)fc * row_stride;
  L.hi = L.lo;
  const double sd = (double)S;

  for (int e0 = 0; e0 < n_ent; e0 += 256 / DYN_MIXED_FREQ_LANES) {
    const int e = e0 + row;
    const bool e_ok = e < n_ent;
    const int ec = e_ok ? e : 0;
    const int n = ec / S + 1, sh = ec % S + 1;
    const double nd = (double)n, ad = (double)sh;
    L.den = nd * ml;
    L.rden = 1.0 / L.den;
    for (int w = w0; w < w1; ++w) {
      const CellRec rec = s_rec[w - w0];
      const double ls = div_by(rec.load * ad, sd, a.r_share);      // the part of the load this type takes
      const Looked r = table_lookup<AXIS, false>(L, ls);
      const double en = (nd * r.v[2]) * a.window_s;
      const double p_ttft = rec.xp99 * r.v[0];
      const double p_tbt = r.v[1] * rec.nonempty;
      const bool ok = f_ok && !r.ov && !(p_ttft > slo_ttft) && !(p_tbt > slo_tbt);
      // least energy of the row's admissible lanes (energies are >= +0: their bits order as integers),
      // lowest frequency among equals; +inf when no lane is admissible
      const uint64_t bits = ok ? (uint64_t)__double_as_longlong(en) : 0x7FF0000000000000ull;
      const uint32_t hi = (uint32_t)(bits >> 32), lo = (uint32_t)bits;
      const uint32_t mh = row_min_u32(hi);
      const uint32_t mlw = row_min_u32(hi == mh ? lo : 0xFFFFFFFFu);
      const uint32_t fsel = row_min_u32((ok && hi == mh && lo == mlw) ? (uint32_t)f : 0xFFu);
      if (f == 0 && e_ok) {
        const size_t o = ((size_t)w * a.G + g) * n_entry + a.types.off[i] + e;
        a.type_energy[o] = __longlong_as_double((long long)(((uint64_t)mh << 32) | mlw));
        a.type_f[o] = fsel == 0xFFu ? (int8_t)-1 : (int8_t)fsel;
      }
    }
  }
}

// Entries of a type that are not twice another.
__host__ __device__ __forceinline__ int own_entries(int n_max, int S) { return n_max / 2 * (S + (S + 1) / 2) + (n_max & 1) * S; }

// The same per-type energies with the frequencies walked by the thread: a thread is (entry, window), takes its
// share of the window's load once and keeps the least admissible energy over the frequencies in ascending order
// (strictly less replaces: the lowest frequency among equals), so nothing crosses lanes and every lane stores.
// The capacities n x max load and their reciprocals, which the other kernel forms per lane and pass, come from an
// LDS table [n_max][n_f] built once per block.  Chosen when that table fits beside the rows.
// 2n instances with 2a shares run at the utilization of n with a: load and capacity are both exactly twice as much, so every
// quotient, table value and comparison is the same to the last bit and the energy exactly twice.  Only the entries that are not twice
// another are looked up, three of four with 8 shares: 36 000 cells, 28 instances and 8 shares 282 us a call, 255 so.
// LDS: as above, then [capacity n_max*n_f] [its reciprocal n_max*n_f]
template <int AXIS>
__global__ __launch_bounds__(256) void mixed_type_walk_kernel(MixedTypeArgs a) {
  extern __shared__ double smem[];
  const int n_rho = a.n_rho, n_f = a.n_f, S = a.n_share;
  const int i = blockIdx.x % a.n_tp;
  const int g = (blockIdx.x / a.n_tp) % a.G;
  const int chunk = blockIdx.x / (a.n_tp * a.G);
  const int n_max = a.types.n_max[i];
  const int n_ent = n_max * S;                     // entries of this type
  if (n_ent == 0) return;                          // block-uniform
  const int w0 = chunk * a.win_per_block;
  const int w1 = min(w0 + a.win_per_block, a.n_window);
  const int n_entry = a.types.off[a.n_tp];

  const int row_stride = (3 * n_rho) | 1;          // see mixed_type_kernel
  double* s_tab = smem;
  const Axis axis = place_axis<AXIS>(s_tab + (size_t)n_f * row_stride, n_rho, a.axis.n_bucket);
  CellRec* s_rec = (CellRec*)axis.end;
  double* s_den = (double*)(s_rec + a.win_per_block);            // [n_max][n_f]
  double* s_rden = s_den + (size_t)n_max * n_f;
  uint16_t* s_js = (uint16_t*)(s_rden + (size_t)n_max * n_f);

  {
    const double* src = a.tab + ((size_t)g * a.n_tp + i) * n_f * 3 * n_rho;   // the type's rows are contiguous
    for (int q = threadIdx.x; q < n_f * 3 * n_rho; q += blockDim.x) {
      const int r = q / (3 * n_rho);
      s_tab[r * row_stride + (q - r * 3 * n_rho)] = src[q];
    }
  }
  stage_axis<AXIS>(a.axis, axis, s_js);
  for (int q = threadIdx.x; q < w1 - w0; q += blockDim.x) s_rec[q] = a.rec[(size_t)(w0 + q) * a.G + g];
  for (int q = threadIdx.x; q < n_max * n_f; q += blockDim.x) {
    const int n = q / n_f + 1, f = q - (n - 1) * n_f;
    const double den = (double)n * a.ml[((size_t)g * a.n_tp + i) * n_f + f];
    s_den[q] = den;
    s_rden[q] = 1.0 / den;
  }
  __syncthreads();

  const double slo_ttft = a.slo_ttft[g], slo_tbt = a.slo_tbt[g];
  Lookup L;
  L.u = 0.0; L.omu = 1.0;
  use_axis<AXIS>(a.axis, axis, s_js, &L);
  const double sd = (double)S;
  // entries that are not twice another: of every two instance counts all shares of the odd one, the odd shares of the even one
  const int per_two = S + (S + 1) / 2, n_own = own_entries(n_max, S);
  const int n_pair = n_own * (w1 - w0);                           // (window, entry), entry fastest
  for (int idx = threadIdx.x; idx < n_pair; idx += blockDim.x) {
    const int dw = idx / n_own, e = idx - dw * n_own, two = e / per_two, in_two = e - two * per_two;
    const int n = 2 * two + (in_two < S ? 1 : 2), sh = in_two < S ? in_two + 1 : 2 * (in_two - S) + 1;
    const double nd = (double)n, ad = (double)sh;
    const CellRec rec = s_rec[dw];
    const double ls = div_by(rec.load * ad, sd, a.r_share);      // the part of the load this type takes
    const double* den = s_den + (size_t)(n - 1) * n_f;
    const double* rden = s_rden + (size_t)(n - 1) * n_f;
    double best = __builtin_inf();
    int bf = -1;
    for (int f = 0; f < n_f; ++f) {                              // ascending: the lowest frequency wins equal energies
      // table_lookup's arithmetic, in the order that lets a wave stop early: its lanes hold neighbouring entries, which
      // are overloaded at much the same frequencies and rarely find less energy above the first admissible one
      const double rho = div_by(ls, den[f], rden[f]);
      bool live = !(rho > L.rho_max);
      if (__ballot(live) == 0) continue;
      double p0, p1;
      const double* tab;
      const double t = find_bracket<AXIS>(L, min_uniform(rho, L.rho_max), [&](int j) {
        tab = s_tab + (size_t)f * row_stride + 3 * j;
        p0 = tab[2]; p1 = tab[5];
      }, [&] { read_now(p0, p1); });
      const double omt = 1.0 - t;
      const double en = (nd * (omt * p0 + t * p1)) * a.window_s;
      live = live && en < best;
      if (__ballot(live) == 0) continue;
      const double pf = omt * tab[0] + t * tab[3], tb = omt * tab[1] + t * tab[4];
      if (live && !(rec.xp99 * pf > slo_ttft) && !(tb * rec.nonempty > slo_tbt)) { best = en; bf = f; }
    }
    const size_t o = ((size_t)(w0 + dw) * a.G + g) * n_entry + a.types.off[i];
    for (int q = 1; q * n <= n_max && q * sh <= S; q *= 2) {      // twice the instances under twice the load: the same utilization to the last bit
      a.type_energy[o + (q * n - 1) * S + (q * sh - 1)] = (double)q * best;
      a.type_f[o + (q * n - 1) * S + (q * sh - 1)] = (int8_t)bf;
    }
  }
}

// One wave per cell.  What bounds it: vector instructions, 8 a candidate (prefix state, instances, shares).  The first type has
// one candidate a state and the last one U + 1 states; going over all of both cost three times the candidates
// (36 000 cells, 8 shares, 16 units of GPUs, three types: 276 us, 124 us so).  LDS: [E_i(n, a) of the cell, n_entry] [D of the previous type] [D of this type]
// [choice per type and state (16-bit: n << 8 | a)], states = (units of GPUs 0..U) x (shares 0..S).
// SMAX >= n_share bounds the unrolled loop over the shares given to a type: the loads of one
// (state, n) are issued together and the running minimum is the only dependence.
template <int SMAX>
__global__ __launch_bounds__(DYN_WAVE) void mixed_combine_kernel(MixedCombineArgs a) {
  extern __shared__ double smem[];
  const int64_t cell = blockIdx.x;
  const int g = (int)(cell % a.G);
  const int S = a.n_share, n_tp = a.types.n_tp, n_entry = a.types.off[n_tp];
  const int32_t bud = a.budget[g];
  const int U = bud > 0 ? min(bud / a.unit, a.u_max) : a.u_max;
  const int S1 = S + 1;
  const int n_state_max = (a.u_max + 1) * S1;
  const int n_state = (U + 1) * S1;
  double* s_c = smem;                                  // [n_entry]
  double* s_d0 = s_c + n_entry;                        // [n_state_max]
  double* s_d1 = s_d0 + n_state_max;
  uint16_t* s_ch = (uint16_t*)(s_d1 + n_state_max);    // [n_tp][n_state_max]
  const double inf = __builtin_inf();

  for (int q = threadIdx.x; q < n_entry; q += DYN_WAVE) s_c[q] = a.type_energy[cell * n_entry + q];
  // D_0 is 0 J with nothing used and +inf elsewhere, so D_1 is the first type's own energies; of the last type's states only
  // those with all shares assigned are asked for
  double* prev = s_d0;
  double* next = s_d1;
  for (int i = 0; i < n_tp; ++i) {
    __syncthreads();
    const int units = max(a.types.units[i], 1), n_max = a.types.n_max[i];   // 0: a type of no instances
    const double* ci = s_c + a.types.off[i];
    uint16_t* ch = s_ch + (size_t)i * n_state_max;
    const bool last = i == n_tp - 1;
    if (i == 0) {
      for (int q = threadIdx.x; q < n_state; q += DYN_WAVE) {
        const int u = q / S1, sh = q - u * S1, n = u / units;
        double best = q == 0 ? 0.0 : inf;
        uint32_t bc = 0;
        if (n >= 1 && n <= n_max && n * units == u && sh >= 1) {
          const double cand = 0.0 + ci[(n - 1) * S + sh - 1];
          if (cand < best) { best = cand; bc = ((uint32_t)n << 8) | (uint32_t)sh; }
        }
        next[q] = best;
        ch[q] = (uint16_t)bc;
      }
      double* t = prev; prev = next; next = t;
      continue;
    }
    for (int q = threadIdx.x; q < (last ? U + 1 : n_state); q += DYN_WAVE) {
      const int st = last ? q * S1 + S : q;
      const int u = last ? q : st / S1, sh = st - u * S1;
      double best = prev[st];                          // the type stays unused
      uint32_t bc = 0;
      for (int n = 1; n <= n_max && n * units <= u; ++n) {
        const double* pr = prev + (u - n * units) * S1 + sh;   // pr[-x]: x shares given to this type
        const double* cn = ci + (n - 1) * S;
#pragma unroll
        for (int x = 1; x <= SMAX; ++x) {
          if (x <= sh) {
            const double cand = pr[-x] + cn[x - 1];    // +inf marks what cannot be done
            if (cand < best) { best = cand; bc = ((uint32_t)n << 8) | (uint32_t)x; }
          }
        }
      }
      next[st] = best;
      ch[st] = (uint16_t)bc;
    }
    double* t = prev; prev = next; next = t;
  }
  __syncthreads();
  double best = inf;                                   // the least energy, the fewest GPUs among equals
  int bu = -1;
  for (int u = threadIdx.x; u <= U; u += DYN_WAVE) {
    const double v = prev[u * S1 + S];
    if (v < best) { best = v; bu = u; }
  }
#pragma unroll
  for (int d = 1; d < DYN_WAVE; d <<= 1) {
    const double ov = __shfl_xor(best, d, DYN_WAVE);
    const int ou = __shfl_xor(bu, d, DYN_WAVE);
    if (ov < best || (ov == best && (uint32_t)ou < (uint32_t)bu)) { best = ov; bu = ou; }
  }
  if (threadIdx.x == 0) {
    a.energy[cell] = best;
    a.ok[cell] = bu >= 0 ? 0 : -1;
    int st = bu >= 0 ? bu * S1 + S : 0;
    for (int i = n_tp - 1; i >= 0; --i) {
      const uint32_t bc = bu >= 0 ? s_ch[(size_t)i * n_state_max + st] : 0u;
      const int n = (int)(bc >> 8), x = (int)(bc & 0xFFu);
      a.n_inst[cell * n_tp + i] = n;
      a.share[cell * n_tp + i] = x;
      a.f_index[cell * n_tp + i] = n > 0 ? (int32_t)a.type_f[cell * n_entry + a.types.off[i] + (n - 1) * S + (x - 1)] : -1;
      st -= n * a.types.units[i] * S1 + x;
    }
  }
}

// The same programme with the shares in registers: a lane holds one count of GPUs of one cell, its D over all shares; 63 / (U + 1)
// cells to a wave (lane 63 stays free of them).  For every number of instances the lane reads the row that many GPUs below from LDS
// once, and every (shares before, shares given) pair of it costs an addition and a minimum.  Nothing else is kept: the
// choices are found again on the way back, at the n_tp states of the best assignment, as the first candidate in the order
// above whose sum is the state's value.
// What bounds it: vector instructions, 2 a candidate and the lanes without one; the row reads.  36 000 cells, 8 shares, 16 units,
// three types: 73 us; 122 us by the kernel above, which stays for more than 62 units of GPUs.
// The shares are numbered from the top (t = s + SMAX - S), so that all of them assigned is t = SMAX whatever S is.
// LDS: [row SMAX + 1 of D per lane, and one of +inf before them; per type after the first] [least total per lane]
constexpr int kRowLanes = DYN_WAVE + 1;
template <int SMAX>
__global__ __launch_bounds__(DYN_WAVE) void mixed_rows_kernel(MixedCombineArgs a) {
  extern __shared__ double smem[];
  constexpr int W = SMAX + 1;
  const double inf = __builtin_inf();
  const int S = a.n_share, skip = SMAX - S, n_tp = a.types.n_tp, n_entry = a.types.off[n_tp];
  const int lane = threadIdx.x, U1 = a.u_max + 1, per_wave = (DYN_WAVE - 1) / U1;
  const int grp = lane / U1, u = lane - grp * U1;
  const int64_t cell = (int64_t)blockIdx.x * per_wave + grp;
  const bool live = grp < per_wave && cell < a.cells;
  const double* te = a.type_energy + (live ? cell : 0) * n_entry;
  double* s_v = smem + (size_t)(n_tp - 1) * kRowLanes * W;       // [DYN_WAVE]

  double cur[W];                                 // D_1: the first type's own energies
  {
    const int units = max(a.types.units[0], 1), n = u / units;   // 0: a type of no instances
    const bool some = live && n >= 1 && n <= a.types.n_max[0] && n * units == u;
    const double* c = te + (some ? (n - 1) * S : 0);
#pragma unroll
    for (int t = 0; t < W; ++t) {
      cur[t] = inf;
      if (t > skip && some) cur[t] = 0.0 + c[t - skip - 1];
      if (t == skip && live && u == 0) cur[t] = 0.0;             // nothing used
    }
  }
  for (int i = 1; i < n_tp; ++i) {
    double* rows = smem + (size_t)(i - 1) * kRowLanes * W;       // row 0: what cannot be done; row 1 + lane
    const int units = max(a.types.units[i], 1), n_end = min(a.types.n_max[i], a.u_max / units);
    const double* ci = te + a.types.off[i];
    const bool last = i == n_tp - 1;
#pragma unroll
    for (int t = 0; t < W; ++t) rows[(1 + lane) * W + t] = cur[t];
    if (lane < W) rows[lane] = inf;
    __syncthreads();
    double c[SMAX];                              // c[x - 1]: the energy of n instances with x shares; the next n's in flight
#pragma unroll
    for (int x = 0; x < SMAX; ++x) c[x] = n_end >= 1 && x < S ? ci[x] : inf;
    for (int n = 1; n <= n_end; ++n) {
      double cn[SMAX], row[SMAX];
      const double* cnext = ci + (size_t)(n < n_end ? n : 0) * S;
#pragma unroll
      for (int x = 0; x < SMAX; ++x) cn[x] = x < S ? cnext[x] : inf;
      const double* from = rows + (size_t)(live && u >= n * units ? 1 + lane - n * units : 0) * W;
#pragma unroll
      for (int t = 0; t < SMAX; ++t) row[t] = from[t];
      if (last) {
#pragma unroll
        for (int x = 1; x <= SMAX; ++x) cur[SMAX] = min_num(cur[SMAX], row[SMAX - x] + c[x - 1]);
      } else {
#pragma unroll
        for (int t = 1; t <= SMAX; ++t) {
#pragma unroll
          for (int x = 1; x <= t; ++x) cur[t] = min_num(cur[t], row[t - x] + c[x - 1]);
        }
      }
#pragma unroll
      for (int x = 0; x < SMAX; ++x) c[x] = cn[x];
    }
  }
  s_v[lane] = cur[SMAX];
  __syncthreads();
  // the least energy and the fewest GPUs that have it: every lane of a cell goes over its cell's values
  const int32_t bud = a.budget[live ? (int)(cell % a.G) : 0];
  const int U = bud > 0 ? min(bud / a.unit, a.u_max) : a.u_max;
  double best = inf;
  int bu = -1;
  for (int q = 0; q <= U; ++q) {
    const double v = s_v[live ? grp * U1 + q : DYN_WAVE - 1];
    if (v < best) { best = v; bu = q; }
  }
  const bool lead = live && u == 0;
  if (lead) {
    a.energy[cell] = best;
    a.ok[cell] = bu >= 0 ? 0 : -1;
  }
  const uint64_t mine = live ? ((1ull << U1) - 1ull) << (grp * U1) : 0ull;   // the cell's lanes
  int su = bu >= 0 ? bu : 0, st = bu >= 0 ? SMAX : skip;         // the state on the way back
  double val = best;
  for (int i = n_tp - 1; i >= 0; --i) {
    const int units = max(a.types.units[i], 1);
    int n = 0, x = 0;
    if (i == 0) {
      if (bu >= 0 && su > 0) { n = su / units; x = st - skip; }
    } else {
      const double* rows = smem + (size_t)(i - 1) * kRowLanes * W;
      const double* at = rows + (size_t)(live ? 1 + grp * U1 + su : 0) * W;
      const int n_cand = min(a.types.n_max[i], a.u_max / units) * S;
      bool open = live && bu >= 0 && at[st] != val;              // else the type is not used
      for (int f0 = 0; f0 < n_cand && __ballot(open) != 0; f0 += U1) {
        const int f = f0 + u, fn = f / S + 1, fx = f - (fn - 1) * S + 1;
        const bool can = open && f < n_cand && fn * units <= su && fx <= st - skip;
        const bool hit = can && at[-fn * units * W + st - fx] + te[a.types.off[i] + f] == val;
        const uint64_t who = __ballot(hit) & mine;
        if (open && who != 0) {
          const int ff = f0 + (int)__builtin_ctzll(who) - grp * U1;
          n = ff / S + 1;
          x = ff - (n - 1) * S + 1;
          open = false;
        }
      }
      if (n > 0) {
        val = at[-n * units * W + st - x];
        su -= n * units;
        st -= x;
      }
    }
    if (lead) {
      a.n_inst[cell * n_tp + i] = n;
      a.share[cell * n_tp + i] = x;
      a.f_index[cell * n_tp + i] = n > 0 ? (int32_t)a.type_f[cell * n_entry + a.types.off[i] + (n - 1) * S + (x - 1)] : -1;
    }
  }
}

size_t type_lds(const MixedTypeArgs& a, int axis) {
  return (size_t)a.n_f * ((3 * a.n_rho) | 1) * sizeof(double) + dyn_axis_lds(a.axis, axis) + (size_t)a.win_per_block * sizeof(CellRec);
}
size_t type_walk_lds(const MixedTypeArgs& a, int axis) {   // plus the capacities of the type with most instances
  int n_max = 0;
  for (int i = 0; i < a.n_tp; ++i) n_max = std::max(n_max, a.types.n_max[i]);
  return type_lds(a, axis) + (size_t)2 * n_max * a.n_f * sizeof(double);
}

}  // namespace

size_t dyn_mixed_combine_lds(int32_t n_tp, int32_t n_entry, int32_t u_max, int32_t n_share) {
  const size_t n_state = (size_t)(u_max + 1) * (n_share + 1);
  return ((size_t)n_entry + 2 * n_state) * sizeof(double) + (size_t)n_tp * n_state * sizeof(uint16_t) + 8;
}

// A type's block takes 256 of its (window, entry) pairs at a time, and the last time what is left.  36 000 cells of 96, 48 and 24 entries
// of their own: 14 windows 260 us (2816 places for 2352 pairs), 16 windows 255 (2816 for 2688).
int32_t dyn_mixed_even_windows(const MixedTypeArgs& a) {
  int32_t best = a.win_per_block;
  int64_t least = INT64_MAX, of = 1;
  for (int32_t w = a.win_per_block; w <= std::min(DYN_MAX_WIN_PER_BLOCK, a.win_per_block + a.win_per_block / 4); ++w) {
    int64_t rounds = 0;
    for (int i = 0; i < a.n_tp; ++i) rounds += ((int64_t)own_entries(a.types.n_max[i], a.n_share) * w + 255) / 256;
    if (least == INT64_MAX || rounds * of < least * w) { least = rounds; of = w; best = w; }
  }
  return best;
}

hipError_t dyn_launch_mixed_types(const MixedTypeArgs& a, hipStream_t s) {
  const int n_chunk = (a.n_window + a.win_per_block - 1) / a.win_per_block;
  const dim3 grid((unsigned)((size_t)n_chunk * a.G * a.n_tp)), block(256);
  int axis = dyn_axis(a.axis);
  if (type_lds(a, axis) > DYN_LDS_BUDGET) axis = DYN_AXIS_SEARCH;
  const size_t lds = type_lds(a, axis);
  if (lds > DYN_LDS_BUDGET) return hipErrorInvalidValue;
  DynTimed timed(DYN_K_MIXED_TYPES, s);
  const size_t lds_walk = type_walk_lds(a, axis);
  if (lds_walk <= DYN_LDS_BUDGET) {
    if (axis == DYN_AXIS_EVEN) hipLaunchKernelGGL(mixed_type_walk_kernel<DYN_AXIS_EVEN>, grid, block, lds_walk, s, a);
    else if (axis == DYN_AXIS_SINGLE) hipLaunchKernelGGL(mixed_type_walk_kernel<DYN_AXIS_SINGLE>, grid, block, lds_walk, s, a);
    else hipLaunchKernelGGL(mixed_type_walk_kernel<DYN_AXIS_SEARCH>, grid, block, lds_walk, s, a);
    return hipGetLastError();
  }
  if (axis == DYN_AXIS_EVEN) hipLaunchKernelGGL(mixed_type_kernel<DYN_AXIS_EVEN>, grid, block, lds, s, a);
  else if (axis == DYN_AXIS_SINGLE) hipLaunchKernelGGL(mixed_type_kernel<DYN_AXIS_SINGLE>, grid, block, lds, s, a);
  else hipLaunchKernelGGL(mixed_type_kernel<DYN_AXIS_SEARCH>, grid, block, lds, s, a);
  return hipGetLastError();
}

template <int SMAX>
bool launch_rows(const MixedCombineArgs& a, hipStream_t s) {   // false: the shape is not for it
  const int U1 = a.u_max + 1;
  const size_t lds = ((size_t)(a.types.n_tp - 1) * kRowLanes * (SMAX + 1) + DYN_WAVE) * sizeof(double);
  if (U1 > DYN_WAVE - 1 || lds > DYN_LDS_BUDGET) return false;
  const int64_t per_wave = (DYN_WAVE - 1) / U1;
  hipLaunchKernelGGL(mixed_rows_kernel<SMAX>, dim3((unsigned)((a.cells + per_wave - 1) / per_wave)), dim3(DYN_WAVE), lds, s, a);
  return true;
}

hipError_t dyn_launch_mixed_combine(const MixedCombineArgs& a, hipStream_t s) {
  const size_t lds = dyn_mixed_combine_lds(a.types.n_tp, a.types.off[a.types.n_tp], a.u_max, a.n_share);
  if (lds > DYN_LDS_BUDGET) return hipErrorInvalidValue;
  DynTimed timed(DYN_K_MIXED_COMBINE, s);
  if (a.n_share <= 4 ? launch_rows<4>(a, s) : a.n_share <= 8 ? launch_rows<8>(a, s) : launch_rows<DYN_MIXED_MAX_SHARES>(a, s)) return hipGetLastError();
  const dim3 grid((unsigned)a.cells), block(DYN_WAVE);
  if (a.n_share <= 4) hipLaunchKernelGGL(mixed_combine_kernel<4>, grid, block, lds, s, a);
  else if (a.n_share <= 8) hipLaunchKernelGGL(mixed_combine_kernel<8>, grid, block, lds, s, a);
  else hipLaunchKernelGGL(mixed_combine_kernel<DYN_MIXED_MAX_SHARES>, grid, block, lds, s, a);
  return hipGetLastError();
}
