// The three controllers of Section IV-B, top down, on the aggregates of a trace:
//   hier_shard_kernel   scale-out/in and shard-up/down.  Per (window, class): the node count of the
//                       window's epoch = ceil(peak load of the epoch / largest profiled load of one node
//                       at the reference configuration), at least one; then the layout (instances, TP)
//                       of least energy at the reference frequency among those that fit the nodes' GPUs
//                       and meet the SLO;
//   hier_freq_kernel    scale-up/down: per tick the frequency of least power among those that meet the
//                       SLO under the tick's load (the reference frequency, counted, if none does);
//                       energy of a (window, class) = its ticks' energies added in time order; window
//                       totals = the classes' energies added in class order.
//   hier_spill_*        (fragmentation rule only) before the others: per epoch, classes in ascending order,
//                       the node counts, the fraction of its arriving load every pool keeps and the loads the
//                       pools serve in every window and tick once the rest has been forwarded to the next class.
// The frequency kernel's tables stay in global memory (they are a few hundred KB and live in L2; copying a class's tables
// to LDS per block was measured to cost more than the look-ups it serves).  Two things matter instead:
// neighbouring lanes share the class and the layout, so that a wave's gathers fall into a few table rows, and the
// kernel takes its look-ups three at a time, level by level (capacity -> grid points -> table values), so that a
// thread waits for a few rounds of loads per three frequencies, not nine.
#include <algorithm>

#include "dyn_hier.h"
#include "dyn_mixed.h"
#include "dyn_device.h"

namespace {

constexpr int kShardWaves = 4;          // of a block of the shard kernel
constexpr size_t kRowsLds = 16 * 1024;  // rows at the reference frequency are staged in LDS up to this
constexpr int kFreqChunk = 3;           // look-ups a thread of the frequency kernel has in flight: four need the registers of a third of the waves (35 us, 27)
constexpr int kSpillLds = 48 * 1024;    // an epoch's window loads are staged in LDS when they fit in this
constexpr int kSpillRun = 8;            // classes whose tick loads a thread fetches ahead of the chain

struct Row { double pf, tb, pw; bool ov; };

// Bracket of a clamped load fraction rc: largest grid index i <= n_rho-2 with grid[i] <= rc.
// EVEN: one multiplication, or one less where rc is just below the point.
template <int AXIS>
__device__ __forceinline__ int bracket(const Lookup& L, double rc) {
  if ((AXIS & ~DYN_AXIS_GLOBAL) != DYN_AXIS_EVEN) return find_index<AXIS>(L, rc);
  int j = (int)min((uint32_t)(int)(rc * L.scale), (uint32_t)(L.n_rho - 2));
  while (j > 0 && L.grid[3 * j] > rc) --j;
  return j;
}

// Linear interpolation in table row `row` (class, TP, frequency) between grid points j and j+1.
template <int AXIS>
__device__ __forceinline__ void interpolate(const double* tab, const Lookup& L, size_t row, int j, double rc, Row* r) {
  double t;
  if ((AXIS & ~DYN_AXIS_GLOBAL) == DYN_AXIS_EVEN) {
    const double* g = L.grid + 3 * j;
    t = div_by(rc - g[0], g[1], g[2]);
  } else {
    const double g0 = L.grid[j + 1], g1 = L.grid[j + 2];
    t = div_by(rc - g0, g1 - g0, L.rinv[j + 1]);             // RN(1 / spacing)
  }
  const double omt = 1.0 - t;
  const double* v = tab + (row * L.n_rho + j) * 3;
  r->pf = omt * v[0] + t * v[3];
  r->tb = omt * v[1] + t * v[4];
  r->pw = omt * v[2] + t * v[5];
}

__device__ __forceinline__ double wave_max_f64(double v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = fmax(v, __shfl_xor(v, d, DYN_WAVE));
  return v;
}

// Largest value of each row of 16 lanes, in all of the row's lanes (rotations by 1, 2, 4 and 8 lanes).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double row_max_f64(double v) {
  v = fmax(v, dpp_f64<0x121>(v));
  v = fmax(v, dpp_f64<0x122>(v));
  v = fmax(v, dpp_f64<0x124>(v));
  return fmax(v, dpp_f64<0x128>(v));
}

// The node count of epoch e for class g (a wave's work; the same in every lane).
__device__ __forceinline__ int32_t epoch_nodes(const HierArgs& a, int e, int g, int lane) {
  const int e0 = e * a.epoch_windows, e1 = min(a.n_window, e0 + a.epoch_windows);
  double peak = 0.0;
  for (int i = e0 + lane; i < e1; i += DYN_WAVE) peak = fmax(peak, a.rec_c[(size_t)i * a.G + g].load);
  peak = row_max_f64(peak);                                  // of 16 lanes, then of the four rows
  peak = fmax(fmax(lane_f64(peak, 0), lane_f64(peak, 16)), fmax(lane_f64(peak, 32), lane_f64(peak, 48)));
  const int inst = max(1, a.gpus_per_node / a.tp[a.tp_ref]);
  const double ml_node = ((double)inst * a.ml[((size_t)g * a.n_tp + a.tp_ref) * a.n_f + a.f_ref]) * a.axis.rho_max;
  const double q = ceil(peak / ml_node);
  return q < 1.0 ? 1 : (q > 2147483647.0 ? 2147483647 : (int32_t)q);
}

// Block = (run of windows, class), one wave per `per_wave` windows after each other.  A lane is a layout; what depends on the class and the
// layout only (capacity and its reciprocal, the rows at the reference frequency, which a block keeps in LDS) is formed once, a wave's
// records and statuses are read together, and the nodes are counted where an epoch begins.  A wave a cell, which did all of that
// for one look-up per lane, took 28 us for 36 000 cells of 48 layouts, bound by its chain of loads.
// The load axis is read from global memory, at most five words a look-up: copies in LDS are no faster where they are small (36 000 cells, 64 even points
// 95.1 us, 95.2) and cost waves where they are not (9000 cells, 64 uneven points, 38 KB: 49 us, 61; 4000 points 64, more than 300).
// LDS: [rows at f_ref n_tp*3*n_rho (ROWS)]
template <bool ROWS, int FORM>
__global__ __launch_bounds__(kShardWaves* DYN_WAVE) void hier_shard_kernel(HierArgs a, int per_wave) {
  constexpr int AXIS = FORM | DYN_AXIS_GLOBAL;
  extern __shared__ double s_rows[];
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DYN_WAVE);
  const int g = blockIdx.x % a.G;
  const int w0 = ((int)(blockIdx.x / a.G) * kShardWaves + wave) * per_wave, w1 = min(w0 + per_wave, a.n_window);
  const size_t row_ref = ((size_t)g * a.n_tp) * a.n_f + a.f_ref;   // of the first TP degree; the next is n_f rows on

  CellRec mine;                                              // lane i: the wave's window i (per_wave <= 64)
  mine.load = mine.xp99 = mine.nonempty = 0.0;
  if (w0 + lane < w1) {
    const size_t cell = (size_t)(w0 + lane) * a.G + g;
    mine = a.rec_c[cell];
    if (a.served_c) mine.load = a.served_c[cell];            // fragmentation rule: loads and node counts come from the spill kernels
    if (a.cstat_c[cell]) atomicOr(a.status, (uint32_t)a.cstat_c[cell]);
  }
  if (ROWS)
    for (int t = wave; t < a.n_tp; t += kShardWaves)
      for (int i = lane; i < 3 * a.n_rho; i += DYN_WAVE) s_rows[t * 3 * a.n_rho + i] = a.tab[(row_ref + (size_t)t * a.n_f) * 3 * a.n_rho + i];

  struct Layout { int64_t gpus; double nd; };
  Lookup L;
  Layout y;
  auto take = [&](int l) {                                   // the constants of layout l
    const int n = a.lay_n[l], ti = a.lay_tp[l];
    y.gpus = (int64_t)n * a.tp[ti];
    y.nd = (double)n;
    L.den = y.nd * a.ml[row_ref + (size_t)ti * a.n_f];
    L.rden = 1.0 / L.den;
    L.lo = ROWS ? s_rows + ti * 3 * a.n_rho : a.tab + (row_ref + (size_t)ti * a.n_f) * 3 * a.n_rho;
    L.hi = L.lo;
  };
  use_axis<AXIS>(a.axis, Axis(), nullptr, &L);
  L.u = 0.0; L.omu = 1.0;
  take(min(lane, a.n_layout - 1));
  const double slo_t = a.slo_ttft[g], slo_b = a.slo_tbt[g];
  __syncthreads();
  int e_now = -1;
  int64_t budget = 0;
  for (int w = w0; w < w1; ++w) {
    const int at = w - w0;
    const double load = lane_f64(mine.load, at), xp99 = lane_f64(mine.xp99, at), nonempty = lane_f64(mine.nonempty, at);
    const size_t cell = (size_t)w * a.G + g;
    const int e = w / a.epoch_windows;
    if (e != e_now) {
      e_now = e;
      const int32_t nodes = a.served_c ? a.nodes[(size_t)e * a.G + g] : epoch_nodes(a, e, g, lane);
      if (!a.served_c && w == e * a.epoch_windows && lane == 0) a.nodes[(size_t)e * a.G + g] = nodes;
      budget = (int64_t)nodes * a.gpus_per_node;
    }
    double best_e = __builtin_inf();
    int best = 0x7FFFFFFF;
    for (int l0 = 0; l0 < a.n_layout; l0 += DYN_WAVE) {
      const int l = l0 + lane;
      if (a.n_layout > DYN_WAVE) take(min(l, a.n_layout - 1));
      const Looked r = table_lookup<AXIS, false>(L, load);
      const bool fits = l < a.n_layout && y.gpus <= budget;
      const bool ok = fits && !(r.ov || xp99 * r.v[0] > slo_t || r.v[1] * nonempty > slo_b);
      const double en = fits ? (y.nd * r.v[2]) * a.window_s : __builtin_inf();
      if (a.lay_energy && l < a.n_layout) {                  // the sequence selection takes it from here
        a.lay_energy[cell * a.n_layout + l] = en;
        a.lay_flags[cell * a.n_layout + l] = ok ? (uint8_t)DYN_F_FEASIBLE : (uint8_t)0;
      }
      if (ok && (best == 0x7FFFFFFF || en < best_e)) { best_e = en; best = l; }   // l ascends per lane
    }
    // least energy, the lowest index among equals; energies are >= +0, so their bits order as integers
    const uint64_t bits = (uint64_t)__double_as_longlong(best_e);
    const bool has = best != 0x7FFFFFFF;
    const uint32_t hi = has ? (uint32_t)(bits >> 32) : 0xFFFFFFFFu;
    const uint32_t most = wave_min_u32(hi);
    const uint32_t lo = has && hi == most ? (uint32_t)bits : 0xFFFFFFFFu;
    const uint32_t least = wave_min_u32(lo);
    const uint32_t l = wave_min_u32(has && hi == most && lo == least ? (uint32_t)best : 0xFFFFFFFFu);
    if (lane == 0) a.layout_sel[cell] = (int32_t)l;          // -1 where no lane has one
  }
}

// Block = (run of windows, run of classes); its cells are its windows' classes, one window after the other.  A thread takes (cell, tick) pairs, ticks fastest, so that
// the ticks of a cell, which share the layout and mostly the bracket, are neighbouring lanes and read the same few lines of the tables.  The cells' capacities per
// frequency and their reciprocals come from a table in LDS (TABLED; a division and a gather less per look-up).  Frequencies and energies meet in LDS: they
// leave it with the classes side by side, and a thread per cell adds its ticks in time order, in chunks of DYN_FREQ_CHUNK.  With one run of
// classes the windows' totals are added here too, in class order.  With a block per class and 256 ticks, results written a class apart
// and a kernel of its own for the sums: 31 + 7.6 us for 432 000 ticks.
// LDS: [load axis] [energy chunk*cells] [capacities, reciprocals cells*n_f each (TABLED)] [instances cells] [frequency chunk*cells] [table row cells] [first tick cells]
//      [class cells] [bucket index]
template <bool TABLED, int AXIS>
__global__ __launch_bounds__(DYN_FREQ_THREADS) __attribute__((amdgpu_waves_per_eu(6, 6))) void hier_freq_kernel(HierArgs a, DynFreqShape f) {
  extern __shared__ double s_freq[];
  const int run = f.run, chunk = f.chunk, most = f.wins * run;
  const int w0 = (int)(blockIdx.x / f.n_run) * f.wins, g0 = (int)(blockIdx.x % f.n_run) * run;
  const int n_g = min(run, a.G - g0), n_w = min(f.wins, a.n_window - w0), n_c = n_w * n_g;
  const Axis axis = place_axis<AXIS>(s_freq, a.n_rho, a.axis.n_bucket);
  double* s_e = axis.end;                                    // [chunk][most]
  double* s_den = s_e + (size_t)chunk * most;                // [most][n_f]
  double* s_rden = s_den + (TABLED ? (size_t)most * a.n_f : 0);
  double* s_nd = s_rden + (TABLED ? (size_t)most * a.n_f : 0);
  int32_t* s_f = (int32_t*)(s_nd + most);                    // [chunk][most]; bit 30: no frequency was admissible
  int32_t* s_row = s_f + chunk * most;                       // first table row of the cell's layout; -1: no layout
  int32_t* s_at = s_row + most;                              // the cell's first tick
  int32_t* s_g = s_at + most;                                // the cell's class
  uint16_t* s_js = (uint16_t*)(s_g + most);
  stage_axis<AXIS>(a.axis, axis, s_js);
  for (int i = threadIdx.x; i < n_c; i += blockDim.x) {
    const int dw = i / n_g, g = g0 + (i - dw * n_g), w = w0 + dw;
    const int l = a.layout_sel[(size_t)w * a.G + g];
    s_row[i] = l < 0 ? -1 : (g * a.n_tp + a.lay_tp[l]) * a.n_f;
    s_nd[i] = l < 0 ? 1.0 : (double)a.lay_n[l];
    s_at[i] = w * a.n_tick * a.G + g;                        // below 2^30
    s_g[i] = g;
  }
  __syncthreads();
  if (TABLED) {
    for (int i = threadIdx.x; i < n_c * a.n_f; i += blockDim.x) {
      const int c = i / a.n_f;
      const double den = s_nd[c] * a.ml[(size_t)max(s_row[c], 0) + (i - c * a.n_f)];
      s_den[i] = den;
      s_rden[i] = 1.0 / den;
    }
    __syncthreads();
  }
  Lookup x;
  use_axis<AXIS>(a.axis, axis, s_js, &x);
  const double rho_max = a.axis.rho_max;
  double sum = 0.0;                                          // thread i: of cell i (at most as many as threads)
  int32_t viol = 0;
  for (int q0 = 0; q0 < a.n_tick; q0 += chunk) {
    const int n_q = min(chunk, a.n_tick - q0);
    int stride = most;                                       // not known to stay the same: the addresses of the sums below are not kept over the look-ups
    asm volatile("" : "+s"(stride));
    for (int i = threadIdx.x; i < n_c * n_q; i += blockDim.x) {
      const int c = i / n_q, q = i - c * n_q;
      const int row0 = s_row[c], at = s_at[c] + (q0 + q) * a.G;
      if (a.cstat_f[at]) atomicOr(a.status, (uint32_t)a.cstat_f[at]);
      if (row0 < 0) {
        s_f[q * stride + c] = -1;
        s_e[q * stride + c] = 0.0;
        continue;
      }
      const CellRec rec = a.rec_f[at];
      const double load = a.served_f ? a.served_f[at] : rec.load;
      const double nd = s_nd[c];
      const int g = s_g[c];
      const double slo_t = a.slo_ttft[g], slo_b = a.slo_tbt[g];
      int bf = -1;
      double bp = __builtin_inf(), pw_ref = 0.0;
      for (int f0 = 0; f0 < a.n_f; f0 += kFreqChunk) {
        double rc[kFreqChunk];
        bool ov[kFreqChunk];
        int j[kFreqChunk];
        Row r[kFreqChunk];
#pragma unroll
        for (int k = 0; k < kFreqChunk; ++k) {               // level 1: capacities
          const int fi = min(f0 + k, a.n_f - 1);
          const double rho = TABLED ? div_by(load, s_den[c * a.n_f + fi], s_rden[c * a.n_f + fi]) : load / (nd * a.ml[row0 + fi]);
          ov[k] = rho > rho_max;
          rc[k] = ov[k] ? rho_max : rho;
        }
#pragma unroll
        for (int k = 0; k < kFreqChunk; ++k) j[k] = bracket<AXIS>(x, rc[k]);   // level 2: the load axis
#pragma unroll
        for (int k = 0; k < kFreqChunk; ++k)                 // level 3: table values
          interpolate<AXIS>(a.tab, x, (size_t)(row0 + min(f0 + k, a.n_f - 1)), j[k], rc[k], &r[k]);
#pragma unroll
        for (int k = 0; k < kFreqChunk; ++k) {               // ascending frequency: the lowest wins equal powers
          const int fi = f0 + k;
          if (fi >= a.n_f) break;
          if (fi == a.f_ref) pw_ref = r[k].pw;
          if (ov[k] || rec.xp99 * r[k].pf > slo_t || r[k].tb * rec.nonempty > slo_b) continue;
          if (bf < 0 || r[k].pw < bp) { bf = fi; bp = r[k].pw; }
        }
      }
      int32_t none = 0;
      if (bf < 0) {                                          // nothing admissible: the reference frequency, counted
        bp = pw_ref;
        bf = a.f_ref;
        none = 1 << 30;
      }
      s_f[q * stride + c] = bf | none;
      s_e[q * stride + c] = (nd * bp) * a.tick_s;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n_c * n_q; i += blockDim.x) {
      const int q = i / n_c, c = i - q * n_c;
      const int32_t v = s_f[q * stride + c];
      a.f_sel[s_at[c] + (q0 + q) * a.G] = v < 0 ? -1 : v & ~(1 << 30);
    }
    if ((int)threadIdx.x < n_c)
      for (int q = 0; q < n_q; ++q) {                        // time order
        sum += s_e[q * stride + threadIdx.x];
        const int32_t v = s_f[q * stride + threadIdx.x];
        viol += v >= 0 ? v >> 30 : 0;
      }
    __syncthreads();
  }
  if ((int)threadIdx.x < n_c) {
    const int dw = threadIdx.x / n_g;
    const size_t cell = (size_t)(w0 + dw) * a.G + g0 + ((int)threadIdx.x - dw * n_g);
    const bool has = s_row[threadIdx.x] >= 0;
    a.energy[cell] = has ? sum : __builtin_inf();
    a.violations[cell] = has ? viol : 0;
    s_e[threadIdx.x] = sum;
  }
  if (f.n_run > 1) return;                                   // the totals are another kernel's
  __syncthreads();
  if ((int)threadIdx.x < n_w) {                              // thread i: window i
    const double* e_w = s_e + threadIdx.x * n_g;
    const int32_t* row_w = s_row + threadIdx.x * n_g;
    double e = 0.0;
    int32_t ninf = 0;
#pragma unroll 4
    for (int g = 0; g < n_g; ++g) {
      if (row_w[g] >= 0) e += e_w[g]; else ++ninf;
    }
    a.win_energy[w0 + threadIdx.x] = e;
    a.win_inf[w0 + threadIdx.x] = ninf;
  }
}

// Fragmentation rule, window level.  One wave per epoch, lanes stride the epoch's windows, classes one after the
// other: what a class forwards arrives at the next.  STAGED (at most one window per lane and the epoch's loads fit in
// LDS): loads and node capacities are copied to LDS up front, the forwarded load stays in a register and the results
// per class are collected in LDS, so the chain over the classes waits for LDS and a short wave reduction per class,
// never for global memory.
template <bool STAGED>
__global__ __launch_bounds__(DYN_WAVE) void hier_spill_epoch_kernel(HierArgs a) {
  extern __shared__ double s_spill[];                        // STAGED: loads [windows of the epoch][G], capacity, its reciprocal, keep [G] each, nodes [G]
  const int e = blockIdx.x, lane = threadIdx.x;
  const int e0 = e * a.epoch_windows, e1 = min(a.n_window, e0 + a.epoch_windows);
  const int G = a.G;
  const int inst = max(1, a.gpus_per_node / a.tp[a.tp_ref]);
  const double rho_max = a.axis.rho_max;
  const double guard = 1.0 - 0x1p-40;
  double* s_load = s_spill;
  double* s_cap = s_spill + (size_t)min(a.epoch_windows, a.n_window) * G;
  double* s_rcap = s_cap + G;                                // RN(1 / capacity)
  double* s_keep = s_rcap + G;
  int32_t* s_nodes = (int32_t*)(s_keep + G);
  if (STAGED) {
    for (int i = lane; i < (e1 - e0) * G; i += DYN_WAVE) s_load[i] = a.rec_c[(size_t)e0 * G + i].load;
    for (int g = lane; g < G; g += DYN_WAVE) {
      s_cap[g] = ((double)inst * a.ml[((size_t)g * a.n_tp + a.tp_ref) * a.n_f + a.f_ref]) * rho_max;
      s_rcap[g] = 1.0 / s_cap[g];
    }
    __syncthreads();
  } else {
    for (int i = e0 + lane; i < e1; i += DYN_WAVE) a.fwd[i] = 0.0;
  }
  const bool mine = e0 + lane < e1;                          // STAGED: this lane's window
  double fwd = 0.0;
  for (int g = 0; g < G; ++g) {
    double arrive = 0.0, peak = 0.0, ml_node;
    if (STAGED) {
      if (mine) arrive = s_load[lane * G + g] + fwd;
      peak = row_max_f64(arrive);                            // lanes without a window hold 0
      if (e1 - e0 > 16) peak = fmax(peak, __shfl_xor(peak, 16, DYN_WAVE));
      if (e1 - e0 > 32) peak = fmax(peak, __shfl_xor(peak, 32, DYN_WAVE));
      ml_node = s_cap[g];
    } else {
      for (int i = e0 + lane; i < e1; i += DYN_WAVE) peak = fmax(peak, a.rec_c[(size_t)i * G + g].load + a.fwd[i]);
      peak = wave_max_f64(peak);
      ml_node = ((double)inst * a.ml[((size_t)g * a.n_tp + a.tp_ref) * a.n_f + a.f_ref]) * rho_max;
    }
    const double q = STAGED ? div_by(peak, ml_node, s_rcap[g]) : peak / ml_node;
    const double fl = floor(q);
    double keep = 1.0;
    int32_t nodes;
    if (g < G - 1 && fl >= 1.0 && fl < q && fl < 2147483647.0) {
      nodes = (int32_t)fl;
      keep = ((fl * ml_node) / peak) * guard;
    } else {
      const double up = ceil(q);
      nodes = up < 1.0 ? 1 : (up > 2147483647.0 ? 2147483647 : (int32_t)up);
    }
    if (STAGED) {
      if (lane == 0) { s_nodes[g] = nodes; s_keep[g] = keep; }
      if (mine) {
        const double served = keep * arrive;
        s_load[lane * G + g] = served;
        fwd = arrive - served;
      }
    } else {
      if (lane == 0) {
        a.nodes[(size_t)e * G + g] = nodes;
        a.keep[(size_t)e * G + g] = keep;
      }
      for (int i = e0 + lane; i < e1; i += DYN_WAVE) {
        const double arr = a.rec_c[(size_t)i * G + g].load + a.fwd[i];
        const double served = keep * arr;
        a.served_c[(size_t)i * G + g] = served;
        a.fwd[i] = arr - served;                             // read again by this lane only
      }
    }
  }
  if (STAGED) {
    __syncthreads();
    for (int i = lane; i < (e1 - e0) * G; i += DYN_WAVE) a.served_c[(size_t)e0 * G + i] = s_load[i];
    for (int g = lane; g < G; g += DYN_WAVE) {
      a.nodes[(size_t)e * G + g] = s_nodes[g];
      a.keep[(size_t)e * G + g] = s_keep[g];
    }
  }
}

// Fragmentation rule, tick level: one thread per tick walks the classes with the kept fractions of the tick's epoch;
// the loads of kSpillRun classes are fetched together, ahead of the chain that links them.
__global__ __launch_bounds__(DYN_WAVE) void hier_spill_tick_kernel(HierArgs a) {
  const int64_t wt = (int64_t)blockIdx.x * DYN_WAVE + threadIdx.x;
  if (wt >= (int64_t)a.n_window * a.n_tick) return;
  const int e = (int)(wt / a.n_tick) / a.epoch_windows;
  const double* keep = a.keep + (size_t)e * a.G;
  const CellRec* rec = a.rec_f + (size_t)wt * a.G;
  double* served_f = a.served_f + (size_t)wt * a.G;
  double fwd = 0.0;
  for (int g0 = 0; g0 < a.G; g0 += kSpillRun) {
    double own[kSpillRun], k[kSpillRun];
#pragma unroll
    for (int c = 0; c < kSpillRun; ++c) {
      const int g = min(g0 + c, a.G - 1);
      own[c] = rec[g].load;
      k[c] = keep[g];
    }
#pragma unroll
    for (int c = 0; c < kSpillRun; ++c) {
      if (g0 + c >= a.G) break;
      const double arr = own[c] + fwd;
      const double served = k[c] * arr;
      served_f[g0 + c] = served;
      fwd = arr - served;
    }
  }
}

template <typename F>
void with_axis(int axis, F&& f) {
  if (axis == DYN_AXIS_EVEN) f(std::integral_constant<int, DYN_AXIS_EVEN>());
  else if (axis == DYN_AXIS_SINGLE) f(std::integral_constant<int, DYN_AXIS_SINGLE>());
  else f(std::integral_constant<int, DYN_AXIS_SEARCH>());
}

}  // namespace

hipError_t dyn_launch_hier_spill(const HierArgs& a, hipStream_t s) {
  const int64_t ticks = (int64_t)a.n_window * a.n_tick;
  const size_t lds = ((size_t)std::min(a.epoch_windows, a.n_window) * a.G + 3 * (size_t)a.G) * sizeof(double) + (size_t)a.G * sizeof(int32_t);
  DynTimed timed(DYN_K_HIER, s);
  if (a.epoch_windows <= DYN_WAVE && lds <= (size_t)kSpillLds)
    hipLaunchKernelGGL(hier_spill_epoch_kernel<true>, dim3((unsigned)a.n_epoch), dim3(DYN_WAVE), lds, s, a);
  else
    hipLaunchKernelGGL(hier_spill_epoch_kernel<false>, dim3((unsigned)a.n_epoch), dim3(DYN_WAVE), 0, s, a);
  hipLaunchKernelGGL(hier_spill_tick_kernel, dim3((unsigned)((ticks + DYN_WAVE - 1) / DYN_WAVE)), dim3(DYN_WAVE), 0, s, a);
  return hipGetLastError();
}

hipError_t dyn_launch_hier_shard(const HierArgs& a, hipStream_t s) {
  // Windows a wave: as many as leave the device about 6000 waves, and no more than 8; the blocks' set-up is by then a small part.
  const int64_t cells = (int64_t)a.n_window * a.G;
  const int per_wave = (int)std::max<int64_t>(1, std::min<int64_t>(8, cells / 6144));
  const int64_t runs = (a.n_window + (int64_t)per_wave * kShardWaves - 1) / ((int64_t)per_wave * kShardWaves);
  const size_t rows = (size_t)a.n_tp * 3 * a.n_rho * sizeof(double);
  // a load axis beyond a compute unit's LDS is refused
  if (dyn_axis_lds(a.axis, a.axis.single_point ? DYN_AXIS_SINGLE : DYN_AXIS_SEARCH) > 160 * 1024) return hipErrorInvalidValue;
  DynTimed timed(DYN_K_HIER, s);
  with_axis(dyn_axis(a.axis), [&](auto x) {
    const dim3 grid((unsigned)(runs * a.G)), block(kShardWaves * DYN_WAVE);
    if (rows <= kRowsLds) hipLaunchKernelGGL((hier_shard_kernel<true, decltype(x)::value>), grid, block, rows, s, a, per_wave);
    else hipLaunchKernelGGL((hier_shard_kernel<false, decltype(x)::value>), grid, block, 0, s, a, per_wave);
  });
  return hipGetLastError();
}

hipError_t dyn_launch_hier_ticks(const HierArgs& a, hipStream_t s) {
  const int axis = dyn_axis(a.axis);
  const DynFreqShape f = dyn_freq_shape(a.n_window, a.G, a.n_tick, a.n_f, dyn_axis_lds(a.axis, axis), a.n_cu);
  {
    DynTimed timed(DYN_K_HIER, s);
    const dim3 grid((unsigned)f.blocks), block(DYN_FREQ_THREADS);
    with_axis(axis, [&](auto x) {
      constexpr int FORM = decltype(x)::value;
      if (f.staged) hipLaunchKernelGGL((hier_freq_kernel<true, FORM>), grid, block, f.lds, s, a, f);
      else if (f.tabled) hipLaunchKernelGGL((hier_freq_kernel<true, FORM | DYN_AXIS_GLOBAL>), grid, block, f.lds, s, a, f);
      else hipLaunchKernelGGL((hier_freq_kernel<false, FORM | DYN_AXIS_GLOBAL>), grid, block, f.lds, s, a, f);
    });
  }
  if (f.n_run > 1) {
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : dyn_launch_window_totals(a.layout_sel, a.energy, a.n_window, a.G, a.win_energy, a.win_inf, s);
  }
  return hipGetLastError();
}
