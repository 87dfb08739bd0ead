// Device-side helpers shared by the HIP sources that look the profile up per thread
// (wave reductions, exact division by a fixed divisor, the table look-up itself).
#ifndef DYN_DEVICE_H_
#define DYN_DEVICE_H_

#include "dyn_internal.h"

namespace {

template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
// Reductions over the 64 lanes of a fully active wave (wave-uniform result): rotations by
// 1, 2, 4, 8 inside each row of 16 lanes leave the row's result in every lane of the row, the
// four row results are then read from lanes 0, 16, 32, 48 and combined as scalars.
__device__ __forceinline__ int wave_sum_i32(int v) {
  v += dpp_mov<0x121>(v);  // row_ror:1
  v += dpp_mov<0x122>(v);  // row_ror:2
  v += dpp_mov<0x124>(v);  // row_ror:4
  v += dpp_mov<0x128>(v);  // row_ror:8
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) +
         __builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48);
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) { return (uint32_t)wave_sum_i32((int)x); }
__device__ __forceinline__ uint32_t wave_or_u32(uint32_t x) {
  int v = (int)x;
  v |= dpp_mov<0x121>(v);
  v |= dpp_mov<0x122>(v);
  v |= dpp_mov<0x124>(v);
  v |= dpp_mov<0x128>(v);
  return (uint32_t)(__builtin_amdgcn_readlane(v, 0) | __builtin_amdgcn_readlane(v, 16) |
                    __builtin_amdgcn_readlane(v, 32) | __builtin_amdgcn_readlane(v, 48));
}
__device__ __forceinline__ int wave_max_i32(int v) {
  v = max(v, dpp_mov<0x121>(v));
  v = max(v, dpp_mov<0x122>(v));
  v = max(v, dpp_mov<0x124>(v));
  v = max(v, dpp_mov<0x128>(v));
  return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
             max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  x = max(x, (uint32_t)dpp_mov<0x121>((int)x));
  x = max(x, (uint32_t)dpp_mov<0x122>((int)x));
  x = max(x, (uint32_t)dpp_mov<0x124>((int)x));
  x = max(x, (uint32_t)dpp_mov<0x128>((int)x));
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)x, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
  const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)x, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
  return max(max(a, b), max(c, d));
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
  x = min(x, (uint32_t)dpp_mov<0x121>((int)x));
  x = min(x, (uint32_t)dpp_mov<0x122>((int)x));
  x = min(x, (uint32_t)dpp_mov<0x124>((int)x));
  x = min(x, (uint32_t)dpp_mov<0x128>((int)x));
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)x, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
  const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)x, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
  return min(min(a, b), min(c, d));
}
// x, which is the same in every lane.  The builtin returns an int: as a half of 64 bits it must not be sign-extended.
__device__ __forceinline__ uint64_t uniform_u64(uint64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t x) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, DYN_WAVE);
  return uniform_u64(x);
}
__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {   // every lane ends with the total
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, DYN_WAVE);
  return v;
}
__device__ __forceinline__ int64_t readlane_i64(int64_t x, int lane) {   // lane must be wave-uniform
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), lane);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double lane_f64(double x, int lane) { return __longlong_as_double((long long)readlane_i64(__double_as_longlong(x), lane)); }
// a / b, correctly rounded, given rb = RN(1 / b): the one division routine of the library.  One multiplication and two fused
// operations are enough for a divisor known beforehand (Brisebarre, Muller, Raina, "Accelerating correctly rounded floating-point division
// when the divisor is known in advance", IEEE Trans. Computers 53, 2004).  Why: scale a and b to [1, 2) and let u = 2^-53, n = rb - 1/b,
// |n| <= u / 2.  If q0 = RN(a * rb) is one of the two doubles around a / b, the residual is exact and Markstein's theorem gives RN(a / b).
// It always is for a >= b: |a * n| < u, half an ulp of the quotient, and the rounding adds no more than the other half.  For a < b (ulp
// u, and |a * n| < u) it can be the next but one.  Let m be the midpoint of two doubles nearest to a / b; a - m * b = k u^2 for an
// integer k, not 0.  Up to |k| = 4, a * rb = m + a * n + k u^2 / b is less than u from m, so q0 is a neighbour of m and with that of
// a / b.  Beyond, a / b is 5 u^2 / b or more from m, and what the last rounding is given is off by less: by |q0 - a / b| * b * |n|, at most
// (a + 1) b u^2 / 4 < 3 u^2 / b, and by the residual's own rounding, at most 2 u^2 / b.  (All pairs of up to 10 bits, and the hardest of 53:
// tests/test_division.py.)  Holds while nothing under- or overflows: the host keeps window lengths, capacities and grid
// spacings within [1e-100, 1e100], which leaves every operand, residual and quotient normal
// (a == 0 gives 0 exactly).
__device__ __forceinline__ double div_by(double a, double b, double rb) {
  const double q0 = a * rb;
  const double e0 = __builtin_fma(-b, q0, a);
  return __builtin_fma(e0, rb, q0);
}

// Lengths counted by exponent and the six bits below it: exact below 64, otherwise a bin is at most 1/64 of its value wide.
constexpr int kCoarseBins = 64 + 26 * 64;          // exponents 6 .. 31
__device__ __forceinline__ int coarse_bin(uint32_t v) {
  const int e = 31 - __builtin_clz(v | 32u);         // 5 below 64
  return e < 6 ? (int)v : (e - 5) * 64 + (int)((v >> (e - 6)) & 63u);
}
// The least value of a bin, and how many bits the values in it differ by.
__device__ __forceinline__ uint32_t coarse_low(int bin, int* bits) {
  const int e = bin / 64 + 5;
  *bits = bin < 64 ? 0 : e - 6;
  return bin < 64 ? (uint32_t)bin : (64u + (uint32_t)(bin & 63)) << (e - 6);
}

// The bin where the running count of `bins` counters (a thread holds PER consecutive ones, zeroes beyond) reaches `need`; *below = the
// count before it.  Block-uniform; `s` is LDS scratch of WAVES + 2 words.
template <int WAVES, int PER>
__device__ __forceinline__ int find_bin(const uint32_t (&k)[PER], int64_t need, uint32_t* s, int64_t* below) {
  const int lane = threadIdx.x & (DYN_WAVE - 1), wave = threadIdx.x / DYN_WAVE;
  uint32_t mine = 0;                                 // a cell has fewer than 2^31 requests
#pragma unroll
  for (int q = 0; q < PER; ++q) mine += k[q];
  uint32_t incl = mine;
#pragma unroll
  for (int d = 1; d < DYN_WAVE; d <<= 1) {
    const uint32_t up = __shfl_up(incl, d, DYN_WAVE);
    if (lane >= d) incl += up;
  }
  if (lane == DYN_WAVE - 1) s[wave] = incl;
  __syncthreads();
  uint32_t run = incl - mine;
  for (int w = 0; w < wave; ++w) run += s[w];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if ((int64_t)run < need && need <= (int64_t)run + k[q]) {   // one thread, one bin
      s[WAVES] = (uint32_t)((int)threadIdx.x * PER + q);
      s[WAVES + 1] = run;
    }
    run += k[q];
  }
  __syncthreads();
  const int bin = (int)s[WAVES];
  *below = s[WAVES + 1];
  __syncthreads();
  return bin;
}

struct Lookup {          // per-thread constants of the table look-up
  double den, rden, rho_max, scale, omu, u;   // scale: buckets (DYN_AXIS_EVEN: load points) per unit of the load axis
  const double *lo, *hi;         // the configuration's two table rows: [n_rho][3] prefill, TBT, power
  const double* grid;            // DYN_AXIS_EVEN: [n_rho - 1][3] load point, spacing, its reciprocal; else the padded load grid
  const double* rinv;            // reciprocal spacings
  const uint16_t* js;            // bucket index
  const int32_t* js_global;      // DYN_AXIS_GLOBAL: the same
  const double* thr;             // DYN_AXIS_SINGLE: the grid point inside each bucket
  int n_rho;
};

// Plain v_max_f64 / v_min_f64 of two values known not to be NaN (no quieting of the operands).
__device__ __forceinline__ double max_num(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double min_num(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// A block's copy of the load axis in LDS, doubles first, then the bucket index.
struct Axis {
  double *grid, *rinv, *thr;     // grid: DYN_AXIS_EVEN [3 * (n_rho - 1)], else [n_rho + 2] and after it rinv [n_rho + 1]; thr: SINGLE [n_bucket + 1]
  double* end;                   // the first double after them
};
template <int AXIS>
__device__ __forceinline__ Axis place_axis(double* at, int n_rho, int n_bucket) {
  Axis x;
  x.grid = at;
  x.rinv = at + (n_rho + 2);
  x.thr = x.rinv + (n_rho + 1);
  x.end = AXIS & DYN_AXIS_GLOBAL ? at : AXIS == DYN_AXIS_EVEN ? at + 3 * (n_rho - 1) : x.thr + (AXIS == DYN_AXIS_SINGLE ? n_bucket + 1 : 0);
  return x;
}
template <int AXIS>
__device__ __forceinline__ void stage_axis(const AxisArgs& a, const Axis& x, uint16_t* js) {
  if (AXIS & DYN_AXIS_GLOBAL) return;
  if (AXIS == DYN_AXIS_EVEN) {
    for (int i = threadIdx.x; i < 3 * (a.n_rho - 1); i += blockDim.x) x.grid[i] = a.even_grid[i];
    return;
  }
  for (int i = threadIdx.x; i < 2 * a.n_rho + 3; i += blockDim.x) x.grid[i] = a.gridpack[i];
  for (int i = threadIdx.x; i <= a.n_bucket; i += blockDim.x) {
    js[i] = (uint16_t)(AXIS == DYN_AXIS_SINGLE ? a.tstart[i] : a.jstart[i]);
    if (AXIS == DYN_AXIS_SINGLE) x.thr[i] = a.thr[i];
  }
}
template <int AXIS>
__device__ __forceinline__ void use_axis(const AxisArgs& a, const Axis& x, const uint16_t* js, Lookup* L) {
  constexpr int FORM = AXIS & ~DYN_AXIS_GLOBAL;
  L->rho_max = a.rho_max;
  L->scale = FORM == DYN_AXIS_EVEN ? a.even_scale : a.bucket_scale;
  L->n_rho = a.n_rho;
  if (AXIS & DYN_AXIS_GLOBAL) {
    L->grid = FORM == DYN_AXIS_EVEN ? a.even_grid : a.gridpack;
    L->rinv = a.gridpack + a.n_rho + 2;
    L->thr = a.thr;
    L->js_global = FORM == DYN_AXIS_SINGLE ? a.tstart : a.jstart;
  } else {
    L->grid = x.grid; L->rinv = x.rinv; L->thr = x.thr; L->js = js;
  }
}

// The lesser of v and the wave-uniform s.
__device__ __forceinline__ double min_uniform(double v, double s) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(v), "s"(s));
  return r;
}
// Values that are read by here: the compiler otherwise moves their loads behind the next branch, a memory latency later.
__device__ __forceinline__ void read_now(double& a) { asm volatile("" : "+v"(a)); }
__device__ __forceinline__ void read_now(double& a, double& b) { asm volatile("" : "+v"(a), "+v"(b)); }
__device__ __forceinline__ void read_now(double& a, double& b, double& c, double& d) { asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d)); }

// The bracket of a load by the bucket index.
template <int AXIS>
__device__ __forceinline__ int find_index(const Lookup& L, double rc) {
  const int b = (int)(fmax(rc, 0.0) * L.scale);
  int j = AXIS & DYN_AXIS_GLOBAL ? L.js_global[b] : (int)L.js[b];
  if ((AXIS & ~DYN_AXIS_GLOBAL) == DYN_AXIS_SINGLE) return j + (rc >= L.thr[b] ? 1 : 0);
  while (j > 0 && L.grid[j + 1] > rc) --j;
  while (j < L.n_rho - 2 && L.grid[j + 2] <= rc) ++j;
  return j;
}
// The bracket of the load axis that rc = min(rho, rho_max) lies in and its weight there; load(j) reads from the table rows what
// the caller wants of load points j and j + 1, read() waits for it.
// EVEN: the bracket is one multiplication away, or one less where rc is just below the load point (dyn_even_scale), which few
// waves meet: everything is read at once and read again in that case.  SINGLE: every bucket holds at most one
// interior grid point, so the bracket is the bucket's start index plus one comparison.  SEARCH: searched from the bucket's index.
// Vector instructions of a look-up of three columns: 50 by SINGLE from three tables side by side, 33 by EVEN from one of triples.
template <int AXIS, typename Load, typename Read>
__device__ __forceinline__ double find_bracket(const Lookup& L, double rc, Load&& load, Read&& read) {
  if (AXIS == DYN_AXIS_EVEN) {
    int j = (int)min((uint32_t)(int)(rc * L.scale), (uint32_t)(L.n_rho - 2));   // a load below 0 goes through the search
    const double* g = L.grid + 3 * j;
    double r0 = g[0], d = g[1], ri = g[2];
    load(j);
    read_now(r0, d);
    read_now(ri);
    read();
    if (__builtin_expect(__ballot(rc < r0) != 0, 0)) {
      while (j > 0 && L.grid[3 * j] > rc) --j;
      g = L.grid + 3 * j;
      r0 = g[0]; d = g[1]; ri = g[2];
      load(j);
    }
    return div_by(rc - r0, d, ri);
  }
  const int j = find_index<AXIS>(L, rc);
  const double r0 = L.grid[j + 1], r1 = L.grid[j + 2];
  load(j);
  return div_by(rc - r0, r1 - r0, L.rinv[j + 1]);
}

// Tables at (f, min(rho, rho_max)) for N loads (>= 0) at once: the window-level kernel's arithmetic.  What the loads wait for in LDS
// they wait for together.  COLUMNS: which of them.
// TWO: both frequency rows are combined (weight 0 on the upper row leaves
// the lower row's value unchanged, so lanes with a profiled frequency may run it too).
constexpr int kPrefill = 1, kTbt = 2, kPower = 4, kAllColumns = 7;
struct Looked {
  double v[3];                   // prefill, TBT, power: those asked for
  bool ov;
};
__device__ __forceinline__ const double* at_point(const double* base, int j) { return (const double*)((const char*)base + __umul24((uint32_t)j, 24u)); }
template <int AXIS, bool TWO, int COLUMNS, int N>
__device__ __forceinline__ void table_lookups(const Lookup& L, const double (&load)[N], Looked (&r)[N]) {
  constexpr int FORM = AXIS & ~DYN_AXIS_GLOBAL;
  double rc[N], r0[N], d[N], ri[N], a[N][6], b[N][6];
  auto read = [&](int i, int j) {
    if (FORM == DYN_AXIS_EVEN) {
      const double* g = at_point(L.grid, j);
      r0[i] = g[0]; d[i] = g[1]; ri[i] = g[2];
    } else {
      r0[i] = L.grid[j + 1]; d[i] = L.grid[j + 2] - r0[i]; ri[i] = L.rinv[j + 1];
    }
    const double* lo = at_point(L.lo, j);
    const double* hi = at_point(L.hi, j);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (!(COLUMNS >> c & 1)) continue;
      a[i][2 * c] = lo[c]; a[i][2 * c + 1] = lo[c + 3];
      if (TWO) { b[i][2 * c] = hi[c]; b[i][2 * c + 1] = hi[c + 3]; }
    }
  };
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double rho = div_by(load[i], L.den, L.rden);
    r[i].ov = rho > L.rho_max;
    rc[i] = min_uniform(rho, L.rho_max);
  }
  if (FORM == DYN_AXIS_EVEN) {
    int j[N];
    bool low = false;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      j[i] = (int)min((uint32_t)(int)(rc[i] * L.scale), (uint32_t)(L.n_rho - 2));
      read(i, j[i]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
      read_now(r0[i], d[i]);
      read_now(ri[i]);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (!(COLUMNS >> c & 1)) continue;
        read_now(a[i][2 * c], a[i][2 * c + 1]);
        if (TWO) read_now(b[i][2 * c], b[i][2 * c + 1]);
      }
      low = low || rc[i] < r0[i];
    }
    if (__builtin_expect(__ballot(low) != 0, 0)) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        while (j[i] > 0 && L.grid[3 * j[i]] > rc[i]) --j[i];
        read(i, j[i]);
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) read(i, find_index<AXIS>(L, rc[i]));
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double t = div_by(rc[i] - r0[i], d[i], ri[i]);
    const double omt = 1.0 - t;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (!(COLUMNS >> c & 1)) continue;
      r[i].v[c] = omt * a[i][2 * c] + t * a[i][2 * c + 1];
      if (TWO) r[i].v[c] = L.omu * r[i].v[c] + L.u * (omt * b[i][2 * c] + t * b[i][2 * c + 1]);
    }
  }
}
template <int AXIS, bool TWO, int COLUMNS = kAllColumns>
__device__ __forceinline__ Looked table_lookup(const Lookup& L, double load) {
  const double one[1] = {load};
  Looked r[1];
  table_lookups<AXIS, TWO, COLUMNS, 1>(L, one, r);
  return r[0];
}

}  // namespace

#endif  // DYN_DEVICE_H_
