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
// a / b, correctly rounded, given rb = RN(1 / b): the one division routine of the library.  One multiplication and two fused
// operations are enough for a divisor known beforehand (Brisebarre, Muller, Raina, "Accelerating correctly rounded floating-point division
// when the divisor is known in advance", IEEE Trans. Computers 53, 2004).  Why: scale a and b to [1, 2) and let u = 2^-53, n = rb - 1/b,
// |n| <= u / 2.  If q0 = RN(a * rb) is one of the two doubles around a / b, the residual is exact and Markstein's theorem gives RN(a / b).
// It always is for a >= b: |a * n| < u, half an ulp of the quotient, and the rounding adds no more than the other half.  For a < b (ulp
// u, and |a * n| < u) it can be the next but one.  Let m be the midpoint of two doubles nearest to a / b; a - m * b = k u^2 for an
// integer k, not 0.  Up to |k| = 4, a * rb = m + a * n + k u^2 / b is less than u from m, so q0 is a neighbour of m and with that of
// a / b.  Beyond, a / b is 5 u^2 / b or more from m, and what the last rounding is given is off by less: by |q0 - a / b| * b * |n|, at most
// (a + 1) b u^2 / 4 < 3 u^2 / b, and by the residual's own rounding, at most 2 u^2 / b.  (All pairs of up to 13 bits, and the hardest of 53:
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
  double den, rden, rho_max, bucket_scale, omu, u;
  const double *lo, *hi;         // the configuration's two table rows: [3][n_rho] prefill, TBT, power
  const double *rgp, *rinv;      // padded load grid and reciprocal spacings
  const uint16_t* js;            // bucket index
  const double* thr;             // SINGLE: the grid point inside each bucket
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

// SINGLE: every bucket of the load axis holds at most one interior grid point, so the bracket
// is the bucket's start index plus one comparison; otherwise the bracket is searched from the
// bucket's index.
// The bracket of the load axis that rc = min(rho, rho_max) lies in, and its weight there.
template <bool SINGLE>
__device__ __forceinline__ int table_bracket(const Lookup& L, double rc, double* t) {
  int jj;
  if (SINGLE) {
    const int b = (int)(rc * L.bucket_scale);
    jj = (int)L.js[b] + (rc >= L.thr[b] ? 1 : 0);
  } else {
    jj = L.js[(int)(fmax(rc, 0.0) * L.bucket_scale)];
    while (jj > 0 && L.rgp[jj + 1] > rc) --jj;
    while (jj < L.n_rho - 2 && L.rgp[jj + 2] <= rc) ++jj;
  }
  const double r0 = L.rgp[jj + 1], r1 = L.rgp[jj + 2];
  *t = div_by(rc - r0, r1 - r0, L.rinv[jj + 1]);
  return jj;
}

// Tables at (f, min(rho, rho_max)) for load `load` (>= 0): the window-level kernel's arithmetic.
// TWO: both frequency rows are combined (weight 0 on the upper row leaves
// the lower row's value unchanged, so lanes with a profiled frequency may run it too).
template <bool SINGLE, bool TWO>
__device__ __forceinline__ bool table_lookup(const Lookup& L, double load, double* pf, double* tb, double* pw) {
  const double rho = div_by(load, L.den, L.rden);
  const bool ov = rho > L.rho_max;
  double t;
  const int jj = table_bracket<SINGLE>(L, ov ? L.rho_max : rho, &t);
  const double omt = 1.0 - t;
  const int n_rho = L.n_rho;
  double x_pf = omt * L.lo[jj] + t * L.lo[jj + 1];
  double x_tb = omt * L.lo[n_rho + jj] + t * L.lo[n_rho + jj + 1];
  double x_pw = omt * L.lo[2 * n_rho + jj] + t * L.lo[2 * n_rho + jj + 1];
  if (TWO) {
    const double b_pf = omt * L.hi[jj] + t * L.hi[jj + 1];
    const double b_tb = omt * L.hi[n_rho + jj] + t * L.hi[n_rho + jj + 1];
    const double b_pw = omt * L.hi[2 * n_rho + jj] + t * L.hi[2 * n_rho + jj + 1];
    x_pf = L.omu * x_pf + L.u * b_pf;
    x_tb = L.omu * x_tb + L.u * b_tb;
    x_pw = L.omu * x_pw + L.u * b_pw;
  }
  *pf = x_pf; *tb = x_tb; *pw = x_pw;
  return ov;
}

}  // namespace

#endif  // DYN_DEVICE_H_
