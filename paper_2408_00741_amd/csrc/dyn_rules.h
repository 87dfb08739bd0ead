// Rules of the host side that depend on sizes and tables only, in plain C++: tests/test_rules.py compiles them on the CPU.
#ifndef DYN_RULES_H_
#define DYN_RULES_H_

#include <cstddef>
#include <cstdint>

// Evenly spaced load points: buckets a little narrower than the spacing, of which every point opens its own and fills at most the first
// 2^-20 (the points' own roundings and the 2^-40 take far less).  A product by a constant is monotone, so only loads in that part of a
// bucket can lie below its point: a wave hardly ever meets one.  Points anywhere in their buckets would do as well for the result, but with
// points 0.3 to 0.9 of a spacing late most loads then are asked twice: 36 000 cells of mixed pools 294 us, 248 by the buckets' index; ticks 562, 486.
// Returns buckets per unit of the load axis, 0 where the points do not lie so.
inline double dyn_even_scale(const double* rho, int32_t n_rho) {
  const double scale = (double)(n_rho - 1) / rho[n_rho - 1] * (1.0 + 0x1p-40);
  for (int32_t q = 1; q < n_rho; ++q) {
    const double x = rho[q] * scale - (double)q;
    if (!(x >= 0.0 && x < 0x1p-20)) return 0.0;
  }
  return scale;
}

#endif  // DYN_RULES_H_
