// noise_tables.h -- host side: the tables of the normal draws (neg2_ln_u24 and
// cossin_2pi_u24 in eco_device.h), computed once.
#pragma once

#include <cmath>
#include <vector>

#include "eco_device.h"

namespace eco {

// The Box-Muller angle table: cos and sin of 2 pi a / 256, a = 0..255.  The
// angle is reduced exactly by quarter turns and octant symmetry, so libm only
// sees arguments in [0, pi / 4] and the multiples of a quarter turn are exact.
inline std::vector<double2> angle_table() {
  std::vector<double2> t(kTrigTable);
  const int quarter = kTrigTable / 4;
  for (int a = 0; a < kTrigTable; ++a) {
    const int q = a / quarter, m = a % quarter;   // a = q quarter + m, m in [0, 64)
    double cb, sb;                                // cos, sin of 2 pi m / 256 in [0, pi / 2)
    if (2 * m <= quarter) {
      const double b = 2.0 * M_PI * (double)m / (double)kTrigTable;
      cb = std::cos(b);
      sb = std::sin(b);
    } else {                                      // pi / 2 - b = 2 pi (64 - m) / 256
      const double b = 2.0 * M_PI * (double)(quarter - m) / (double)kTrigTable;
      cb = std::sin(b);
      sb = std::cos(b);
    }
    const double c = q == 0 ? cb : (q == 1 ? -sb : (q == 2 ? -cb : sb));
    const double s = q == 0 ? sb : (q == 1 ? cb : (q == 2 ? -sb : -cb));
    t[a] = make_double2(c, s);
  }
  return t;
}

// The logarithm table: entry i stands for f in [1 + i / 256, 1 + (i + 1) / 256) with
// {1/c, -2 ln c}, 1/c of 28 bits behind the point for c in the middle (c = 1 and 2 at
// the ends), and the logarithm that of c / 2 from kLogFold on.  Of the 1/c next to the
// middle's the one whose logarithm lies nearest to a double is taken, so that the
// table adds no rounding of its own.
inline std::vector<double2> log_table() {
  std::vector<double2> t(kLogTable);
  for (int i = 0; i < kLogTable; ++i) {
    const long double fold = i >= kLogFold ? 2.0L : 1.0L;
    const double c = i == 0 ? 1.0 : (i == kLogTable - 1 ? 2.0 : 1.0 + (i + 0.5) / kLogTable);
    const int span = (i == 0 || i == kLogTable - 1) ? 0 : 64;
    long double best = 1.0L;
    for (int n = -span; n <= span; ++n) {
      const double ic = (std::nearbyint(0x1p28 / c) + n) * 0x1p-28;
      const long double l = 2.0L * std::log((long double)ic * fold);
      const long double off = l == 0.0L ? 0.0L : std::fabs(((long double)(double)l - l) / l);
      if (off < best) {
        best = off;
        t[i] = make_double2(ic, (double)l);
      }
    }
  }
  return t;
}

// Both, as the kernels hold them.
inline std::vector<double2> noise_tables() {
  std::vector<double2> t = angle_table(), l = log_table();
  t.insert(t.end(), l.begin(), l.end());
  return t;
}

}  // namespace eco
