// The kernels' arithmetic of the normal draws (csrc/eco_device.h) on the CPU, against the
// long double functions of libm: largest relative errors, in units of 2^-53, printed as
//   ln <over every u1>  radius <sqrt(-2 ln u1) over every u1, for the reciprocal square
//   root off by -2^-24, 0, 2^-24>  cossin <over every u2>  normal <over pairs of draws>
#include "noise_tables.h"

#include <cstdio>

double rsq_off = 0.0;

static double units(double got, long double want) {
  return want == 0.0L ? (got == 0.0 ? 0.0 : 1e300) : (double)(std::fabs(((long double)got - want) / want) * 0x1p53L);
}

// cos, sin of 2 pi j 2^-24, the angle first reduced to an eighth of a turn in integers.
static void exact(uint32_t j, long double& c, long double& s) {
  const uint32_t quarter = 1u << 22, q = (j + quarter / 2) / quarter;
  const long double x = 2.0L * 3.14159265358979323846264338327950288L * ((long double)j - (long double)q * quarter) * 0x1p-24L;
  const long double a = std::cos(x), b = std::sin(x);
  c = (q & 3) == 0 ? a : ((q & 3) == 1 ? -b : ((q & 3) == 2 ? -a : b));
  s = (q & 3) == 0 ? b : ((q & 3) == 1 ? a : ((q & 3) == 2 ? -b : -a));
}

int main() {
  using namespace eco;
  const std::vector<double2> tab = noise_tables();
  const uint32_t all = 1u << 24;
  double ln = 0.0, radius = 0.0, cs = 0.0, normal = 0.0;
  for (uint32_t m = 1; m < all; ++m) {   // m = 2^24: ln 1, below
    const double y = neg2_ln_u24(m, tab.data() + kTrigTable);
    const long double want = -2.0L * std::log((long double)m * 0x1p-24L), root = std::sqrt(want);
    ln = std::fmax(ln, units(y, want));
    for (int k = -1; k <= 1; ++k) {
      rsq_off = k * 0x1p-24;
      radius = std::fmax(radius, units(sqrt_small(y), root));
    }
  }
  rsq_off = 0.0;
  const bool one = neg2_ln_u24(all, tab.data() + kTrigTable) == 0.0 && sqrt_small(0.0) > 0.0 && sqrt_small(0.0) < 0x1p-499;
  for (uint32_t j = 0; j < all; ++j) {
    double c, s;
    long double ce, se;
    cossin_2pi_u24(j, tab.data(), c, s);
    exact(j, ce, se);
    if (j % (all / 4) == 0) {   // the quarter turns: exact
      const uint32_t q = j / (all / 4);
      ce = q == 0 ? 1 : (q == 2 ? -1 : 0);
      se = q == 1 ? 1 : (q == 3 ? -1 : 0);
    }
    cs = std::fmax(cs, std::fmax(units(c, ce), units(s, se)));
  }
  for (uint32_t i = 0; i < 1u << 20; ++i) {
    double z[4];
    gauss4k(0x9E3779B9u, 42u, i, 3u, 5u, 7u, tab.data(), z);
    const uint4 x = philox10(i, 3u, 5u, 7u, 0x9E3779B9u, 42u);
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
    for (int p = 0; p < 2; ++p) {
      const long double r = std::sqrt(-2.0L * std::log((long double)((w[2 * p] >> 8) + 1) * 0x1p-24L));
      long double c, s;
      exact(w[2 * p + 1] >> 8, c, s);
      if ((w[2 * p] >> 8) + 1 == all || (w[2 * p + 1] >> 8) % (all / 4) == 0) continue;
      normal = std::fmax(normal, std::fmax(units(z[2 * p], r * c), units(z[2 * p + 1], r * s)));
    }
  }
  std::printf("ln %.4f radius %.4f cossin %.4f normal %.4f one %d\n", ln, radius, cs, normal, (int)one);
  return 0;
}
