// Host test of root.hpp against the square root and the division of the C
// library, from estimates as bad as 2^-14.
#include <math.h>
#include <stdio.h>
#include <random>
#include "root.hpp"

int main() {
  std::mt19937_64 rng(1);
  std::uniform_real_distribution<double> U(0, 1);
  const double range[5][3] = {{-40, 13, 0}, {-300, -40, 0}, {-960, -300, 0}, {-1021, -960, 0x1p-52}, {-1070, -1022, 0x1p-27}};
  int bad = 0;
  for (const double bits : {-14.0, -20.0, -26.0})
    for (const double(&lim)[3] : range) {
      double worst = 0, worstq = 0;
      for (int i = 0; i < 200000; ++i) {
        const double d = (1 + U(rng)) * exp2(lim[0] + (lim[1] - lim[0]) * U(rng));
        const double y = (double)((1.0L / sqrtl((long double)d)) * (1.0L + (long double)((2 * U(rng) - 1) * exp2(bits))));
        const double t = (U(rng) - 0.5) * exp2(40 * U(rng) - 20) * sqrt(d);
        double r;
        const double g = cfog::sqrt_rcp(d, y, r), s = sqrt(d);
        const double q = cfog::quotient(t, g, r);
        worst = fmax(worst, fabs(g - s) / s);
        worstq = fmax(worstq, fabs(q - t / g) / fabs(t / g));
      }
      // exact where the limit is 0; quotients by the root g that was found
      const bool ok = worst <= lim[2] && worstq <= lim[2];
      if (!ok) ++bad;
      printf("%s estimate 2^%g d 2^[%g, %g]: root %.3g quotient %.3g\n", ok ? "ok" : "FAIL", bits, lim[0], lim[1], worst, worstq);
    }
  return bad ? 1 : 0;
}
