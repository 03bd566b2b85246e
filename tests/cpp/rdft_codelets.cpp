// Host check of the real-input DFT codelets (dft.hpp) against the definition.
#include "dft.hpp"
#include <cmath>
#include <complex>
#include <cstdio>
using namespace cfog;
template <int R> double check() {
  float x[R];
  float2 X[R / 2 + 1];
  for (int i = 0; i < R; ++i) x[i] = std::sin(1.3 * i * i + 0.2);
  rdft<R>(x, X);
  double err = 0;
  for (int k = 0; k <= R / 2; ++k) {
    std::complex<double> s = 0;
    for (int n = 0; n < R; ++n) s += (double)x[n] * std::polar(1.0, -2 * M_PI * n * k / R);
    err = std::max(err, std::abs(s - std::complex<double>(X[k].x, X[k].y)));
  }
  if (X[0].y != 0.f || (R % 2 == 0 && X[R / 2].y != 0.f)) err = 1;  // real by construction
  std::printf("R=%d err=%.3g\n", R, err);
  return err;
}
int main() {
  double e = 0;
#define C(R) e = std::max(e, check<R>());
  C(2) C(3) C(4) C(5) C(8) C(9) C(10) C(12) C(15) C(16) C(20) C(24)
  return e < 1e-5 ? 0 : 1;
}
