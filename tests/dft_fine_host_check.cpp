// Host check of the DFTs that rotate by both parts of their constants (dft.h, FINE): against a
// direct DFT in double precision their root-mean-square error over seeded inputs must be below
// that of the ones with rounded constants.  Prints one line per length.
#include <cmath>
#include <complex>
#include <cstdio>
#include <random>

#include "dft.h"

using namespace lddmm::dft;

template <int R>
static bool check() {
  std::mt19937 gen(2000 + R);
  std::normal_distribution<float> nd;
  std::complex<double> w[R];
  for (int k = 0; k < R; ++k) w[k] = std::polar(1.0, -2.0 * M_PI * k / R);
  double plain = 0.0, fine = 0.0, size = 0.0;
  for (int n = 0; n < 20000; ++n) {
    float2 v[R], f[R];
    std::complex<double> x[R];
    for (int i = 0; i < R; ++i) {
      v[i] = f[i] = make_float2(nd(gen), nd(gen));
      x[i] = {v[i].x, v[i].y};
    }
    Dft<R>::run(v);
    Dft<R, true>::run(f);
    for (int m = 0; m < R; ++m) {
      std::complex<double> s = 0.0;
      for (int p = 0; p < R; ++p) s += x[p] * w[p * m % R];
      plain += std::norm(s - std::complex<double>(v[m].x, v[m].y));
      fine += std::norm(s - std::complex<double>(f[m].x, f[m].y));
      size += std::norm(s);
    }
  }
  std::printf("R=%2d rms error %.4e, with both parts %.4e\n", R, std::sqrt(plain / size),
              std::sqrt(fine / size));
  return fine < plain;
}

int main() { return check<8>() & check<9>() & check<16>() & check<18>() ? 0 : 1; }
