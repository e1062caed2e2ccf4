// Host check of div_by (divide.h) against the division: random values over its whole range, whole
// multiples of h and their neighbours, the ends of the range and what lies past them.  Prints one
// line per set and exits non-zero at the first difference.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <limits>
#include <random>

#include "divide.h"

using namespace lddmm;

static int bad = 0;

static void same(double a, double h) {
  const double want = a / h, got = div_by(a, h, 1.0 / h);
  if (got == want) return;                        // -0 and 0 are one position
  if (bad++ < 5) std::printf("  %a / %a: %a, not %a\n", a, h, got, want);
}

int main() {
  std::mt19937_64 gen(7);
  auto value = [&](double lo, double hi) {        // log-uniform, random mantissa and sign
    const double e = std::uniform_real_distribution<double>(std::log2(lo), std::log2(hi))(gen);
    double x = std::exp2(e);
    uint64_t b;
    std::memcpy(&b, &x, 8);
    b = (b & ~((1ull << 52) - 1)) | (gen() & ((1ull << 52) - 1)) | (gen() & (1ull << 63));
    std::memcpy(&x, &b, 8);
    return x;
  };
  for (int i = 0; i < 4000000; ++i) same(value(1e-200, 1e199), std::fabs(value(1e-99, 1e99)));
  std::printf("whole range: %d differ\n", bad);
  const double inf = std::numeric_limits<double>::infinity();
  for (int i = 0; i < 400000; ++i) {              // positions: multiples of h and their neighbours
    const double h = std::fabs(value(1e-3, 1e3)), a = h * (double)(gen() % 4096);
    for (double x : {a, std::nextafter(a, inf), std::nextafter(a, -inf), -a}) same(x, h);
  }
  std::printf("multiples: %d differ\n", bad);
  for (double h : {1e-100, 0.05, 1.0, 1.0 + 0x1p-52, 2.0 - 0x1p-52, 1e100}) {
    for (double a : {0.0, 1e-200, 1.0, 1.0 - 0x1p-53, 9.99e199, -9.99e199}) same(a, h);
    // past the range: far outside every grid, or not finite, as the division's
    for (double a : {1e200, -1e200, 1e300, 1.7e308, -1.7e308, inf, -inf}) {
      const double want = a / h, got = div_by(a, h, 1.0 / h);
      if (!(got * want > 0.0) || !(std::fabs(got) >= 1e99) || !(std::fabs(want) >= 1e99)) ++bad;
    }
    if (!std::isnan(div_by(std::nan(""), h, 1.0 / h))) ++bad;
    for (double a : {5e-324, 1e-310, 1e-250})     // below it: the sign
      if (div_by(a, h, 1.0 / h) < 0.0 || div_by(-a, h, 1.0 / h) > 0.0) ++bad;
  }
  std::printf("ends: %d differ\n", bad);
  for (double h : {5e-324, 1e-310, 9e-101, 1.1e100, 1.7e308})
    if (div_by_fits(h)) ++bad;
  for (double h : {1e-100, 0.05, 1e100})
    if (!div_by_fits(h)) ++bad;
  std::printf("%s\n", bad ? "FAILED" : "ok");
  return bad ? 1 : 0;
}
