// The arithmetic of a Cholesky pivot (common.hpp) on the host, against sqrt and
// division: pivots over the range its comment states, a starting value off by up
// to 2^-20, operands of any size beside it.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "common.hpp"

static uint64_t state = 1;
static uint64_t next() {
  state += 0x9E3779B97F4A7C15ull;
  uint64_t z = state;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
static double unit() { return double(next() >> 11) * 0x1.0p-53; }
static int64_t ulps(double a, double b) {
  int64_t x, y;
  std::memcpy(&x, &a, 8);
  std::memcpy(&y, &b, 8);
  return x > y ? x - y : y - x;
}

int main() {
  int64_t root_off = 0, inv_most = 0, div_off = 0, div_most = 0, n = 0;
  for (int i = 0; i < 4000000; ++i) {
    double d = std::exp2((unit() * 2.0 - 1.0) * 664.0) * (1.0 + unit());  // 1e-200 .. 1e200
    if (i % 5 == 0) {  // beside a square: roots next to a rounding boundary
      const double r = 1.0 + unit();
      d = r * r * std::exp2(double(2 * (int(next() % 600) - 300)));
      d = std::nextafter(d, i % 2 ? 0.0 : 1e300);
    }
    const double y = 1.0 / std::sqrt(d) * (1.0 + (unit() * 2.0 - 1.0) * 0x1.0p-20);
    const hef::Pivot p = hef::pivot_from(d, y);
    root_off += p.root != std::sqrt(d);
    const int64_t iu = ulps(p.inv, 1.0 / p.root);
    inv_most = iu > inv_most ? iu : inv_most;
    const double x = p.root * std::exp2((unit() * 2.0 - 1.0) * 60.0) * (i % 2 ? 1.0 : -1.0);
    const int64_t du = ulps(hef::div_pivot(x, p), x / p.root);
    div_off += du != 0;
    div_most = du > div_most ? du : div_most;
    ++n;
  }
  std::printf("pivots %lld root_off %lld inv_ulps %lld div_off %lld div_ulps %lld\n", (long long)n,
              (long long)root_off, (long long)inv_most, (long long)div_off, (long long)div_most);
  return 0;
}
