// The constant-culling search (pa_search.hpp) against the bisection that defines it,
// where evaluations are as wrong as their bound allows: random non-decreasing curves
// with flat stretches next to the target, and an error of up to eta0 + eta1 x at x, a
// fixed function of x, that is mostly at one of its ends.  eta1 is large, so that the
// bound at a large step exceeds the one at the crossing many times over.  argv: the
// searches and the evaluations per round.  Prints the searches that differ in outcome
// or in any bit of lo, and the searches.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "pa_search.hpp"

struct Curve {
  std::vector<double> x, y;  // a broken line, both ascending
  double eta0, eta1;
  uint64_t salt;

  double exact(double at) const {
    if (at <= x.front()) return y.front();
    if (at >= x.back()) return y.back();
    const size_t i = std::upper_bound(x.begin(), x.end(), at) - x.begin();
    const double f = (at - x[i - 1]) / (x[i] - x[i - 1]);
    return y[i - 1] + f * (y[i] - y[i - 1]);
  }
  double eps(double at) const {
    uint64_t h;
    std::memcpy(&h, &at, 8);
    h = (h ^ salt) * 0x9E3779B97F4A7C15ull;
    h ^= h >> 29;
    h *= 0xBF58476D1CE4E5B9ull;
    h ^= h >> 32;
    const double u = (h & 3u) == 0 ? (double)((h >> 8) & 0xFFFF) / 32768.0 - 1.0 : (h & 4u) ? 0.999 : -0.999;
    return exact(at) + u * (eta0 + eta1 * at);
  }
};

int main(int, char** argv) {
  const int n = std::atoi(argv[1]), lanes = std::atoi(argv[2]);
  std::mt19937_64 g(77 + lanes);
  std::uniform_real_distribution<> u01(0.0, 1.0);
  int bad = 0;
  for (int t = 0; t < n; ++t) {
    const double rem = 5.0, target = 0.3;
    const double cross = rem * std::exp(-6.0 * u01(g));
    Curve c;
    c.salt = g();
    c.eta0 = std::exp(-14.0 + 6.0 * u01(g));
    c.eta1 = std::exp(-12.0 + 6.0 * u01(g));
    // up to the target, flat or slowly rising stretches above it, then up
    const double eta = c.eta0 + c.eta1 * cross;
    c.x = {0.0, cross};
    c.y = {0.0, target - eta * u01(g)};
    double x = cross, y = target;
    for (int k = 0; k < 3; ++k) {
      x += (rem - x) * 0.02 * u01(g);
      y += eta * 6.0 * u01(g);
      c.x.push_back(x);
      c.y.push_back(y);
      x += (rem - x) * 0.6 * u01(g);
      c.x.push_back(x);
      c.y.push_back(y);
    }
    c.x.push_back(rem);
    c.y.push_back(std::max(y, 0.5) + 0.4);
    int want = c.eps(0.0) > target ? -1 : c.eps(rem) <= target ? 1 : 2;
    double lo = 0.0, hi = rem;
    for (int k = 0; want == 2 && k < 64; ++k) {
      const double mid = lo + 0.5 * (hi - lo);
      if (c.eps(mid) <= target) lo = mid;
      else hi = mid;
    }
    pa::CullSearch s;
    s.eta0 = c.eta0;
    s.eta1 = c.eta1;
    pa::cull_start(s, rem, target, c.eps(0.0), cross * std::exp(2.0 * u01(g) - 1.0), lanes);
    for (int r = 0; s.result == 0 && r < 100; ++r) {
      for (int k = 0; k < s.n; ++k) s.e[k] = c.eps(s.x[k]);
      pa::cull_advance(s);
    }
    if (s.result != want || (want == 2 && std::memcmp(&s.lo, &lo, 8) != 0)) ++bad;
  }
  std::printf("%d %d\n", bad, n);
  return 0;
}
