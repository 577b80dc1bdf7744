// The constant-culling search (pa_search.hpp) against the bisection that defines
// it: 64 halvings of [0, rem], lo + (hi - lo)/2, each decided by an evaluation.
// Energy levels of many shapes (Gaussian, one-sided, a few levels, heavy tails),
// widths and sizes, culling targets from 0.001 to 0.95, short and long ranges,
// populations above and below the target size.  Evaluations: sequential double
// sums over the levels (one rounding per level), or sums in extended precision
// rounded once (argument "exact"), as the device's exact sums.  Prints the number
// of searches whose outcome or lo differs in any bit, the searches, the
// evaluations and the most rounds.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "pa_search.hpp"

struct Levels {
  std::vector<double> arg, cnt;
  double R;
};

template <typename Sum>
double eps(const Levels& l, double db) {
  std::vector<double> w(l.arg.size());
  Sum S = 0, acc = 0;
  for (size_t i = 0; i < w.size(); ++i) {
    w[i] = std::exp(-db * l.arg[i]);
    S = S + l.cnt[i] * (Sum)w[i];
  }
  for (size_t i = 0; i < w.size(); ++i) {
    const double tau = (l.R * w[i]) / (double)S;
    if (tau < 1.0) acc = acc + l.cnt[i] * (Sum)(1.0 - tau);
  }
  return (double)acc / l.R;
}

template <typename Sum>
int run(int n, int lanes) {
  std::mt19937_64 g(20240 + lanes);
  int bad = 0, most = 0;
  long evals = 0;
  for (int t = 0; t < n; ++t) {
    const int R0 = (int)std::exp(std::uniform_real_distribution<>(0.0, std::log(2e4))(g));
    const double sigma = std::exp(std::uniform_real_distribution<>(0.0, std::log(80.0))(g));
    const double unit = t % 3 == 0 ? 2.0 : t % 3 == 1 ? 1.0 / 16 : 1e-6 * sigma;
    std::normal_distribution<> normal(0.0, sigma);
    std::vector<long long> lev(R0);
    for (auto& v : lev) {
      double e = normal(g);
      if (t % 5 == 1) e = std::fabs(e);
      if (t % 5 == 2) e = std::floor(e / (3 * sigma)) * sigma;
      if (t % 5 == 3 && (g() & 7) == 0) e *= 8;
      v = std::llround(e / unit);
    }
    std::sort(lev.begin(), lev.end());
    Levels l;
    double mean = 0;
    for (size_t i = 0; i < lev.size();) {
      size_t j = i;
      while (j < lev.size() && lev[j] == lev[i]) ++j;
      l.arg.push_back(unit * (double)(lev[i] - lev[0]));
      l.cnt.push_back((double)(j - i));
      mean += l.arg.back() * l.cnt.back() / R0;
      i = j;
    }
    l.R = t % 7 == 0 ? R0 + R0 / 50 : t % 7 == 1 ? std::max(1, R0 - R0 / 40) : R0;
    const double target = t % 4 == 0   ? 0.1
                          : t % 4 == 1 ? 0.02
                          : t % 4 == 2 ? 0.5
                                       : std::uniform_real_distribution<>(0.001, 0.95)(g);
    const double rem = t % 6 == 0 ? 1e-3 : t % 6 == 1 ? 40.0 : 5.0;
    const double e0 = eps<Sum>(l, 0.0);
    int want = -1;
    double lo = 0, hi = rem;
    if (e0 <= target) {
      want = 1;
      if (eps<Sum>(l, rem) > target) {
        want = 2;
        for (int k = 0; k < 64; ++k) {
          const double mid = lo + 0.5 * (hi - lo);
          if (eps<Sum>(l, mid) <= target) lo = mid;
          else hi = mid;
        }
      }
    }
    pa::CullSearch s;
    pa::cull_eta(s, mean * 1.001, sizeof(Sum) > 8 ? 0.0 : (double)l.arg.size(), R0 / l.R);
    // guesses near, far below and far above the crossing
    const double guess = target * 2.5 * std::sqrt(2 * std::log(R0 + 2.0)) / (mean > 0 ? mean : 1);
    pa::cull_start(s, rem, target, e0, t % 11 == 0 ? guess * 1e-3 : t % 11 == 1 ? guess * 30 : guess,
                   lanes);
    int rounds = 0;
    for (; s.result == 0 && rounds < 100; ++rounds) {
      for (int k = 0; k < s.n; ++k) s.e[k] = eps<Sum>(l, s.x[k]);
      evals += s.n;
      pa::cull_advance(s);
    }
    if (s.result != want || (want == 2 && std::memcmp(&s.lo, &lo, 8) != 0)) ++bad;
    most = std::max(most, rounds);
  }
  std::printf("%d %d %ld %d\n", bad, n, evals, most);
  return bad;
}

int main(int argc, char** argv) {
  const int n = std::atoi(argv[1]), lanes = std::atoi(argv[2]);
  if (argc > 3 && !std::strcmp(argv[3], "exact")) return run<long double>(n, lanes) != 0;
  return run<double>(n, lanes) != 0;
}
