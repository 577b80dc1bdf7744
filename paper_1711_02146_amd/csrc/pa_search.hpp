// pa_search.hpp -- the constant-culling step (Sec. III.C) as a search for the
// end point of 64 bisection halvings, for the host and the device alike.
//
// The step is defined by the sequential bisection of [0, rem]: mid = lo +
// (hi - lo)/2, lo = mid if eps(mid) <= target, else hi = mid, 64 times, where
// eps is the culling fraction as evaluated in floating point.  CullSearch
// returns the same lo, bit for bit, from far fewer evaluations:
//   - The exact culling fraction sum_i max(0, 1 - tau_i) / R never falls as the
//     step grows.  tau_i = R w_i / sum w, w_i = exp(-x (E_i - E_min)), changes
//     at the rate tau_i (<E>_w - E_i); the replicas with tau_i < 1 are those
//     above some energy, and the sum of tau_i (<E>_w - E_i) over them is minus
//     a covariance of E with an increasing function of E.
//   - An evaluation is off by at most eta(x) = eta0 + eta1 x (cull_eta).  So if
//     eps(a) + 2 eta(a) <= target, every mid <= a has eps(mid) <= target; if eps(x) -
//     eta(x) - eta(c) > target, every mid from x to c has eps(mid) > target.  With c =
//     rem this holds for every mid from some x = far up, with c = far for every mid
//     from some b <= far to far, so for all from b up.  (far lies next to the crossing
//     after a round or two, so eta(far) is hardly more than eta(b).)  Those halvings
//     are decided without an evaluation.
//   - A first few rounds of up to kCullLanes evaluations close [a, b] in on the
//     crossing by interpolation; the halvings left between a and b (about the
//     last twelve) are evaluated, three at a time where evaluations run side by
//     side: the candidates of the next halvings on every outcome, each formed
//     from the (lo, hi) that the sequential search would hold there.
// An interpolation that goes wrong costs rounds, never a bit.
#pragma once

#ifndef PA_HD
#define PA_HD
#endif
// (device: every index into the small arrays a constant, so that they stay in registers)
#ifdef __clang__
#define PA_UNROLL _Pragma("unroll")
#else
#define PA_UNROLL
#endif

namespace pa {

constexpr int kCullLanes = 7;      // evaluations per round where they run side by side
constexpr int kCullSerial = 3;     // most of a round where they run one after another
constexpr int kCullInterp = 6;     // rounds of interpolation at most
constexpr int kCullHalvings = 64;

struct CullSearch {
  double rem, target;
  double eta0, eta1;               // error bound of an evaluation at x: eta0 + eta1 x
  double lo, hi;                   // the bisection's interval after `it` halvings
  double a, b;                     // decided: taken at and below a, not taken at and above b
  double far;                      // not taken at and above, by the bound at rem (b <= far)
  double x[kCullLanes];            // candidates of the round
  double e[kCullLanes];            // their culling fractions
  double px[4], pe[4];             // evaluated points next to the crossing, ascending in x: two
                                   // with e <= target, then two above it
  int n, it, round, n_left, n_right;  // of those points, how many on each side
  int result;                      // 0 running, 1 the whole range, 2 bisected (lo), -1 impossible
  int lanes;                       // kCullLanes or kCullSerial
  int pad;
};

// Error bound of an evaluation at x, in units of 2^-53 with a quarter to spare:
// each weight is off by at most x d + 4 units (d = E - E_min: the rounding of
// the argument, and of exp within two ulp), the sum of the weights by their
// weighted mean plus the rounding of the additions, tau by both and two
// roundings, the terms 1 - tau by one each.  The weighted mean of d is at most
// its plain mean; `mean_d` may exceed it.  adds: roundings that a sum of the
// evaluation accumulates (0 for exact sums); ratio: R~ / R.
PA_HD inline void cull_eta(CullSearch& s, double mean_d, double adds, double ratio) {
  const double u = 1.25 * 0x1p-53;
  s.eta0 = u * (16.0 + 2.0 * adds + 4.0 * ratio);
  s.eta1 = u * 2.0 * mean_d;
}

// Start: eps0 = eps(0), guess: a step thought to be near the crossing (any
// positive number serves).  The first round evaluates rem and a spread of steps
// around the guess.  lanes: kCullLanes, or kCullSerial for evaluations made one
// after another (fewer of them in all, in more rounds).
PA_HD inline void cull_start(CullSearch& s, double rem, double target, double eps0, double guess,
                             int lanes) {
  s.lanes = lanes;
  s.rem = rem;
  s.target = target;
  s.lo = 0.0;
  s.hi = rem;
  s.a = 0.0;       // eps(0) <= target: mid = 0 occurs only as lo itself
  s.b = 2.0 * rem;
  s.far = 2.0 * rem;
  s.it = 0;
  s.round = 0;
  s.result = eps0 > target ? -1 : 0;
  s.px[1] = 0.0;
  s.pe[1] = eps0;
  s.n_left = 1;
  s.n_right = 0;
  s.x[0] = rem;
  s.n = lanes;
  double f = lanes == kCullLanes ? 0.55 : 0.8;
  PA_UNROLL
  for (int k = 1; k < kCullLanes; ++k) {
    const double c = guess * f;
    s.x[k] = c < rem ? c : rem;
    f *= lanes == kCullLanes ? 1.3 : 1.6;
  }
}

// The halvings from (lo, hi, it) on that need no evaluation; returns the first
// mid that does, or a negative number when all 64 are done.  A mid that rounds to
// an end of the interval repeats that end's outcome (lo was taken, hi was not).
PA_HD inline double cull_walk(const CullSearch& s, double& lo_io, double& hi_io, int& it_io) {
  const double a = s.a, b = s.b;
  double lo = lo_io, hi = hi_io, mid = -1.0;
  int it = it_io;
  while (it < kCullHalvings) {
    mid = lo + 0.5 * (hi - lo);
    int known = mid <= a || mid <= lo ? 1 : mid >= b || mid >= hi ? 0 : -1;
    if (known < 0) {
      PA_UNROLL
      for (int k = 0; k < kCullLanes; ++k)
        if (k < s.n && s.x[k] == mid) known = s.e[k] <= s.target ? 1 : 0;
      if (known < 0) break;
    }
    if (known) lo = mid;
    else hi = mid;
    ++it;
  }
  lo_io = lo;
  hi_io = hi;
  it_io = it;
  return it < kCullHalvings ? mid : -1.0;
}

// The points next to the crossing after a round (its candidates ascend, some
// may repeat; rem, the first round's candidate 0, is the upper end).
PA_HD inline void cull_points(CullSearch& s) {
  if (s.round == 0) {
    s.px[2] = s.x[0];
    s.pe[2] = s.e[0];
    s.n_right = 1;
  }
  const double x2 = s.px[2], e2 = s.pe[2];
  int above = 0;  // candidates seen above the target
  PA_UNROLL
  for (int k = 0; k < kCullLanes; ++k) {
    if (k >= s.n || (k == 0 && s.round == 0)) continue;
    const double x = s.x[k], e = s.e[k];
    if (above == 0 && e <= s.target) {
      if (x > s.px[1]) {
        s.px[0] = s.px[1];
        s.pe[0] = s.pe[1];
        s.px[1] = x;
        s.pe[1] = e;
        s.n_left = 2;
      }
    } else if (above == 0) {
      if (x < x2) {
        s.px[3] = x2;
        s.pe[3] = e2;
        s.px[2] = x;
        s.pe[2] = e;
        s.n_right = 2;
      }
      above = 1;
    } else if (above == 1 && x > s.px[2]) {
      s.px[3] = x;
      s.pe[3] = e;
      above = 2;
    }
  }
}

// Estimate of the crossing between the inner two points, by inverse
// interpolation through all of them.
PA_HD inline double cull_estimate(const CullSearch& s) {
  const double xl = s.px[1], xr = s.px[2], t = s.target;
  const double el = s.pe[1], er = s.pe[2];
  const double mid = xl + (xr - xl) * ((t - el) / (er - el));
  double r = mid;
  // Neville's scheme on x as a function of e: (1, 2), then with 0, then with 3
  double r012 = mid, r123 = mid;
  if (s.n_left == 2 && s.pe[0] < el) {
    const double p01 = s.px[0] + (xl - s.px[0]) * ((t - s.pe[0]) / (el - s.pe[0]));
    r012 = p01 + (mid - p01) * ((t - s.pe[0]) / (er - s.pe[0]));
    r = r012;
  }
  if (s.n_right == 2 && s.pe[3] > er) {
    const double p23 = xr + (s.px[3] - xr) * ((t - er) / (s.pe[3] - er));
    r123 = mid + (p23 - mid) * ((t - el) / (s.pe[3] - el));
    r = s.n_left == 2 && s.pe[0] < el
            ? r012 + (r123 - r012) * ((t - s.pe[0]) / (s.pe[3] - s.pe[0]))
            : r123;
  }
  return r > xl && r < xr ? r : mid > xl && mid < xr ? mid : xl + 0.5 * (xr - xl);
}

// The round's results are in s.e[0 .. n): decide what they decide, and either
// finish (s.result) or set the candidates of the next round.
PA_HD inline void cull_advance(CullSearch& s) {
  if (s.result != 0) return;
  if (s.round == 0 && s.e[0] <= s.target) {
    s.result = 1;
    return;
  }
  const double eta_rem = s.eta0 + s.eta1 * s.rem;
  PA_UNROLL
  for (int k = 0; k < kCullLanes; ++k) {
    if (k >= s.n) continue;
    const double eta = s.eta0 + s.eta1 * s.x[k];
    if (s.e[k] + 2.0 * eta <= s.target && s.x[k] > s.a) s.a = s.x[k];
    if (s.e[k] - (eta + eta_rem) > s.target && s.x[k] < s.far) s.far = s.x[k];
  }
  const double eta_far = s.eta0 + s.eta1 * (s.far < s.rem ? s.far : s.rem);
  PA_UNROLL
  for (int k = 0; k < kCullLanes; ++k) {
    if (k >= s.n) continue;
    const double eta = s.eta0 + s.eta1 * s.x[k];
    if (s.e[k] - (eta + eta_far) > s.target && s.x[k] < s.b) s.b = s.x[k];
  }
  if (s.round < kCullInterp) cull_points(s);
  ++s.round;
  const double first = cull_walk(s, s.lo, s.hi, s.it);
  if (first < 0.0) {
    s.result = 2;
    return;
  }
  const double xr = s.px[2], width = xr - s.px[1];
  // the uncertain stretch around the crossing, where evaluations decide
  const double rise = s.n_right ? s.pe[2] - s.pe[1] : 0.0;
  const double zone = rise > 0.0 ? 3.0 * (s.eta0 + s.eta1 * xr) * width / rise : 0.0;
  if (s.round < kCullInterp && width > 8.0 * zone && zone > 0.0) {
    const double r = cull_estimate(s);
    // around the estimate, outermost first, by parts of the bracket and at least
    // a few zones; a candidate outside the interval repeats the bracket's end
    const bool first_round = s.round == 1, wide = s.lanes == kCullLanes;
    PA_UNROLL
    for (int k = 0; k < kCullLanes; ++k) {
      const int q = wide ? k - 3 : k - 1;  // -3..3, or -1, 0, 1
      const int m = q < 0 ? -q : q;
      const double f = !wide ? (first_round ? 5e-2 : s.round == 2 ? 1e-4 : 1e-7)
                       : m == 3 ? (first_round ? 0.12 : 1e-2)
                       : m == 2 ? (first_round ? 4e-3 : 1e-5)
                                : (first_round ? 5e-5 : 1e-9);
      double step = m == 0 ? 0.0 : f * width;
      if (step < zone * (double)m) step = zone * (double)m;
      const double c = q < 0 ? r - step : r + step;
      s.x[k] = c <= s.px[1] ? s.px[1] : c >= xr ? xr : c;
    }
    s.n = s.lanes;
    return;
  }
  // the next halvings' candidates on every outcome (one after another: only the
  // next one): node k of the tree has the children 2k + 1 (not taken) and 2k + 2
  // (taken); a branch that ends repeats the root's candidate
  const int most = s.lanes == kCullLanes ? kCullLanes : 1;
  double qlo[kCullLanes], qhi[kCullLanes], qmid[kCullLanes];
  int qit[kCullLanes];
  PA_UNROLL
  for (int k = 0; k < kCullLanes; ++k) {
    if (k >= most) continue;
    const int up = (k - 1) / 2;
    double lo = s.lo, hi = s.hi;
    int it = s.it;
    bool live = true;
    if (k > 0) {
      live = qmid[up] >= 0.0;
      lo = (k & 1) ? qlo[up] : qmid[up];
      hi = (k & 1) ? qmid[up] : qhi[up];
      it = qit[up] + 1;
    }
    qmid[k] = live ? cull_walk(s, lo, hi, it) : -1.0;
    qlo[k] = lo;
    qhi[k] = hi;
    qit[k] = it;
  }
  // (after the walks, which still look the last round's candidates up)
  PA_UNROLL
  for (int k = 0; k < kCullLanes; ++k)
    if (k < most) s.x[k] = qmid[k] >= 0.0 ? qmid[k] : first;
  s.n = most;
}

}  // namespace pa
