// Energy panels for the response of Eq. (RPA) at finite broadening.
//
// Every weight of the transition sum is 1 / (x - D + i eta) with x = w
// (resonant) or x = -w (anti-resonant): a function of the transition energy D
// that is analytic except for the poles at x + i eta, one per frequency.  On
// an interval (a panel) that stays clear of the poles it is a short Chebyshev
// series in D,
//   1 / (z - y) = (1 / s) (1 + 2 sum_{i >= 1} r^-i T_i(y)),
//   s = sqrt(z - 1) sqrt(z + 1),  r = z + s,  |r| > 1,
// so the sum over the transitions of a panel is needed only for the basis
// functions T_0 .. T_{n-1}, whatever the number of frequencies.  The panels
// of a side depend on the frequencies and the broadening alone: they cover
// the whole energy axis, are as wide as the convergence of the series allows
// (about the broadening between the frequencies, growing with the distance
// outside), and end on both sides, kPanelFar from the frequencies, in an
// unbounded panel, on which
//   1 / (x - D + i eta) = -(u / S) / (1 - zeta u),  u = S / (D - c),
//   zeta = (x - c + i eta) / S,
// is u times a series in 2u - 1 (c lies beyond the frequencies on the other
// side of the panel, so 0 < u <= 1 and Re zeta > 0).  There Im W falls as u^2
// and its series only as u: the imaginary part keeps u times the relative
// accuracy.  Bounded panels keep it whole, so they cover every energy that
// occurs (a handful more per side: their width grows with the distance).
//
// Host code without HIP, so that it can be compiled and checked alone.
#pragma once

#include <algorithm>
#include <cmath>
#include <complex>
#include <limits>
#include <vector>

namespace qcx {

// kind 0: y = (D - c) s on |y| <= 1, basis T_i(y)
// kind 1: u = s / (D - c), y = 2u - 1, basis u T_i(y)
struct PanelDesc {
  double c, s;
  int kind, pad;
};

// Series lengths: the FP32-accumulated products use 16 terms, the FP64 ones
// 32.  One layout serves both: the remainder after 16 terms is below
// kPanelTol of the weight, and the remainder after 32 below its square,
// kPanelTol^2 = 1e-16, the rounding of FP64.
constexpr int kPanelTerms = 16, kPanelTerms64 = 32;
constexpr double kPanelTol = 1e-8;
constexpr double kPanelFar = 1e4;  // Hartree; the deepest core level lies above -5e3

// Remainder of the series after kPanelTerms terms relative to |1 / (z - y)|;
// |r| is the sum of the semi-axes of the ellipse with foci -1 and 1 through z.
inline double panel_remainder(std::complex<double> z) {
  const double x = z.real(), y2 = z.imag() * z.imag();
  const double m = std::sqrt((x - 1.0) * (x - 1.0) + y2), p = std::sqrt((x + 1.0) * (x + 1.0) + y2);
  const double a = 0.5 * (m + p);
  if (!(a > 1.0)) return std::numeric_limits<double>::infinity();
  const double r = a + std::sqrt(a * a - 1.0);
  const double r2 = r * r, r4 = r2 * r2, r8 = r4 * r4;
  return 2.0 / (r8 * r8) / (std::sqrt(m * p) * (1.0 - 1.0 / r)) * (std::sqrt(x * x + y2) + 1.0);
}

// Panels of one side for poles at x[0] <= x[1] <= ... (+ i eta), eta > 0:
// panel p holds edge[p - 1] <= D < edge[p] (unbounded outside).  Returns
// false if more than max_panels are needed or the numbers leave the range in
// which the recurrences are safe; the caller then sums the transitions
// directly.
inline bool panel_side(const std::vector<double>& x, double eta, int max_panels,
                       std::vector<double>& edge, std::vector<PanelDesc>& desc) {
  edge.clear();
  desc.clear();
  const double lo = x.front(), hi = x.back();
  const double span = std::max(hi - lo, eta);
  if (!(eta > 0.0) || !std::isfinite(span) || !(span < 1e12 * eta) ||
      !(std::max(std::fabs(lo), std::fabs(hi)) < 1e9 * eta))
    return false;
  using cd = std::complex<double>;
  // unbounded panel from X away from the poles (dir = +1 right, -1 left)
  auto unbounded = [&](double X, int dir) {
    PanelDesc d{};
    d.kind = 1;
    d.c = dir > 0 ? lo - span : hi + span;
    d.s = X - d.c;
    return d;
  };
  auto unbounded_ok = [&](double X, int dir) {
    const PanelDesc d = unbounded(X, dir);
    const cd zeta = cd((dir > 0 ? hi : lo) - d.c, eta) / d.s;
    return std::abs(zeta) < 1.0 && panel_remainder(2.0 / zeta - 1.0) <= kPanelTol;
  };
  // on a bounded panel the pole whose real part is nearest to the centre
  // lies on the smallest ellipse, so it alone decides
  auto bounded_ok = [&](double a, double h) {
    const double c = a + h;
    const auto it = std::lower_bound(x.begin(), x.end(), c);
    double d = std::numeric_limits<double>::infinity();
    if (it != x.end()) d = *it - c;
    if (it != x.begin()) d = std::min(d, c - *(it - 1));
    return panel_remainder(cd(d, eta) / h) <= kPanelTol;
  };
  // left end
  double far = kPanelFar;
  while (!unbounded_ok(lo - far, -1)) {
    far *= 2.0;
    if (!(far < 1e6 * std::max(span, kPanelFar))) return false;
  }
  double a = lo - far;
  desc.push_back(unbounded(a, -1));
  edge.push_back(a);
  const double h_min = 0.25 * eta;  // converges wherever the poles are
  double h = h_min;
  while (!(a >= hi + kPanelFar && unbounded_ok(a, 1))) {
    if ((int)desc.size() + 2 > max_panels) return false;
    // widest panel from a: the previous width while it still just fits
    // (between dense frequencies), else a bracket refined by bisection
    if (!(bounded_ok(a, h) && !bounded_ok(a, 1.05 * h))) {
      double g0 = h_min, g1 = h_min;
      if (bounded_ok(a, h)) g0 = g1 = h;
      do {
        g0 = g1;
        g1 *= 2.0;
      } while (bounded_ok(a, g1));  // ends: the poles are a finite distance away
      for (int i = 0; i < 12; ++i) {
        const double m = 0.5 * (g0 + g1);
        (bounded_ok(a, m) ? g0 : g1) = m;
      }
      h = g0;
    }
    const double b = a + 2.0 * h;
    if (!(b > a)) return false;
    PanelDesc d{};
    d.c = a + h;
    d.s = 1.0 / h;
    desc.push_back(d);
    edge.push_back(b);
    a = b;
  }
  desc.push_back(unbounded(a, 1));
  return true;
}

// Ranges of rows of G whose pairs' moments are held at once: rows [0, n) in whole
// tiles of `tile` rows, at most `most` pairs (one tile at least).  The tiles are
// those of the moments kernels (16 rows for each put the FP64 moments of 1024 G
// and 1000 frequencies at 14 GB; two take 1.8).
constexpr int kPanBinRows = 8, kPanBin64Rows = 2;  // FP32, FP64
struct PanelRange {
  int g0, g1, task0, n_task;  // rows and their tiles in the task list
  long b0;                    // upper-triangle index of the first pair
  int nb, nbp;                // pairs, padded to 128
};
inline void panel_ranges(int n, int tile, long most, bool diag, std::vector<PanelRange>& out) {
  auto first = [&](int g) { return diag ? (long)g : (long)g * n - (long)g * (g - 1) / 2; };
  out.clear();
  for (int g = 0; g < n;) {
    PanelRange r{};
    r.g0 = g;
    r.g1 = std::min(n, g + tile);
    while (r.g1 < n && first(std::min(n, r.g1 + tile)) - first(g) <= most) r.g1 = std::min(n, r.g1 + tile);
    r.b0 = first(g);
    r.nb = (int)(first(r.g1) - r.b0);
    r.nbp = (r.nb + 127) / 128 * 128;
    out.push_back(r);
    g = r.g1;
  }
}

// Are the panels the cheaper route?  Estimated seconds of the direct sum, which
// costs rows x transitions x columns, and of the panels, whose sum over the
// transitions is formed once (16 or 32 terms each), followed by rows x panels x
// columns; their dozen small launches cost as much as a whole small problem.
// The rates are least squares fits to both routes timed on MI355X at 70 random
// sizes (3^3 to 8^3 k points, 20 to 181 G, 8 to 450 frequencies; nine in ten
// within 12% of the time, the direct sum's within 30%).  Where the rule took the panels they
// never lost by more than 19%; where it did not they would have won by 47% at
// most.
struct PanelWork {
  bool fp64, fp32;  // else split-BF16
  bool diag;        // only the squares
  int n_t, n_g, n_w;
};
inline bool panels_pay(const PanelWork& k, int n_panels) {
  auto up = [](double x, double m) { return std::ceil(x / m) * m; };
  const double n_t = k.n_t, n_g = k.n_g, rows = 2.0 * k.n_w;
  const double pairs = k.diag ? n_g : n_g * (n_g + 1) / 2, p = std::min((double)n_panels, n_t);
  if (k.fp64) {
    const double direct = 17e-6 + rows * 2 * pairs * n_t / 2.3e13 + n_t * pairs / 3.3e11;
    return 176e-6 + 0.96e-9 * n_t + n_t * pairs / 2.9e11 + p * pairs / 6.2e10 +
               up(rows, 160) * up((k.diag ? 1 : 2) * pairs, 128) * p / 1.6e12 <
           direct;
  }
  const double rp = up(rows, 128), direct = k.fp32 ? 66e-6 + rp * 2 * pairs * n_t / 6.75e13 + 0.87e-9 * n_t + rp * n_t / 4.3e11
                                                   : 60e-6 + rp * 2 * pairs * n_t / 1.64e14 + rp * n_t / 3.9e11;
  // in FP32 the panels are the more accurate route (rms 1e-7 against 1.3e-7 to
  // 1.5e-6): they may take 15% longer
  return 236e-6 + 0.5e-9 * n_t + n_t * pairs / 1.0e12 + up(rows, 160) * 2 * n_g * p / 2.5e11 +
             up(rows, 32) * up(2 * pairs, 256) * p / (k.fp32 ? 1.27e13 : 3.7e13) <
         (k.fp32 ? 1.15 : 1.0) * direct;
}

// Can panels be taken at all, by what is known before their plan is made (which
// takes 0.1 ms of host time at 128 frequencies, 2 ms at a broadening of 6 meV)?
// w_max is the largest |w| (Hartree).
inline bool panels_possible(const PanelWork& k, double eta, double w_max) {
  // the squares alone below FP64 gain little (their direct sum is a small part
  // of the pair densities they come from)
  if (k.n_t < 2 || !(eta > 0.0) || (k.diag && !k.fp64)) return false;
  // a broadening far below the energies (nothing below this was measured) is
  // left to the direct sum
  if (!k.fp64 && !(eta >= 1e-4 * std::max(1.0, w_max))) return false;
  // below about 10,000 transitions a direct FP32 sum in many splits can be as
  // accurate (its error grows with the transitions, this route's does not)
  if (k.fp32 && k.n_t < 10000) return false;
  return panels_pay(k, 2);  // no plan has fewer
}

// The same panels for poles at -x[j] + i eta (the anti-resonant side).
inline void panel_mirror(const std::vector<double>& edge, const std::vector<PanelDesc>& desc,
                         std::vector<double>& m_edge, std::vector<PanelDesc>& m_desc) {
  m_edge.assign(edge.rbegin(), edge.rend());
  for (double& e : m_edge) e = -e;
  m_desc.assign(desc.rbegin(), desc.rend());
  for (PanelDesc& d : m_desc) {
    d.c = -d.c;
    if (d.kind == 1) d.s = -d.s;
  }
}

}  // namespace qcx
