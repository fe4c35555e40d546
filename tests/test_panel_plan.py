"""The energy panels of the response (csrc/panel_plan.h, host code without HIP):
compiled here, checked against the weights 1 / (x - D + i eta) themselves."""
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2603_12326_amd" / "csrc"

# reads eta, n, x[n]; prints one line per side: ok, panels, worst relative
# remainder of 16 and of 32 terms, 1 if the edges ascend
_PROGRAM = r"""
#include "panel_plan.h"
#include <cstdio>
using namespace qcx;
using cd = std::complex<double>;
int main() {
  double eta; int n;
  if (scanf("%lf %d", &eta, &n) != 2) return 1;
  std::vector<double> x(n);
  for (double& v : x) if (scanf("%lf", &v) != 1) return 1;
  std::sort(x.begin(), x.end());
  std::vector<double> e0, e; std::vector<PanelDesc> d0, d;
  const bool ok = panel_side(x, eta, 4096, e0, d0);
  for (int side = 0; side < 2; ++side) {
    if (!ok) { printf("0 0 0 0 0\n"); continue; }
    e = e0; d = d0;
    if (side) panel_mirror(e0, d0, e, d);
    double m16 = 0, m32 = 0; bool asc = d.size() == e.size() + 1;
    for (size_t q = 1; q < e.size(); ++q) asc = asc && e[q] > e[q - 1];
    for (size_t q = 0; q < d.size(); ++q)
      for (int k = 0; k <= 12; ++k) {
        double D;  // inside the panel, the unbounded ones out to 1e8 eta
        if (q == 0) D = e[0] - eta * std::pow(10.0, k - 4);
        else if (q == e.size()) D = e[q - 1] + eta * std::pow(10.0, k - 4);
        else D = e[q - 1] + (e[q] - e[q - 1]) * k / 12.0;
        double y, wt = 1;
        if (d[q].kind) { const double u = d[q].s / (D - d[q].c); y = 2 * u - 1; wt = u; }
        else y = (D - d[q].c) * d[q].s;
        if (std::fabs(y) > 1 + 1e-9) asc = false;
        for (int j = 0; j < n; j += 1 + n / 40) {
          const cd w(side ? -x[j] : x[j], eta);
          cd z, amp;
          if (d[q].kind) { const cd ze = (w - d[q].c) / d[q].s; z = 2.0 / ze - 1.0; amp = -(1 / d[q].s) * (2.0 / ze); }
          else { z = (w - d[q].c) * d[q].s; amp = d[q].s; }
          const cd s = std::sqrt(z - 1.0) * std::sqrt(z + 1.0), r = 1.0 / (z + s);
          amp /= s;
          double t0 = 1, t1 = y; cd sum = amp, pw = r, s16;
          for (int i = 1; i < kPanelTerms64; ++i) {
            sum += 2.0 * amp * pw * t1;
            if (i == kPanelTerms - 1) s16 = sum;
            pw *= r;
            const double t2 = 2 * y * t1 - t0; t0 = t1; t1 = t2;
          }
          const cd ex = 1.0 / (w - D);
          m16 = std::max(m16, std::abs(s16 * wt - ex) / std::abs(ex));
          m32 = std::max(m32, std::abs(sum * wt - ex) / std::abs(ex));
        }
      }
    printf("%d %zu %.3e %.3e %d\n", (int)ok, d.size(), m16, m32, (int)asc);
  }
}
"""

HA = 27.211386245988


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx
    d = tmp_path_factory.mktemp("panel")
    (d / "p.cpp").write_text(_PROGRAM)
    subprocess.run([gxx, "-O1", "-std=c++20", f"-I{CSRC}", str(d / "p.cpp"), "-o", str(d / "p")], check=True)
    return d / "p"


def _sides(program, x, eta):
    text = f"{eta!r} {len(x)} " + " ".join(repr(float(v)) for v in x)
    out = subprocess.run([str(program)], input=text, capture_output=True, text=True, check=True).stdout
    return [[float(v) for v in line.split()] for line in out.strip().split("\n")]


_RNG = np.random.default_rng(5)
_LISTS = dict(
    dense=(np.linspace(0, 60, 400), 0.1), sparse=(np.array([0.0, 7.0, 50.0]), 0.1),
    one=(np.array([10.0]), 0.1), zero=(np.array([0.0]), 0.3), thousand=(np.linspace(0, 100, 1000), 0.1),
    wide=(np.linspace(0, 20, 33), 2.0), negative=(np.linspace(-30, 25, 77), 0.2),
    unsorted=(_RNG.uniform(0, 40, 150), 0.15), repeated=(np.repeat([3.0, 3.0, 12.0], 20), 0.1),
    near=(5.0 + 1e-9 * np.arange(10), 0.1), far=(np.array([500.0, 500.5]), 0.5))


@pytest.mark.parametrize("name", list(_LISTS))
def test_series_meets_its_remainder(program, name):
    """Every weight, at points across every panel of both sides, within the
    planned remainder: 1e-8 after 16 terms; 1e-16 after 32, of which rounding
    leaves the conditioning of D - x (1e-13 covers |x| / eta <= 1000 x 2^-53)."""
    w, eta = _LISTS[name]
    for ok, n, m16, m32, asc in _sides(program, w / HA, eta / HA):
        assert ok == 1 and asc == 1
        assert 2 <= n <= 4096
        assert m16 <= 1.0e-8 * (1 + 1e-3)
        assert m32 <= 1.0e-13


def test_refuses_what_it_cannot_cover(program):
    """No broadening, or more panels than the limit: the caller sums directly."""
    assert _sides(program, np.linspace(0, 1, 5), 0.0)[0][0] == 0
    assert _sides(program, np.linspace(0, 100, 20000), 1e-4)[0][0] == 0
