"""The imaginary part of the panel series (csrc/panel_plan.h) by itself: the
loss far from every pole comes from Im 1 / (x - D + i eta) = -eta / (x - D)^2,
a small part of the weight, which has to keep its own relative accuracy at
every transition energy that occurs."""
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2603_12326_amd" / "csrc"
HA = 27.211386245988

# reads eta, n, x[n], m, D[m]; per side the worst relative error of the
# imaginary part after 16 and 32 terms
_PROGRAM = r"""
#include "panel_plan.h"
#include <cstdio>
using namespace qcx;
using cd = std::complex<double>;
int main() {
  double eta; int n, m;
  if (scanf("%lf %d", &eta, &n) != 2) return 1;
  std::vector<double> x(n);
  for (double& v : x) if (scanf("%lf", &v) != 1) return 1;
  if (scanf("%d", &m) != 1) return 1;
  std::vector<double> D(m);
  for (double& v : D) if (scanf("%lf", &v) != 1) return 1;
  std::sort(x.begin(), x.end());
  std::vector<double> e0, e; std::vector<PanelDesc> d0, d;
  if (!panel_side(x, eta, 4096, e0, d0)) return 2;
  for (int side = 0; side < 2; ++side) {
    e = e0; d = d0;
    if (side) panel_mirror(e0, d0, e, d);
    double worst[2] = {0, 0};
    for (double en : D) {
      const size_t q = std::upper_bound(e.begin(), e.end(), en) - e.begin();
      double y, wt = 1;
      if (d[q].kind) { const double u = d[q].s / (en - d[q].c); y = 2 * u - 1; wt = u; }
      else y = (en - d[q].c) * d[q].s;
      for (int j = 0; j < n; j += 1 + n / 20) {
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
        const double re = w.real() - en, ex = -eta / (re * re + eta * eta);
        worst[0] = std::max(worst[0], std::fabs(s16.imag() * wt / ex - 1));
        worst[1] = std::max(worst[1], std::fabs(sum.imag() * wt / ex - 1));
      }
    }
    printf("%.3e %.3e\n", worst[0], worst[1]);
  }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx
    d = tmp_path_factory.mktemp("panel")
    (d / "p.cpp").write_text(_PROGRAM)
    subprocess.run([gxx, "-O1", "-std=c++20", f"-I{CSRC}", str(d / "p.cpp"), "-o", str(d / "p")], check=True)
    return d / "p"


@pytest.mark.parametrize("w,eta", [
    (np.linspace(0, 60, 400), 0.1), (np.linspace(0, 30, 300), 0.1), (np.linspace(0, 1, 300), 0.003),
    (np.array([10.0]), 0.1), (np.array([1.0, 1.2]), 1e-4), (np.linspace(-30, 25, 77), 0.2),
    (np.linspace(0, 20, 33), 2.0)], ids=["60eV", "30eV", "gap", "one", "narrow", "negative", "wide"])
def test_imaginary_part(program, w, eta):
    """Transition energies from 0.01 eV to 100 keV, core levels included.  With
    the remainder 1e-8 of the weight after 16 terms the imaginary part's is
    below 1e-8 (16 / |s| + 2 / |z - 1|)(|z| + 1) <= 5e-7 for every pole that
    the plan admits (|z| >= 1.7); after 32 terms 1e-14 with the rounding of
    32 terms."""
    D = np.concatenate([np.geomspace(0.01, 1e5, 700), w[w > 0][:50] + 0.01]) / HA
    text = f"{eta / HA!r} {len(w)} " + " ".join(repr(float(v / HA)) for v in w)
    text += f" {len(D)} " + " ".join(repr(float(v)) for v in D)
    out = subprocess.run([str(program)], input=text, capture_output=True, text=True, check=True).stdout
    for line in out.strip().split("\n"):
        e16, e32 = map(float, line.split())
        assert e16 <= 5e-7
        assert e32 <= 1e-13
