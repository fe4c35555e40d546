"""Which route the response takes (panels_pay of csrc/panel_plan.h, host code
without HIP) against the time of both, measured on MI355X."""
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2603_12326_amd" / "csrc"
HA = 27.211386245988

# reads lines: precision (0 FP64, 1 FP32, 2 split), diag, n_t, n_g, n_w, eta, w_max
# (0 .. w_max evenly), n_panels (0: of the plan); prints the panels of a side, the
# choice, and what is known of it before the plan
_PROGRAM = r"""
#include "panel_plan.h"
#include <cstdio>
using namespace qcx;
int main() {
  int prec, diag, n_t, n_g, n_w, n_p; double eta, top;
  while (scanf("%d %d %d %d %d %lf %lf %d", &prec, &diag, &n_t, &n_g, &n_w, &eta, &top, &n_p) == 8) {
    std::vector<double> x(n_w), e; std::vector<PanelDesc> d;
    for (int i = 0; i < n_w; ++i) x[i] = n_w > 1 ? top * i / (n_w - 1) : top;
    if (!n_p && panel_side(x, eta, 4096, e, d)) n_p = (int)d.size();
    const PanelWork k{prec == 0, prec == 1, diag != 0, n_t, n_g, n_w};
    printf("%d %d %d\n", n_p, (int)panels_pay(k, n_p), (int)panels_possible(k, eta, top));
  }
}
"""

# precision, transitions, G, frequencies, broadening and last frequency (eV),
# us by the direct sum, us through panels
_MEASURED = [
    (2, 43904, 51, 77, 0.23, 45, 218, 339), (2, 27648, 73, 78, 0.28, 45, 240, 368), (2, 27648, 60, 106, 0.17, 45, 239, 329),
    (2, 65536, 48, 68, 0.09, 45, 287, 403), (2, 65536, 113, 400, 0.1, 60, 4400, 1000), (2, 65536, 95, 105, 0.13, 45, 1089, 607),
    (1, 16464, 32, 110, 0.09, 45, 146, 366), (1, 16464, 35, 80, 0.15, 45, 156, 299), (1, 16464, 27, 133, 0.14, 45, 158, 293),
    (1, 24576, 38, 37, 0.13, 45, 168, 273), (1, 24576, 181, 155, 0.1, 60, 4089, 1120), (1, 10368, 91, 224, 0.21, 45, 733, 368),
    (0, 16464, 41, 51, 0.17, 45, 188, 324), (0, 10368, 48, 94, 0.12, 45, 215, 318), (0, 24576, 38, 37, 0.13, 45, 246, 369),
    (0, 6000, 152, 77, 0.24, 45, 1800, 921), (0, 24576, 138, 12, 0.27, 45, 1983, 1120), (0, 3072, 27, 128, 0.2, 40, 45, 250),
    (0, 65536, 113, 400, 0.1, 60, 31400, 3900)]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx
    d = tmp_path_factory.mktemp("route")
    (d / "p.cpp").write_text(_PROGRAM)
    subprocess.run([gxx, "-O1", "-std=c++20", f"-I{CSRC}", str(d / "p.cpp"), "-o", str(d / "p")], check=True)
    return d / "p"


def _run(program, lines):
    text = "\n".join(f"{p} {d} {t} {g} {w} {eta / HA!r} {top / HA!r} {n}" for p, d, t, g, w, eta, top, n in lines)
    out = subprocess.run([str(program)], input=text, capture_output=True, text=True, check=True).stdout
    return [tuple(map(int, line.split())) for line in out.strip().split("\n")]


def test_faster_route_is_taken(program):
    """Sizes at which one route takes at least a quarter more than the other."""
    got = _run(program, [(p, 0, t, g, w, eta, top, 0) for p, t, g, w, eta, top, _, _ in _MEASURED])
    for m, (_, panels, _) in zip(_MEASURED, got):
        assert bool(panels) == (m[7] < m[6]), m


def test_no_plan_where_panels_cannot_be_taken(program):
    """Calls that panels never serve are known as such before any plan is made:
    small problems, the diagonal below FP64, few FP32 transitions, a vanishing
    broadening.  And nothing that pays with its own plan is lost."""
    never = [(0, 0, 3072, 27, 128, 0.2, 40, 0), (2, 0, 3072, 27, 128, 0.2, 40, 0), (2, 1, 27648, 4096, 400, 0.1, 60, 0),
             (1, 1, 65536, 4096, 400, 0.1, 60, 0), (1, 0, 9999, 181, 400, 0.1, 60, 0), (2, 0, 65536, 113, 400, 0.002, 60, 1),
             (2, 0, 65536, 113, 400, 0.0, 60, 1), (0, 0, 65536, 113, 400, 0.0, 60, 1), (0, 0, 1296, 60, 100, 0.1, 60, 0)]
    assert [r[2] for r in _run(program, never)] == [0] * len(never)
    rng = np.random.default_rng(4)
    many = [(p, d, int(t), int(g), int(w), float(eta), float(rng.uniform(30, 60)), 0)
            for p in (0, 1, 2) for d in (0, 1) if p == 0 or not d
            for t, g, w, eta in zip(np.exp(rng.uniform(7, 11.5, 150)), np.exp(rng.uniform(2, 6.5, 150)),
                                    np.exp(rng.uniform(1, 6.5, 150)), rng.uniform(0.08, 0.3, 150)) if p != 1 or t >= 10000]
    got = _run(program, many)
    assert sum(r[1] for r in got) > 100
    assert all(r[2] >= r[1] for r in got)
