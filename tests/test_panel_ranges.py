"""Ranges of rows whose moments the panel route holds at once (panel_ranges of
csrc/panel_plan.h, host code without HIP)."""
import shutil
import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2603_12326_amd" / "csrc"

_PROGRAM = r"""
#include "panel_plan.h"
#include <cstdio>
using namespace qcx;
int main() {
  int n, fp64, diag; long most;
  printf("%d %d\n", kPanBinRows, kPanBin64Rows);
  while (scanf("%d %d %d %ld", &n, &fp64, &diag, &most) == 4) {
    std::vector<PanelRange> r;
    panel_ranges(n, diag ? 128 : fp64 ? kPanBin64Rows : kPanBinRows, most, diag, r);
    for (const PanelRange& x : r) printf("%d %d %ld %d %d ", x.g0, x.g1, x.b0, x.nb, x.nbp);
    printf("\n");
  }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx
    d = tmp_path_factory.mktemp("ranges")
    (d / "p.cpp").write_text(_PROGRAM)
    subprocess.run([gxx, "-O1", "-std=c++20", f"-I{CSRC}", str(d / "p.cpp"), "-o", str(d / "p")], check=True)
    return d / "p"


_CASES = [(n, f, d, m) for n in (1, 2, 15, 16, 17, 113, 300, 749, 1024, 4096) for f, d in ((0, 0), (1, 0), (1, 1))
          for m in (1, 200, 2100, 9000, 1 << 40)]


def test_ranges(program):
    """The ranges cover the rows in order, hold every pair once, stay within
    what may be held unless they are a single tile, and are as long as that
    allows."""
    text = "\n".join(" ".join(map(str, c)) for c in _CASES)
    lines = subprocess.run([str(program)], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    rows = list(map(int, lines[0].split()))
    for (n, f, diag, most), line in zip(_CASES, lines[1:]):
        tile = 128 if diag else rows[f]
        v = list(map(int, line.split()))
        r = [v[i:i + 5] for i in range(0, len(v), 5)]
        at = pair = 0
        for i, (g0, g1, b0, nb, nbp) in enumerate(r):
            assert g0 == at and g1 > g0 and b0 == pair
            assert nb == sum(1 if diag else n - g for g in range(g0, g1)) and nb <= nbp < nb + 128 and nbp % 128 == 0
            assert g0 % tile == 0 and (g1 - g0 <= tile or nb <= most)
            if g1 < n:
                assert nb + sum(1 if diag else n - g for g in range(g1, min(n, g1 + tile))) > most
            at, pair = g1, pair + nb
        assert at == n


def test_moments_of_many_rows_fit(program):
    """1024 G in FP64 (32 terms of 8 bytes, two parts, 1700 entries) and 4096 G
    in three bf16 planes: 4 GiB hold every range."""
    for n, f, per in ((1024, 1, 32 * 8 * 2 * 1700), (4096, 0, 96 * 2 * 600)):
        out = subprocess.run([str(program)], input=f"{n} {f} 0 {(4 << 30) // per}", capture_output=True, text=True,
                             check=True).stdout.split("\n")[1].split()
        assert max(map(int, out[3::5])) * per <= 4 << 30
