"""The three nearest triangles that a lane of the 3D closest-triangle search
keeps, on the host: what it hands on is always a triangle that it was shown.  A
mesh with non-finite markers can leave it with fewer than three, or with none."""
import os
import subprocess

import pytest

from paper_1906_03065_amd import build

MAIN = r"""
#include <cmath>
#include <cstdio>
#include "k_lb.h"
#include "k_ibm.h"
#include "k_ibm3d.h"
int main() {
  int n;
  while (scanf("%d", &n) == 1) {
    lb::Nearest3 a;
    float tol, d;
    int q;
    if (scanf("%f", &tol) != 1) return 1;
    for (int k = 0; k < n; k++) {
      if (scanf("%f %d", &d, &q) != 2) return 1;
      a.add(d, q);
    }
    printf("%d %d %d %d\n", a.within(tol), a.q0, a.q1, a.q2);
  }
}
"""
NONE = 3.0e38  # the least distance of a lane that was shown nothing


@pytest.fixture(scope="module")
def select(tmp_path_factory):
    d = tmp_path_factory.mktemp("sel")
    src, exe = d / "sel.hip", d / "sel"
    src.write_text(MAIN)
    csrc = os.path.join(os.path.dirname(build.__file__), "csrc")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call([build.HIPCC, *flags, "-I", csrc, "-o", str(exe), str(src)], stderr=subprocess.DEVNULL)

    def run(tol, shown):
        text = f"{len(shown)} {tol} " + " ".join(f"{d} {q}" for d, q in shown)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        return [int(v) for v in out.split()]

    return run


@pytest.mark.parametrize("shown,kept", [
    ([], []), ([("nan", 4), ("nan", 0)], []), ([("inf", 3)], []),
    ([("nan", 7), (2.0, 5)], [5]), ([(2.0, 5), ("nan", 7), (1.0, 9)], [9, 5]),
    ([(4.0, 0), (3.0, 1), (2.0, 2), (1.0, 3)], [3, 2, 1]), ([(1.0, 8), (1.0, 2)], [8, 2]),
])
@pytest.mark.parametrize("tol", [0.5, 1.0, 2.5, NONE, 3.3e38, "inf"])
def test_only_triangles_that_were_shown(select, shown, kept, tol):
    n, *q = select(tol, shown)
    assert q == kept + [-1] * (3 - len(kept))
    dist = {i: float(d) for d, i in shown}
    assert n == sum(dist[i] <= float(tol) for i in kept)
