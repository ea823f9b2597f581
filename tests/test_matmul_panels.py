"""Panel sizes of the matrix engine under a short workspace: the library's host code, compiled alone (no GPU)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_11112_amd", "csrc")
MAIN = r"""
#include <stdio.h>
#include <stdlib.h>
#include "panels.h"
int main(int, char **v) {
  const int64_t tm = atoll(v[1]), tn = atoll(v[2]);
  int64_t pm = spdz::up(atoll(v[3]), tm), pn = spdz::up(atoll(v[4]), tn);
  for (int k = 0; k < 200; k++) {
    printf("%lld %lld\n", (long long)pm, (long long)pn);
    if (!spdz::smaller_panel(pm, pn, tm, tn)) return 0;
  }
  return 1;
}
"""


@pytest.fixture(scope="module")
def panels(tmp_path_factory):
    d = tmp_path_factory.mktemp("panels")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "panels")], check=True)
    return str(d / "panels")


# tiles of 64 WM x 64 WN for the engine's three tilings
@pytest.mark.parametrize("tm,tn", [(256, 256), (256, 128), (128, 128)])
@pytest.mark.parametrize("M,N", [(1, 1), (256, 256), (200, 250), (257, 1), (1, 100000), (4096, 4096), (4095, 8193),
                                 (768, 640), (1 << 40, 3), (3, 1 << 40), (1 << 31, 1 << 31)])
def test_panels_shrink_to_one_tile(panels, tm, tn, M, N):
    """Every step is smaller, in whole tiles, and the steps end at one tile, after at most log2 of the tiles."""
    run = subprocess.run([panels, str(tm), str(tn), str(M), str(N)], capture_output=True, text=True, timeout=20)
    assert run.returncode == 0, run.stdout[-200:]
    steps = [tuple(map(int, line.split())) for line in run.stdout.splitlines()]
    assert steps[0] == (-(-M // tm) * tm, -(-N // tn) * tn) and steps[-1] == (tm, tn)
    for (m0, n0), (m1, n1) in zip(steps, steps[1:]):
        assert m1 % tm == 0 and n1 % tn == 0 and m1 <= m0 and n1 <= n0 and (m1, n1) != (m0, n0)
    assert len(steps) <= 2 + (steps[0][0] // tm).bit_length() + (steps[0][1] // tn).bit_length()
