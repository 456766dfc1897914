"""The GEMMs' rules (csrc/a3_gemm_tiles.h), compiled for the CPU.  Which tile a workgroup takes: every tile exactly once, and no
XCD (workgroup id % 8) with more than its share, unless that still fits its 32 CUs - one more would cost a second round.
Which tile a product runs in: one that took at most a tenth longer than the best of the six on an MI355X."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "a3_gemm_tiles.h"
int main() {
  for (int n_wt = 1; n_wt <= 150; n_wt += n_wt < 40 ? 1 : 11)
    for (int n_xt = 1; n_xt <= 66; n_xt += n_xt < 20 ? 1 : 5) {
      const int gm = gemm_tile_group(n_wt, n_xt), grid = (int)gemm_tile_grid(n_wt, n_xt);
      std::vector<int> seen(n_wt * n_xt, 0);
      int per_xcd[8] = {0};
      for (int id = 0; id < grid; ++id) {
        int wt = -1, xt = -1;
        if (!gemm_tile_of(n_wt, n_xt, gm, id, wt, xt)) continue;
        if (wt < 0 || wt >= n_wt || xt < 0 || xt >= n_xt) return std::printf("%d x %d: tile (%d, %d)\n", n_wt, n_xt, wt, xt), 1;
        ++seen[wt * n_xt + xt];
        ++per_xcd[id % 8];
      }
      for (int s : seen)
        if (s != 1) return std::printf("%d x %d: a tile taken %d times\n", n_wt, n_xt, s), 1;
      for (int x = 0; x < 8; ++x)
        if (per_xcd[x] > 32 && per_xcd[x] > (n_wt * n_xt + 7) / 8) return std::printf("%d x %d: XCD %d takes %d tiles\n", n_wt, n_xt, x, per_xcd[x]), 1;
    }
  return 0;
}
"""


# (weight rows, activation rows, reduction): us of the projection in the tiles 256x256, 256x192, 256x128, 128x192, 128x128, 128x64
MEASURED = {
    (6144, 1500, 4096): [88, 72, 100, 82, 94, 112],
    (6144, 1860, 4096): [92, 76, 104, 88, 100, 136],
    (6144, 2050, 4096): [94, 130, 107, 120, 126, 154],
    (4608, 1500, 3584): [76, 62, 50, 70, 58, 78],
    (4608, 2650, 3584): [84, 72, 96, 82, 92, 123],
    (4096, 1500, 4096): [83, 68, 55, 48, 63, 69],
    (4096, 3000, 4096): [94, 81, 108, 93, 103, 137],
    (4096, 2650, 14336): [275, 223, 313, 257, 299, 403],
}


def _run(tmp_path, program):
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(program)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2511_17560_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True)


pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")


def test_every_tile_once_and_evenly_over_the_xcds(tmp_path):
    res = _run(tmp_path, PROGRAM)
    assert res.returncode == 0, res.stdout


def test_choice_is_near_the_measured_best(tmp_path):
    calls = "".join(f'std::printf("%d ", gemm_choose_tile({w}, {x}, {k // 64}, 1).tile);' for w, x, k in MEASURED)
    res = _run(tmp_path, '#include <cstdio>\n#include "a3_gemm_tiles.h"\nint main() { ' + calls + " }")
    for (shape, us), tile in zip(MEASURED.items(), map(int, res.stdout.split())):
        assert us[tile] <= 1.1 * min(us), (shape, tile)
