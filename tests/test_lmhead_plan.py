"""The LM-head tile kernel is compiled for the row-tile heights that calls reach:
lmhead_least_height, by which the others are left out, against every row count."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "paper_2608_03447_amd/csrc/asd_plan.h"
using namespace asd;
int main() {
    int64_t least[300];
    for (int64_t& h : least) h = 1 << 20;
    for (int64_t rows = 129; rows <= 256 * 299; ++rows) {
        const int64_t t = lmhead_row_tiles(rows), h = lmhead_tile_height(rows);
        if (h < 5 || h > 8 || t * 32 * h < rows || (t - 1) * 32 * h >= rows) return 1;
        if (h < least[t]) least[t] = h;
    }
    for (int64_t t = 298; t >= 2; --t) {
        if (least[t + 1] < least[t]) least[t] = least[t + 1];      // of t row tiles or more
        if (least[t] != lmhead_least_height(t)) return 2;
    }
    std::printf("%d %d\n", (int)lmhead_least_height(3), (int)lmhead_least_height(kLmheadFewRowTiles + 1));
    return 0;
}
"""


def test_every_row_count_reaches_a_compiled_height(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src = tmp_path / "heights.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "heights")
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", ROOT,
                    "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include", str(src),
                    "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0
    assert run.stdout.split() == ["6", "7"]
