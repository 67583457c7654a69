"""LDS of the wave kernels' rows, compiled for the CPU from the library's own
header: whatever the grid, the depth and the number of segments, the window and
the segments' lengths stay within the 64 KB that a launch has without asking, and
the window holds whole waves of records."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1802_01070_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include "pct_internal.h"
using namespace pct;
int main()
{
    long cases = 0, bad = 0;
    const int extents[] = {1, 3, 64, 256, 1000, 3200, 30000, 1 << 30};
    const double pitches[] = {1e-3, 0.02, 0.3, 1.0, 8.0};
    const int segments[] = {1, 2, 63, 64, 65, 220, 1000, 2345, kMaxRowSegments, kMaxRowSegments + 3};
    for (int nx : extents) for (int ny : extents) for (int nz : extents)
        for (double pitch : pitches) for (double pz : pitches) for (double depth : {1.0, 80.0, 220.0, 2000.0})
            for (int k : segments) {
                pct_grid g{nx, ny, nz, {pitch, pitch, pz}, {0, 0, 0}};
                const int span = record_span(g, depth, k);
                ++cases;
                if (span < kWave || span % kWave != 0 || record_bytes(k, span) > 65536) {
                    if (bad++ == 0) std::printf("%d %d %d %g %g %g %d: %d, %zu\n", nx, ny, nz, pitch, pz, depth, k, span, record_bytes(k, span));
                }
            }
    std::printf("%ld cases, %ld bad\n", cases, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_a_rows_window_fits_the_lds_of_a_launch(tmp_path):
    src, exe = tmp_path / "span.cpp", tmp_path / "span"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-I", os.path.join(CSRC, "..", "..", "include"), "-o",
                    str(exe), str(src)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
