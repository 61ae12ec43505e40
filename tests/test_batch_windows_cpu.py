"""The batch's fixed-point coordinates on the host: for every point the window and
the first tap's distance are those of the plan's floating-point expressions, bit
for bit, moved by the cells between the shared and the own bin's start."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SRC = r"""
#include "internal.h"
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
int main()
{
    std::mt19937_64 r(1);
    long bad = 0, n = 0;
    for (int w = 2; w <= 8; ++w)
        for (int own : {6, 8, 11, 12, 16, 17, 23, 32})
            for (int m : {8, 16, 29, 32}) {
                const int P = (w + 1) / 2;
                for (int it = 0; it < 20000; ++it) {
                    // anywhere, or within units of single precision of a window's edge
                    const double f = r() % 4 ? (double)(r() % (1ull << 53)) / (double)(1ull << 53)
                                             : (w & 1 ? 0.5 : 0.0) + ((int)(r() % 65) - 32) *
                                                   std::ldexp(1.0, -20 - (int)(r() % 8));
                    const double gc = (double)(r() % 1000 + 1) + f;
                    const int l = (int)gc, c = l / own * own, o = c - l / m * m;
                    const float u = (float)(gc - (double)c), v = u + (float)P;
                    const float s = std::ceil(v - (float)(0.5 * w)), d = s - v;
                    float e;
                    const int q = mn::fix_coord(u, P, o), t = mn::fix_start(q, w, e);
                    const bool ok = t == (int)s + o && e == d && t >= 0 && t <= m + 1 && q > 0 &&
                                    q < (1 << 29);
                    if (!ok && ++bad < 5) std::printf("w %d own %d m %d gc %.17g\n", w, own, m, gc);
                    ++n;
                }
            }
    std::printf("%ld points, %ld differ\n", n, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
def test_fixed_point_windows(tmp_path):
    src, exe = tmp_path / "w.cpp", tmp_path / "w"
    src.write_text(SRC)
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17",
                    "-I" + os.path.join(ROOT, "paper_2102_08463_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
