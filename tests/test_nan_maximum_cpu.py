"""max_nan (csrc/df_nan.hpp), the running maximum of the vertex symmetry check and of the
screening certificate: a NaN stays, wherever it enters.  Host build of the same header."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include "df_nan.hpp"
int main() {
    // the 64-lane xor butterfly with a NaN in one lane, finite values elsewhere
    for (int bad = -1; bad < 64; ++bad) {
        float v[64], u[64];
        for (int l = 0; l < 64; ++l) v[l] = l == bad ? NAN : (float)((l * 37) % 64);
        for (int off = 1; off < 64; off <<= 1) {
            for (int l = 0; l < 64; ++l) u[l] = df::max_nan(v[l], v[l ^ off]);
            for (int l = 0; l < 64; ++l) v[l] = u[l];
        }
        for (int l = 0; l < 64; ++l)
            if (bad < 0 ? v[l] != 63.f : v[l] == v[l]) return printf("lane %d of NaN %d\n", l, bad), 1;
    }
    // a serial maximum, the NaN at either end, infinities ordered
    if (df::max_nan(df::max_nan(0.f, NAN), 5.f) == df::max_nan(df::max_nan(0.f, NAN), 5.f)) return 2;
    if (df::max_nan(5.f, NAN) == df::max_nan(5.f, NAN)) return 3;
    if (df::max_nan(5.f, INFINITY) != INFINITY || df::max_nan(-INFINITY, 5.f) != 5.f) return 4;
    return 0;
}
"""


def test_a_nan_reaches_every_lane(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    inc = os.path.join(ROOT, "paper_1507_00895_amd", "csrc")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", inc, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)
