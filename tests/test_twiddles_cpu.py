"""The FP32 twiddle constants w = c (1 + i t), compiled on the host: every root
the transforms use is within sqrt(2) 2^-25 of w, the most that the two
roundings of a (cos, sin) pair in FP32 leave."""
import math
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2609_03027_amd", "csrc")
SIDES = (16, 24, 32, 48, 96, 128, 256, 512)


def _compile_and_run(src, tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    f = tmp_path / "t.cpp"
    f.write_text(src)
    exe = str(tmp_path / "t")
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(f), "-o", exe], check=True,
                   capture_output=True, text=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout


def test_roots_as_exact_as_rounded_pairs(tmp_path):
    lines = "\n".join(f"for (int n = 0; n < {s} / 2; ++n) out(n, {s});" for s in SIDES)
    out = _compile_and_run(
        '#include <cstdio>\n#include "roots.h"\n'
        "static void out(int n, int L) { const epic::Root r = epic::root_of(n, L);"
        ' printf("%d %d %.17g %.17g\\n", n, L, (double)r.t, (double)r.c); }\n'
        "int main() {" + lines + "}\n", tmp_path)
    assert len(out.splitlines()) == sum(SIDES) // 2
    for line in out.splitlines():
        n, side, t, c = (float(x) for x in line.split())
        if 4 * n == side:
            assert c * t == 1.0 and c <= 2.0 ** -40
            continue
        a = 2.0 * math.pi * n / side
        err = math.hypot(c - math.cos(a), c * t - math.sin(a))
        assert err <= math.sqrt(2.0) * 2.0 ** -25, (n, side, err)
