"""The bracket of the Soft-TopK threshold: wide enough, and finite, for every target sum that a call may name."""
import math
import subprocess

import pytest

from paper_2605_06676_amd import build as B

PROGRAM = """
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include "lkv_bracket.h"
int main(int n, char** v) {
  for (int i = 2; i < n; ++i)
    printf("%.17g\\n", lkv::bracket_margin(atoi(v[1]), strtod(v[i], nullptr), [](float x) { return std::log2(x); }));
}
"""

PARTS = [5e-324, 1e-310, 2.3e-308, 1e-300, 1e-100, 1e-45, 1e-40, 1e-39, 1e-38, 1e-30, 1e-6, 0.25, 0.5, 0.75, 1.0, 7.3, 1000.5]


@pytest.mark.parametrize("n", [1, 2, 1000, 16384, 1 << 22])
def test_margin(tmp_path, n):
    (tmp_path / "margin.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", B.CSRC, str(tmp_path / "margin.cpp"), "-o", str(tmp_path / "margin")], check=True)
    parts = PARTS + [n / 2, n * (1 - 2.0 ** -30), math.nextafter(n, 0)]
    out = subprocess.run([str(tmp_path / "margin"), str(n)] + [repr(float(p)) for p in parts], check=True, capture_output=True, text=True)
    for part, got in zip(parts, map(float, out.stdout.split())):
        needed = 1 + max(0.0, math.log(n) - math.log(2) - math.log(part))
        # fp32: four roundings of numbers up to 2^10.1
        assert needed <= got <= needed + 0.0015, (part, got, needed)
