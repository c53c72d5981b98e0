"""Division by a launch constant (csrc/div_const.hpp), compiled for the host: the
quotient of every divisor a box can have, at the multiples of it (and their
neighbours) where a wrong reciprocal shows first, up to the largest index."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1707_08900_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <initializer_list>
#include "div_const.hpp"
int main() {
    unsigned long long bad = 0, n = 0;
    const uint32_t top = 0x7fffffffu;
    auto at = [&](const fd6::DivConst& c, uint32_t x) {
        if (x <= top) ++n, bad += x / c != x / c.d;
    };
    for (uint32_t d = 2; d <= 4200; ++d) {
        const fd6::DivConst c = fd6::div_const(d);
        const uint32_t last = top / d;
        for (uint32_t q = 1; q <= 64; ++q)
            for (const uint32_t m : {q, last - q, last / 64 * q, last - q * 97 % last}) {
                at(c, m * d);
                at(c, m * d - 1);
                at(c, m * d + 1);
            }
        at(c, 0);
        at(c, d - 1);
        at(c, top);
        at(c, last * d);
        at(c, last * d - 1);
    }
    printf("%llu %llu\n", n, bad);
}
"""


def test_quotients_are_exact(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "h.cpp", tmp_path / "h"
    src.write_text(HARNESS)
    subprocess.run([cxx, "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", str(src), "-o",
                    str(exe)], check=True)
    n, bad = map(int, subprocess.run([str(exe)], capture_output=True, text=True,
                                     check=True).stdout.split())
    assert n > 3_000_000 and bad == 0
