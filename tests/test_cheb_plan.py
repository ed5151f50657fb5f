"""The storage plan of the Chebyshev expansions, built with the host compiler and
its undefined-behaviour checks (conversions out of range end the program)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1203_6836_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include "cheb_plan.h"
int main() {
    for (int N : {1, 2, 3, 45, 128, 2048, 11585, 11586, 16384, 23170, 32768})
        for (int m : {2, 3, 4, 5, 36, 50, 1024, 1025, 1250, 4088}) {
            const int s = sp2::cheb_stored(N, m);
            std::printf("%d %d %d %d\\n", N, m, s, sp2::cheb_multiples(m, s));
        }
    return 0;
}
"""


def test_stored_polynomials_over_the_sizes(tmp_path):
    """N = 1 to 32768: at least one stored polynomial and at most 32 or
    ceil(sqrt(m)), s + 2 matrices within 32 GiB or five, all m coefficients
    covered by the multiples, and no conversion out of range (32 GiB are 2^32
    matrices of N = 1)."""
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "plan.cpp").write_text(PROGRAM)
    exe = tmp_path / "plan"
    subprocess.run([cxx, "-std=c++17", "-fsanitize=undefined,float-cast-overflow", "-fno-sanitize-recover=all", "-I", CSRC,
                    str(tmp_path / "plan.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    rows = [tuple(map(int, l.split())) for l in r.stdout.splitlines()]
    assert len(rows) == 110
    for N, m, s, q in rows:
        assert s in (1, 2, 4, 8, 12, 16, 20, 24, 28, 32)
        assert s == 1 or (s - 1) ** 2 < m
        assert (s + 2) * 8 * N * N <= max(32 << 30, 5 * 8 * N * N)
        assert (q + 1) * s >= m and q * s < m
