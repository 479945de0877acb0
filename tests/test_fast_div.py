"""Host check of FastDiv (csrc/launch_util.hpp), the quotient by a
multiplication that the seam pass indexes with: compiled with hipcc for the
host, run on the CPU and compared with the division.  Exact for every
0 <= n < 2^31; the values where a rounded reciprocal would fail first are the
multiples of the divisor and their predecessors."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2003_12621_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"

SRC = r"""
#include <climits>
#include <cstdio>
#include "launch_util.hpp"
using namespace fftsplit;

int main() {
    long long bad = 0, seen = 0;
    auto check = [&](int d) {
        const FastDiv f = fast_div(d);
        auto at = [&](long long n) {
            if (n < 0 || n > INT_MAX) return;
            ++seen;
            bad += f.quotient(int(n)) != int(n / d);
        };
        const long long top = INT_MAX / d;
        for (long long q = 0; q <= top && q < 200; ++q)
            for (long long e = -1; e <= 1; ++e) {
                at(q * d + e);
                at((top - q) * d + e);
            }
        for (long long n = 0; n <= INT_MAX; n += 1000003) at(n);
        at(INT_MAX);
    };
    for (int d = 1; d <= 4096; ++d) check(d);
    for (int b = 12; b < 31; ++b)
        for (int e = -1; e <= 1; ++e) check((1 << b) + e);
    check(INT_MAX);
    check(INT_MAX - 1);
    std::printf("seen=%lld bad=%lld\n", seen, bad);
    return bad ? 1 : 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_quotients(tmp_path):
    src = tmp_path / "fast_div.hip"
    src.write_text(SRC)
    exe = tmp_path / "fast_div"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert " bad=0" in r.stdout
