"""The descriptor's reciprocals (csrc/desc.hpp `recip`): the kernels divide
positions below 2^31 by an index's extent with one multiplication and a
shift.  Compiled for the host and checked against the division itself: every
divisor up to 4096, powers of two and their neighbours, the largest extents,
each at the positions where a quotient steps and at the ends of the range."""
import shutil
import subprocess

import pytest

from conftest import ROOT

SOURCE = r"""
#include <initializer_list>
#include <stdio.h>
#include "paper_1607_00145_amd/csrc/desc.hpp"
static bool check(int64_t n)
{
    const gett::Recip r = gett::recip(n);
    const uint64_t top = 2147483647ull;   // positions are below 2^31 - 1
    auto one = [&](uint64_t v) {
        return v > top || ((v * r.mag) >> 32 >> r.sh) == v / (uint64_t)n;
    };
    for (uint64_t k = 0; k < 300; ++k) {
        const uint64_t q = k < 100 ? k : (top / n) * k / 299;   // multiples over the whole range
        const uint64_t v = q * n;
        if (!one(v) || !one(v + n - 1) || (v > 0 && !one(v - 1))) return false;
    }
    return one(top) && one(top - 1) && one(top / 2);
}
int main()
{
    if (gett::recip(1).mag != 0 || gett::recip(0).mag != 0) return 1;
    for (int64_t n = 2; n <= 4096; ++n)
        if (!check(n)) { printf("%lld\n", (long long)n); return 2; }
    for (int b = 1; b < 31; ++b)
        for (int64_t n = (1ll << b) - 1; n <= (1ll << b) + 1; ++n)
            if (n > 1 && !check(n)) { printf("%lld\n", (long long)n); return 3; }
    for (int64_t n : {2147483647ll, 2147483646ll, 1431655765ll, 1073741825ll, 715827883ll})
        if (!check(n)) { printf("%lld\n", (long long)n); return 4; }
    return 0;
}
"""


def test_reciprocal_divides(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("g++ not found")
    src, exe = tmp_path / "recip.cpp", tmp_path / "recip"
    src.write_text(SOURCE)
    subprocess.run([cxx, "-std=c++17", "-O1", f"-I{ROOT}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)
