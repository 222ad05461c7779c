"""The tempering call's exchange rows (host code, no GPU): the threshold that row,
cut and zero give is that of the formula for every energy difference, for pairs
so close that a row holds all of them, pairs whose thresholds turn to 1 and to 0
inside it, the denormal end of exp, and rows longer than a pair needs."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1709_04394_amd", "csrc")

DRIVER = r"""
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "pt_rows.hpp"
using namespace mcs;
static long ones, zeros, bad;
static void pair(double b0, double b1, int64_t mmax, int64_t more)
{
    const PtPair p = pt_pair(b0, b1, mmax);
    const int64_t row = std::min(p.cut + 1 + more, mmax + 1);
    std::vector<uint64_t> x((size_t)row);
    const uint64_t round0 = (1ull << 40) - 3;
    pt_row(b0, b1, p, row, round0, x.data());
    if (x[0] >> kPtZeroBits != round0 || p.cut > mmax || p.zero > mmax + 1) ++bad;
    for (int64_t m = 1; m <= mmax; ++m) {
        const uint64_t want = (uint64_t)std::ceil(std::ldexp(std::exp((b0 - b1) * (double)(4 * m)), 32));
        const uint64_t got = pt_threshold(x.data(), (int)row, (int)m);
        if (got != want && ++bad < 5) fprintf(stderr, "b %a %a m %lld: %llu, not %llu\n", b0, b1, (long long)m, (unsigned long long)got, (unsigned long long)want);
        ones += want == 1 && m >= row;
        zeros += want == 0 && m >= row;
    }
}
int main()
{
    const int L[] = {4, 8, 16, 32, 64, 128, 512};
    srand(3);
    for (int l : L) {
        const int64_t mmax = (int64_t)l * l;
        for (int64_t more : {0, 1, 1000}) {
            for (double d : {0.2 / 31, 0.2 / 999, 0.01, 0.35, 2.4, 37.0, 1e-9, 1e-17, 1e3, 1e300, 5e-324, 186.0, 186.28})
                pair(0.0, d, mmax, more), pair(0.37, 0.37 + d, mmax, more);
            // an m at each place between -746 and -744, and around -22.5
            for (double x : {744.0, 744.4400719213812, 745.0, 745.13, 745.1332191019412, 745.14, 746.0, 22.5, 22.18070977791825})
                for (int m : {1, 2, 3, 7, 1000, 4095})
                    for (double e : {-1e-13, 0.0, 1e-13}) pair(0.0, x * (1.0 + e) / (4.0 * m), mmax, more);
            for (int i = 0; i < 20; ++i) {
                const double b = rand() / 1e9;
                pair(b, b + std::exp(rand() / 1.1e8 - 15.0), mmax, more);
            }
        }
    }
    printf("ones %ld zeros %ld bad %ld\n", ones, zeros, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_rows_give_the_formula(tmp_path):
    src, exe = tmp_path / "rows.cpp", str(tmp_path / "rows")
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wall", "-I", CSRC, str(src), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, (r.stdout, r.stderr)
    ones, zeros = int(r.stdout.split()[1]), int(r.stdout.split()[3])
    assert ones > 0 and zeros > 0  # differences beyond a row, of either kind
