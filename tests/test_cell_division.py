"""The division by a grid's cell counts (a multiplication and a shift, common.hpp) against exact
integer division: compiled for the host from the header's own text, over divisors and dividends at
and next to the multiples, up to 2^31 - 1."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1908_01682_amd", "csrc")

MAIN = r"""
#include <cstdint>
#include <cstdio>
#include <random>
#define __host__
#define __device__
%s
int main()
{
    std::mt19937_64 r(1);
    long bad = 0;
    auto check = [&](int n, int x) {
        unsigned mul;
        int shift;
        make_divisor(n, mul, shift);
        bad += divide_by(x, mul, shift) != x / n;
    };
    for (int t = 0; t < 600000; ++t) {
        int n = t < 5000 ? t + 1 : int((r() & 0x7fffffff) >> (r() %% 31));
        if (n < 1) n = 1;
        const int q = int(r() %% (0x7fffffffu / unsigned(n) + 1));
        check(n, 0), check(n, 0x7fffffff), check(n, int(r() & 0x7fffffff)), check(n, q * n);
        if (q) check(n, q * n - 1);
    }
    printf("%%ld\n", bad);
    return bad != 0;
}
"""


def test_divide_by_is_exact(tmp_path):
    text = open(os.path.join(CSRC, "common.hpp")).read()
    i = text.index("__host__ __device__ inline int divide_by")
    j = text.index("template <typename R>\n__device__ __forceinline__ bool finite_r")
    src, exe = str(tmp_path / "t.cpp"), str(tmp_path / "t")
    with open(src, "w") as f:
        f.write(MAIN % text[i:j])
    subprocess.check_call(["g++", "-O2", "-o", exe, src])
    assert subprocess.run([exe], capture_output=True, text=True).stdout.strip() == "0"
