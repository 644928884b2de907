"""The fixed-point scale of the capacity loss's probability sums (csrc/capacity_scale.h), compiled for the host: over every number of
assignments that the library accepts the sum of as many ones stays within 64 bits, no bit is given away, and batches below 2^26
assignments keep 2^38."""
import os
import subprocess

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "capacity_scale.h"
int main(int argc, char **argv)
{
    for (int i = 1; i < argc; ++i) std::printf("%d\n", slicemoe::capacity_fraction_bits(std::atoll(argv[i])));
}
"""


def test_the_sum_of_as_many_ones_fits_64_bits(tmp_path):
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04286_amd", "csrc")
    (tmp_path / "scale.cpp").write_text(SRC)
    exe = str(tmp_path / "scale")
    subprocess.check_call(["g++", "-std=c++17", "-I", csrc, str(tmp_path / "scale.cpp"), "-o", exe])
    sizes = sorted({n + o for b in range(0, 31) for n in (1 << b, 3 << b >> 1) for o in (-1, 0, 1)} | {2**31 - 1})   # up to T S k < 2^31
    sizes = [n for n in sizes if 1 <= n < 2**31]
    bits = list(map(int, subprocess.check_output([exe, *map(str, sizes)], text=True).split()))
    for n, f in zip(sizes, bits):
        assert n << f < 2**64, (n, f)
        assert f == 38 or n << (f + 1) >= 2**64, (n, f)
        assert n >= 2**26 or f == 38, (n, f)
