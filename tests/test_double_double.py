"""The double-double primitives of the 6j evaluation, compiled for the host, against exact fractions."""
import os
import random
import subprocess
from fractions import Fraction

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2107_13952_amd", "csrc")

SOURCE = r'''
#include <cstdio>
#include "dd.hpp"
int main() {
  double a, b;
  while (std::scanf("%lf %lf", &a, &b) == 2) {
    const eprl::dd q = eprl::dd_ratio(a, b);
    std::printf("%a %a\n", q.hi, q.lo);
  }
}
'''


@pytest.fixture(scope="module")
def ratio(tmp_path_factory):
    path = tmp_path_factory.mktemp("dd")
    src, exe = str(path / "ratio.cpp"), str(path / "ratio")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", CSRC, "-o", exe, src], check=True)
    return exe


def test_ratio_has_all_bits(ratio):
    # Ratios of the Racah series: products of three or four factors up to 400, signed.  Both words of the
    # quotient rounded to nearest: half an ulp of a second word that is half an ulp of the first, 2^-106
    # (and 2^-40 of that for the rounding of the corrections).
    rng = random.Random(11)
    pairs = [(-rng.randint(1, 402) * rng.randint(1, 400) * rng.randint(1, 400) * rng.randint(1, 400),
              rng.randint(1, 400) * rng.randint(1, 400) * rng.randint(1, 400) * rng.choice([1, rng.randint(1, 400)]))
             for _ in range(20000)]
    pairs += [(-a, b) for a in range(1, 60) for b in range(1, 60)]
    out = subprocess.run([ratio], input="\n".join(f"{a} {b}" for a, b in pairs), capture_output=True, text=True, check=True)
    worst = 0
    for (a, b), line in zip(pairs, out.stdout.split("\n")):
        hi, lo = (Fraction(float.fromhex(v)) for v in line.split())
        exact = Fraction(a, b)
        worst = max(worst, abs(hi + lo - exact) / abs(exact))
    assert worst <= Fraction(1, 2 ** 106) * (1 + Fraction(1, 2 ** 40)), float(worst * 2 ** 106)
