"""The slice denominators of the gain estimates (device code), compiled for the host from the same
source text: where a solve's slices have no common denominator the value is the correctly rounded
quotient, as a division gives it, for every integer numerator below 2^62 in magnitude and every
denominator below 2^31; a product with the rounded reciprocal is not."""
import os
import random
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
DEVICE_HPP = os.path.join(HERE, "..", "paper_2608_03695_amd", "csrc", "device.hpp")

MAIN = r"""
int main() {
  long long a, S;
  long cases = 0, wrong = 0, products = 0;
  while (scanf("%lld %lld", &a, &S) == 2) {
    const double x = (double)a, d = (double)S;
    const SliceRecip q{1.0 / d, d}, whole{(double)(a % 1000), 0.0};
    cases++;
    wrong += q.of(x) != x / d || whole.of(x) != x * (double)(a % 1000);
    products += x * (1.0 / d) != x / d;
  }
  printf("%ld %ld %ld\n", cases, wrong, products);
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_quotients_are_rounded_once(tmp_path):
    src = open(DEVICE_HPP).read()
    a, b = src.index("struct SliceRecip"), src.index("// end of the slice denominators")
    cpp, exe = tmp_path / "q.cpp", tmp_path / "q"
    cpp.write_text("#include <cmath>\n#include <cstdio>\nusing std::fma;\n#define __device__\n"
                   "#define __host__\n" + src[a:b] + MAIN)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", str(cpp), "-o", str(exe)],
                   check=True)
    rnd = random.Random(11)
    top = 2 ** 31 - 1
    dens = [1, 2, 3, 5, 7, top, top - 1, 2 ** 30, 2 ** 30 + 1] + [rnd.randint(1, top) for _ in range(300)]
    cases = []
    for S in dens:
        for bits in range(1, 63):
            a = rnd.getrandbits(bits) - (1 << bits - 1) * rnd.randint(0, 1)
            # numerators of any size, next to multiples of S and next to halves of the last place
            cases += [(a, S), (a // S * S + rnd.randint(-1, 1), S), ((a | 1) * S >> 1, S)]
    cases = [(a, S) for a, S in cases if abs(a) < 2 ** 62]
    out = subprocess.run([str(exe)], input="".join(f"{a} {S}\n" for a, S in cases),
                         capture_output=True, text=True, check=True).stdout.split()
    assert [int(x) for x in out[:2]] == [len(cases), 0]
    assert int(out[2]) > len(cases) // 100   # the plain products differ in many of them
