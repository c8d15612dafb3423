"""Ranges of examples of the fp16 EK-FAC squares, on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_37842_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "ekfac_plan.h"
int main() {
  long long N, T, i, o;
  while (std::scanf("%lld %lld %lld %lld", &N, &T, &i, &o) == 4)
    std::printf("%d %d\n", eogp::sq16_splits(N, T, i, o), eogp::sq16_min_splits(N, i, o));
}
"""


@pytest.fixture(scope="module")
def ranges(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("ekfac")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", f"-I{CSRC}", str(src), "-o", str(exe)], check=True,
                   capture_output=True, text=True)

    def ask(*case):
        out = subprocess.run([str(exe)], input=" ".join(map(str, case)), check=True, capture_output=True, text=True)
        return tuple(int(x) for x in out.stdout.split())
    return ask


@pytest.mark.parametrize("N,T,d_in,d_out,expect", [
    (256, 512, 769, 2304, 8), (200, 300, 2048, 2048, 8), (32, 512, 2304, 2304, 8), (128, 512, 3073, 768, 8),
    (32, 512, 2048, 2048, 2), (64, 128, 2048, 2048, 2),     # two ranges fill the chip, few tokens
    (64, 12, 769, 2304, 8),                                  # fewest ranges, but they fill it badly
    (31, 512, 769, 2304, 5), (64, 512, 3073, 3073, 1),      # few examples; tiles that fill it alone
])
def test_ranges(ranges, N, T, d_in, d_out, expect):
    assert ranges(N, T, d_in, d_out)[0] == expect


def test_ranges_fit_the_examples(ranges):
    for N in (0, 1, 3, 31, 32, 33, 1000):
        for d in (1, 128, 129, 1000, 2048, 5000):
            sp, least = ranges(N, 100, d, d)
            assert 1 <= least <= 32 and 1 <= sp <= 32 and (sp == least or sp * 4 <= N)
