"""Which second stages of few rows stream P past a shared Z, on the host: both sides of the
rule at sizes where one of the two kernels was measured a tenth or more faster."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_37842_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "gemm_plan.h"
int main() {
  long long M, N, K, sp, products;
  while (std::scanf("%lld %lld %lld %lld %lld", &M, &N, &K, &sp, &products) == 5) {
    const eogp::FewRowsPlan p = eogp::few_rows_plan(M, N, K, (int)sp, (int)products);
    std::printf("%d %d %lld\n", p.use ? 1 : 0, p.splits, (long long)p.kc);
  }
}
"""
# (rows, m, k, products, the stream is the faster)
MEASURED = [
    (1, 16384, 1024, 1, False), (16, 16384, 300, 1, False), (32, 32768, 2048, 1, False),
    (128, 32768, 1024, 1, False), (72, 16384, 4096, 1, False), (128, 8192, 4096, 1, False),
    (128, 4096, 4096, 1, False), (96, 16384, 2500, 1, False),
    (16, 512, 256, 1, True), (1, 2048, 2048, 1, True), (16, 8192, 4096, 1, True),
    (16, 16384, 8192, 1, True), (1, 16384, 16384, 1, True), (64, 16384, 4096, 1, True),
    (64, 65536, 32768, 1, True), (128, 2048, 700, 1, True), (128, 4096, 256, 1, True),
    (128, 16384, 8192, 1, True), (16, 32768, 16384, 1, True),
    (128, 800, 300, 3, False), (96, 16384, 300, 3, False), (128, 2048, 128, 3, False),
    (1, 800, 300, 3, True), (64, 4096, 256, 3, True), (128, 2048, 700, 3, True),
    (128, 16384, 1024, 3, True), (128, 32768, 16384, 3, True),
    (64, 800, 300, 3, False), (64, 800, 300, 2, True), (128, 16384, 300, 2, False), (128, 16384, 1024, 2, True),
    # tiled units that leave a grid rounded down to the XCDs in a second round, and neighbours that don't
    (87, 2680, 785, 1, True), (128, 2688, 1024, 1, True), (128, 3200, 700, 1, True), (128, 1472, 1300, 1, True),
    (128, 3648, 2500, 1, True), (65, 2680, 300, 3, True), (128, 2688, 785, 2, True), (128, 1024, 785, 3, True),
    (128, 800, 785, 2, False),
    # more groups than CUs: rounds of either kernel
    (1, 32768, 12000, 1, True), (16, 16392, 12000, 1, True), (32, 32768, 8400, 1, True),
    (128, 20000, 10240, 1, False), (65, 32760, 20480, 1, False), (128, 32768, 10240, 1, False),
    (128, 20000, 11264, 1, True), (128, 16384, 16384, 1, True), (16, 32760, 18432, 1, False),
    (48, 20000, 14336, 1, True),
    # 224 to 256 groups: rows of P a multiple of 8 KB apart, and others
    (64, 16384, 8192, 1, True), (128, 8200, 8192, 1, False), (87, 16392, 8192, 1, False),
    (64, 8200, 4096, 1, False), (16, 16392, 8192, 1, False),
]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("few_rows")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", f"-I{CSRC}", str(src), "-o", str(exe)], check=True,
                   capture_output=True, text=True)

    def ask(rows, m, k, products, splits=8):
        out = subprocess.run([str(exe)], input=f"{rows} {k} {m} {splits} {products}\n", check=True,
                             capture_output=True, text=True).stdout
        return tuple(int(x) for x in out.split())
    return ask


@pytest.mark.parametrize("rows,m,k,products,stream", MEASURED)
def test_measured_sizes(plan, rows, m, k, products, stream):
    assert bool(plan(rows, m, k, products)[0]) == stream


@pytest.mark.parametrize("m", [8, 200, 512, 520, 4104, 65536, 1000000])
@pytest.mark.parametrize("k", [1, 256, 257, 8192, 100000])
@pytest.mark.parametrize("splits", [1, 3, 8])
def test_ranges_cover_the_depth(plan, m, k, splits):
    for rows in (1, 33, 65, 128):
        use, sp, kc = plan(rows, m, k, 1, splits)
        assert 1 <= sp <= splits and kc % 64 == 0 and (sp - 1) * kc < m <= sp * kc
    assert plan(129, m, k, 1, splits)[0] == 0
