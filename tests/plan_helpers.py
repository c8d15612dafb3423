"""The scoring call's own plan (host header score_plan.h), asked from a test."""
import functools
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_37842_amd", "csrc")

# stdin: one call a line, "N Q topk tiled ws U k_0 .. k_(U-1)"; stdout: nqt rt n_rng grid n_blocks
# n_steps, the total of its workspace, and the first module of every range
PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "score_plan.h"
using namespace eogp;
int main() {
  long long N, Q, topk, tiled, ws, U;
  while (std::scanf("%lld %lld %lld %lld %lld %lld", &N, &Q, &topk, &tiled, &ws, &U) == 6) {
    std::vector<int64_t> k(U);
    for (auto& x : k) { long long v; if (std::scanf("%lld", &v) != 1) return 1; x = v; }
    const PassCfg c = choose_cfg(N, Q, (int)U, k.data(), (int)topk, tiled != 0, ws < 0 ? ~size_t(0) : (size_t)ws);
    const ScoreLayout L = score_layout(N, Q, (int)U, k.data(), (int)topk, c);
    std::vector<int32_t> rng(MAX_RNG + 1, 0);
    if (U > 1) module_ranges(k.data(), (int)U, L.n_steps, L.n_rng, rng.data());
    else rng[1] = 1;
    std::printf("%d %d %d %lld %lld %lld %zu", c.nqt, c.rt, L.n_rng, (long long)L.grid,
                (long long)row_blocks(N, c.rt), (long long)L.n_steps, L.total);
    for (int r = 0; r <= L.n_rng; ++r) std::printf(" %d", rng[r]);
    std::printf("\n");
  }
}
"""


@functools.lru_cache(maxsize=None)
def _program():
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tempfile.mkdtemp(prefix="score_plan_")
    src, exe = os.path.join(d, "plan.cpp"), os.path.join(d, "plan")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", f"-I{CSRC}", src, "-o", exe], check=True, capture_output=True, text=True)
    return exe


def score_plans(calls):
    """Plans of calls (N, Q, topk, tiled, workspace bytes or -1 for any, ks)."""
    text = "".join(f"{N} {Q} {topk} {int(tiled)} {ws} {len(ks)} {' '.join(map(str, ks))}\n"
                   for N, Q, topk, tiled, ws, ks in calls)
    out = subprocess.run([_program()], input=text, check=True, capture_output=True, text=True).stdout
    plans = []
    for line in out.splitlines():
        v = [int(x) for x in line.split()]
        plans.append(dict(nqt=v[0], rt=v[1], n_rng=v[2], grid=v[3], n_blocks=v[4], n_steps=v[5], total=v[6],
                          rng=v[7:]))
    return plans


def score_plan(N, Q, ks, topk, tiled=True, ws=-1):
    return score_plans([(N, Q, topk, tiled, ws, ks)])[0]
