"""The scoring call's plan, on the host: the workgroups of a pass over several modules share
its units evenly, and the block size is the one with the shorter schedule."""
import math
import random

import pytest

from plan_helpers import score_plan, score_plans

XCDS, CUS = 8, 256


def most_units(plan):
    """The most units that one workgroup walks, as the kernel deals them: contiguous
    shares to the XCDs (workgroup b on XCD b % 8), at a fixed stride within a share."""
    units, G = plan["n_blocks"] * plan["n_rng"], plan["grid"]
    shares = XCDS if G >= XCDS and G % XCDS == 0 else 1
    chunk = -(-units // shares)
    seen, most = 0, 0
    for b in range(G):
        x = b % shares
        end = min((x + 1) * chunk, units)
        got = len(range(x * chunk + b // shares, end, G // shares))
        seen, most = seen + got, max(most, got)
    assert seen == units, (plan, seen)
    return most


def calls():
    rng = random.Random(5)
    out = [(N, 16, 10, True, -1, [k] * U) for U, N, k in
           [(2, 30_000, 8192), (2, 60_000, 8192), (2, 100_000, 8192), (3, 40_000, 8192), (5, 25_000, 8192),
            (7, 30_000, 8192), (48, 20_000, 8192), (48, 5_000, 8192), (112, 5_000, 8192), (107, 9_723, 256),
            (26, 30_877, 12_800), (9, 121_564, 11_776), (54, 36_168, 16_384), (2, 1, 64), (64, 300, 64)]]
    for _ in range(200):
        U = int(math.exp(rng.uniform(math.log(2), math.log(200))))
        N = int(math.exp(rng.uniform(0, math.log(2_000_000))))
        ks = [64 * rng.randint(1, 200) for _ in range(U)]
        out.append((N, rng.randint(1, 64), rng.randint(1, 256), rng.random() < 0.5, -1, ks))
    return out


def test_units_are_shared_evenly():
    """A plan of one round runs in one: no workgroup has more than its share rounded up."""
    for c, p in zip(calls(), score_plans(calls())):
        units = p["n_blocks"] * p["n_rng"]
        assert p["grid"] <= CUS and (units >= XCDS or p["grid"] == units)
        assert most_units(p) == -(-units // CUS), (c, p)
        assert p["rng"][0] == 0 and p["rng"][-1] == len(c[5])
        assert all(a < b for a, b in zip(p["rng"], p["rng"][1:]))


@pytest.mark.parametrize("U,N,k", [(2, 30_000, 8192), (2, 60_000, 8192), (2, 100_000, 8192), (3, 30_000, 8192),
                                   (3, 50_000, 8192), (5, 25_000, 8192), (7, 30_000, 8192), (12, 60_000, 8192),
                                   (48, 20_000, 8192), (48, 30_000, 8192), (112, 5_000, 8192)])
def test_block_size_has_the_shorter_schedule(U, N, k):
    """The longest workgroup's steps (those of four tiles weigh 1.75 of two) against every
    number of ranges at both block sizes: within a tenth of the shortest."""
    steps = U * k // 512

    def length(rt, r):
        units = -(-N // (256 * rt)) * r
        return -(-units // CUS) * (steps / U * -(-U // r) + 1) * (1.75 if rt == 4 else 1.0)

    p = score_plan(N, 16, [k] * U, 100)
    took = most_units(p) * (max(b - a for a, b in zip(p["rng"], p["rng"][1:])) * steps / U + 1) * (
        1.75 if p["rt"] == 4 else 1.0)
    best = min(length(rt, r) for rt in (2, 4) for r in range(1, min(U, 64) + 1))
    assert took <= 1.1 * best, (p, took, best)
