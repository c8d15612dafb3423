"""Every variant of the scoring pass against the oracle, exactly: 16 and 32
queries per pass, two and (tiled) four row tiles per wave, one and several
modules, dots of 32 and 64 bits, both store layouts, rows requested by halves
and whole steps, module ends inside a step, ties that fill the candidate lists,
and a workspace that holds only the 16-query layout. Each case names the variant
it is for and asserts that the plan takes it."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_37842_amd import eogp as E
from plan_helpers import score_plan
from tiled_helpers import tiled_from_rows

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def d(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def store(N, ks, Q, seed):
    g = np.random.default_rng(seed)
    codes = g.integers(0, 256, size=(N, sum(ks) // 8), dtype=np.uint8)
    scales = np.exp(g.standard_normal((N, len(ks)))).astype(np.float16)
    return codes, scales, g.standard_normal((Q, sum(ks))).astype(np.float32)


def check(codes, scales, ks, Y, topk, tiled):
    N = codes.shape[0]
    print(f"[score] N={N} ks={ks[:3]}x{len(ks)} Q={Y.shape[0]} topk={topk} tiled={tiled}", flush=True)
    sc = d(scales.view(np.int16))
    if tiled:
        got = E.eogp_score_topk_tiled(d(tiled_from_rows(codes)), sc, N, ks, d(Y), topk, full_scores=True)
    else:
        got = E.eogp_score_topk(d(codes), sc, ks, d(Y), topk, full_scores=True)
    torch.cuda.synchronize()
    ref = O.score(codes, scales.view(np.uint16), ks, Y)
    oi, ov = O.topk(ref, topk)
    assert np.array_equal(got[2].cpu().numpy(), ref.astype(np.float32))
    assert np.array_equal(got[0].cpu().numpy(), oi)
    assert np.array_equal(got[1].cpu().numpy(), ov)


@pytest.mark.parametrize("tiled", [True, False])
@pytest.mark.parametrize("N,ks,Q,topk,rt,nqt", [
    (19, [1024], 5, 10, 2, 1),               # fewer rows than a tile
    (5000, [2048], 16, 100, 2, 1),           # 16 queries, two tiles per wave
    (5000, [2048], 40, 100, 2, 2),           # 32 queries, then a last pass of 16
    (270_000, [512], 16, 200, 2, 1),         # three rounds of two-tile blocks
    (270_000, [512], 33, 128, 2, 2),
    (140_001, [512], 16, 200, 4, 1),         # four tiles per wave, an unfinished last block
    (140_001, [512], 33, 100, 4, 2),
    (140_001, [1024], 64, 128, 4, 2),
    (500_001, [512], 16, 256, 4, 1),         # several blocks per workgroup: requests run on
    (500_001, [512], 33, 100, 4, 2),
    (3000, [512, 1024], 16, 200, 2, 1),      # several modules
    (3000, [512, 1024, 512], 20, 37, 2, 2),  # several modules, 32 queries
    (30_000, [512] * 3, 33, 100, 2, 2),
    (70_001, [512] * 3, 16, 100, 4, 1),      # several modules, four tiles per wave
    (70_001, [512] * 3, 33, 100, 4, 2),
    (90_001, [512] * 20, 20, 10, 4, 2),      # several units per workgroup
    (700, [66048], 20, 10, 2, 1),            # one module whose dots take 64 bits
    (1100, [1 << 18, 512], 20, 10, 2, 1),    # 64-bit dots of several modules
])
def test_score_pass_variants(N, ks, Q, topk, rt, nqt, tiled):
    plan = score_plan(N, Q, ks, topk, tiled)
    assert (plan["rt"], plan["nqt"]) == (rt if tiled else 2, nqt)      # the kernel this case is for
    if N in (500_001, 90_001) and tiled:
        assert plan["n_blocks"] * plan["n_rng"] > plan["grid"]
    codes, scales, Y = store(N, ks, Q, N + Q)
    check(codes, scales, ks, Y, topk, tiled)


@pytest.mark.parametrize("N,ks", [(140_001, [576]), (140_001, [64]), (30_001, [320, 64, 704])])
@pytest.mark.parametrize("Q", [16, 33])
def test_score_many_rows_end_inside_a_step(N, ks, Q):
    """Row-major modules that end inside a half step, over more blocks than one round."""
    codes, scales, Y = store(N, ks, Q, N + Q)
    check(codes, scales, ks, Y, 20, False)


@pytest.mark.parametrize("N,ks,Q", [
    (300, [64], 20), (33, [576], 17), (5, [320, 64, 704], 40), (1030, [832, 448], 16), (1, [64], 3),
])
def test_score_module_ends_inside_a_step(N, ks, Q):
    codes, scales, Y = store(N, ks, Q, N)
    check(codes, scales, ks, Y, 7, False)


@pytest.mark.parametrize("ks", [[320, 64, 704], [512, 1024], [1024, 64, 64, 576, 512, 448]])
@pytest.mark.parametrize("Q", [5, 16, 33])
@pytest.mark.parametrize("stride", [8192, 16384, 8192 + 8])
def test_score_rows_far_apart(ks, Q, stride):
    """Rows a multiple of 8 KB apart are requested a whole step at a time, others by halves;
    what lies between the rows is not read into any score."""
    N = 1100
    codes, scales, Y = store(N, ks, Q, stride + Q)
    wide = torch.randint(0, 256, (N, stride), device=DEV, dtype=torch.uint8)
    rows = wide[:, :sum(ks) // 8]
    rows.copy_(d(codes))
    got = E.eogp_score_topk(rows, d(scales.view(np.int16)), ks, d(Y), 9, full_scores=True)
    torch.cuda.synchronize()
    ref = O.score(codes, scales.view(np.uint16), ks, Y)
    oi, ov = O.topk(ref, 9)
    assert np.array_equal(got[2].cpu().numpy(), ref.astype(np.float32))
    assert np.array_equal(got[0].cpu().numpy(), oi) and np.array_equal(got[1].cpu().numpy(), ov)


@pytest.mark.parametrize("Q,topk", [(16, 256), (32, 128), (7, 1)])
def test_score_ties_and_infinite_scales(Q, topk):
    """Few distinct rows (every list fills with equal keys; the smaller index
    wins) and infinite scales."""
    codes, scales, Y = store(9000, [512], Q, 3)
    codes[:] = codes[np.arange(9000) % 3]
    scales[:] = scales[np.arange(9000) % 3]
    check(codes, scales, [512], Y, topk, True)
    scales[100:140] = np.inf
    check(codes, scales, [512], Y, topk, False)


@pytest.mark.parametrize("topk", [1, 2, 63, 64, 65, 127, 170, 171, 256])
@pytest.mark.parametrize("N,ks", [(9000, [512]), (1500, [512] * 8)])
def test_score_merge_sizes(N, ks, topk):
    """The merge's list of the other waves' entries ends inside, at and past one round
    of 512 (3 topk entries beside the topk kept)."""
    codes, scales, Y = store(N, ks, 3, topk)
    check(codes, scales, ks, Y, topk, True)


@pytest.mark.parametrize("ks", [[1024], [512, 512]])
def test_score_workspace_of_the_16_query_layout(ks):
    """A workspace too small for the 32-query pass runs the 16-query one, with
    the same results; one byte less than that is refused."""
    N, Q, topk = 4000, 48, 20
    codes, scales, Y = store(N, ks, Q, 5)
    c, s, y = d(codes), d(scales.view(np.int16)), d(Y)
    idx, sc, _ = E.eogp_score_topk(c, s, ks, y, topk)
    L = E.load()
    karr = (E.c_i64 * len(ks))(*ks)
    full = E.eogp_score_topk_workspace_size(N, Q, ks, topk)
    assert score_plan(N, Q, ks, topk, False) == dict(score_plan(N, Q, ks, topk, False, full), nqt=2, total=full)
    less = score_plan(N, Q, ks, topk, False, 0)["total"]          # the 16-query layout
    assert less < full and score_plan(N, Q, ks, topk, False, full - 1)["nqt"] == 1
    ws = torch.empty(full, dtype=torch.uint8, device=DEV)
    for nbytes in (full, full - 1, less):
        i2, s2 = torch.full_like(idx, -7), torch.zeros_like(sc)
        st = L.eogp_score_topk(E._ptr(c), codes.shape[1], E._ptr(s), N, len(ks), karr, E._ptr(y), sum(ks), Q, topk,
                               E._ptr(i2), E._ptr(s2), None, E._ptr(ws), nbytes, E._stream())
        assert st == 0
        torch.cuda.synchronize()
        assert torch.equal(i2, idx) and torch.equal(s2, sc)
    assert L.eogp_score_topk(E._ptr(c), codes.shape[1], E._ptr(s), N, len(ks), karr, E._ptr(y), sum(ks), Q, topk,
                             E._ptr(idx), E._ptr(sc), None, E._ptr(ws), less - 1, E._stream()) == -4
