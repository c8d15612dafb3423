"""Calls that must not cost more than a call with more to do: each test times
both on the same card, in turn, and compares medians."""
import statistics

import pytest
import torch

from paper_2609_37842_amd import eogp as E

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def times(*calls, passes=20, rounds=9):
    """Median time of one pass of each call, in microseconds."""
    for f in calls:
        f()
    got = [[] for _ in calls]
    for _ in range(rounds):
        for f, out in zip(calls, got):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            t0.record()
            for _ in range(passes):
                f()
            t1.record()
            torch.cuda.synchronize()
            out.append(t0.elapsed_time(t1) * 1e3 / passes)
    return [statistics.median(x) for x in got]


def random_store(N, k, Q, seed=1):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    codes = torch.randint(0, 256, (N, k // 8), device=DEV, dtype=torch.uint8, generator=g)
    scales = torch.rand((N, 1), device=DEV, generator=g).add_(0.5).half().view(torch.int16)
    return codes, scales, torch.randn((Q, k), device=DEV, generator=g)


@pytest.mark.parametrize("N,k", [(256, 128), (20000, 128), (20000, 2048)])
def test_one_query_costs_no_more_than_sixteen(N, k):
    """Lists of the fifteen queries that do not exist take no selection of their own."""
    codes, scales, Y = random_store(N, k, 16)

    def call(Q):
        ws = torch.empty(E.eogp_score_topk_workspace_size(N, Q, [k], 10), dtype=torch.uint8, device=DEV)
        idx = torch.empty((Q, 10), dtype=torch.int64, device=DEV)
        top = torch.empty((Q, 10), device=DEV)
        return lambda: E.eogp_score_topk(codes, scales, [k], Y[:Q], 10, out_idx=idx, out_score=top, ws=ws)

    one, sixteen = times(call(1), call(16))
    print(f"[times] N={N} k={k}: one query {one:.1f} us, sixteen {sixteen:.1f} us", flush=True)
    assert one <= sixteen


def layout_calls(N, k, Q, topk=10):
    """One scoring call on a row-major store and one on a tiled store of N codes."""
    rows, scales, Y = random_store(N, k, Q)
    tiles = torch.randint(0, 256, (E.tiled_store_bytes(N, [k]),), device=DEV, dtype=torch.uint8)
    idx = torch.empty((Q, topk), dtype=torch.int64, device=DEV)
    top = torch.empty((Q, topk), device=DEV)
    ws = torch.empty(E.eogp_score_topk_workspace_size(N, Q, [k], topk), dtype=torch.uint8, device=DEV)
    return (lambda: E.eogp_score_topk(rows, scales, [k], Y, topk, out_idx=idx, out_score=top, ws=ws),
            lambda: E.eogp_score_topk_tiled(tiles, scales, N, [k], Y, topk, out_idx=idx, out_score=top, ws=ws))


def test_row_major_store_is_read_in_whole_loads():
    """Row-major codes are read 16 bytes per lane; in pieces of 4 and 8 a pass took
    1.6 times as long as over the tiled layout."""
    rows, tiled = times(*layout_calls(473_050, 6144, 16))
    print(f"[times] 473,050 x 6,144 bits, 16 queries: row-major {rows:.1f} us, tiled {tiled:.1f} us", flush=True)
    assert rows <= 1.4 * tiled


def test_short_modules_cost_what_their_bits_cost():
    """The same bits and dots in one long module and in many short ones: what ends a
    module (its dots written) is not a chain of waits."""
    N, Q, topk = 200_000, 16, 10
    scales = torch.rand((N, 64), device=DEV).add_(0.5).half().view(torch.int16)
    codes = torch.randint(0, 256, (E.tiled_store_bytes(N, [512] * 64),), device=DEV, dtype=torch.uint8)
    Y = torch.randn((Q, 64 * 512), device=DEV)
    idx = torch.empty((Q, topk), dtype=torch.int64, device=DEV)
    top = torch.empty((Q, topk), device=DEV)

    def call(U):
        ks = [64 * 512 // U] * U
        s = scales[:, :U].contiguous()
        ws = torch.empty(E.eogp_score_topk_workspace_size(N, Q, ks, topk), dtype=torch.uint8, device=DEV)
        return lambda: E.eogp_score_topk_tiled(codes, s, N, ks, Y, topk, out_idx=idx, out_score=top, ws=ws)

    few, many = times(call(4), call(64))
    dots = 60 * N * Q * 4                       # bytes that 60 more modules write, and read again
    print(f"[times] 200,000 x 32,768 bits: 4 modules {few:.1f} us, 64 modules {many:.1f} us", flush=True)
    assert many <= few + 2 * dots / 4e6         # 384 us at 4 TB/s (301 measured; as a chain 487)


def test_a_quarter_more_codes_cost_no_second_round():
    """Two modules: 25,600 codes fit the same round of workgroups as 20,480."""
    Q, topk, ks = 16, 10, [8192, 8192]
    Y = torch.randn((Q, sum(ks)), device=DEV)
    idx = torch.empty((Q, topk), dtype=torch.int64, device=DEV)
    top = torch.empty((Q, topk), device=DEV)

    def call(N):
        codes = torch.randint(0, 256, (E.tiled_store_bytes(N, ks),), device=DEV, dtype=torch.uint8)
        scales = torch.rand((N, 2), device=DEV).add_(0.5).half().view(torch.int16)
        ws = torch.empty(E.eogp_score_topk_workspace_size(N, Q, ks, topk), dtype=torch.uint8, device=DEV)
        return lambda: E.eogp_score_topk_tiled(codes, scales, N, ks, Y, topk, out_idx=idx, out_score=top, ws=ws)

    less, more = times(call(20_480), call(25_600))
    print(f"[times] 2 x 8,192 bits: 20,480 codes {less:.1f} us, 25,600 codes {more:.1f} us", flush=True)
    assert more <= 1.25 * less


def test_one_query_writes_no_dots_of_the_other_fifteen():
    """Several short modules, where the dots between pass and fold are most of the traffic."""
    N, U, topk = 200_000, 30, 10
    ks = [512] * U
    codes = torch.randint(0, 256, (E.tiled_store_bytes(N, ks),), device=DEV, dtype=torch.uint8)
    scales = torch.rand((N, U), device=DEV).add_(0.5).half().view(torch.int16)
    Y = torch.randn((16, sum(ks)), device=DEV)

    def call(Q):
        ws = torch.empty(E.eogp_score_topk_workspace_size(N, Q, ks, topk), dtype=torch.uint8, device=DEV)
        idx = torch.empty((Q, topk), dtype=torch.int64, device=DEV)
        top = torch.empty((Q, topk), device=DEV)
        return lambda: E.eogp_score_topk_tiled(codes, scales, N, ks, Y[:Q], topk, out_idx=idx, out_score=top, ws=ws)

    one, sixteen = times(call(1), call(16))
    print(f"[times] 30 x 512 bits, 200,000 codes: one query {one:.1f} us, sixteen {sixteen:.1f} us", flush=True)
    assert one <= 0.8 * sixteen


def test_rows_a_power_of_two_apart_cost_little_more():
    """Row-major rows 16 KB apart (16 modules of 8,192 bits) against rows 64 bytes more."""
    N, U, Q, topk = 20_000, 16, 4, 10
    ks = [8192] * U
    scales = torch.rand((N, U), device=DEV).add_(0.5).half().view(torch.int16)
    Y = torch.randn((Q, sum(ks)), device=DEV)
    ws = torch.empty(E.eogp_score_topk_workspace_size(N, Q, ks, topk), dtype=torch.uint8, device=DEV)
    idx = torch.empty((Q, topk), dtype=torch.int64, device=DEV)
    top = torch.empty((Q, topk), device=DEV)

    def call(pad):
        codes = torch.randint(0, 256, (N, 1024 * U + pad), device=DEV, dtype=torch.uint8)[:, :1024 * U]
        return lambda: E.eogp_score_topk(codes, scales, ks, Y, topk, out_idx=idx, out_score=top, ws=ws)

    even, odd = times(call(0), call(64))
    print(f"[times] 16 x 8,192 bits row-major: 16 KB apart {even:.1f} us, 64 bytes more {odd:.1f} us", flush=True)
    assert even <= 1.25 * odd


def test_short_rows_pack_no_slower_than_their_bytes():
    """Rows of 64 coordinates carry an eighth of the bytes of rows of 512: packing them
    takes no longer."""
    N = 100_000
    X = torch.randn((N, 1024), device=DEV)
    scales = torch.empty((N, 1), dtype=torch.int16, device=DEV)

    def call(k):
        x, codes = X[:, :k].contiguous(), torch.empty((N, k // 8), dtype=torch.uint8, device=DEV)
        return lambda: E.eogp_sign_pack(x, codes, scales)

    t64, t256, t1024 = times(call(64), call(256), call(1024))
    print(f"[times] pack 100,000 rows: of 64 {t64:.1f} us, of 256 {t256:.1f} us, of 1,024 {t1024:.1f} us", flush=True)
    # 410 MB are read for rows of 1,024: at 3 TB/s or better (2.2 when every row paid for eight chunks)
    assert t1024 <= 137 and t64 <= 0.8 * t1024


@pytest.mark.parametrize("m,k", [(32768, 1024), (16384, 4096)])
def test_128_rows_cost_no_more_than_129(m, k):
    """Up to 128 rows a kernel of their own may run; not where the one for more is faster."""
    Z = torch.randn((129, m), device=DEV).half()
    Pt = torch.randn((k, m), device=DEV).mul_(m ** -0.5).half()
    ws = torch.empty(E.eogp_pca_project_workspace_size(129, m, k, E.F16, E.PREC_FAST), dtype=torch.uint8, device=DEV)
    X = torch.empty((129, k), device=DEV)
    few, more = times(lambda: E.eogp_pca_project(Z[:128], Pt, X=X[:128], ws=ws),
                      lambda: E.eogp_pca_project(Z, Pt, X=X, ws=ws))
    print(f"[times] {m} -> {k}: 128 rows {few:.1f} us, 129 rows {more:.1f} us", flush=True)
    assert few <= 1.08 * more
