"""The fp16 squares of the EK-FAC pass over ranges of examples: modules whose blocks end inside a
wave's 64 x 64 or a workgroup's 128 x 128, examples without tokens, ranges without examples, few
examples, and a workspace with room for the fewest ranges only."""
import pytest
import torch

from paper_2609_37842_amd import eogp as E

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inputs(N, T, d_in, d_out, long_one):
    g = torch.Generator(device=DEV)
    g.manual_seed(N + T + d_in + d_out)
    lens = torch.randint(0, max(2, T // 8) if long_one else T + 1, (N,), device=DEV, generator=g)
    lens[N // 2] = T                             # one example may hold most of the tokens
    lens[0] = 0
    lens[N - 1] = 0
    mask = (torch.arange(T, device=DEV)[None, :] < lens[:, None]).to(torch.uint8)
    a = torch.randn((N, T, d_in), device=DEV, generator=g)
    ds = torch.randn((N, T, d_out), device=DEV, generator=g)
    QA = torch.randn((d_in, d_in), device=DEV, generator=g) * d_in ** -0.5
    QS = torch.randn((d_out, d_out), device=DEV, generator=g) * d_out ** -0.5
    return a, ds, mask, QA, QS


def reference(a, ds, mask, QA, QS):
    sq = torch.zeros((ds.shape[2], a.shape[2]), device=DEV, dtype=torch.float64)
    for i in range(a.shape[0]):
        on = mask[i].bool()
        S, A = ds[i][on].double() @ QS.double(), a[i][on].double() @ QA.double()
        sq += (S.t().contiguous() @ A).square_()
    return sq


@pytest.mark.parametrize("N,T,d_in,d_out,long_one", [
    (3, 9, 32, 32, False),            # fewer examples than one range's four
    (31, 20, 65, 33, False),          # one below the range rule's 32
    (32, 17, 129, 64, False),
    (97, 40, 63, 127, True),          # ranges without examples around the long one
    (130, 24, 257, 96, False),
    (64, 16, 769, 300, True),
])
def test_squares_over_ranges(N, T, d_in, d_out, long_one):
    """Tolerance: inputs, bases and rotated tokens are each rounded to fp16 once (2^-11): 3e-3 of
    the norm bounds the squares, as for the pass as a whole."""
    print(f"[ekfac] N={N} T={T} {d_in}x{d_out}", flush=True)
    x = inputs(N, T, d_in, d_out, long_one)
    one = E.eogp_ekfac_eigenvalues(*x, prec=E.PREC_F16)
    two = E.eogp_ekfac_eigenvalues(*x, prec=E.PREC_F16)
    torch.cuda.synchronize()
    want = reference(*x)
    assert ((one.double() - want).norm() / want.norm()).item() <= 3e-3
    assert torch.equal(one, two)


def test_smaller_workspace():
    """769 x 2,304 and 64 examples prefer eight ranges; room for five is enough, less is refused."""
    N, T, d_in, d_out = 64, 12, 769, 2304
    x = inputs(N, T, d_in, d_out, False)
    size, sums = E.eogp_ekfac_workspace_size(N, T, d_in, d_out), 4 * d_in * d_out
    ws = torch.empty(size, dtype=torch.uint8, device=DEV)
    full = E.eogp_ekfac_eigenvalues(*x, prec=E.PREC_F16, ws=ws)
    few = E.eogp_ekfac_eigenvalues(*x, prec=E.PREC_F16, ws=ws[:size - 2 * sums])
    torch.cuda.synchronize()
    # the same products, summed over other ranges: fp32 sums of 64 squares
    assert ((full - few).norm() / full.norm()).item() <= 1e-6
    with pytest.raises(Exception):
        E.eogp_ekfac_eigenvalues(*x, prec=E.PREC_F16, ws=ws[:size - 4 * sums])
