"""The second stage of a small batch (at most 128 rows: the kernel that streams
P past a shared Z) against 64-bit products: edges of the row tiles, column and
K remainders, every operand type, padded strides, with and without scratch."""
import pytest
import torch

from paper_2609_37842_amd import eogp as E

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# Relative row error: operands rounded once (2^-9 bf16, 2^-12 fp16, each at most
# sqrt(2) for two rounded operands, a factor 2 for the row's spread), the split
# modes' 16 bits, or only the fp32 sums.
TOL = {"exact": 4e-6, "f16": 2 * 2 ** -12, "bf16": 2 * 2 ** -8, "split": 3e-5}


@pytest.mark.parametrize("rows", [1, 16, 32, 33, 64, 65, 128, 129])
@pytest.mark.parametrize("m,k,z,p,prec,tol", [
    (512, 256, "f16", "f16", E.PREC_FAST, "exact"),
    (1032, 300, "bf16", "bf16", E.PREC_FAST, "exact"),      # K and column remainders
    (4096, 257, "f32", "f16", E.PREC_FAST, "f16"),
    (4104, 1024, "f32", "f16", E.PREC_ACCURATE, "split"),
    (2048, 130, "f32", "bf16", E.PREC_ACCURATE, "split"),
    (2056, 511, "f32", "f32", E.PREC_ACCURATE, "split"),
    (264, 64, "f32", "f32", E.PREC_FAST, "bf16"),
    (200, 40, "f32", "bf16", E.PREC_FAST, "bf16"),
])
def test_pca_few_rows(rows, m, k, z, p, prec, tol):
    print(f"[pca] rows={rows} m={m} k={k} z={z} p={p}", flush=True)
    dt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
    g = torch.Generator(device=DEV)
    g.manual_seed(rows * 1000 + m)
    # rows of Z and P inside wider buffers: what lies beyond must not matter
    Zb = torch.full((rows, m + 24), float("nan"), device=DEV, dtype=dt[z])
    Pb = torch.full((k, m + 16), float("nan"), device=DEV, dtype=dt[p])
    Zb[:, :m] = torch.randn((rows, m), device=DEV, generator=g)
    Pb[:, :m] = torch.randn((k, m), device=DEV, generator=g) * m ** -0.5
    Z, Pt = Zb[:, :m], Pb[:, :m]
    want = Z.double() @ Pt.double().t().contiguous()
    Xb = torch.full((rows, k + 5), 7.0, device=DEV)
    X = E.eogp_pca_project(Z, Pt, X=Xb[:, :k], prec=prec)
    torch.cuda.synchronize()
    err = ((X.double() - want).norm(dim=1) / want.norm(dim=1)).max().item()
    assert err <= TOL[tol], err
    assert torch.all(Xb[:, k:] == 7.0)
    if p != "f32":      # without scratch: no split of K
        L, Y = E.load(), torch.empty((rows, k), device=DEV)
        st = L.eogp_pca_project(E._ptr(Z), E._DTYPE_CODE[Z.dtype], Z.stride(0), rows, m, E._ptr(Pt),
                                E._DTYPE_CODE[Pt.dtype], Pt.stride(0), k, E._ptr(Y), k, prec, None, 0, E._stream())
        assert st == 0
        torch.cuda.synchronize()
        assert ((Y.double() - want).norm(dim=1) / want.norm(dim=1)).max().item() <= TOL[tol]
