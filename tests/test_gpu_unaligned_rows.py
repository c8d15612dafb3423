"""Token rows that start at any fp32 element, and PCA matrices whose sizes are no
multiples of the tiles, against 64-bit products. Gaps between rows hold NaN."""
import pytest
import torch

from paper_2609_37842_amd import eogp as E

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def rows(shape, ld, off, g, scale):
    """[N, T, d] view, tokens ld apart, starting `off` elements into a buffer of NaN."""
    N, T, d = shape
    buf = torch.full((N * T * ld + off + ld,), float("nan"), device=DEV)
    x = buf[off:off + N * T * ld].view(N, T, ld)[:, :, :d]
    x.copy_(torch.randn(shape, device=DEV, generator=g) * scale)
    return x


@pytest.mark.parametrize("prec,tol", [(E.PREC_ACCURATE, 4e-5), (E.PREC_F16, 2e-3), (E.PREC_FAST, 1.2e-2)])
@pytest.mark.parametrize("d_in,d_out,ld_a,ld_g,off", [
    (769, 128, 769, 128, 0),      # unpadded odd rows
    (65, 33, 65, 35, 1),          # rows shorter than a K slice's multiple, base off by one element
    (96, 64, 97, 66, 3),          # whole K slices, odd strides
    (31, 300, 31, 301, 2),        # one ragged K slice only
])
def test_first_stage_rows_at_any_element(d_in, d_out, ld_a, ld_g, off, prec, tol):
    print(f"[rows] d={d_in}x{d_out} ld={ld_a},{ld_g} off={off} prec={prec}", flush=True)
    N, T = 5, 37
    m = min(700, d_in * d_out // 2)
    g = torch.Generator(device=DEV)
    g.manual_seed(d_in + off)
    a, ds = rows((N, T, d_in), ld_a, off, g, 1.0), rows((N, T, d_out), ld_g, off, g, 0.5)
    mask = (torch.arange(T, device=DEV)[None, :] < torch.tensor([37, 1, 20, 0, 36], device=DEV)[:, None]).to(torch.uint8)
    QA = torch.randn((d_in, d_in), device=DEV, generator=g) * d_in ** -0.5
    QS = torch.randn((d_out, d_out), device=DEV, generator=g) * d_out ** -0.5
    lam = torch.rand((d_out, d_in), device=DEV, generator=g) + 0.5
    plan = E.eogp_plan_create(lam, 0.1, m, QA, QS)
    flat, w = plan.retained()
    Z = E.eogp_rotate_retain_planned(plan, a, ds, mask, prec=prec)
    torch.cuda.synchronize()
    plan.close()
    j, k = flat.long() // d_in, flat.long() % d_in
    for i in range(N):
        on = mask[i].bool()
        S, A = ds[i][on].double() @ QS.double(), a[i][on].double() @ QA.double()
        want = (S.t().contiguous() @ A)[j, k] * w.double()
        err = (Z[i].double() - want).norm() / max(want.norm().item(), 1e-30)
        assert (err.item() <= tol) if on.any() else torch.all(Z[i] == 0)


@pytest.mark.parametrize("m,k", [(1032, 300), (264, 255), (4096, 513), (40, 24)])
@pytest.mark.parametrize("z,p,tol", [("f16", "f16", 4e-6), ("bf16", "bf16", 4e-6), ("f32", "f16", 5e-4)])
def test_pca_sizes_off_the_tiles(m, k, z, p, tol):
    """More rows than the small-batch kernel takes; K and column remainders."""
    dt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
    g = torch.Generator(device=DEV)
    g.manual_seed(m + k)
    Zb = torch.full((300, m + 8), float("nan"), device=DEV, dtype=dt[z])
    Pb = torch.full((k, m + 8), float("nan"), device=DEV, dtype=dt[p])
    Zb[:, :m] = torch.randn((300, m), device=DEV, generator=g)
    Pb[:, :m] = torch.randn((k, m), device=DEV, generator=g) * m ** -0.5
    X = E.eogp_pca_project(Zb[:, :m], Pb[:, :m], prec=E.PREC_FAST)
    torch.cuda.synchronize()
    want = Zb[:, :m].double() @ Pb[:, :m].double().t().contiguous()
    assert ((X.double() - want).norm(dim=1) / want.norm(dim=1)).max().item() <= tol
