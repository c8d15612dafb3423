"""The random second stage and the sign packing at the edges of their load paths: rows that end
inside a 16-byte piece, rows, signs and codes at any element or byte, every width of the
register transforms, chunks with one element or none."""
import numpy as np
import pytest
import torch

from oracle import eogp_oracle as O
from paper_2609_37842_amd import eogp as E
from paper_2609_37842_amd import synth as S
from tiled_helpers import tiled_from_rows

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print(msg, flush=True)


@pytest.mark.parametrize("m,k", [
    (513, 3), (1022, 1024), (1025, 1), (2047, 2046), (2049, 515), (4093, 4096), (4097, 2), (8190, 77),
    (8193, 4099), (16381, 8192), (16385, 6), (32767, 32768), (32769, 33), (65533, 65536),
    (65537, 1001),      # four chunks: the third holds one element, the fourth none
    (98307, 5),         # the last chunk holds three
])
def test_srht_edges(m, k):
    """Entries of unit variance and sums of m terms each scaled by 1/sqrt(k): fp32 butterflies over
    log2 p <= 17 levels err by at most about 17 x 6e-8 of a row's norm, so 2e-6."""
    say(f"[srht] m={m} k={k}")
    p, N = O.srht_width(m), 3
    signs, rows = S.srht_draws(11, m + k, m, p, k)
    rows[k // 2] = p if k > 2 else rows[k // 2]
    Zb = torch.from_numpy(np.random.default_rng(m).standard_normal((N, m + 5)).astype(np.float32)).to(DEV)
    sb = torch.zeros(m + 3, dtype=torch.int8, device=DEV)
    sb[3:] = torch.from_numpy(signs).to(DEV)
    rb = torch.zeros(k + 1, dtype=torch.int32, device=DEV)
    rb[1:] = torch.from_numpy(np.asarray(rows, np.int32)).to(DEV)
    Xb = torch.full((N, k + 3), 7.0, device=DEV)
    E.eogp_srht_project(Zb[:, 1:m + 1], sb[3:], rb[1:], X=Xb[:, 1:k + 1])
    torch.cuda.synchronize()
    Xg = Xb.cpu().numpy()
    assert np.all(Xg[:, 0] == 7.0) and np.all(Xg[:, k + 1:] == 7.0)
    Xg = Xg[:, 1:k + 1]
    good = np.asarray(rows) < p
    assert np.all(np.isnan(Xg[:, ~good]))
    ref = O.srht_project(Zb[:, 1:m + 1].cpu().numpy(), signs, np.where(good, rows, 0))
    rms = np.sqrt(m / k)                         # of an entry of the transform of unit-variance values
    err = np.abs(Xg[:, good] - ref[:, good]).max() / rms
    say(f"   max err {err:.2e} of the rms")
    assert err <= 1e-5                           # the largest of up to 2e5 entries, five times the rms bound


@pytest.mark.parametrize("k", [1, 3, 7, 8, 9, 253, 256, 259, 1023, 1024, 1029, 2047, 2049, 4096, 4099, 8192, 8195, 16640])
@pytest.mark.parametrize("shift", [0, 1])
def test_sign_pack_edges(k, shift):
    """Codes are exact; a scale may differ by one fp16 step (2^-10) from the rounded fp64 mean."""
    say(f"[sign_pack] k={k} shift={shift}")
    N, nb = 5, (k + 7) // 8
    X = np.random.default_rng(k).standard_normal((N, k + 3)).astype(np.float32)
    X[0, shift] = -0.0
    X[1, shift + k - 1] = 0.0
    Xd = torch.from_numpy(X).to(DEV)[:, shift:shift + k]
    codes = torch.full((N, nb + 4 + (-nb) % 4), 0xA5, dtype=torch.uint8, device=DEV)
    scales = torch.empty((N, 1), dtype=torch.int16, device=DEV)
    E.eogp_sign_pack(Xd, codes[:, shift:shift + nb], scales)
    torch.cuda.synchronize()
    x = X[:, shift:shift + k]
    got = codes.cpu().numpy()
    assert np.array_equal(got[:, shift:shift + nb], np.packbits(x >= 0, axis=1, bitorder="little"))
    assert np.all(got[:, :shift] == 0xA5) and np.all(got[:, shift + nb:] == 0xA5)
    ref = np.abs(x.astype(np.float64)).mean(1)
    assert np.all(np.abs(scales.cpu().numpy().view(np.float16)[:, 0] - ref) <= ref * 2.0 ** -10)


@pytest.mark.parametrize("k", [512, 1024, 1536, 2048, 2560, 4096, 4608, 8704])
def test_sign_pack_tiled_row_lengths(k):
    """Every number of chunks that a wave requests at once: the tiled codes and scales are the
    row-major ones, which test_sign_pack_edges checks."""
    say(f"[sign_pack_tiled] k={k}")
    N = 37
    X = torch.from_numpy(np.random.default_rng(k).standard_normal((N, k)).astype(np.float32)).to(DEV)
    rows, s0 = E.eogp_sign_pack(X)
    tiles = torch.zeros(E.tiled_store_bytes(N, [k]), dtype=torch.uint8, device=DEV)
    s1 = torch.empty((N, 1), dtype=torch.int16, device=DEV)
    E.eogp_sign_pack_tiled(X, tiles, 0, k // 512, 0, s1)
    torch.cuda.synchronize()
    assert np.array_equal(tiles.cpu().numpy(), tiled_from_rows(rows.cpu().numpy()))
    assert torch.equal(s0.view(torch.int16).view(-1), s1.view(-1))
