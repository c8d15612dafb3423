"""The calls whose time counts: the sizes, types and options that a user of the library runs.

Each case is one pass through the public entry points of paper_2609_37842_amd.eogp. The sizes are
those of the workloads this repository names (tiny 64x64, GPT-2 small, OLMo-2 1B and 32B, and the
scoring stores), and `draw` gives odd sizes of the same ranges.

Kinds of case
  roundtrip    a small module stored and queried at once: every step of the path on small inputs
  block_store  one GPT-2 block (4 linear modules) stored: shared token list, first stage, PCA, codes
  query        query examples of one module: first stage and PCA, left unquantised
  first_stage  the first stage of one module, with its own token list
  pca          the second stage of one module from cached coordinates
  srht_store   EOGP-R: the random second stage and the codes
  ekfac        corrected eigenvalues of one module from a batch (the fitting pass)
  score        query projections against a store of packed codes, per-query top-k

Inputs follow the repository's generators: activations with log-normal channel variances,
output-gradients with a low-rank part, prefix masks of random length, log-normal corrected
eigenvalues, random codes with log-normal fp16 scales. The bases and P have independent
N(0, 1/d) entries, which is how the entries of a random orthonormal matrix of these widths are
distributed (no step of the path uses exact orthonormality).
"""
import functools
import math
import random

import numpy as np
import torch

from paper_2609_37842_amd import eogp as E

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
PRECS = {"fast": E.PREC_FAST, "accurate": E.PREC_ACCURATE, "f16": E.PREC_F16}
GPT2_BLOCK = ((769, 2304), (769, 768), (769, 3072), (3073, 768))
DAMPING = 0.1


def listed():
    return [
        # a small store-and-query roundtrip in the default precision: the latency of the whole path
        dict(name="tiny_roundtrip", kind="roundtrip", d_in=64, d_out=64, N=256, T=16, m=512, k=128,
             Q=8, topk=10),
        # the flagship store step: one GPT-2 block, 1,250 examples and 16 queries in one batch
        dict(name="gpt2_block_store", kind="block_store", N=1266, T=512, len_lo=64, m=16384,
             k=8192),
        # 16 query examples of GPT-2's widest module: few tokens, the PCA matrix read for 16 rows
        dict(name="gpt2_query", kind="query", d_in=769, d_out=3072, N=16, T=512, len_lo=64,
             m=16384, k=8192, dtype="f32", prec="f16", z="f16", pad=True),
        # the default precision on rows as a model leaves them (769 wide, no padding)
        dict(name="gpt2_accurate", kind="first_stage", d_in=769, d_out=768, N=128, T=512,
             len_lo=64, m=16384, dtype="f32", prec="accurate", z="f32", pad=False),
        # OLMo-2 1B's wide projection, bf16 inputs in the fp16 mode
        dict(name="olmo1b_up", kind="first_stage", d_in=2048, d_out=8192, N=256, T=1024, len_lo=64,
             m=32768, dtype="bf16", prec="f16", z="f16", pad=True),
        # OLMo-2 32B's attention projection, bf16 throughout, unpadded sequences
        dict(name="olmo32b_q_bf16", kind="first_stage", d_in=5120, d_out=5120, N=24, T=2048,
             len_lo=2048, m=65536, dtype="bf16", prec="fast", z="f32", pad=True),
        # OLMo-2 32B's second stage for one batch: 4.3 GB of P for 64 rows
        dict(name="olmo32b_pca", kind="pca", N=64, m=65536, k=32768, z="f16", p="f16",
             prec="fast"),
        # EOGP-R on a GPT-2 module
        dict(name="gpt2_srht_store", kind="srht_store", N=1266, m=16384, k=8192, tiled=True),
        # the EK-FAC fitting pass of a GPT-2 module
        dict(name="gpt2_ekfac", kind="ekfac", d_in=769, d_out=2304, N=256, T=512, len_lo=64,
             dtype="f32", prec="f16", pad=True),
        # serving: 16 queries over 4M stored codes, one pass of the store
        dict(name="score_16q", kind="score", N=4 * 1024 * 1024, U=1, k=16384, Q=16, topk=100,
             tiled=True, ragged=False),
        # an attribution job: 512 queries over 1M stored codes
        dict(name="score_512q", kind="score", N=1024 * 1024, U=1, k=16384, Q=512, topk=100,
             tiled=True, ragged=False),
        # the GPT-2 store: 20,000 examples, 48 modules, the 16 queries of a step
        dict(name="score_modules", kind="score", N=20000, U=48, k=8192, Q=16, topk=100, tiled=True,
             ragged=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["roundtrip", "query", "first_stage", "first_stage", "pca", "srht_store", "ekfac",
                       "score", "score", "score"])
    if kind == "roundtrip":
        d_in, d_out = _log(rng, 17, 160), _log(rng, 16, 160)
        m = min(_log(rng, 64, 2000), d_in * d_out)
        return dict(kind=kind, d_in=d_in, d_out=d_out, N=_log(rng, 8, 400), T=_log(rng, 4, 48), m=m,
                    k=64 * rng.randint(1, max(1, min(m // 64, 16))), Q=rng.randint(1, 24),
                    topk=rng.randint(1, 20))
    if kind in ("query", "first_stage", "ekfac"):
        bf16 = rng.random() < 0.4
        wide = 4096 if kind == "first_stage" else 2304
        d_in, d_out = _log(rng, 129, wide), _log(rng, 128, wide)
        if bf16:   # 16-bit rows start on 16-byte boundaries
            d_in, d_out = d_in // 8 * 8, d_out // 8 * 8
        T = _log(rng, 48, 1024)
        N = 16 if kind == "query" else _log(rng, 9, 256)
        N = min(N, max(4, 100000 // T))
        prec = rng.choice(["f16", "f16", "fast"] if bf16 else ["f16", "f16", "accurate"])
        c = dict(kind=kind, d_in=d_in, d_out=d_out, N=N, T=T, len_lo=rng.choice([1, T // 4, T]),
                 dtype="bf16" if bf16 else "f32", prec=prec, pad=bf16 or rng.random() < 0.7)
        if kind != "ekfac":
            c["m"] = min(_log(rng, 1000, 32768) // 8 * 8, d_in * d_out // 8 * 8)
            c["z"] = "f16" if kind == "query" else rng.choice(["f32", "f16"])
        if kind == "query":
            c["k"] = 8 * _log(rng, 16, max(17, c["m"] // 16))
        return c
    if kind == "pca":
        m, k = 8 * _log(rng, 100, 4096), _log(rng, 300, 16384)
        p = rng.choice(["f16", "f16", "bf16", "f32"])
        z = rng.choice(["f32", p])
        N = _log(rng, 5, 2000)
        return dict(kind=kind, N=N, m=m, k=k, z=z, p=p, prec=rng.choice(["fast", "accurate"]) if z == "f32" else "fast")
    if kind == "srht_store":
        m = _log(rng, 700, 60000)
        p = 1 << (m - 1).bit_length()
        return dict(kind=kind, N=_log(rng, 16, 1500), m=m, k=512 * rng.randint(1, max(1, p // 1024)),
                    tiled=rng.random() < 0.5)
    tiled = rng.random() < 0.6
    U = rng.choice([1, 1, _log(rng, 2, 112)])
    k = 512 * _log(rng, 1, 48) if tiled else 64 * _log(rng, 2, 256)
    N = _log(rng, 700, 2000000)
    N = max(300, min(N, int(4e9 / (U * k / 8))))
    Q = _log(rng, 1, 300)
    Q = max(1, min(Q, int(16 * 2.5e10 / (U * k / 8 * N))))
    return dict(kind="score", N=N, U=U, k=k, Q=Q, topk=_log(rng, 1, 256), tiled=tiled,
                ragged=U > 1 and rng.random() < 0.5)


# ---- inputs ------------------------------------------------------------------------------------
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + 7919 * int(stream) + 17) & 0x7FFFFFFFFFFFFFFF)
    return g


def _tokens(seed, stream, N, T, d_in, d_out, dtype, pad):
    """acts [N, T, d_in] and out_grads [N, T, d_out]; with `pad` their rows sit in a wider buffer
    whose row length is a multiple of 128 bytes."""
    el = 32 if dtype == torch.float32 else 64
    g = _gen(seed, stream)
    ld_a = -(-d_in // el) * el if pad else d_in
    ld_g = -(-d_out // el) * el if pad else d_out
    a = torch.zeros((N, T, ld_a), device=DEV, dtype=dtype)
    ds = torch.zeros((N, T, ld_g), device=DEV, dtype=dtype)
    sd = torch.empty(d_in, device=DEV).log_normal_(0.0, 1.0, generator=g).sqrt()
    step = max(1, (1 << 27) // (T * max(d_in, d_out)))
    for i in range(0, N, step):
        n = min(N, i + step) - i
        x = torch.randn((n, T, d_in), device=DEV, generator=g).mul_(sd)
        if d_in % 2:
            x[:, :, -1] = 1.0                   # an attributed bias is a constant input channel
        a[i:i + n, :, :d_in] = x
        y = torch.randn((n, T, d_out), device=DEV, generator=g).mul_(0.01)
        u = torch.randn((n, 8, d_out), device=DEV, generator=g).mul_(0.01)
        c = torch.randn((n, T, 8), device=DEV, generator=g).mul_(8 ** -0.5)
        ds[i:i + n, :, :d_out] = y.baddbmm_(c, u)
    return a[:, :, :d_in], ds[:, :, :d_out]


def _mask(seed, stream, N, T, lo):
    lens = torch.randint(lo, T + 1, (N,), device=DEV, generator=_gen(seed, stream))
    return (torch.arange(T, device=DEV)[None, :] < lens[:, None]).to(torch.uint8).contiguous()


def _basis(seed, stream, d):
    return torch.randn((d, d), device=DEV, generator=_gen(seed, stream)).mul_(d ** -0.5)


def _eigvals(seed, stream, d_out, d_in, tokens):
    g = _gen(seed, stream)
    sig = torch.empty(d_out, device=DEV).log_normal_(0.0, 1.0, generator=g)
    alp = torch.empty(d_in, device=DEV).log_normal_(0.0, 1.0, generator=g)
    xi = torch.randn((d_out, d_in), device=DEV, generator=g)
    return (sig[:, None] * alp[None, :] * torch.exp(0.25 * xi) * (1.2e-4 * tokens)).contiguous()


def _damping(tokens):
    return DAMPING * 1.2e-4 * tokens * math.exp(1.03)


def _directions(seed, stream, k, m, dtype):
    out = torch.empty((k, m), device=DEV, dtype=dtype)
    g, step = _gen(seed, stream), max(1, (1 << 28) // m)
    for i in range(0, k, step):
        n = min(k, i + step) - i
        out[i:i + n] = torch.randn((n, m), device=DEV, generator=g).mul_(m ** -0.5)
    return out


def _module(seed, stream, d_in, d_out, m, tokens):
    """What the fit of one module hands over: bases, corrected eigenvalues, damping."""
    return dict(Q_A=_basis(seed, stream, d_in), Q_S=_basis(seed, stream + 1, d_out),
                lam=_eigvals(seed, stream + 2, d_out, d_in, tokens), damping=_damping(tokens), m=m)


def _plan(f):
    return E.eogp_plan_create(f["lam"], f["damping"], f["m"], f["Q_A"], f["Q_S"])


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device=DEV)


def _module_bits(c):
    """Bits of each module of a scoring case; ragged ones differ from module to module."""
    unit = 512 if c["tiled"] else 64
    if not c["ragged"]:
        return [c["k"]] * c["U"]
    return [max(unit, c["k"] - unit * ((3 * u) % 5)) for u in range(c["U"])]


def _raw(c, seed):
    """The inputs of a case as plain tensors."""
    kind, r = c["kind"], {}
    if kind == "roundtrip":
        r["fit"] = _module(seed, 1, c["d_in"], c["d_out"], c["m"], c["T"])
        r["a"], r["ds"] = _tokens(seed, 10, c["N"], c["T"], c["d_in"], c["d_out"], torch.float32, False)
        r["qa"], r["qds"] = _tokens(seed, 11, c["Q"], c["T"], c["d_in"], c["d_out"], torch.float32, False)
        r["mask"] = _mask(seed, 12, c["N"], c["T"], max(1, c["T"] // 2))
        r["Pt"] = _directions(seed, 13, c["k"], c["m"], torch.float32)
    elif kind == "block_store":
        mean = 0.5 * (c["len_lo"] + c["T"])
        r["mask"] = _mask(seed, 12, c["N"], c["T"], c["len_lo"])
        r["mods"] = []
        for i, (d_in, d_out) in enumerate(GPT2_BLOCK):
            a, ds = _tokens(seed, 100 + i, c["N"], c["T"], d_in, d_out, torch.float32, True)
            r["mods"].append(dict(fit=_module(seed, 200 + 8 * i, d_in, d_out, c["m"], mean), a=a, ds=ds,
                                  Pt=_directions(seed, 300 + i, c["k"], c["m"], torch.float16)))
    elif kind in ("query", "first_stage", "ekfac"):
        mean = 0.5 * (c["len_lo"] + c["T"])
        r["a"], r["ds"] = _tokens(seed, 10, c["N"], c["T"], c["d_in"], c["d_out"], DTYPES[c["dtype"]],
                                  c["pad"])
        r["mask"] = _mask(seed, 12, c["N"], c["T"], c["len_lo"]) if c["len_lo"] < c["T"] else None
        r["fit"] = _module(seed, 1, c["d_in"], c["d_out"], c.get("m", 1), mean)
        if kind == "query":
            r["Pt"] = _directions(seed, 13, c["k"], c["m"], torch.float16)
    elif kind == "pca":
        r["Z"] = torch.randn((c["N"], c["m"]), device=DEV, generator=_gen(seed, 1)).to(DTYPES[c["z"]])
        r["Pt"] = _directions(seed, 2, c["k"], c["m"], DTYPES[c["p"]])
    elif kind == "srht_store":
        p = 1 << (c["m"] - 1).bit_length()
        r["Z"] = torch.randn((c["N"], c["m"]), device=DEV, generator=_gen(seed, 1))
        r["signs"] = (torch.randint(0, 2, (c["m"],), device=DEV, generator=_gen(seed, 2)) * 2 - 1).to(torch.int8)
        r["rows"] = torch.randperm(p, device=DEV, generator=_gen(seed, 3))[:c["k"]].to(torch.int32)
    else:
        ks = _module_bits(c)
        shape = (E.tiled_store_bytes(c["N"], ks),) if c["tiled"] else (c["N"], sum(ks) // 8)
        n = math.prod(shape)
        words = torch.randint(-(1 << 62), 1 << 62, (-(-n // 7),), device=DEV, generator=_gen(seed, 1))
        r["codes"] = words.view(torch.uint8).view(-1, 8)[:, :7].reshape(-1)[:n].reshape(shape).contiguous()
        r["scales"] = torch.randn((c["N"], c["U"]), device=DEV, generator=_gen(seed, 2)).exp_().half()
        r["Y"] = torch.randn((c["Q"], sum(ks)), device=DEV, generator=_gen(seed, 3))
        r["ks"] = ks
    return r


def prepare(c, seed):
    kind, s = c["kind"], _raw(c, seed)
    s["case"] = dict(c)
    if kind == "roundtrip":
        s["plan"] = _plan(s["fit"])
        n = max(E.eogp_rotate_retain_workspace_size(s["plan"], max(c["N"], c["Q"]), c["T"]),
                E.eogp_pca_project_workspace_size(max(c["N"], c["Q"]), c["m"], c["k"], E.F32, E.PREC_ACCURATE),
                E.eogp_score_topk_workspace_size(c["N"], c["Q"], [c["k"]], c["topk"]))
        s["ws"] = _bytes(n)
    elif kind == "block_store":
        N, T, m, k = c["N"], c["T"], c["m"], c["k"]
        n = E.eogp_pca_project_workspace_size(N, m, k, E.F16, E.PREC_FAST)
        for md in s["mods"]:
            md["plan"] = _plan(md.pop("fit"))
            n = max(n, E.eogp_rotate_retain_workspace_size(md["plan"], N, T))
        s["ws"], s["ws_pca"] = _bytes(n), _bytes(n)
        s["Z"] = [torch.empty((N, m), device=DEV, dtype=torch.float16) for _ in s["mods"]]
        s["X"] = torch.empty((N, len(s["mods"]) * k), device=DEV)
        s["codes"] = torch.zeros(E.tiled_store_bytes(N, [k] * len(s["mods"])), device=DEV, dtype=torch.uint8)
        s["scales"] = torch.empty((N, len(s["mods"])), device=DEV, dtype=torch.int16)
    elif kind in ("query", "first_stage"):
        N, T = c["N"], c["T"]
        s["plan"] = _plan(s.pop("fit"))
        s["Z"] = torch.empty((N, c["m"]), device=DEV, dtype=DTYPES[c["z"]])
        s["ws"] = _bytes(E.eogp_rotate_retain_workspace_size(s["plan"], N, T))
        if kind == "query":
            s["ws_pca"] = _bytes(E.eogp_pca_project_workspace_size(N, c["m"], c["k"], E.F16, E.PREC_FAST))
            s["X"] = torch.empty((N, c["k"]), device=DEV)
    elif kind == "ekfac":
        s["ws"] = _bytes(E.eogp_ekfac_workspace_size(c["N"], c["T"], c["d_in"], c["d_out"]))
        s["sq"] = torch.empty((c["d_out"], c["d_in"]), device=DEV)
    elif kind == "pca":
        s["ws"] = _bytes(E.eogp_pca_project_workspace_size(c["N"], c["m"], c["k"], E._DTYPE_CODE[s["Pt"].dtype],
                                                           PRECS[c["prec"]]))
        s["X"] = torch.empty((c["N"], c["k"]), device=DEV)
    elif kind == "srht_store":
        s["X"] = torch.empty((c["N"], c["k"]), device=DEV)
        s["ws"] = _bytes(E.eogp_srht_project_workspace_size(c["N"], c["m"]))
        n = E.tiled_store_bytes(c["N"], [c["k"]])
        s["codes"] = torch.zeros(n, device=DEV, dtype=torch.uint8) if c["tiled"] else \
            torch.empty((c["N"], c["k"] // 8), device=DEV, dtype=torch.uint8)
        s["scales"] = torch.empty((c["N"], 1), device=DEV, dtype=torch.int16)
    else:
        s["ws"] = _bytes(E.eogp_score_topk_workspace_size(c["N"], c["Q"], s["ks"], c["topk"]))
        s["idx"] = torch.empty((c["Q"], c["topk"]), device=DEV, dtype=torch.int64)
        s["top"] = torch.empty((c["Q"], c["topk"]), device=DEV)
    return s


# ---- one pass ----------------------------------------------------------------------------------
def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "roundtrip":
        Z = E.eogp_rotate_retain_planned(s["plan"], s["a"], s["ds"], s["mask"], ws=s["ws"])
        X = E.eogp_pca_project(Z, s["Pt"], prec=E.PREC_ACCURATE, ws=s["ws"])
        codes, scales = E.eogp_sign_pack(X)
        Zq = E.eogp_rotate_retain_planned(s["plan"], s["qa"], s["qds"], ws=s["ws"])
        Y = E.eogp_pca_project(Zq, s["Pt"], prec=E.PREC_ACCURATE, ws=s["ws"])
        idx, top, _ = E.eogp_score_topk(codes, scales, [c["k"]], Y, c["topk"], ws=s["ws"])
        return dict(Z=Z, X=X, codes=codes, scales=scales.view(torch.float16), Y=Y, top=top)
    if kind == "block_store":
        N, T, k, prec = c["N"], c["T"], c["k"], E.PREC_F16
        E.eogp_compact_tokens(s["mask"], N, T, prec, s["ws"])
        steps = k // 512
        for u, md in enumerate(s["mods"]):
            Z, X = s["Z"][u], s["X"][:, u * k:(u + 1) * k]
            E.eogp_rotate_retain_compacted(md["plan"], md["a"], md["ds"], s["ws"], Z=Z, prec=prec)
            E.eogp_pca_project(Z, md["Pt"], X=X, ws=s["ws_pca"])
            E.eogp_sign_pack_tiled(X, s["codes"], 0, steps * len(s["mods"]), steps * u, s["scales"][:, u:u + 1])
        return dict(Z=s["Z"], X=s["X"], codes=s["codes"], scales=s["scales"].view(torch.float16))
    if kind in ("query", "first_stage"):
        E.eogp_rotate_retain_planned(s["plan"], s["a"], s["ds"], s["mask"], Z=s["Z"], prec=PRECS[c["prec"]], ws=s["ws"])
        if kind == "first_stage":
            return dict(Z=s["Z"])
        E.eogp_pca_project(s["Z"], s["Pt"], X=s["X"], ws=s["ws_pca"])
        return dict(Z=s["Z"], X=s["X"])
    if kind == "ekfac":
        E.eogp_ekfac_eigenvalues(s["a"], s["ds"], s["mask"], s["fit"]["Q_A"], s["fit"]["Q_S"], sq_sum=s["sq"],
                                 prec=PRECS[c["prec"]], ws=s["ws"])
        return dict(sq=s["sq"])
    if kind == "pca":
        E.eogp_pca_project(s["Z"], s["Pt"], X=s["X"], prec=PRECS[c["prec"]], ws=s["ws"])
        return dict(X=s["X"])
    if kind == "srht_store":
        E.eogp_srht_project(s["Z"], s["signs"], s["rows"], X=s["X"], ws=s["ws"])
        if c["tiled"]:
            E.eogp_sign_pack_tiled(s["X"], s["codes"], 0, c["k"] // 512, 0, s["scales"])
        else:
            E.eogp_sign_pack(s["X"], s["codes"], s["scales"])
        return dict(X=s["X"], codes=s["codes"], scales=s["scales"].view(torch.float16))
    if c["tiled"]:
        E.eogp_score_topk_tiled(s["codes"], s["scales"], c["N"], s["ks"], s["Y"], c["topk"], out_idx=s["idx"],
                                out_score=s["top"], ws=s["ws"])
    else:
        E.eogp_score_topk(s["codes"], s["scales"], s["ks"], s["Y"], c["topk"], out_idx=s["idx"],
                          out_score=s["top"], ws=s["ws"])
    return dict(idx=s["idx"], top=s["top"])


# ---- what a pass cannot do without -------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _axes(d_out, d_in, m):
    """|J| and |K|: rows and columns that the m largest corrected eigenvalues touch (one sample)."""
    g = np.random.default_rng([d_out, d_in, m])
    lam = (g.lognormal(0, 1, (d_out, 1)) * g.lognormal(0, 1, (1, d_in))
           * np.exp(0.25 * g.standard_normal((d_out, d_in), dtype=np.float32))).reshape(-1)
    at = np.argpartition(-lam, m - 1)[:m] if m < lam.size else np.arange(lam.size)
    return len(np.unique(at // d_in)), len(np.unique(at % d_in))


def _first_stage_work(N, T, len_lo, d_in, d_out, m, el, zel):
    tok = N * 0.5 * (len_lo + T)
    J, K = _axes(d_out, d_in, m)
    return (tok * (d_in + d_out) * el + 4 * (d_out * J + d_in * K) + N * m * zel,
            2 * tok * (d_out * J + d_in * K) + 2 * tok * m)


SIZE = {"f32": 4, "bf16": 2, "f16": 2}


def work(c):
    kind = c["kind"]
    if kind == "roundtrip":
        N = c["N"] + c["Q"]
        b, f = _first_stage_work(N, c["T"], c["T"] // 2, c["d_in"], c["d_out"], c["m"], 4, 4)
        return dict(bytes=b + 4 * c["m"] * c["k"] + N * c["k"] * 4 + c["N"] * c["k"] / 8,
                    flops=f + 2 * N * c["m"] * c["k"] + 2 * c["Q"] * c["N"] * c["k"])
    if kind == "block_store":
        b = f = 0.0
        for d_in, d_out in GPT2_BLOCK:
            bb, ff = _first_stage_work(c["N"], c["T"], c["len_lo"], d_in, d_out, c["m"], 4, 2)
            b += bb + c["m"] * c["k"] * 2 + c["N"] * c["k"] * (4 + 1 / 8)
            f += ff + 2 * c["N"] * c["m"] * c["k"]
        return dict(bytes=b, flops=f)
    if kind in ("query", "first_stage"):
        b, f = _first_stage_work(c["N"], c["T"], c["len_lo"], c["d_in"], c["d_out"], c["m"],
                                 SIZE[c["dtype"]], SIZE[c["z"]])
        if kind == "query":
            b += 2 * c["m"] * c["k"] + 4 * c["N"] * c["k"]
            f += 2 * c["N"] * c["m"] * c["k"]
        return dict(bytes=b, flops=f)
    if kind == "ekfac":
        tok = c["N"] * 0.5 * (c["len_lo"] + c["T"])
        i, o = c["d_in"], c["d_out"]
        return dict(bytes=tok * (i + o) * SIZE[c["dtype"]] + 4 * (i * i + o * o + i * o),
                    flops=2 * tok * (i * i + o * o + i * o))
    if kind == "pca":
        return dict(bytes=c["N"] * c["m"] * SIZE[c["z"]] + c["m"] * c["k"] * SIZE[c["p"]] + 4 * c["N"] * c["k"],
                    flops=2 * c["N"] * c["m"] * c["k"])
    if kind == "srht_store":
        p = 1 << (c["m"] - 1).bit_length()
        return dict(bytes=c["N"] * (4 * c["m"] + 4 * c["k"] + c["k"] / 8 + 2),
                    flops=c["N"] * p * math.log2(p))
    bits = sum(_module_bits(c))
    return dict(bytes=c["N"] * (bits / 8 + 2 * c["U"]) + 4 * c["Q"] * bits + 12 * c["Q"] * c["topk"],
                flops=2 * c["Q"] * c["N"] * bits)


def tolerance(c):
    """About four times the error that each path showed against `exact`. In the 16-bit modes inputs,
    bases and rotated tokens are each rounded once (fp16 5.5e-4 of a row of Z, bf16 3.3e-3; the EK-FAC
    sums average over examples: fp16 1.5e-4); an fp16 Z is rounded once more (2e-4). The PCA rounds
    neither a 16-bit Z nor a 16-bit P (1e-6, the fp32 sums). A code byte may differ where one of its 8
    coordinates lies within the error of zero (the share that differs per bit is the error times
    sqrt(2/pi) / 2), and a scale by one fp16 step where the mean lies at a rounding boundary. Scores
    are exact integers, scaled and summed in 64 bits in a stated order."""
    kind, prec = c["kind"], c.get("prec")
    if kind == "score":
        return "exact"
    if kind == "srht_store":                     # 1.1e-7, the fp32 sums
        return dict(rel=1e-5, max=2e-3, differ=1e-4)
    if kind == "roundtrip":                      # 7.6e-6
        return dict(rel=2e-4, max=2e-3, differ=2e-3)
    if kind == "block_store":
        return dict(rel=2.2e-3, max=0.05, differ=8e-3)
    if kind == "pca":
        if c["z"] == c["p"] and c["p"] != "f32":
            return dict(rel=5e-6, max=1e-4)
        if prec == "accurate":
            return dict(rel=4e-5, max=1e-3)
        return dict(rel=1.2e-3, max=0.02) if c["p"] == "f16" else dict(rel=1.3e-2, max=0.2)
    if kind == "ekfac":
        rel = {"accurate": 5e-5, "f16": 6e-4, "fast": 6e-3}[prec]
        return dict(rel=rel, max=50 * rel)
    rel = {"accurate": 1e-3 if c["z"] == "f16" else 3e-5, "f16": 2.2e-3, "fast": 1.4e-2}[prec]
    return dict(rel=rel, max=25 * rel)


# ---- the same in 64 bits, by plain torch -------------------------------------------------------
def _exact_first_stage(fit, a, ds, mask):
    lam, d_in = fit["lam"], a.shape[2]
    order = torch.sort(lam.reshape(-1), descending=True, stable=True).indices[:fit["m"]]
    jr, kr = order // d_in, order % d_in
    J, jp = torch.unique(jr, return_inverse=True)
    K, kp = torch.unique(kr, return_inverse=True)
    w = (lam.reshape(-1)[order].double() + fit["damping"]).rsqrt()
    QS, QA = fit["Q_S"][:, J].double(), fit["Q_A"][:, K].double()
    out = torch.empty((a.shape[0], fit["m"]), device=DEV, dtype=torch.float64)
    for i in range(a.shape[0]):
        on = mask[i].bool() if mask is not None else slice(None)
        S, A = ds[i][on].double() @ QS, a[i][on].double() @ QA
        out[i] = (S.t().contiguous() @ A)[jp, kp] * w
    return out


def _pow2(e):
    """2^e in 64 bits, exactly (a power function may be an ulp off, which moves ties)."""
    return ((e.long() + 1023) << 52).view(torch.float64)


def _exact_scores(r, c, q0, q1):
    """Top scores of queries q0..q1: the query in 15-bit fixed point per module, as the library
    states it; integers below 2^53, so 64-bit floating arithmetic is exact."""
    ks, N = r["ks"], c["N"]
    Yi, f, lo = [], [], 0
    for k in ks:
        y = r["Y"][q0:q1, lo:lo + k].double()
        e = torch.frexp(y.abs().amax(1)).exponent
        f.append(14 - e)
        Yi.append(torch.round(y * _pow2(14 - e)[:, None]))
        lo += k
    top = torch.full((q1 - q0, c["topk"]), -math.inf, device=DEV, dtype=torch.float64)
    idx = torch.full((q1 - q0, c["topk"]), -1, device=DEV, dtype=torch.int64)
    shifts = torch.arange(8, device=DEV, dtype=torch.uint8)
    steps, step = sum(ks) // 512, max(32, (1 << 26) // sum(ks) // 32 * 32)
    for i in range(0, N, step):
        n = min(N, i + step) - i
        if c["tiled"]:   # blocks of 32 rows x 64 bytes; 16-byte piece p of a row at (p % 2, p // 2)
            t = -(-n // 32)
            b = r["codes"][i // 32 * steps * 2048:][:t * steps * 2048].view(t, steps, 2, 2, 32, 16)
            b = b.permute(0, 4, 1, 3, 2, 5).reshape(t * 32, steps * 64)[:n]
        else:
            b = r["codes"][i:i + n]
        sc, lo = torch.zeros((q1 - q0, n), device=DEV, dtype=torch.float64), 0
        for u, k in enumerate(ks):
            bits = (b[:, lo // 8:(lo + k) // 8, None] >> shifts & 1).reshape(n, k).double()
            dot = Yi[u] @ (2 * bits - 1).t().contiguous()
            sc += dot * r["scales"][i:i + n, u].double() * _pow2(-f[u])[:, None]
            lo += k
        both = torch.cat([top, sc], 1)
        ids = torch.cat([idx, torch.arange(i, i + n, device=DEV).expand(q1 - q0, n)], 1)
        top, at = torch.topk(both, c["topk"], dim=1)
        idx = torch.gather(ids, 1, at)
    return top


def exact(c, seed):
    kind = c["kind"]
    if kind == "score" and c["N"] * sum(_module_bits(c)) > 1.8e10:
        return None                              # expanding the bits would take too long
    r = _raw(c, seed)
    if kind == "roundtrip":
        Z = _exact_first_stage(r["fit"], r["a"], r["ds"], r["mask"])
        Zq = _exact_first_stage(r["fit"], r["qa"], r["qds"], None)
        P = r["Pt"].double().t().contiguous()
        X = Z @ P
        return dict(Z=Z, X=X, codes=None, scales=X.abs().mean(1, keepdim=True), Y=Zq @ P, top=None)
    if kind == "block_store":
        Zs, Xs, sc = [], [], []
        for md in r["mods"]:
            Z = _exact_first_stage(md["fit"], md["a"], md["ds"], r["mask"])
            X = Z @ md["Pt"].double().t().contiguous()
            Zs.append(Z)
            Xs.append(X)
            sc.append(X.abs().mean(1))
        return dict(Z=Zs, X=torch.cat(Xs, 1), codes=None, scales=torch.stack(sc, 1))
    if kind in ("query", "first_stage"):
        Z = _exact_first_stage(r["fit"], r["a"], r["ds"], r["mask"])
        if kind == "first_stage":
            return dict(Z=Z)
        return dict(Z=Z, X=Z @ r["Pt"].double().t().contiguous())
    if kind == "ekfac":
        QA, QS = r["fit"]["Q_A"].double(), r["fit"]["Q_S"].double()
        sq = torch.zeros((c["d_out"], c["d_in"]), device=DEV, dtype=torch.float64)
        for i in range(c["N"]):
            on = r["mask"][i].bool() if r["mask"] is not None else slice(None)
            S, A = r["ds"][i][on].double() @ QS, r["a"][i][on].double() @ QA
            sq += (S.t().contiguous() @ A).square_()
        return dict(sq=sq)
    if kind == "pca":
        X = torch.empty((c["N"], c["k"]), device=DEV, dtype=torch.float64)
        Z, step = r["Z"].double(), max(1, (1 << 28) // c["m"])
        for i in range(0, c["k"], step):
            X[:, i:i + step] = Z @ r["Pt"][i:i + step].double().t().contiguous()
        return dict(X=X)
    if kind == "srht_store":
        p = 1 << (c["m"] - 1).bit_length()
        v = torch.zeros((c["N"], p), device=DEV, dtype=torch.float64)
        v[:, :c["m"]] = r["Z"].double() * r["signs"].double()
        h = 1
        while h < p:                             # Walsh-Hadamard in Sylvester order
            v = v.view(c["N"], p // (2 * h), 2, h)
            v = torch.stack([v[:, :, 0] + v[:, :, 1], v[:, :, 0] - v[:, :, 1]], 2)
            h *= 2
        X = v.reshape(c["N"], p)[:, r["rows"].long()] * c["k"] ** -0.5
        return dict(X=X, codes=None, scales=X.abs().mean(1, keepdim=True))
    n = max(1, (1 << 29) // c["N"])
    top = torch.cat([_exact_scores(r, c, q, min(c["Q"], q + n)) for q in range(0, c["Q"], n)])
    return dict(idx=None, top=top)
