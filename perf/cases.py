"""The work a user has this library do, as cases that can be timed and compared.

A serving loop appends a few rows per generated token (encode + pack), encodes prompts in chunks,
reads the cache back (decode of keys with the rotary embedding, decode of values, attention of one
query position straight over the codes), and a codebook is learnt by steps of assignment and
moving-average update over all stages.  Shapes come from the repository's workloads: rows of 1024
channels (8 kv heads x 128), of 128 channels (one head), of 4096 channels (32 heads, K = 4096),
groups of 32, depth 8, K = 2048, and the ablation grid (depth 4 / 6 / 8, K = 1024 / 2048).

Inputs are synthetic in the repository's manner: Gaussian rows with log-normal channel scales; keys
carry 2 % outlier channels of 20 times the scale.  Codebooks are built here with plain torch / numpy
from rows of the same distribution (picked rows, one centroid step per stage), so that they depend
on the seed alone.
"""
import math

import numpy as np
import torch

from paper_2410_15704_amd import binding as b

DHAT = 32


def listed():
    return [
        # one generated token: its key row is quantized and packed (bench.py's append leg)
        dict(name="append_1_row", op="encode", N=1, d=1024, dtype="bf16", grouping="strided", depth=8, K=2048, pack=True),
        # one step of a batch of 48 sequences, values
        dict(name="append_48_rows", op="encode", N=48, d=1024, dtype="bf16", grouping="contiguous", depth=8, K=2048, pack=True),
        # a ragged prompt chunk, keys
        dict(name="prefill_1500_rows", op="encode", N=1500, d=1024, dtype="bf16", grouping="strided", depth=8, K=2048, pack=True),
        # a whole 32k prompt, keys: the repository's benchmark workload
        dict(name="encode_32768_rows", op="encode", N=32768, d=1024, dtype="bf16", grouping="strided", depth=8, K=2048, pack=False),
        # multi-head attention without shared kv heads: 128 groups per row, a codebook of two LDS pieces
        dict(name="encode_mha_k4096", op="encode", N=6000, d=4096, dtype="fp16", grouping="strided", depth=8, K=4096, pack=False),
        # one head per row at a smaller setting of the ablation grid: quantize, reconstruct in fp32
        dict(name="heads_depth6_round_trip", op="roundtrip", N=50001, d=128, dtype="bf16", grouping="strided", depth=6, K=1024),
        # reading a long cache back: rotated keys from int16 codes, values from packed codes
        dict(name="decode_keys_rope", op="decode", N=262144, d=1024, grouping="strided", depth=8, K=2048, form="rope"),
        dict(name="decode_values_packed", op="decode", N=262144, d=1024, grouping="contiguous", depth=8, K=2048, form="packed"),
        # reading a short cache back
        dict(name="decode_3000_rows", op="decode", N=3000, d=1024, grouping="contiguous", depth=8, K=2048, form="int16"),
        # one query position over the codes of a long and of a short context, 8 kv heads x 4 queries
        dict(name="attn_131072_tokens", op="attn", N=131072, Hkv=8, rep=4, K=2048, packed=True),
        dict(name="attn_2100_tokens", op="attn", N=2100, Hkv=8, rep=4, K=2048, packed=False),
        # one step of codebook learning over all stages
        dict(name="train_step", op="train", M=1048576, depth=8, K=2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["encode", "encode", "encode", "encode", "roundtrip", "decode", "decode", "attn", "attn", "train"])
    grouping = rng.choice(["strided", "contiguous"])
    if op == "encode":
        d = rng.choice([128, 1024, 1024, 1024, 4096])
        dtype = rng.choice(["bf16", "bf16", "fp16", "fp32"])
        K = 4096 if d == 4096 else rng.choice([1024, 2048, 2048])
        top = {128: 262144, 1024: 32768, 4096: 4096}[d]
        return dict(op=op, N=_log_int(rng, 1, top), d=d, dtype=dtype, grouping=grouping, depth=8, K=K, pack=rng.random() < 0.5)
    if op == "roundtrip":
        return dict(op=op, N=_log_int(rng, 64, 131072), d=128, dtype=rng.choice(["bf16", "fp32"]), grouping=grouping,
                    depth=rng.choice([4, 6, 8]), K=rng.choice([256, 1024, 2048]))
    if op == "decode":
        d = rng.choice([128, 1024, 1024, 4096])
        K = 4096 if d == 4096 else 2048
        form = rng.choice(["int16", "packed", "rope"])
        return dict(op=op, N=_log_int(rng, 1, 262144 * 1024 // d), d=d, grouping=grouping, depth=8, K=K, form=form)
    if op == "attn":
        return dict(op=op, N=_log_int(rng, 100, 131072), Hkv=8, rep=rng.choice([1, 4, 8]), K=2048, packed=rng.random() < 0.5)
    return dict(op=op, M=_log_int(rng, 32768, 1048576), depth=rng.choice([4, 6, 8]), K=rng.choice([1024, 2048]))


# ---- inputs ------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _scales(d, keys, g):
    """Per-channel scales: keys log-normal(0, 1) with 2 % of the channels times 20, values
    log-normal(0, 0.5)."""
    sigma = torch.exp((1.0 if keys else 0.5) * torch.randn(d, device="cuda", generator=g))
    if keys:
        sigma[torch.randperm(d, device="cuda", generator=g)[: max(1, d // 50)]] *= 20.0
    return sigma


def _groups(X, strided):
    """Rows scaled by their std and split into groups of 32: float32 [rows * G][32]."""
    Z = X.float()
    Z = Z / Z.std(dim=1, unbiased=False, keepdim=True)
    n, d = Z.shape
    G = d // DHAT
    Z = Z.view(n, DHAT, G).transpose(1, 2) if strided else Z.view(n, G, DHAT)
    return Z.reshape(n * G, DHAT).contiguous()


def _nearest(R, C):
    c2 = (C * C).sum(1)
    return torch.cat([(c2 - 2.0 * (r @ C.t())).argmin(1) for r in R.split(8192)])


def _codebooks(Z, depth, K, g):
    """Codebooks [depth][K][32]: per stage K picked rows of the residuals and one centroid step."""
    V = Z.shape[0]
    C = torch.empty((depth, K, DHAT), device="cuda")
    R = Z
    for s in range(depth):
        c = R[torch.randperm(V, device="cuda", generator=g)[:K]].clone()
        a = _nearest(R, c).cpu().numpy()
        r = R.cpu().numpy().astype(np.float64)
        cnt = np.bincount(a, minlength=K)
        tot = np.stack([np.bincount(a, weights=r[:, j], minlength=K) for j in range(DHAT)], 1)
        mean = torch.from_numpy((tot / np.maximum(cnt, 1)[:, None]).astype(np.float32)).cuda()
        c = torch.where(torch.from_numpy(cnt > 0).cuda()[:, None], mean, c)
        C[s] = c
        R = R - c[_nearest(R, c)]
    return C


def _rows(N, sigma, g, dtype):
    X = torch.empty((N, sigma.numel()), dtype=dtype, device="cuda")
    for i in range(0, N, 16384):
        n = min(16384, N - i)
        X[i:i + n] = (torch.randn((n, sigma.numel()), device="cuda", generator=g) * sigma).to(dtype)
    return X


_TORCH = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}


def _grouping(case):
    return b.STRIDED if case["grouping"] == "strided" else b.CONTIGUOUS


def prepare(case, seed):
    g = _gen(seed)
    op, depth, K = case["op"], case.get("depth", 8), case["K"]
    s = dict(case=case)
    if op in ("encode", "roundtrip"):
        # a context with codebooks learnt from other rows of the same distribution, and the new rows
        keys = case["grouping"] == "strided"
        sigma = _scales(case["d"], keys, g)
        dt = _TORCH[case["dtype"]]
        C = _codebooks(_groups(_rows(max(1, 16384 * DHAT // case["d"]), sigma, g, dt), keys), depth, K, g)
        s["q"] = b.Quantizer(d=case["d"], dhat=DHAT, depth=depth, K=K, grouping=_grouping(case),
                             in_dtype=b.DTYPES[case["dtype"]], out_dtype=b.F32 if op == "roundtrip" else b.F16)
        s["q"].set_codebooks(C)
        s["X"] = _rows(case["N"], sigma, g, dt)
    elif op == "decode":
        N, G = case["N"], case["d"] // DHAT
        shrink = 0.6 ** torch.arange(depth, device="cuda", dtype=torch.float32)
        C = torch.randn((depth, K, DHAT), device="cuda", generator=g) * shrink[:, None, None]
        s["q"] = b.Quantizer(d=case["d"], dhat=DHAT, depth=depth, K=K, grouping=_grouping(case))
        s["q"].set_codebooks(C)
        s["codes"] = torch.randint(0, K, (N, G, depth), dtype=torch.int16, device="cuda", generator=g)
        s["std"] = torch.exp(0.5 * torch.randn(N, device="cuda", generator=g)).half()
        s["out"] = torch.empty((N, case["d"]), dtype=torch.float16, device="cuda")
        if case["form"] == "packed":
            s["codes"] = s["q"].pack(s["codes"])
        elif case["form"] == "rope":
            s["cos"], s["sin"] = _rope_tables(torch.arange(N, device="cuda") % 32768)
    elif op == "attn":
        N, Hkv, Hq = case["N"], case["Hkv"], case["Hkv"] * case["rep"]
        rows = N * Hkv
        shrink = 0.6 ** torch.arange(8, device="cuda", dtype=torch.float32)
        for which, grouping in (("k", b.STRIDED), ("v", b.CONTIGUOUS)):
            q = b.Quantizer(d=128, dhat=DHAT, depth=8, K=K, grouping=grouping)
            q.set_codebooks(torch.randn((8, K, DHAT), device="cuda", generator=g) * shrink[:, None, None])
            codes = torch.randint(0, K, (rows, 4, 8), dtype=torch.int16, device="cuda", generator=g)
            s["q" + which] = q
            s["codes" + which] = q.pack(codes) if case["packed"] else codes
            s["std" + which] = (torch.rand(rows, device="cuda", generator=g) + 0.5).half()
        s["cos"], s["sin"] = _rope_tables(torch.arange(N, device="cuda"))
        s["query"] = torch.randn((Hq, 128), device="cuda", generator=g)
        s["ws_bytes"] = b.rvq_attn_workspace_bytes(N, Hq, Hkv)
        s["ws"] = torch.empty(s["ws_bytes"] // 4, device="cuda")
        s["out"] = torch.empty((Hq, 128), device="cuda")
    else:
        # per-head key rows, already scaled and grouped, and the moving averages of a running training
        M = case["M"]
        sigma = _scales(128, True, g)
        Z = _groups(_rows((M + 3) // 4 + 4096, sigma, g, torch.bfloat16), True)
        C = _codebooks(Z[:16384].contiguous(), depth, K, g)
        s["R0"] = Z[16384:16384 + M].contiguous()
        s["q"] = b.Quantizer(d=DHAT, dhat=DHAT, depth=depth, K=K, scale=0)
        s["q"].set_codebooks(C)
        s["codes"] = torch.empty((M, 1, depth), dtype=torch.int16, device="cuda")
        s["cs"] = [torch.full((K,), M / K, device="cuda") for _ in range(depth)]
        s["es"] = [C[i] * (M / K) for i in range(depth)]
    return s


def _rope_tables(pos):
    ang = pos.double()[:, None] * (10000.0 ** (-torch.arange(64, device="cuda").double() / 64.0))[None, :]
    return torch.cos(ang).float(), torch.sin(ang).float()


# ---- one pass ----------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    op = case["op"]
    if op == "encode":
        codes, std, _ = s["q"].encode(s["X"])
        if case["pack"]:
            return codes, std, s["q"].pack(codes)
        return codes, std
    if op == "roundtrip":
        codes, std, _ = s["q"].encode(s["X"])
        return codes, std, s["q"].decode(codes, std)
    if op == "decode":
        if case["form"] == "packed":
            return s["q"].decode_packed(s["codes"], s["std"], out=s["out"])
        if case["form"] == "rope":
            return s["q"].decode_rope(s["codes"], s["std"], s["cos"], s["sin"], 128, out=s["out"])
        return s["q"].decode(s["codes"], s["std"], out=s["out"])
    if op == "attn":
        b.rvq_attn_decode(s["qk"].ctx, s["qv"].ctx, s["query"], case["Hkv"] * case["rep"], case["Hkv"], s["codesk"], s["stdk"],
                          s["codesv"], s["stdv"], case["N"], s["cos"], s["sin"], 128 ** -0.5, s["out"], s["ws"], s["ws_bytes"],
                          packed=1 if case["packed"] else 0)
        return s["out"]
    # a step of train.ema_train_online: every stage assigns, passes its residual on and is updated
    q, depth, M, codes = s["q"], case["depth"], case["M"], s["codes"]
    R = s["R0"]
    for i in range(depth):
        _, _, res = q.encode(R, want_residual=True, stages=(i, i + 1), codes=codes)
        b.rvq_ema_update(q.ctx, i, R, codes.data_ptr() + 2 * i, depth, M, 0.99, 1e-5, s["cs"][i], s["es"][i])
        R = res.view(M, DHAT)
    return codes, q.get_codebooks(), s["cs"], s["es"]


def work(case):
    """Inputs and codebooks read once, outputs written once; a multiply and an add per codeword
    element and vector for the search, an add per gathered element for the decode."""
    op, depth, K = case["op"], case.get("depth", 8), case["K"]
    book = depth * K * DHAT * 4
    if op in ("encode", "roundtrip"):
        N, d = case["N"], case["d"]
        V = N * d // DHAT
        esz = 4 if case["dtype"] == "fp32" else 2
        nbytes = N * d * esz + book + V * depth * 2 + N * 2
        flops = 2 * DHAT * K * depth * V
        if op == "roundtrip":
            nbytes += N * d * 4
            flops += V * DHAT * depth
        elif case["pack"]:
            nbytes += V * _record_bytes(depth, K)
        return dict(bytes=nbytes, flops=flops)
    if op == "decode":
        N, d = case["N"], case["d"]
        V = N * d // DHAT
        per = _record_bytes(depth, K) if case["form"] == "packed" else 2 * depth
        return dict(bytes=V * per + N * 2 + N * d * 2 + book + (N * 64 * 8 if case["form"] == "rope" else 0), flops=V * DHAT * depth)
    if op == "attn":
        N, Hkv, Hq = case["N"], case["Hkv"], case["Hkv"] * case["rep"]
        per = 4 * (_record_bytes(8, K) if case["packed"] else 16) + 2
        return dict(bytes=2 * N * Hkv * per + N * 64 * 8 + 2 * book + Hq * 128 * 8, flops=N * Hkv * 128 * 16 + 4 * N * Hq * 128)
    M = case["M"]
    # R0 in, codes out; codebooks, counts and sums in and out
    return dict(bytes=M * DHAT * 4 + M * depth * 2 + 4 * book, flops=2 * DHAT * K * depth * M)


def _record_bytes(depth, K):
    return (depth * max(1, (K - 1).bit_length()) + 7) // 8


def tolerance(case):
    """About four times what the library showed against the same path in 64 bits: 2e-6 to 7e-6 of the
    codes are near-ties that fall the other way, fp16 outputs differ where a sum rounds to the other
    neighbour, sums over the codes carry fp32 rounding and the near-ties of the stages before."""
    op = case["op"]
    if op == "encode":
        return dict(rel=2e-5, max=3e-3, differ=3e-5)  # std in fp16, codes, packed bytes
    if op == "roundtrip":
        return dict(rel=2e-3, max=0.99, differ=3e-5)  # a near-tie that falls the other way reconstructs another vector
    if op == "decode":
        return dict(rel=3e-5, max=4e-3)
    if op == "attn":
        return dict(rel=2e-6, max=2e-5)
    return dict(rel=3e-5, max=2e-3, differ=3e-5)
