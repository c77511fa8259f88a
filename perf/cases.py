"""Performance cases of the codec: encode, random-access decode and fused attention.

The shapes are those of the workloads (`paper_2605_11478_amd/workloads.py`:
GPT-2-small, TinyLlama-1.1B, the 32k-context cache, the d = 128 stress cache
and the fp32 toy) and of the paper's rate axis (`bench.py --rate-axis`); the
input law is theirs too: per-channel log-normal scales with two outlier
channels per head.  The shared codebook of a code (d, k, N) is built once per
process, as a program that loads its codebook file would have it; the cache,
the queries, the token ids and the rotation come from the seed.
"""
import functools
import math

import numpy as np
import torch

import paper_2605_11478_amd as fq

DTYPES = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
DEVICE = "cuda"


def listed():
    return [
        # One decode step of one TinyLlama layer at batch 8: the new token's K
        # and V rows (8 x 4 heads) are encoded, one call each.  The smallest
        # calls there are.
        {"name": "append_tinyllama", "op": "append", "d": 64, "k": 4, "N": 256, "dtype": "bf16",
         "rows": 32, "heads": 4, "fused_kv": False},
        # Prefill of GPT-2-small: the K cache of 12 layers x 12 heads x 1024
        # tokens at 2 bits per coordinate.
        {"name": "encode_gpt2", "op": "encode", "d": 64, "k": 4, "N": 256, "dtype": "fp16",
         "rows": 147456, "heads": 144, "fused_kv": False},
        # Prefill of TinyLlama at 3 bits: 22 layers x batch 8 x 4 heads x 2048.
        {"name": "encode_tinyllama_k2", "op": "encode", "d": 64, "k": 2, "N": 64,
         "dtype": "bf16", "rows": 1441792, "heads": 88, "fused_kv": False},
        # The 32k-context cache at half a bit (the benchmark's encode):
        # 22 layers x batch 4 x 4 heads x 32768.
        {"name": "encode_long32k", "op": "encode", "d": 64, "k": 8, "N": 16, "dtype": "bf16",
         "rows": 11534336, "heads": 88, "fused_kv": False},
        # One layer of the stress cache: 8 heads x 131072 tokens, d = 128,
        # 3 bits with the large codebook.
        {"name": "encode_stress", "op": "encode", "d": 128, "k": 4, "N": 4096, "dtype": "bf16",
         "rows": 1048576, "heads": 8, "fused_kv": False},
        # A point of the rate axis off the tuned codes: 1.25 bits, k = 8, on
        # the GPT-2-shaped cache.
        {"name": "encode_rate_k8n1024", "op": "encode", "d": 64, "k": 8, "N": 1024,
         "dtype": "fp16", "rows": 147456, "heads": 144, "fused_kv": False},
        # fp32 rows, ragged count, taken out of a fused K|V projection (row
        # stride 2 d): the toy code.
        {"name": "encode_fp32_strided", "op": "encode", "d": 64, "k": 2, "N": 16,
         "dtype": "fp32", "rows": 4095, "heads": 1, "fused_kv": True},
        # Random access into the 32k cache: 65536 token ids (the benchmark's
        # decode).
        {"name": "decode_ids_long32k", "op": "decode", "d": 64, "k": 8, "N": 16, "dtype": "bf16",
         "rows": 65536, "cache": 2097152, "ids": True},
        # The whole GPT-2 cache back to fp32 rows.
        {"name": "decode_all_gpt2", "op": "decode", "d": 64, "k": 4, "N": 256, "dtype": "fp16",
         "rows": 147456, "cache": 147456, "ids": False},
        # Decode attention of one TinyLlama layer in a serving loop (kept
        # workspace): batch 8 x 4 KV heads, 8 query heads each, a cache filled
        # to an odd length.
        {"name": "attn_layer_tinyllama", "op": "attn", "d": 64, "k": 4, "N": 256,
         "dtype": "bf16", "groups": 32, "G": 8, "T": 1999, "T_stride": 2048,
         "keep_workspace": True},
        # Decode attention over the whole 32k cache (the benchmark's attention).
        {"name": "attn_long32k", "op": "attn", "d": 64, "k": 8, "N": 16, "dtype": "bf16",
         "groups": 352, "G": 8, "T": 32768, "T_stride": 32768, "keep_workspace": True},
        # One layer of the stress cache: few groups, the longest context,
        # d = 128, the call as the README writes it (no workspace passed).
        {"name": "attn_stress", "op": "attn", "d": 128, "k": 4, "N": 4096, "dtype": "bf16",
         "groups": 8, "G": 4, "T": 131072, "T_stride": 131072, "keep_workspace": False},
    ]


# (d, k, N): the workloads' codes, the rate axis and d = 128 codes of the tests,
# with the most rows that one encode of them is given.
CODES = [
    (64, 2, 16, 1 << 20), (64, 2, 64, 2 << 20), (64, 4, 256, 2 << 20), (64, 8, 16, 11534336),
    (64, 8, 64, 4 << 20), (64, 1, 16, 1 << 20), (64, 8, 256, 300000), (64, 8, 1024, 300000),
    (64, 8, 4096, 147456), (64, 16, 4096, 147456), (64, 32, 16384, 32768),
    (128, 4, 4096, 1 << 20), (128, 4, 256, 262144), (128, 8, 256, 131072),
]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    d, k, N, most = rng.choice(CODES)
    dtype = rng.choice(["bf16", "bf16", "fp16", "fp16", "fp32"])
    case = {"op": rng.choice(["append", "encode", "encode", "decode", "attn", "attn"]), "d": d, "k": k,
            "N": N, "dtype": dtype}
    if case["op"] in ("append", "encode"):
        lo, hi = (1, 1024) if case["op"] == "append" else (1024, most)
        if dtype == "fp32":
            hi = min(hi, 1 << 20)
        case.update(rows=_log(rng, lo, hi), heads=rng.choice([1, 4, 8, 12]),
                    fused_kv=rng.random() < 0.25)
    elif case["op"] == "decode":
        cache = _log(rng, 1024, min(most, 1 << 20))
        ids = rng.random() < 0.5
        case.update(rows=_log(rng, 1, 1 << 18) if ids else cache, cache=cache, ids=ids)
    else:
        groups = _log(rng, 1, 512)
        longest = min(131072, max(64, min(most, 4 << 20) // groups))
        T = _log(rng, 64, longest)
        case.update(groups=groups, G=rng.choice([1, 4, 8]), T=T,
                    T_stride=T + rng.choice([0, 1, 49]), keep_workspace=rng.random() < 0.5)
    return case


# ------------------------------------------------------------------ inputs --
@functools.lru_cache(maxsize=None)
def _codebook(d, k, N):
    if k >= 32:  # large blocks: sampled blocks of unit vectors (a Lloyd build takes minutes)
        g = np.random.default_rng(1000 * k + N)
        x = g.standard_normal((N, d))
        c = x[:, :k] / np.linalg.norm(x, axis=1, keepdims=True)
        return torch.from_numpy(c.astype(np.float16).astype(np.float32)).to(DEVICE)
    iters = 8 if N <= 256 else 4
    C, _ = fq.build_codebook(d, k, N, 1, M=max(20000, 4 * N), restarts=1, iters=iters)
    return torch.from_numpy(C).to(DEVICE)


def _rotation(d, seed):
    return torch.from_numpy(fq.build_rotation(d, seed + 2)).to(DEVICE)


def _rows(gen, n, d, heads, dtype, fused_kv=False):
    """n cache rows of `heads` heads' channel laws, head-major; fused_kv: a view of rows 2 d wide."""
    heads = min(heads, n)
    sigma = torch.exp(0.5 * torch.randn(heads, d, generator=gen, device=DEVICE))
    loud = torch.rand(heads, d, generator=gen, device=DEVICE).argsort(1)[:, :2]
    sigma.scatter_(1, loud, 10.0 * sigma.gather(1, loud))
    out = torch.empty(n, 2 * d if fused_kv else d, dtype=DTYPES[dtype], device=DEVICE)[:, :d]
    for h in range(heads):
        a, b = n * h // heads, n * (h + 1) // heads
        out[a:b] = torch.randn(b - a, d, generator=gen, device=DEVICE) * sigma[h]
    return out


def prepare(case, seed):
    d, k, N, op = case["d"], case["k"], case["N"], case["op"]
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    s = {"case": case, "C": _codebook(d, k, N), "R": _rotation(d, seed)}
    if op in ("append", "encode"):
        s["x"] = [_rows(gen, case["rows"], d, case["heads"], case["dtype"], case["fused_kv"])
                  for _ in range(2 if op == "append" else 1)]
    elif op == "decode":
        x = _rows(gen, case["cache"], d, 8, case["dtype"])
        s["payload"], s["norms"] = fq.encode(x, k, N, s["R"], s["C"])
        s["ids"] = (torch.randint(0, case["cache"], (case["rows"],), generator=gen, device=DEVICE)
                    if case["ids"] else None)
    else:
        groups, Ts = case["groups"], case["T_stride"]
        s["kv"] = []
        for _ in range(2):
            x = _rows(gen, groups * Ts, d, min(groups, 88), case["dtype"])
            payload, norms = fq.encode(x, k, N, s["R"], s["C"])
            s["kv"] += [payload.view(groups, Ts, -1), norms.view(groups, Ts)]
        s["q"] = torch.randn(groups, case["G"], d, generator=gen,
                             device=DEVICE).to(DTYPES[case["dtype"]])
        s["workspace"] = None
        if case["keep_workspace"]:
            need = fq.attn_workspace_bytes(groups, case["G"], case["T"], d, k, N)
            s["workspace"] = torch.zeros(max(need, 1), dtype=torch.uint8, device=DEVICE)
    return s


def run(s):
    case = s["case"]
    d, k, N, R, C = case["d"], case["k"], case["N"], s["R"], s["C"]
    if case["op"] in ("append", "encode"):
        return [fq.encode(x, k, N, R, C) for x in s["x"]]
    if case["op"] == "decode":
        return fq.decode(s["payload"], s["norms"], d, k, N, R, C, token_ids=s["ids"])
    kp, kn, vp, vn = s["kv"]
    return fq.attn_decode(s["q"], kp, kn, vp, vn, case["T"], k, N, R, C, workspace=s["workspace"])


# ------------------------------------------------------------------ figures --
def _payload(d, k, N):
    return (d // k * int(math.log2(N)) + 7) // 8


def work(case):
    """Each input read once and each output written once; the products of the
    rotation, of the search as its definition states it (all N codewords of
    every block) and of attention."""
    d, k, N, op = case["d"], case["k"], case["N"], case["op"]
    P, es = _payload(d, k, N), 4 if case["dtype"] == "fp32" else 2
    tables = 4 * (d * d + N * k)
    if op in ("append", "encode"):
        calls = 2 if op == "append" else 1
        return {"bytes": calls * (case["rows"] * (d * es + P + 2) + tables),
                "flops": calls * case["rows"] * (2 * d * d + 2 * d * N)}
    if op == "decode":
        per = P + 2 + 4 * d + (8 if case["ids"] else 0)
        return {"bytes": case["rows"] * per + tables, "flops": case["rows"] * 2 * d * d}
    tokens, heads = case["groups"] * case["T"], case["groups"] * case["G"]
    return {"bytes": 2 * tokens * (P + 2) + heads * d * (es + 4) + tables,
            "flops": 4 * tokens * case["G"] * d + 4 * heads * d * d}


def tolerance(case):
    """Encode: the float64 nearest codeword and the rounded norm, so the same
    bytes.  Decode: sums of d float32 products (1.5e-7 against float64).
    Attention: softmax weights rounded to binary16 (up to 8e-5 against float64,
    1.2e-4 between two orders of the same sums)."""
    if case["op"] in ("append", "encode"):
        return "exact"
    if case["op"] == "decode":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 5e-4, "max": 1e-2}


# --------------------------------------------------------- float64 reference --
def _exact_encode(x, R, C, k, N):
    n, d = x.shape
    nb, w = d // k, int(math.log2(N))
    P = _payload(d, k, N)
    R, C = R.double(), C.double()
    c2 = (C * C).sum(1)
    step = max(1, (1 << 27) // (nb * N))
    bits = torch.arange(w, device=DEVICE)
    weights = 1 << torch.arange(8, device=DEVICE)
    payload = torch.empty(n, P, dtype=torch.uint8, device=DEVICE)
    norms = np.empty(n, dtype=np.int16)
    for a in range(0, n, step):
        xc = x[a:a + step].double()
        nu = xc.square().sum(1).sqrt()
        y = (xc / torch.where(nu > 0, nu, 1.0)[:, None]) @ R.T.contiguous()
        score = torch.addmm(c2[None, :], y.reshape(-1, k), C.T.contiguous(), alpha=-2.0)
        idx = score.argmin(1).view(-1, nb) * (nu > 0)[:, None]
        stream = ((idx[:, :, None] >> bits) & 1).view(len(xc), nb * w)
        stream = torch.nn.functional.pad(stream, (0, 8 * P - nb * w))
        payload[a:a + step] = (stream.view(-1, P, 8) * weights).sum(2).to(torch.uint8)
        norms[a:a + step] = nu.cpu().numpy().astype(np.float16).view(np.int16)
    return payload, torch.from_numpy(norms)


def _exact_rows(payload, norms, R, C, d, k, N):
    nb, w = d // k, int(math.log2(N))
    bits = (payload.long()[:, :, None] >> torch.arange(8, device=DEVICE)) & 1
    bits = bits.view(len(payload), -1)[:, :nb * w].reshape(-1, nb, w)
    idx = (bits << torch.arange(w, device=DEVICE)).sum(2)
    y = C.double()[idx].view(-1, d)
    return (y @ R.double()) * norms.view(torch.float16).double()[:, None]


def exact(case, seed):
    s = prepare(case, seed)
    d, k, N, R, C = case["d"], case["k"], case["N"], s["R"], s["C"]
    if case["op"] in ("append", "encode"):
        return [_exact_encode(x, R, C, k, N) for x in s["x"]]
    if case["op"] == "decode":
        payload, norms = s["payload"], s["norms"]
        if s["ids"] is not None:
            payload, norms = payload[s["ids"]], norms[s["ids"]]
        return torch.cat([_exact_rows(p, h, R, C, d, k, N)
                          for p, h in zip(payload.split(1 << 17), norms.split(1 << 17))])
    kp, kn, vp, vn = (t[:, :case["T"]] for t in s["kv"])
    out = torch.empty(case["groups"], case["G"], d, dtype=torch.float64, device=DEVICE)
    for g in range(case["groups"]):
        K = _exact_rows(kp[g], kn[g], R, C, d, k, N)
        V = _exact_rows(vp[g], vn[g], R, C, d, k, N)
        p = torch.softmax((s["q"][g].double() @ K.T.contiguous()) / math.sqrt(d), dim=1)
        out[g] = p @ V
    return out
