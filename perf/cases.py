"""The attention work that programs of this library have it do, as cases to be timed.

Every case is one call of a public entry point over one transformer layer (a batched decode is one call
for the whole batch), on seeded inputs of the shapes and value structure of ``workloads.py``.  The listed
cases take one point each of the ranges that ``draw`` spreads cases over: pre-caching of contexts
(``encode``, ``layer``, ``rope``), the query's prefill (``prefill``, one request or several at once, and
``tree``, a scaling factor per node), and generation (``decode``), in bf16 on the Llama-3-8B head shape
(32 query and 8 KV heads of 128), on the other head shapes that the library takes, and in fp32.
"""
import math
import random

import torch

from paper_2502_05431_amd import binding as B
from paper_2502_05431_amd import workloads as W

DEV = "cuda:0"

# Everything a case may say, with the value it has where a case says nothing.
DEFAULTS = {
    "op": "prefill",            # encode | prefill | decode | tree | rope | layer
    "dtype": "bf16",
    "heads": 32, "kv_heads": 8, "head_dim": 128,
    "prefix": 32,               # tokens of the shared prefix
    "chunks": 20, "chunk_len": 512,   # contexts and their (mean) length
    "ragged": False,            # contexts of different lengths: 1/4 to 7/4 of chunk_len
    "rows": 64,                 # query rows of a prefill
    "own": 0,                   # own tokens in front of the query rows (a decode: generated so far)
    "batch": 1,                 # requests of a decode or a prefill
    "mixed": False,             # requests of a batch with different numbers of contexts: 1 to 2 * chunks - 1
    "lse": False,               # the LogSumExp output is asked for
    "prefix_rows": False,       # encode: the prefix's own rows are computed too
    "nodes": "per_context",     # tree: per_context | grouped | random
    "keys": "plain",            # plain | outliers (a few channels x8) | offsets (a mean per context)
    "hidden": 4096, "intermediate": 14336,   # layer
}


def listed():
    return [
        # the smallest call: the fp32 configuration, a 16-token query over four contexts of 32 tokens (launches and latency)
        {"name": "fp32_small_prefill", "op": "prefill", "dtype": "f32", "heads": 4, "kv_heads": 2, "head_dim": 64, "prefix": 8,
         "chunks": 4, "chunk_len": 32, "rows": 16, "lse": True},
        # pre-caching in fp32, the precision a user checks a model with: eight retrieved passages of different lengths
        {"name": "fp32_encode", "op": "encode", "dtype": "f32", "chunks": 8, "chunk_len": 512, "ragged": True, "lse": True},
        # a retrieval query on the head shape of the models with 256-wide heads (16 query, 8 KV heads)
        {"name": "d256_prefill", "op": "prefill", "heads": 16, "kv_heads": 8, "head_dim": 256},
        # a retrieval query: 64 rows over 20 passages of 512 tokens
        {"name": "rag_prefill", "op": "prefill"},
        # a generated token of the same request
        {"name": "rag_decode", "op": "decode", "own": 100},
        # pre-caching of the same passages through one whole transformer layer
        {"name": "rag_layer", "op": "layer"},
        # pre-caching of a 128K context, 64 contexts of 2048 tokens: the largest call
        {"name": "long_encode", "op": "encode", "chunks": 64, "chunk_len": 2048, "keys": "outliers"},
        # the 256-row query over it
        {"name": "long_prefill", "op": "prefill", "chunks": 64, "chunk_len": 2048, "rows": 256, "keys": "outliers"},
        # many-shot examples as they come: 512 short contexts of different lengths
        {"name": "manyshot_encode", "op": "encode", "chunks": 512, "chunk_len": 256, "ragged": True, "keys": "offsets"},
        # serving: one token for each of 32 requests whose contexts differ in number
        {"name": "batch_decode", "op": "decode", "batch": 32, "chunks": 8, "chunk_len": 1024, "mixed": True, "own": 64},
        # the query of the 128K context with a scaling factor per context
        {"name": "tree_prefill", "op": "tree", "chunks": 64, "chunk_len": 2048, "rows": 256, "keys": "outliers"},
        # positions and cache write in front of the pre-caching of the many-shot examples
        {"name": "rope_cache", "op": "rope", "chunks": 512, "chunk_len": 256, "ragged": True},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# (query heads, KV heads, head_dim): the matrix-core shapes beside the Llama one, and the others
OTHER_FLASH = [(8, 8, 128), (16, 8, 128), (16, 2, 128)]
OTHER_BF16 = [(16, 8, 256), (32, 8, 64), (6, 2, 40), (4, 2, 64), (8, 8, 96), (12, 2, 128)]
OTHER_F32 = [(4, 2, 64), (6, 2, 40), (2, 2, 256), (32, 8, 128), (16, 8, 256)]


def draw(rng):
    op = rng.choice(["encode"] * 6 + ["prefill"] * 7 + ["decode"] * 7 + ["tree", "tree", "rope", "rope", "layer"])
    shape = rng.random()
    c = {"op": op, "prefix": rng.choice([0, 7, 32, 32, 32, 64])}
    if shape < 0.60 or op == "layer":
        c.update(dtype="bf16", heads=32, kv_heads=8, head_dim=128)
        limit = 131072                                   # context tokens of one call
    elif shape < 0.72:
        h = rng.choice(OTHER_FLASH)
        c.update(dtype="bf16", heads=h[0], kv_heads=h[1], head_dim=h[2])
        limit = 65536
    elif shape < 0.86:
        h = rng.choice(OTHER_BF16)
        c.update(dtype="bf16", heads=h[0], kv_heads=h[1], head_dim=h[2])
        limit = 4096 if op == "encode" else 10240
    else:
        h = rng.choice(OTHER_F32)
        c.update(dtype="f32", heads=h[0], kv_heads=h[1], head_dim=h[2])
        limit = 4096
    c["ragged"] = rng.random() < 0.6
    c["keys"] = rng.choice(["plain", "outliers", "offsets"]) if c["dtype"] == "bf16" else "plain"
    c["lse"] = rng.random() < 0.3
    if op == "layer":
        limit = 8192
    total = _log_int(rng, 128, limit)
    c["chunk_len"] = min(_log_int(rng, 32, 2048 if op == "encode" else 8192), total)
    c["chunks"] = max(1, total // c["chunk_len"])
    if op == "encode":
        c["prefix_rows"] = c["prefix"] > 0 and rng.random() < 0.3
    elif op in ("prefill", "tree"):
        c["rows"] = _log_int(rng, 1, 256 if limit > 10240 else 64)
        c["own"] = rng.choice([0, 0, 0, rng.randint(1, 200)])
    if op == "tree":
        c["chunks"] = min(c["chunks"], 256)
        c["nodes"] = rng.choice(["per_context", "grouped", "random"])
    elif op in ("prefill", "decode"):
        c["batch"] = rng.choice([1, 1, _log_int(rng, 1, 32)]) if op == "decode" else rng.choice([1, 1, 1, rng.randint(2, 4)])
        c["mixed"] = c["batch"] > 1 and rng.random() < 0.6
        c["chunks"] = max(1, min(c["chunks"], (2 if op == "decode" else 1) * limit // (c["batch"] * c["chunk_len"])))
        if op == "decode":
            c["own"] = rng.randint(0, 320)
    return c


def _full(case):
    return {**DEFAULTS, **case}


def chunk_lens(case):
    """The context lengths of every request of the case: a list of lists."""
    c = _full(case)
    rng = random.Random("%(chunks)d %(chunk_len)d %(batch)d" % c)
    out = []
    for _ in range(c["batch"]):
        n = rng.randint(1, 2 * c["chunks"] - 1) if c["mixed"] else c["chunks"]
        lo, hi = max(1, c["chunk_len"] // 4), max(1, c["chunk_len"] * 7 // 4)
        out.append([rng.randint(lo, hi) if c["ragged"] else c["chunk_len"] for _ in range(n)])
    return out


def _spec(c, lens):
    own = 0 if c["op"] in ("encode", "rope", "layer") else c["own"] + (1 if c["op"] == "decode" else c["rows"])
    kw = {"plain": dict(k_scale=1.0 if c["dtype"] == "f32" else c["head_dim"] ** -0.5), "outliers": dict(outlier_channels=4, outlier_gain=8.0),
          "offsets": dict(chunk_key_mean_std=0.5)}[c["keys"]]
    return W.WorkloadSpec(name="case", cfg=0, dtype=c["dtype"], n_q_heads=c["heads"], n_kv_heads=c["kv_heads"], head_dim=c["head_dim"],
                          prefix_len=c["prefix"], chunk_lens=tuple(lens), q_len=own, decode_steps=0, **kw)


def _cu(lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    return cu, torch.tensor(cu, dtype=torch.int32, device=DEV)


def _floats(nbytes):
    return torch.empty(max(64, (nbytes + 3) // 4), dtype=torch.float32, device=DEV)


def _nodes(c, n):
    if c["nodes"] == "per_context":
        return W.tree_per_context(n, 0.85)
    return W.tree_grouped(n, 8, 0.9, 0.85) if c["nodes"] == "grouped" else W.tree_random(n, 11)


def prepare(case, seed):
    c = _full(case)
    lens = chunk_lens(c)
    dtype = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    hq, hkv, d = c["heads"], c["kv_heads"], c["head_dim"]
    shape = B.make_shape(hq, hkv, d, dtype)
    s = {"op": c["op"], "shape": shape, "dtype": dtype}
    if c["op"] in ("prefill", "decode", "tree"):
        rows = 1 if c["op"] == "decode" else c["rows"]
        self_len = c["own"] + rows
        reqs, qs = [], []
        for b, ls in enumerate(lens):
            r = W.make_request(_spec(c, ls), DEV, run_index=seed, request=b)
            ks, vs = r.chunk_views()
            reqs.append(B.Request(r.k_prefix if c["prefix"] else None, r.v_prefix if c["prefix"] else None, ks, vs, r.k_self, r.v_self,
                                  self_len, r.temperature, r.scale))
            qs.append(r.q_self[c["own"]:].clone())
        q = torch.stack(qs) if c["batch"] > 1 or c["op"] == "decode" else qs[0]
        if c["op"] == "decode":
            q = q.reshape(c["batch"], hq, d)
        s.update(reqs=reqs, q=q.contiguous(), out=torch.empty_like(q))
        if c["lse"]:
            s["lse"] = torch.empty((c["batch"], hq) if c["op"] == "decode" else (c["batch"], hq, rows) if c["batch"] > 1 else (hq, rows),
                                   dtype=torch.float32, device=DEV)
        longest = max(sum(ls) for ls in lens)
        if c["op"] == "tree":
            nodes = _nodes(c, c["chunks"])
            s["tree"] = B.make_tree(nodes, DEV)
            s["ws"] = _floats(B.tree_workspace_bytes(shape, longest, len(nodes), rows))
        else:
            op = B.APE_OP_DECODE if c["op"] == "decode" else B.APE_OP_PREFILL
            s["ws"] = _floats(B.workspace_bytes(op, shape, c["batch"], rows, longest))
        return s
    s["cu"], s["cu_dev"] = _cu(lens[0])
    m = s["cu"][-1]
    if c["op"] == "encode":
        r = W.make_request(_spec(c, lens[0]), DEV, run_index=seed)
        s.update(q=r.q_ctx, k=r.k_ctx, v=r.v_ctx, out=torch.empty_like(r.q_ctx), kp=r.k_prefix if c["prefix"] else None,
                 vp=r.v_prefix if c["prefix"] else None)
        if c["prefix_rows"]:
            s.update(qp=r.q_prefix, outp=torch.empty_like(r.q_prefix))
        if c["lse"]:
            s["lse"] = torch.empty((hq, m), dtype=torch.float32, device=DEV)
        return s
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)

    def normal(*sizes, scale=1.0):
        return (torch.randn(sizes, generator=gen, device=DEV, dtype=torch.float32) * scale).to(dtype).contiguous()

    if c["op"] == "rope":
        s.update(offset=c["prefix"], q=normal(m, hq, d), k=normal(m, hkv, d), v=normal(m, hkv, d))
        s["cache"] = [torch.empty_like(s["k"]), torch.empty_like(s["v"])]
        s["q_rot"] = torch.empty_like(s["q"])
        s["tables"] = [torch.tensor([t[a:a + 1].data_ptr() for a in s["cu"][:-1]], dtype=torch.int64, device=DEV) for t in s["cache"]]
        return s
    hid, inter = c["hidden"], c["intermediate"]
    s["weights"] = [(1.0 + 0.1 * normal(hid).float()).to(dtype), normal((hq + 2 * hkv) * d, hid, scale=hid ** -0.5),
                    normal(hid, hq * d, scale=(hq * d) ** -0.5), (1.0 + 0.1 * normal(hid).float()).to(dtype),
                    normal(2 * inter, hid, scale=hid ** -0.5), normal(hid, inter, scale=inter ** -0.5)]
    s["layer"] = B.layer_weights(hid, inter, 1e-5, 500000.0, *s["weights"])
    s.update(x=normal(m, hid), kp=normal(c["prefix"], hkv, d) if c["prefix"] else None, vp=normal(c["prefix"], hkv, d) if c["prefix"] else None)
    s.update(k=torch.empty((m, hkv, d), dtype=dtype, device=DEV), v=torch.empty((m, hkv, d), dtype=dtype, device=DEV), y=torch.empty_like(s["x"]))
    s["ws"] = _floats(B.layer_workspace_bytes(shape, hid, inter, m))
    return s


def run(s):
    op, lse = s["op"], s.get("lse")
    if op == "encode":
        B.encode_chunks(s["shape"], s.get("qp"), s["kp"], s["vp"], s["q"], s["k"], s["v"], s["cu"], s["cu_dev"], s.get("outp"), s["out"], None, lse)
        return [s["out"], s.get("outp"), lse]
    if op == "decode":
        B.attention_decode(s["shape"], s["reqs"], s["q"], s["out"], lse, s["ws"])
        return [s["out"], lse]
    if op == "tree":
        B.attention_tree(s["shape"], s["reqs"][0], s["tree"], s["q"], s["out"], lse, s["ws"])
        return [s["out"], lse]
    if op == "prefill":
        if len(s["reqs"]) > 1:
            B.attention_prefill_batch(s["shape"], s["reqs"], s["q"], s["out"], lse, s["ws"])
        else:
            B.attention_prefill(s["shape"], s["reqs"][0], s["q"], s["out"], lse, s["ws"])
        return [s["out"], lse]
    if op == "rope":
        B.rope_write_cache(s["shape"], s["q"], s["k"], s["v"], s["cu"], s["cu_dev"], s["offset"], 500000.0, s["q_rot"], *s["tables"])
        return [s["q_rot"], *s["cache"]]
    B.layer_encode(s["shape"], s["layer"], s["x"], s["kp"], s["vp"], s["cu"], s["cu_dev"], s["k"], s["v"], s["y"], s["ws"])
    return [s["y"], s["k"], s["v"]]


def work(case):
    """Every input read once, every output written once; the two products of attention over the visible (row, token) pairs."""
    c = _full(case)
    es = 4 if c["dtype"] == "f32" else 2
    hq, hkv, d, p = c["heads"], c["kv_heads"], c["head_dim"], c["prefix"]
    kv, qo = 2 * hkv * d * es, 2 * hq * d * es           # bytes of a token's K and V, of a row's Q and output
    lens = chunk_lens(c)
    m = sum(lens[0])
    pairs = sum(n * p + n * (n + 1) // 2 for n in lens[0]) + (p * (p + 1) // 2 if c["prefix_rows"] else 0)
    if c["op"] == "encode":
        return {"bytes": m * (kv + qo + (4 * hq if c["lse"] else 0)) + p * (kv + (qo if c["prefix_rows"] else 0)), "flops": 4 * hq * d * pairs}
    if c["op"] == "rope":
        return {"bytes": m * (kv + qo) + m * kv, "flops": 6 * m * (hq + hkv) * d // 2}
    if c["op"] == "layer":
        hid, inter = c["hidden"], c["intermediate"]
        params = hid * ((hq + 2 * hkv) * d + hq * d + 3 * inter)
        return {"bytes": es * (params + 2 * hid + 2 * m * hid) + (m + p) * kv, "flops": 2 * m * params + 4 * hq * d * pairs}
    rows = 1 if c["op"] == "decode" else c["rows"]
    nbytes = flops = 0
    for ls in lens:
        seen = rows * (sum(ls) + p + c["own"]) + rows * (rows + 1) // 2
        nbytes += (sum(ls) + p + c["own"] + rows) * kv + rows * (qo + (4 * hq if c["lse"] else 0))
        flops += 4 * hq * d * seen
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the outputs were seen to be off by against 64-bit references of the same inputs."""
    c = _full(case)
    if c["dtype"] == "f32":
        return {"rel": 5e-6, "max": 1e-4}                # seen: 1.2e-6 and 1.2e-5 (sums of up to 4096 fp32 terms)
    if c["op"] == "rope":
        return {"rel": 1e-4, "max": 0.04}                # seen: 1.1e-5, single roundings to bf16 that fall the other way (0.0078)
    if c["op"] == "layer":
        return {"rel": 1.3e-2, "max": 0.1}               # seen: 3.3e-3 and 0.017 (bf16 between the four products of the layer)
    return {"rel": 1e-2, "max": 0.1}                     # seen: 2.4e-3 and 0.022 (bf16 probabilities, output rounded to bf16)
