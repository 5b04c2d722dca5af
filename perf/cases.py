"""The work that users of this library have it do, as cases that can be timed.

Three kinds of case, all through the public entry points of ``paper_2510_07535_amd.binding``:

  verify   one verify-step attention of one layer (``owl_verify_attn``): N drafted tokens of each
           sequence over a paged K/V cache
  round    one decoding iteration of a small batch: Prepare, the verify attention of several layers,
           greedy acceptance, the K/V commit of every layer
  drafter  one step of the drafter's recurrent cell (``owl_drafter_cell``), weights in the tiled layout

A case is a dict of plain values; ``prepare`` draws its inputs on the GPU from a seed, ``run`` is one pass.
"""
import math

import numpy as np
import torch

from paper_2510_07535_amd import binding as B
from paper_2510_07535_amd import workloads as W

PAGE = 16
DEV = "cuda:0"
_CODE = {"bf16": B.OWL_BF16, "f16": B.OWL_F16, "f32": B.OWL_F32}
_TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}

# The largest case of the list reads 2.4 GB and does 2.5e11 operations; drawn cases stay below both.
_MOST_BYTES, _MOST_FLOPS = 2.3e9, 1.6e11


def _verify(name, dtype, out, hq, hkv, d, batch, ctx_lo, ctx_hi, tree, n, lens_seed=0, outliers=False, paged=True):
    """``ctx_lo`` .. ``ctx_hi``: context lengths (``lens_seed`` draws the ones in between); ``tree``: chain, tree
    (random, at most 6 deep) or hybrid (a random tree with a chain of a fifth of the nodes under its deepest leaf)."""
    case = {"kind": "verify", "dtype": dtype, "out": out, "hq": hq, "hkv": hkv, "d": d, "batch": batch, "ctx_lo": ctx_lo,
            "ctx_hi": ctx_hi, "tree": tree, "n": n, "lens_seed": lens_seed, "outliers": outliers, "paged": paged}
    return dict(case, name=name) if name else case


def _round(name, dtype, hq, hkv, d, batch, ctx_lo, ctx_hi, nodes, layers, lens_seed=0):
    case = {"kind": "round", "dtype": dtype, "hq": hq, "hkv": hkv, "d": d, "batch": batch, "ctx_lo": ctx_lo,
            "ctx_hi": ctx_hi, "nodes": nodes, "layers": layers, "lens_seed": lens_seed}
    return dict(case, name=name) if name else case


def _drafter(name, dtype, d_in, d, states, rows):
    case = {"kind": "drafter", "dtype": dtype, "d_in": d_in, "d": d, "states": states, "rows": rows}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the small correctness shape: fp32, contiguous cache, one short sequence; latency and launches only
        _verify("tiny_chain4_f32", "f32", "f32", 4, 1, 64, 1, 512, 512, "chain", 4, paged=False),
        # a tree on a short prompt in fp16, the paper's inference type, answer in fp16 for the next layer; odd length
        _verify("8b_tree60_5k_f16", "f16", "f16", 32, 8, 128, 1, 5003, 5003, "tree", 60),
        # sequence (non-tree) verification of six tokens on an 8B-shaped layer at 32K
        _verify("8b_chain6_32k", "bf16", "f32", 32, 8, 128, 1, 32768, 32768, "chain", 6),
        # plain decoding, the one-token case of the same call, at 64K with a bf16 answer
        _verify("8b_decode1_64k", "bf16", "bf16", 32, 8, 128, 1, 65536, 65536, "chain", 1),
        # the paper's tree size on an 8B-shaped layer at 64K
        _verify("8b_tree60_64k", "bf16", "f32", 32, 8, 128, 1, 65536, 65536, "tree", 60),
        # 70B-shaped layer, tree and chain in one draft, keys with outliers, at the 128K limit
        _verify("70b_hybrid40_128k", "bf16", "f32", 64, 8, 128, 1, 131072, 131072, "hybrid", 40, outliers=True),
        # what one of eight GPUs does of that layer when its KV heads are sharded
        _verify("70b_hybrid40_128k_1of8", "bf16", "f32", 8, 1, 128, 1, 131072, 131072, "hybrid", 40, outliers=True),
        # serving: sixteen sequences of very different lengths, each with its own tree, one page pool
        _verify("8b_batch16_tree26", "bf16", "f32", 32, 8, 128, 16, 8192, 65536, "tree", 26, lens_seed=5),
        # one decoding iteration of four users: 30 drafted nodes + 30 extra tokens each, four layers
        _round("8b_round_batch4_f16", "f16", 32, 8, 128, 4, 3001, 16001, 30, 4, lens_seed=2),
        # one level of tree drafting (top-k 10) with the paper's cell width
        _drafter("drafter_12288_p10", "bf16", 12288, 12288, 10, 10),
        # the first drafting step, from the hidden state of an 8B-shaped target, ten children, fp16
        _drafter("drafter_4096_p1_f16", "f16", 4096, 12288, 1, 10),
        # a level of four users' trees drafted together: forty states at once
        _drafter("drafter_12288_p40", "bf16", 12288, 12288, 40, 40),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Verify steps three times in five, decoding iterations and drafter steps once each."""
    kind = rng.choice(["verify", "verify", "verify", "round", "drafter"])
    if kind == "drafter":
        d = 16 * _log_int(rng, 128, 768)
        square = d if d % 32 == 0 else d - 16
        d_in = rng.choice([square, 4096, 8192, 32 * _log_int(rng, 64, 384)])
        states = rng.choice([1, 10, _log_int(rng, 2, 48)])
        rows = min(64, max(states, rng.choice([10, states, rng.randint(1, 64)])))
        return _drafter(None, rng.choice(["bf16", "f16"]), d_in, d, states, rows)
    hq, hkv = rng.choice([(32, 8), (64, 8), (32, 8), (64, 8), (16, 4), (8, 2), (4, 1), (32, 4), (16, 2), (8, 1)])
    d = rng.choice([128, 128, 128, 128, 64])
    dtype = rng.choice(["bf16", "bf16", "f16"])
    if kind == "round":
        batch = _log_int(rng, 1, 12)
        lo, hi = sorted((_log_int(rng, 600, 40000), _log_int(rng, 600, 40000)))
        case = _round(None, dtype, hq, hkv, d, batch, lo, hi, rng.randint(4, 32), rng.randint(1, 4), rng.randrange(1 << 20))
    elif rng.random() < 0.1:                             # fp32 serves small shapes
        case = _verify(None, "f32", "f32", 4 * rng.randint(1, 4), 1, rng.choice([64, 128]), 1, *([_log_int(rng, 200, 2000)] * 2),
                       "chain", rng.randint(1, 8), paged=rng.random() < 0.5)
    else:
        tree = rng.choice(["chain", "tree", "tree", "hybrid"])
        n = _log_int(rng, 1, 16) if tree == "chain" else rng.randint(8, 64)
        batch = 1 if rng.random() < 0.6 else _log_int(rng, 2, 32)
        hi = _log_int(rng, 400, 131072)
        lo = hi if batch == 1 else _log_int(rng, max(100, hi // 8), hi)
        case = _verify(None, dtype, rng.choice(["f32", dtype]), hq, hkv, d, batch, lo, hi, tree, n, rng.randrange(1 << 20),
                       dtype == "bf16" and rng.random() < 0.25)
    while (w := work(case))["bytes"] > _MOST_BYTES or w["flops"] > _MOST_FLOPS:
        case["ctx_hi"] = case["ctx_hi"] * 3 // 4
        case["ctx_lo"] = min(case["ctx_lo"], case["ctx_hi"])
    return case


def _lens(case):
    """Context lengths: the two ends, and seeded ones between them."""
    lo, hi, b = case["ctx_lo"], case["ctx_hi"], case["batch"]
    if b == 1:
        return np.array([hi], np.int32)
    r = np.random.Generator(np.random.Philox(key=case["lens_seed"] ^ 0x5EED))
    lens = r.integers(lo, hi, size=b, endpoint=True)
    lens[:2] = hi, lo
    return r.permutation(lens).astype(np.int32)


def _tree(kind, n, rng):
    if kind == "chain" or n < 2:
        return W.chain_tree(n)
    if kind == "hybrid":
        return W.hybrid_tree(n - max(1, n // 5), max(1, n // 5), rng)
    return W.random_tree(n, 6, rng)


def _cache(case, lens, n, gen, layers=1, outliers=False):
    """Paged K/V pools of N(0, 1) values ([page][Hkv][16][D]) whose pages are scattered over the pool."""
    hkv, d = case["hkv"], case["d"]
    pages = [(int(l) + n + PAGE - 1) // PAGE for l in lens]
    total, width = sum(pages), max(pages)
    order = torch.randperm(total, generator=gen, device=DEV, dtype=torch.int32)
    table = torch.full((len(pages), width), -1, dtype=torch.int32, device=DEV)
    at = 0
    for b, p in enumerate(pages):
        table[b, :p] = order[at:at + p]
        at += p
    pools = []
    for _ in range(layers):
        k = torch.randn((total, hkv, PAGE, d), generator=gen, device=DEV, dtype=_TORCH[case["dtype"]])
        v = torch.randn((total, hkv, PAGE, d), generator=gen, device=DEV, dtype=_TORCH[case["dtype"]])
        if outliers:                                     # one cached position in twenty has keys eight times as large
            hot = torch.rand((total, 1, PAGE, 1), generator=gen, device=DEV) < 0.05
            for b, l in enumerate(lens):                 # (the drafted tokens' own rows have not)
                for pos in range(int(l), int(l) + n):
                    hot[table[b, pos // PAGE].long(), 0, pos % PAGE, 0] = False
            k *= 1.0 + 7.0 * hot
        pools.append((k, v))
    return pools, table, total, width


def _desc(case, n, width, total, lens, out):
    hkv, d = case["hkv"], case["d"]
    return B.make_desc(batch=case["batch"], n_draft=n, n_q_heads=case["hq"], n_kv_heads=hkv, head_dim=d,
                       max_pages_per_seq=width, max_ctx_len=int(lens.max()), qkv_dtype=_CODE[case["dtype"]],
                       scale=1.0 / math.sqrt(d), kv_stride_page=hkv * PAGE * d, kv_stride_head=PAGE * d, kv_stride_token=d,
                       n_pool_pages=total, out_dtype=_CODE[out])


def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)


def _queries(case, n, gen):
    return torch.randn((case["batch"], n, case["hq"], case["d"]), generator=gen, device=DEV, dtype=_TORCH[case["dtype"]])


def _prepare_verify(case, seed):
    gen, rng = torch.Generator(DEV).manual_seed(seed), np.random.Generator(np.random.Philox(key=seed))
    lens, n = _lens(case), case["n"]
    pools, table, total, width = _cache(case, lens, n, gen, outliers=case["outliers"])
    s = {"kind": "verify", "desc": _desc(case, n, width, total, lens, case["out"]), "q": _queries(case, n, gen)}
    s["k"], s["v"] = pools[0]
    s["table"] = table
    if not case["paged"]:                                # a plain [token][Hkv][D] array, no page table
        s["table"] = None
        s["k"], s["v"] = (x.transpose(1, 2).contiguous() for x in pools[0])
        s["desc"].kv_stride_head, s["desc"].kv_stride_token = case["d"], case["hkv"] * case["d"]
    s["lens"] = _i32(lens)
    s["parent"] = _i32(np.stack([_tree(case["tree"], n, rng) for _ in lens]))
    s["out"] = torch.empty((case["batch"], n, case["hq"], case["d"]), dtype=_TORCH[case["out"]], device=DEV)
    s["workspace"] = torch.empty(B.owl_verify_attn_workspace_size(s["desc"]), dtype=torch.uint8, device=DEV)
    s["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    return s


def _prepare_round(case, seed):
    gen, rng = torch.Generator(DEV).manual_seed(seed), np.random.Generator(np.random.Philox(key=seed))
    lens, b, n = _lens(case), case["batch"], case["nodes"]
    pools, table, total, width = _cache(case, lens, 2 * n, gen, layers=case["layers"])
    s = {"kind": "round", "desc": _desc(case, 2 * n, width, total, lens, case["dtype"]), "pools": pools, "table": table, "n": n}
    s["q"] = [_queries(case, 2 * n, gen) for _ in pools]
    s["lens"] = _i32(lens)
    trees = np.stack([W.random_tree(n, 8, rng) for _ in range(b)])
    # what the target model says, and drafted tokens that agree with it on the path to one random node
    tokens, said, root = (rng.integers(0, 128256, size=x) for x in ((b, 2 * n), (b, 2 * n), (b,)))
    for i in range(b):
        node = int(rng.integers(n // 2, n))
        while node >= 0:
            up = int(trees[i, node])
            tokens[i, node] = said[i, up] if up >= 0 else root[i]
            node = up
    s["tree"], s["tokens"], s["said"], s["root"] = _i32(trees), _i32(tokens), _i32(said), _i32(root)
    z32 = lambda *shape: torch.zeros(shape, dtype=torch.int32, device=DEV)
    s["parent"], s["depth"], s["pos"] = z32(b, 2 * n), z32(b, 2 * n), z32(b, 2 * n)
    s["mask"] = torch.zeros((b, 2 * n), dtype=torch.int64, device=DEV)
    s["accepted"], s["n_accept"], s["bonus"], s["last"], s["new_lens"] = z32(b, 2 * n), z32(b), z32(b), z32(b), z32(b)
    s["outs"] = [torch.empty_like(q) for q in s["q"]]
    s["workspace"] = torch.empty(B.owl_verify_attn_workspace_size(s["desc"]), dtype=torch.uint8, device=DEV)
    s["status"] = z32(1)
    return s


def _prepare_drafter(case, seed):
    gen, dt = torch.Generator(DEV).manual_seed(seed), _TORCH[case["dtype"]]
    d_in, d, p, m, vocab = case["d_in"], case["d"], case["states"], case["rows"], 4096
    randn = lambda *shape, dtype=torch.float32: torch.randn(shape, generator=gen, device=DEV, dtype=dtype)
    s = {"kind": "drafter"}
    s["desc"] = B.DrafterDesc(d_in=d_in, d=d, n_states=p, n_rows=m, vocab=vocab, dtype=_CODE[case["dtype"]],
                              alpha=B.owl_drafter_alpha(8, d), eps=1e-5, w_layout=B.OWL_W_TILED)
    w = randn(4, d, d_in, dtype=dt)
    w *= 1.0 / math.sqrt(d_in)
    s["w"] = torch.empty(B.owl_drafter_tiled_weight_bytes(s["desc"]), dtype=torch.uint8, device=DEV)
    B.owl_drafter_tile_weights(s["desc"], w, s["w"])     # once, when a program loads its weights
    s["h"], s["z"], s["emb"] = randn(p, d_in, dtype=dt), randn(p, d), randn(vocab, d, dtype=dt)
    s["tokens"] = torch.randint(0, vocab, (m,), generator=gen, device=DEV, dtype=torch.int32)
    s["parent_row"] = torch.randint(0, p, (m,), generator=gen, device=DEV, dtype=torch.int32)
    s["affine"] = [1.0 + 0.1 * randn(d), 0.1 * randn(d), 1.0 + 0.1 * randn(d), 0.1 * randn(d)]
    s["h_out"], s["h_out_f32"], s["z_out"] = torch.empty((m, d), dtype=dt, device=DEV), torch.empty((m, d), device=DEV), torch.empty((m, d), device=DEV)
    s["workspace"] = torch.empty(B.owl_drafter_cell_workspace_size(s["desc"]), dtype=torch.uint8, device=DEV)
    s["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    return s


def prepare(case, seed):
    return {"verify": _prepare_verify, "round": _prepare_round, "drafter": _prepare_drafter}[case["kind"]](case, seed)


def run(s):
    if s["kind"] == "verify":
        B.owl_verify_attn(s["desc"], s["q"], s["k"], s["v"], s["table"], s["lens"], s["parent"], s["out"], s["workspace"], s["status"])
        return {"out": s["out"], "status": s["status"]}
    if s["kind"] == "drafter":
        B.owl_drafter_cell(s["desc"], s["h"], s["z"], s["tokens"], s["parent_row"], s["w"], s["emb"], *s["affine"],
                           s["h_out"], s["h_out_f32"], s["z_out"], s["workspace"], s["status"])
        return {"h": s["h_out"], "h_f32": s["h_out_f32"], "z": s["z_out"], "status": s["status"]}
    B.owl_prepare_spec_tree(s["tree"], s["lens"], s["parent"], s["mask"], s["depth"], s["pos"], s["status"])
    for q, (k, v), out in zip(s["q"], s["pools"], s["outs"]):
        B.owl_verify_attn(s["desc"], q, k, v, s["table"], s["lens"], s["parent"], out, s["workspace"], s["status"])
    B.owl_accept_greedy(s["tokens"], s["parent"], s["root"], s["said"], s["n"], s["accepted"], s["n_accept"], s["bonus"],
                        s["last"], s["status"])
    for k, v in s["pools"]:
        B.owl_commit_kv(s["desc"], k, v, s["table"], s["lens"], s["accepted"], s["n_accept"], s["new_lens"], s["status"])
    return {x: s[x] for x in ("parent", "mask", "depth", "pos", "outs", "accepted", "n_accept", "bonus", "last", "new_lens",
                              "pools", "status")}


def work(case):
    if case["kind"] == "drafter":
        d_in, d, p, m = (case[x] for x in ("d_in", "d", "states", "rows"))
        # weights, states, embedding rows, affine pairs; three outputs a row
        return {"bytes": 8 * d * d_in + p * (2 * d_in + 4 * d) + 2 * m * d + 16 * d + 10 * m * d, "flops": 8 * p * d * d_in}
    lens = _lens(case).astype(np.int64)
    n = case["n"] if case["kind"] == "verify" else 2 * case["nodes"]
    layers = case.get("layers", 1)
    size = 4 if case["dtype"] == "f32" else 2
    out = 4 if case.get("out", case["dtype"]) == "f32" else 2
    cached = int((lens + n).sum())
    rows = case["batch"] * n * case["hq"]
    moved = 2 * 2 * case["batch"] * 4 * case["hkv"] * case["d"] * size if case["kind"] == "round" else 0     # four accepted rows
    return {"bytes": layers * (2 * cached * case["hkv"] * case["d"] * size + rows * case["d"] * (size + out) + moved) + 4 * cached // PAGE,
            "flops": layers * 4 * cached * case["hq"] * n * case["d"]}


def tolerance(case):
    """About four times what was seen between split sizes (another order of sums and other softmax references) and
    against the same path in 64 bits: bf16 2.3e-3 with an fp32 and 3.1e-3 with a bf16 answer, at most 1.9e-2 at one
    value; fp16 4.8e-4 and 2.0e-3; fp32 7e-7 and 2.5e-6.  Drafter: 3.4e-7 in the fp32 outputs; in the 16-bit one a sum
    in another order moves a few values by one unit in the last place (bf16 1.4e-4, fp16 1.2e-5)."""
    if case["kind"] == "drafter":
        return {"rel": 6e-4, "max": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-4, "max": 1.2e-3}
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-5}
    return {"rel": 1e-2, "max": 8e-2} if case["dtype"] == "bf16" else {"rel": 2e-3, "max": 8e-3}
