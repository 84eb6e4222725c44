"""What is timed of this library: a decode round's steps as a serving program
calls them, over the sizes that such programs meet.

A case is a dict of plain values.  Its `kind` says which public entry points a
pass goes through:

  draft    prepare_block_draft_attn: one-pass attention of the draft block
  verify   prepare_tree_verify_attn: ancestor-masked attention of the tree
  accept   prepare_greedy_accept, with the root entropy: row argmax and walk
  sample   glance_sample_accept: row draws at a temperature, and the walk
  tree     prepare_build_tree: the draft tree from the drafter's logits
  round    draft, verify, greedy acceptance and commit, one after another on
           one stream, as a serving loop issues them

The prepared calls (arguments marshalled once, workspace and outputs kept) are
what a decode loop holds; inputs are resident on the GPU, as its caches are.

Context lengths of a ragged batch are spread between `ctx_lo` and `ctx` by the
golden ratio, so that the work of a case does not depend on the seed; all
values, trees and planted tokens do.
"""

import heapq
import math
import random

import torch

import paper_2609_00355_amd as G

PATH_STRIDE = 16  # holds any accepted path of a tree of depth <= 15
DEPTH_CAP = 15    # offsets of a 16-row draft block

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    qwen = {"hq": 28, "hkv": 4, "d": 128, "dtype": "bf16"}
    return [
        # the smallest round: the tiny fp32 decoder on which losslessness is
        # audited; a handful of dependent launches, latency and nothing else
        {"name": "round tiny fp32", "kind": "round", "batch": 1, "ctx": 256, "ctx_lo": 256, "hq": 4, "hkv": 1,
         "d": 64, "dtype": "f32", "block": 8, "n": 16, "vocab": 1000},
        # interactive use, one sequence: the draft of a short prompt
        {"name": "draft 2k x1", "kind": "draft", "batch": 1, "ctx": 2048, "ctx_lo": 2048, "n": 16, "lse": False, **qwen},
        # interactive use: the 64-row verify of a page-sized prompt
        {"name": "verify 4k x1", "kind": "verify", "batch": 1, "ctx": 4096, "ctx_lo": 4096, "n": 64, "lse": False, **qwen},
        # long grounded documents, a small batch: the headline draft and verify
        {"name": "draft 16k x4", "kind": "draft", "batch": 4, "ctx": 16384, "ctx_lo": 16384, "n": 16, "lse": False, **qwen},
        {"name": "verify 16k x4", "kind": "verify", "batch": 4, "ctx": 16384, "ctx_lo": 16384, "n": 64, "lse": False, **qwen},
        # a smaller target (64-wide heads) with odd, ragged lengths, a tree that
        # fills no whole tile, and the log-sum-exp asked for
        {"name": "verify ragged d64 x3", "kind": "verify", "batch": 3, "ctx": 11003, "ctx_lo": 1037, "n": 37, "lse": True,
         "hq": 28, "hkv": 4, "d": 64, "dtype": "bf16"},
        # the audit of losslessness at the target's own shape, in fp32
        {"name": "verify fp32 4k x1", "kind": "verify", "batch": 1, "ctx": 4096, "ctx_lo": 4096, "n": 64, "lse": True,
         "hq": 28, "hkv": 4, "d": 128, "dtype": "f32"},
        # acceptance over the target's vocabulary: the headline batch, and a
        # vocabulary whose rows are not aligned to any vector
        {"name": "accept 152064 x4", "kind": "accept", "batch": 4, "n": 64, "vocab": 152064, "dtype": "bf16"},
        {"name": "accept 50257 x2", "kind": "accept", "batch": 2, "n": 33, "vocab": 50257, "dtype": "bf16"},
        # the sampling walk at temperature 1, headline batch
        {"name": "sample 152064 x4", "kind": "sample", "batch": 4, "n": 64, "vocab": 152064, "dtype": "bf16",
         "temperature": 1.0},
        # the tree builder on the drafter's rows, headline batch
        {"name": "tree 152064 x4", "kind": "tree", "batch": 4, "horizon": 15, "vocab": 152064, "budget": 63, "dtype": "bf16"},
        # a loaded server: sixteen sequences of 2k to 32k tokens, a whole round
        {"name": "round ragged x16", "kind": "round", "batch": 16, "ctx": 32768, "ctx_lo": 2048, "block": 16, "n": 64,
         "vocab": 152064, **qwen},
    ]


# Query heads, KV heads and head dimension of a few decoders.
HEADS = [(28, 4, 128), (28, 4, 128), (16, 2, 128), (8, 1, 128), (4, 4, 128), (28, 4, 64), (4, 1, 64), (6, 3, 64)]
VOCABS = [1000, 32000, 50257, 65536, 128256, 151936, 152063, 152064]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _vocab(rng):
    return rng.choice(VOCABS) if rng.random() < 0.5 else _log_int(rng, 1000, 152064)


def draw(rng):
    """One more case of the listed ones' ranges; none costs more than the ragged round."""
    kind = rng.choice(["draft", "verify", "verify", "draft", "accept", "sample", "tree", "round"])
    if kind in ("draft", "verify", "round"):
        dtype = "f32" if rng.random() < 0.25 else "bf16"
        hq, hkv, d = rng.choice(HEADS)
        batch = _log_int(rng, 1, 16)
        ctx = _log_int(rng, 200, 32768)
        ctx = min(ctx, (200_000 if dtype == "bf16" else 4096) // batch)
        ctx_lo = ctx if rng.random() < 0.3 else max(1, int(ctx * rng.uniform(0.05, 1.0)))
        c = {"kind": kind, "batch": batch, "ctx": ctx, "ctx_lo": ctx_lo, "hq": hq, "hkv": hkv, "d": d, "dtype": dtype}
        if kind == "draft":
            return {**c, "n": rng.choice([1, 4, 8, 16, 16, 24, 32, rng.randint(2, 32)]), "lse": rng.random() < 0.3}
        if kind == "verify":
            return {**c, "n": rng.choice([64, 64, 32, rng.randint(2, 64)]), "lse": rng.random() < 0.3}
        n = rng.choice([64, 32, rng.randint(4, 64)])
        vocab = _vocab(rng)
        while batch * n * vocab > 8 * 64 * 152064:
            n = max(1, n // 2)
        return {**c, "block": rng.choice([8, 16]), "n": n, "vocab": vocab}
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    batch = _log_int(rng, 1, 16)
    vocab = _vocab(rng)
    if kind == "tree":
        return {"kind": kind, "batch": batch, "horizon": rng.choice([15, 7, rng.randint(2, 15)]), "vocab": vocab,
                "budget": rng.choice([63, 31, 15, rng.randint(5, 63)]), "dtype": dtype}
    n = rng.choice([64, 64, 32, rng.randint(2, 64)])
    if kind == "accept":
        return {"kind": kind, "batch": batch, "n": n, "vocab": vocab, "dtype": dtype}
    return {"kind": kind, "batch": min(batch, 8), "n": n, "vocab": vocab, "dtype": dtype,
            "temperature": rng.choice([1.0, 1.0, 0.7, 1.3])}


# ------------------------------------------------------------------- inputs
def _lens(case):
    lo, hi, n = case["ctx_lo"], case["ctx"], case["batch"]
    if lo == hi:
        return [hi] * n
    lens = [lo + int((hi - lo) * ((0.6180339887 * (i + 1)) % 1.0)) for i in range(n)]
    lens[-1] = hi
    return lens


def _tree(n, vocab, rng):
    """A tree of n nodes grown best first: a deep likely spine with side branches."""
    n_kids, depth, parents = [0], [0], [-1]
    heap = [(-1.0, 0)]
    while len(parents) < n:
        s, v = heapq.heappop(heap)
        for r in range(rng.choice((1, 2, 4))):
            if len(parents) == n:
                break
            c = len(parents)
            parents.append(v)
            depth.append(depth[v] + 1)
            n_kids[v] += 1
            n_kids.append(0)
            if depth[c] < DEPTH_CAP:
                heapq.heappush(heap, (s * rng.uniform(0.5, 0.95) * 2.0 ** -r, c))
    tokens = [rng.randrange(vocab)] + [0] * (n - 1)
    used = set()
    for c in range(1, n):
        t = rng.randrange(vocab)
        while (parents[c], t) in used:
            t = rng.randrange(vocab)
        used.add((parents[c], t))
        tokens[c] = t
    return parents, tokens, depth


def _trees(case, rng):
    got = [_tree(case["n"], case.get("vocab", 152064), rng) for _ in range(case["batch"])]
    dev = {"dtype": torch.int32, "device": "cuda"}
    return torch.tensor([g[0] for g in got], **dev), torch.tensor([g[1] for g in got], **dev), got


def _attention(case, n, gen):
    """Queries, caches and new keys and values: unit normal, so that the scaled
    scores have unit spread.  The cache has room for the rows a round commits."""
    dt, b, hq, hkv, d = DTYPES[case["dtype"]], case["batch"], case["hq"], case["hkv"], case["d"]
    cap = case["ctx"] + (PATH_STRIDE if case["kind"] == "round" else 0)

    def normal(*shape):
        return torch.randn(shape, generator=gen, dtype=dt, device="cuda")

    return {"q": normal(b, n, hq, d), "k_ctx": normal(b, hkv, cap, d), "v_ctx": normal(b, hkv, cap, d),
            "k_new": normal(b, n, hkv, d), "v_new": normal(b, n, hkv, d)}


def _verified_logits(case, trees, rng, gen):
    """Rows ~ N(0, 2); a row whose node has children carries one child's token
    above its maximum with a probability that falls from 0.9 to 0.5 with depth."""
    rows = torch.randn((case["batch"], case["n"], case["vocab"]), generator=gen, dtype=DTYPES[case["dtype"]], device="cuda")
    rows *= math.sqrt(2.0)
    top = rows.float().amax(-1) if case["dtype"] == "bf16" else rows.amax(-1)
    at = []
    for b, (parents, tokens, depth) in enumerate(trees):
        kids = {}
        for c in range(1, case["n"]):
            kids.setdefault(parents[c], []).append(c)
        deepest = max(depth) or 1
        for v, cs in sorted(kids.items()):
            if rng.random() < 0.9 - 0.4 * depth[v] / deepest:
                at.append((b, v, tokens[rng.choice(cs)]))
    if at:
        b, v, t = (torch.tensor(x, device="cuda") for x in zip(*at))
        rows[b, v, t] = (top[b, v] + 1.0).to(rows.dtype)
    return rows


def _peaked_rows(batch, n, vocab, dtype, rng, gen):
    """A confident model's rows: N(0, 1) background and four likely tokens a row,
    whose logits fall from 16 in the first row to 8 in the last."""
    rows = torch.randn((batch, n, vocab), generator=gen, dtype=DTYPES[dtype], device="cuda")
    at, val = [], []
    for b in range(batch):
        for j in range(n):
            top = 16.0 - 8.0 * j / max(n - 1, 1)
            for r, t in enumerate(rng.sample(range(vocab), min(4, vocab))):
                at.append((b, j, t))
                val.append(top - 1.5 * r - rng.uniform(0.0, 0.5))
    b, j, t = (torch.tensor(x, device="cuda") for x in zip(*at))
    rows[b, j, t] = torch.tensor(val, device="cuda").to(rows.dtype)
    return rows


def _inputs(case, seed):
    rng = random.Random(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    s = {"kind": kind}
    if kind in ("draft", "verify", "round"):
        s["lens"] = torch.tensor(_lens(case), dtype=torch.int32, device="cuda")
    if kind in ("verify", "accept", "sample", "round"):
        s["parents"], s["tokens"], trees = _trees(case, rng)
    if kind in ("draft", "round"):
        s["draft"] = _attention(case, case["block"] if kind == "round" else case["n"], gen)
    if kind in ("verify", "round"):
        s["verify"] = _attention(case, case["n"], gen)
    if kind in ("accept", "round"):
        s["logits"] = _verified_logits(case, trees, rng, gen)
    if kind == "sample":
        s["logits"] = _peaked_rows(case["batch"], case["n"], case["vocab"], case["dtype"], rng, gen)
    if kind == "tree":
        s["logits"] = _peaked_rows(case["batch"], case["horizon"], case["vocab"], case["dtype"], rng, gen)
        s["roots"] = torch.tensor([rng.randrange(case["vocab"]) for _ in range(case["batch"])], dtype=torch.int32, device="cuda")
    return s


def _attn_args(a):
    return a["q"], a["k_ctx"], a["v_ctx"], a["k_new"], a["v_new"]


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("draft", "verify"):
        a = s[kind]
        b, n, hq, _ = a["q"].shape
        s["lse"] = torch.empty((b, n, hq), dtype=torch.float32, device="cuda") if case["lse"] else None
    if kind == "draft":
        s["call"], s["out"], _ = G.prepare_block_draft_attn(*_attn_args(s["draft"]), s["lens"], lse=s["lse"])
    elif kind == "verify":
        s["call"], s["out"], _ = G.prepare_tree_verify_attn(*_attn_args(s["verify"]), s["lens"], s["parents"], lse=s["lse"])
    elif kind == "accept":
        s["call"], s["out"] = G.prepare_greedy_accept(s["logits"], s["parents"], s["tokens"], path_stride=PATH_STRIDE,
                                                      want_entropy=True)
    elif kind == "sample":
        s["temperature"], s["seed"] = case["temperature"], seed
        s["workspace"] = torch.empty(G.glance_accept_workspace_size(case["batch"], case["n"], case["vocab"]),
                                     dtype=torch.uint8, device="cuda")
        s["out"] = G.glance_sample_accept(s["logits"], s["parents"], s["tokens"], s["temperature"], s["seed"], 0,
                                          path_stride=PATH_STRIDE, workspace=s["workspace"])
    elif kind == "tree":
        s["call"], s["out"] = G.prepare_build_tree(s["logits"], s["roots"], case["budget"])
    else:
        s["ctx_lens"] = s["lens"].clone()
        s["call_draft"], s["out_draft"], _ = G.prepare_block_draft_attn(*_attn_args(s["draft"]), s["ctx_lens"])
        s["call_verify"], s["out_verify"], _ = G.prepare_tree_verify_attn(*_attn_args(s["verify"]), s["ctx_lens"], s["parents"])
        s["call_accept"], s["out_accept"] = G.prepare_greedy_accept(s["logits"], s["parents"], s["tokens"],
                                                                    path_stride=PATH_STRIDE)
    return s


def run(s):
    kind = s["kind"]
    if kind in ("draft", "verify"):
        s["call"]()
        return {"out": s["out"], "lse": s["lse"]} if s["lse"] is not None else {"out": s["out"]}
    if kind in ("accept", "tree"):
        s["call"]()
        return s["out"]
    if kind == "sample":
        return G.glance_sample_accept(s["logits"], s["parents"], s["tokens"], s["temperature"], s["seed"], 1,
                                      path_stride=PATH_STRIDE, outputs=s["out"], workspace=s["workspace"])
    # The lengths go back to where the round began, so that a pass repeats it
    # (the rows it committed lie behind them).
    s["ctx_lens"].copy_(s["lens"])
    s["call_draft"]()
    s["call_verify"]()
    s["call_accept"]()
    v, acc = s["verify"], s["out_accept"]
    G.glance_commit_path(v["k_new"], v["v_new"], acc["accept_len"], acc["accept_path"], v["k_ctx"], v["v_ctx"], s["ctx_lens"])
    return {"draft": s["out_draft"], "verify": s["out_verify"], "accept": acc, "ctx_lens": s["ctx_lens"],
            "k_ctx": v["k_ctx"], "v_ctx": v["v_ctx"]}


# ------------------------------------------------------ work and tolerances
def _attn_work(case, n):
    esz = 4 if case["dtype"] == "f32" else 2
    keys = sum(_lens(case))
    b, hq, hkv, d = case["batch"], case["hq"], case["hkv"], case["d"]
    moved = 2 * keys * hkv * d + 2 * b * n * hq * d + 2 * b * n * hkv * d  # caches; queries and output; new keys and values
    return moved * esz + 4 * b, 4.0 * d * hq * n * (keys + b * n / 4)


def work(case):
    """Inputs read once, outputs written once, and the two products of attention.
    Acceptance, sampling and tree building read their logits once."""
    kind = case["kind"]
    esz = 4 if case["dtype"] == "f32" else 2
    nbytes = flops = 0.0
    if kind in ("draft", "round"):
        x, y = _attn_work(case, case["block"] if kind == "round" else case["n"])
        nbytes, flops = nbytes + x, flops + y
    if kind in ("verify", "round"):
        x, y = _attn_work(case, case["n"])
        nbytes, flops = nbytes + x, flops + y
    if kind in ("accept", "sample", "round"):
        nbytes += case["batch"] * (case["n"] * (case["vocab"] * esz + 12) + 4 * PATH_STRIDE + 8)
    if kind == "tree":
        nbytes += case["batch"] * (case["horizon"] * case["vocab"] * esz + 12 * (case["budget"] + 1))
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "sample":
        return "exact"  # draws and walk are whole numbers, defined bit for bit
    if kind == "accept":
        return {"rel": 1e-5, "max": 1e-4}  # whole numbers exact; the entropy is a 32-bit sum
    if kind == "tree":
        # scores are 32-bit sums; strings within their rounding may swap places
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}  # 5e-7 from the 64-bit values
    # probabilities and outputs rounded to bf16: 2.3e-3 from the 64-bit values
    return {"rel": 1e-2, "max": 0.05}


# ------------------------------------------------------- 64-bit definitions
def _exact_attention(a, lens, n, case, parents=None):
    b, hq, hkv, d = case["batch"], case["hq"], case["hkv"], case["d"]
    group = hq // hkv
    out = torch.empty((b, n, hq, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((b, n, hq), dtype=torch.float64, device="cuda")
    for i in range(b):
        sees = torch.ones((n, n), dtype=torch.bool)
        if parents is not None:
            sees = torch.eye(n, dtype=torch.bool)
            for v in range(1, n):
                sees[v] |= sees[parents[i][v]]
        sees = sees.cuda().repeat_interleave(group, 0)
        for g in range(hkv):
            k = torch.cat([a["k_ctx"][i, g, :lens[i]], a["k_new"][i, :, g]]).double()
            v = torch.cat([a["v_ctx"][i, g, :lens[i]], a["v_new"][i, :, g]]).double()
            q = a["q"][i, :, g * group:(g + 1) * group].reshape(n * group, d).double()
            s = (q @ k.t()) / math.sqrt(d)
            s[:, lens[i]:].masked_fill_(~sees, -math.inf)
            total = torch.logsumexp(s, 1)
            out[i, :, g * group:(g + 1) * group] = (torch.exp(s - total[:, None]) @ v).reshape(n, group, d)
            lse[i, :, g * group:(g + 1) * group] = total.reshape(n, group)
    return out, lse


def _exact_scores(logits, budget):
    """Scores of the `budget` best strings of each sequence, best first."""
    b, horizon, vocab = logits.shape
    k = min(budget, vocab)
    got = torch.zeros((b, budget + 1), dtype=torch.float64)
    for i in range(b):
        z = logits[i].double()
        lq = (torch.topk(z, k, -1).values - torch.logsumexp(z, -1, keepdim=True)).cpu().tolist()
        heap = [(-lq[0][0], 1, (0,), 0.0)]
        for node in range(1, budget + 1):
            s, length, ranks, base = heapq.heappop(heap)
            got[i, node] = -s
            if length < horizon:
                heapq.heappush(heap, (s - lq[length][0], length + 1, ranks + (0,), -s))
            if ranks[-1] + 1 < k:
                r = ranks[-1] + 1
                heapq.heappush(heap, (-(base + lq[length - 1][r]), length, ranks[:-1] + (r,), base))
    return got


def exact(case, seed):
    kind = case["kind"]
    if kind == "sample":
        return None  # whole numbers only
    s = _inputs(case, seed)
    if kind == "accept":
        z = s["logits"][:, 0].double()
        p = torch.log_softmax(z, -1)
        h = -(torch.exp(p) * p).sum(-1)
        return {"argmax": None, "accept_len": None, "accept_path": None, "next_root": None, "root_entropy": h}
    if kind == "tree":
        return {"parents": None, "tokens": None, "scores": _exact_scores(s["logits"], case["budget"])}
    lens = _lens(case)
    parents = s["parents"].cpu().tolist() if "parents" in s else None
    if kind == "round":
        return {"draft": _exact_attention(s["draft"], lens, case["block"], case)[0],
                "verify": _exact_attention(s["verify"], lens, case["n"], case, parents)[0],
                "accept": None, "ctx_lens": None, "k_ctx": None, "v_ctx": None}
    out, lse = _exact_attention(s[kind], lens, case["n"], case, parents)
    return {"out": out, "lse": lse} if case["lse"] else {"out": out}
