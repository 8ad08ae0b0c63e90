"""The calls whose speed matters to a user of this library, as cases that can be prepared, run and compared.

A decoding loop with draft trees makes, per iteration: the tree tensors once, one attention call per layer, the teacher
head (or its logits), and the epilogue (gather, acceptance, commit).  Programs that keep branch caches add the
replication and the commit by path indices.  `kind` says which part a case is:

  step    tensorize_tree -> tree_verify_attention for each layer -> (lm_head_argmax ->) verify_epilogue
  attn    one layer's tree_verify_attention, the call that is made most often by far
  head    lm_head_argmax: hidden states of the nodes -> the teacher's greedy choice
  branch  replicate_branches, then commit_path_indices from one of the branches

Sizes are this repository's benchmark and test configurations, or lie between them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2603_08088_amd import api, synth

BLOCK = synth.BLOCK
DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _attn(name, **kw):
    c = dict(name=name, kind="attn", B=1, T=60, n_lo=60, Hq=32, Hkv=8, d=128, dtype="bf16", P=2048, P_lo=2048, paged=True,
             tail=False, tree="topk", depth=6)
    c.update(kw)
    c["n_lo"] = kw.get("n_lo", c["T"])
    c["P_lo"] = kw.get("P_lo", c["P"])
    return c


def _step(name, **kw):
    c = _attn(name, kind="step", paged=False, layers=32, V=32000, D=0)
    c.update(kw)
    c["n_lo"] = kw.get("n_lo", c["T"])
    c["P_lo"] = kw.get("P_lo", c["P"])
    del c["tail"]
    return c


def listed():
    return [
        # the smallest complete step, fp32: what a unit test or a toy model runs; nothing but latency and launches
        _step("step_tiny_f32", T=15, Hq=4, Hkv=4, d=64, dtype="f32", P=128, layers=1, V=1000, tree="bfs", depth=4),
        # one user, a 7B-class teacher: all 32 layers of a step and the acceptance from the teacher's logits
        _step("step_gqa_b1", B=1, T=60, P=2048, layers=32),
        # a small serving batch of ragged sequences, the head fused with the greedy choice; four of the layers
        _step("step_ragged_b8_head", B=8, T=60, P=8192, P_lo=512, paged=True, layers=4, D=4096),
        # one long document, large tree, tree rows written in place behind the prefix
        _attn("attn_long_b1", B=1, T=128, P=32768, paged=False, tail=True, tree="bfs", depth=8),
        # a full serving batch, small tree: reading the cache is all there is
        _attn("attn_b32_t8", B=32, T=8, P=4096, tree="spine", depth=4),
        # the same batch with a tree of the usual size
        _attn("attn_b32_t32", B=32, T=32, P=4096, tree="spine", depth=6),
        # the same batch with the largest budget of the benchmark's sweep: its headline
        _attn("attn_b32_t128", B=32, T=128, P=4096, tree="spine", depth=10),
        # fp32 throughout, for a teacher that is checked or run at full precision; odd sizes
        _attn("attn_f32_b2", B=2, T=33, n_lo=29, Hq=16, Hkv=4, dtype="f32", P=1003, P_lo=771, tree="bfs", depth=6),
        # models with heads of 64: bf16, a few ragged sequences
        _attn("attn_d64_b4", B=4, T=48, n_lo=41, Hq=32, Hkv=8, d=64, P=1500, P_lo=900, tree="topk", depth=6),
        # the head of one user's step: 60 rows, the weights are streamed once
        dict(name="head_b1", kind="head", B=1, T=60, n_lo=60, D=4096, V=32000, packed=True),
        # the head of a full batch of large trees
        dict(name="head_b32", kind="head", B=32, T=128, n_lo=128, D=4096, V=32000, packed=True),
        # branch caches: four branches per sequence, and the general commit that reorders every row
        dict(name="branch_reorder", kind="branch", B=8, N=4, T=60, P=2040, P_lo=2040, Hkv=8, d=128, dtype="bf16", layers=8, fast=False),
    ]


# ---------------------------------------------------------------------------------------------------------------
def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost(c):
    w = work(c)
    # fp32 and heads of 64 are priced as vector arithmetic
    return max(w["bytes"] / 8e12, w["flops"] / (1e15 if c["kind"] == "head" or (c["dtype"] == "bf16" and c.get("d") == 128) else 2e12))


def draw(rng):
    most = {"attn": 2.8e-4, "step": 5e-4, "head": 1.0e-3, "branch": 2.5e-4}
    kind = rng.choice(["attn", "attn", "attn", "step", "head", "branch"])
    while True:
        if kind == "head":
            B = _log(rng, 1, 32)
            T = _log(rng, 1, 256)
            c = dict(kind=kind, B=B, T=T, n_lo=rng.randint(max(1, (3 * T) // 4), T), D=128 * _log(rng, 8, 40),
                     V=rng.choice([32000, _log(rng, 1000, 64000)]), packed=rng.random() < 0.7)
        elif kind == "branch":
            P = _log(rng, 100, 4096)
            c = dict(kind=kind, B=_log(rng, 1, 16), N=rng.randint(1, 4), T=_log(rng, 4, 128), P=P, P_lo=rng.randint(max(1, P // 4), P), Hkv=rng.choice([4, 8]),
                     d=rng.choice([64, 128]), dtype=rng.choice(["bf16", "bf16", "f32"]), layers=rng.randint(1, 16), fast=rng.random() < 0.5)
        else:
            dtype, d = rng.choice([("bf16", 128)] * 6 + [("bf16", 64), ("f32", 64), ("f32", 128)])
            Hq, Hkv = rng.choice([(32, 8), (32, 8), (32, 8), (8, 2), (8, 8), (4, 2), (16, 4), (32, 32)])
            T, P = _log(rng, 1, 256), _log(rng, 64, 32768)
            c = dict(kind=kind, B=_log(rng, 1, 32), T=T, n_lo=rng.randint(max(1, (3 * T) // 4), T), Hq=Hq, Hkv=Hkv, d=d,
                     dtype=dtype, P=P, P_lo=rng.choice([P, rng.randint(max(1, P // 16), P)]), paged=rng.random() < 0.7,
                     tree=rng.choice(["topk", "bfs", "spine"]), depth=rng.randint(3, 10))
            if kind == "attn":
                c["tail"] = rng.random() < 0.25
            else:
                c.update(layers=rng.randint(1, 8), V=rng.choice([32000, _log(rng, 1000, 64000)]), D=0)
                if c["dtype"] == "bf16" and rng.random() < 0.5:
                    c["D"] = 128 * _log(rng, 8, 32)
        if _cost(c) <= most[kind]:
            return c


# ---------------------------------------------------------------------------------------------------------------
def _spread(lo, hi, n):
    """n whole numbers from hi down to lo, evenly."""
    return [hi] if n == 1 else [int(round(hi - (hi - lo) * i / (n - 1))) for i in range(n)]


def _elem(c):
    return 4 if c["dtype"] == "f32" else 2


def _attn_work(c):
    e = _elem(c)
    by = fl = 0
    # which length meets which tree is drawn by the seed: the mean of the products stands for it
    P, n = _spread(c["P_lo"], c["P"], c["B"]), _spread(c["n_lo"], c["T"], c["B"])
    for b in range(c["B"]):
        by += (2 * P[b] + 2 * n[b]) * c["Hkv"] * c["d"] * e + 2 * n[b] * c["Hq"] * c["d"] * e
        fl += 4 * c["Hq"] * c["d"] * n[b] * (sum(P) / c["B"] + n[b])
    return by, fl


def work(c):
    kind = c["kind"]
    if kind == "attn":
        by, fl = _attn_work(c)
        return {"bytes": by, "flops": fl}
    if kind == "head":
        rows = sum(_spread(c["n_lo"], c["T"], c["B"]))
        return {"bytes": 2 * c["V"] * c["D"] + 2 * rows * c["D"] + 8 * rows, "flops": 2 * rows * c["V"] * c["D"]}
    if kind == "step":
        by, fl = _attn_work(c)
        rows = sum(_spread(c["n_lo"], c["T"], c["B"]))
        by, fl = by * c["layers"], fl * c["layers"]
        if c["D"]:
            by, fl = by + 2 * c["V"] * c["D"] + 2 * rows * c["D"], fl + 2 * rows * c["V"] * c["D"]
        else:
            by += 4 * rows * c["V"]
        # the root and about half of a path are committed
        by += 4 * c["layers"] * c["B"] * (1 + c["depth"] // 2) * c["Hkv"] * c["d"] * _elem(c)
        return {"bytes": by, "flops": fl}
    row = 2 * c["layers"] * c["Hkv"] * c["d"] * _elem(c)      # K and V of one position
    Ps = _spread(c["P_lo"], c["P"], c["B"])
    moved = sum(c["N"] * (P % BLOCK) + (_branch_rows(c) + (P % BLOCK) if c["fast"] else P + _branch_rows(c)) for P in Ps)
    return {"bytes": 2 * moved * row, "flops": 0}


def _branch_rows(c):
    return min(6, c["T"])


def tolerance(c):
    if c["kind"] == "branch":
        return "exact"
    if c["kind"] == "head":
        # the margins are planted, so the choices are the same; the maxima are fp32 sums of bf16 products in another order
        # (against float64: rel 3.3e-7, max 1.2e-6)
        return {"rel": 1.3e-6, "max": 5e-6}
    if c["dtype"] == "f32":         # against float64: rel 5.6e-7, max 9.5e-6
        return {"rel": 2.5e-6, "max": 4e-5}
    # probabilities and outputs are rounded to bf16 (against float64: rel 0.0023, max 0.018 where a batch mixes short and long prefixes)
    return {"rel": 1e-2, "max": 0.07}


# ---------------------------------------------------------------------------------------------------------------
def _tree(rng, c, T):
    if c["tree"] == "topk" and T <= 10 * c["depth"]:
        return synth.tree_eagle(rng, T, c["depth"], 10)
    if c["tree"] == "spine":
        return synth.tree_spine_leaves(T, c["depth"])
    return synth.tree_bfs(rng, T, c["depth"], 4)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


class _Draw:
    """Seeded draws: whole numbers on the host, values on the GPU."""

    def __init__(self, seed):
        self.rng = np.random.default_rng(seed)
        self.gen = torch.Generator(device=DEV).manual_seed(seed)

    def normal(self, shape, dtype, scale=1.0):
        x = torch.empty(shape, dtype=dtype, device=DEV).normal_(generator=self.gen)
        return x.mul_(scale) if scale != 1.0 else x


def _sequences(c, dr):
    """Trees, prefix lengths and (paged) block tables of a batch."""
    B, T = c["B"], c["T"]
    s = {"case": c}
    ns = [int(x) for x in dr.rng.permutation(_spread(c["n_lo"], T, B))]
    Ps = [int(x) for x in dr.rng.permutation(_spread(c["P_lo"], c["P"], B))]
    parents = [_tree(dr.rng, c, n) for n in ns]
    parent = np.zeros((B, T), dtype=np.int32)
    for b, p in enumerate(parents):
        parent[b, :len(p)] = p
    s["parents"], s["Ps"], s["P_max"] = parents, Ps, max(Ps)
    s["parent"], s["n_nodes"], s["prefix_len"] = _dev(parent), _dev(np.asarray([len(p) for p in parents], np.int32)), _dev(np.asarray(Ps, np.int32))
    room = max(c["depth"] + 1, T)
    s["P_cap"], s["block_table"], s["num_blocks"] = max(Ps) + room, None, 0
    if c["paged"]:
        need = [-(-(P + room) // BLOCK) for P in Ps]
        # a table row reaches as far as the longest sequence may; the entries behind a sequence's own blocks are 0
        width = -(-(max(Ps) + room) // BLOCK)
        s["num_blocks"] = sum(need) + 16
        ids = dr.rng.permutation(s["num_blocks"]).astype(np.int32)
        table = np.zeros((B, width), dtype=np.int32)
        at = 0
        for b, n in enumerate(need):
            table[b, :n] = ids[at:at + n]
            at += n
        s["block_table"] = _dev(table)
        s["capacity"] = _dev(np.asarray([n * BLOCK for n in need], np.int32))
    else:
        s["capacity"] = _dev(np.full(B, s["P_cap"], np.int32))
    s["cache_shape"] = (s["num_blocks"], c["Hkv"], BLOCK, c["d"]) if c["paged"] else (B, s["P_cap"], c["Hkv"], c["d"])
    return s


def _prepare_attn(c, dr):
    s = _sequences(c, dr)
    dt, B, T = DTYPES[c["dtype"]], c["B"], c["T"]
    s["q"] = dr.normal((B, T, c["Hq"], c["d"]), dt)
    s["kt"] = None if c["tail"] else dr.normal((B, T, c["Hkv"], c["d"]), dt)
    s["vt"] = None if c["tail"] else dr.normal((B, T, c["Hkv"], c["d"]), dt)
    s["kc"], s["vc"] = dr.normal(s["cache_shape"], dt), dr.normal(s["cache_shape"], dt)
    # made once per step and used by every layer
    s["bitmask"] = api.build_tree_mask(s["parent"], s["n_nodes"], want_dense=False, want_depth=False)["bitmask"]
    s["out"] = torch.empty_like(s["q"])
    s["lse"] = torch.empty((B, c["Hq"], T), dtype=torch.float32, device=DEV)
    s["desc"] = api.attn_desc(s["q"], s["kt"], s["kc"], s["block_table"], s["P_max"])
    s["ws"] = torch.empty((max(256, api.tree_verify_attention_workspace_bytes(s["desc"])),), dtype=torch.uint8, device=DEV)
    return s


def _run_attn(s):
    return api.tree_verify_attention(s["q"], s["kc"], s["vc"], s["prefix_len"], s["kt"], s["vt"], s["bitmask"], s["n_nodes"],
                                     P_max=s["P_max"], block_table=s["block_table"], out=s["out"], lse=s["lse"],
                                     workspace=s["ws"], desc=s["desc"])


def _prepare_step(c, dr):
    s = _sequences(c, dr)
    dt, B, T, L, V, D = DTYPES[c["dtype"]], c["B"], c["T"], c["layers"], c["V"], c["D"]
    W = c["depth"] + 1
    rets = [synth.build_retrieve(p, W) for p in s["parents"]]
    s["L_max"], s["W"] = T, W       # a tree has at most T leaves
    tokens = np.zeros((B, T), dtype=np.int32)
    choice = dr.rng.integers(0, V, size=(B, T)).astype(np.int32)    # the teacher's planted choice at every node
    for b, p in enumerate(s["parents"]):
        tokens[b, :len(p)] = synth.draw_tokens(dr.rng, p, V)
        path = [int(x) for x in rets[b][int(dr.rng.integers(len(rets[b])))] if x >= 0]
        a = int(dr.rng.integers(0, len(path)))
        for i in range(a):                                          # the first a draft tokens of a path are accepted
            choice[b, path[i]] = tokens[b, path[i + 1]]
    s["tokens"] = _dev(tokens)
    s["tokens3"] = s["tokens"].reshape(B, T, 1)
    s["q"] = dr.normal((L, B, T, c["Hq"], c["d"]), dt)
    s["kt"], s["vt"] = dr.normal((L, B, T, c["Hkv"], c["d"]), dt), dr.normal((L, B, T, c["Hkv"], c["d"]), dt)
    s["kc"], s["vc"] = dr.normal((L,) + s["cache_shape"], dt), dr.normal((L,) + s["cache_shape"], dt)
    picks = _dev(choice)
    if D:
        s["hidden"], s["weight"] = _head_inputs(dr, B, T, D, V, picks)
        s["weight"] = api.pack_lm_head(s["weight"])
        s["logits"] = None
        s["post_ws"] = _head_workspace(B, T, V)
    else:
        s["logits"] = dr.normal((B, T, V), torch.float32)
        s["logits"].scatter_add_(2, picks.long()[..., None], torch.full((B, T, 1), 12.0, device=DEV))
        s["post_ws"] = torch.empty((max(256, api.evaluate_posterior_workspace_bytes(B, T, V)),), dtype=torch.uint8, device=DEV)
    i32 = dict(dtype=torch.int32, device=DEV)
    s["tree_out"] = dict(bitmask=torch.empty((B, T, (T + 63) // 64), dtype=torch.int64, device=DEV),
                         dense=torch.empty((B, 1, T, T), dtype=torch.uint8, device=DEV), depth=torch.empty((B, T), **i32),
                         status=torch.empty((B,), **i32), position_ids=torch.empty((B, T), **i32),
                         retrieve=torch.empty((B, s["L_max"], W), **i32), n_paths=torch.empty((B,), **i32))
    s["gather_out"] = dict(safe=torch.empty((B, s["L_max"], W), **i32),
                           pvalid=torch.empty((B, s["L_max"], W), dtype=torch.uint8, device=DEV),
                           gathered=torch.empty((B, s["L_max"], W, 1), **i32))
    s["post_out"] = dict(argmax=torch.empty((B, T), **i32), len=torch.empty((B, s["L_max"]), **i32), best=torch.empty((B,), **i32),
                         accept_len=torch.empty((B,), **i32), acc_nodes=torch.empty((B, W), **i32), bonus=torch.empty((B,), **i32))
    s["commit_out"] = dict(prefix_len_out=torch.empty((B,), **i32), slot_map=torch.empty((B, W), **i32), status=torch.empty((B,), **i32))
    s["out"] = torch.empty_like(s["q"])
    s["desc"] = api.attn_desc(s["q"][0], s["kt"][0], s["kc"][0], s["block_table"], s["P_max"])
    s["ws"] = torch.empty((max(256, api.tree_verify_attention_workspace_bytes(s["desc"])),), dtype=torch.uint8, device=DEV)
    # a layer's part of each tensor, as the layer's module holds it
    s["layer"] = [(s["q"][l], s["kc"][l], s["vc"][l], s["kt"][l], s["vt"][l], s["out"][l]) for l in range(L)]
    return s


def _run_step(s):
    c = s["case"]
    tree = api.tensorize_tree(s["parent"], s["n_nodes"], s["prefix_len"], s["L_max"], s["W"], out=s["tree_out"])
    for q, kc, vc, kt, vt, out in s["layer"]:
        api.tree_verify_attention(q, kc, vc, s["prefix_len"], kt, vt, tree["bitmask"], s["n_nodes"], P_max=s["P_max"],
                                  block_table=s["block_table"], out=out, want_lse=False, workspace=s["ws"], desc=s["desc"])
    if c["D"]:
        api.lm_head_argmax(s["hidden"], s["weight"], s["n_nodes"], V=c["V"], workspace=s["post_ws"], finish=False)
    # the new lengths go to a buffer of their own: the step can be repeated on the same prefix
    gather, post, commit = api.verify_epilogue(s["logits"], s["tokens"], tree["retrieve"], s["n_nodes"], s["kt"], s["vt"], s["kc"],
                                               s["vc"], s["prefix_len"], s["capacity"], block_table=s["block_table"],
                                               src=s["tokens3"], workspace=s["post_ws"], gather_out=s["gather_out"],
                                               post_out=s["post_out"], commit_out=s["commit_out"], head_V=c["V"] if c["D"] else 0)
    return {"attention": s["out"], "tree": tree, "gather": gather, "posterior": post, "commit": commit, "k_cache": s["kc"], "v_cache": s["vc"]}


def _head_workspace(B, T, V):
    return torch.empty((max(256, int(api.lib().etv_lm_head_argmax_workspace_bytes(B, T, V))),), dtype=torch.uint8, device=DEV)


def _head_inputs(dr, B, T, D, V, picks):
    """Hidden states and head weights with a clear choice per node, as a trained teacher has: the logits are ~N(0, 1) and the
    picked one stands about 8 above them."""
    weight = dr.normal((V, D), torch.bfloat16, 1.0 / math.sqrt(D))
    hidden = dr.normal((B, T, D), torch.bfloat16)
    hidden += 8.0 * weight[picks.long().reshape(-1)].reshape(B, T, D)
    return hidden, weight


def _prepare_head(c, dr):
    B, T, D, V = c["B"], c["T"], c["D"], c["V"]
    picks = _dev(dr.rng.integers(0, V, size=(B, T)).astype(np.int32))
    hidden, weight = _head_inputs(dr, B, T, D, V, picks)
    ns = dr.rng.permutation(_spread(c["n_lo"], T, B)).astype(np.int32)
    return {"case": c, "hidden": hidden, "weight": api.pack_lm_head(weight) if c["packed"] else weight, "n_nodes": _dev(ns),
            "ws": _head_workspace(B, T, V),
            "out": dict(argmax=torch.empty((B, T), dtype=torch.int32, device=DEV),
                        maxval=torch.empty((B, T), dtype=torch.float32, device=DEV))}


def _run_head(s):
    return api.lm_head_argmax(s["hidden"], s["weight"], s["n_nodes"], V=s["case"]["V"], workspace=s["ws"], out=s["out"])


def _prepare_branch(c, dr):
    B, N, L, dt = c["B"], c["N"], c["layers"], DTYPES[c["dtype"]]
    Ps = [int(x) for x in dr.rng.permutation(_spread(c["P_lo"], c["P"], B))]
    held = [-(-P // BLOCK) for P in Ps]                       # blocks of the committed caches
    width = -(-(max(Ps) + c["T"]) // BLOCK)
    free = sum(N * (-(-(P + c["T"]) // BLOCK) - P // BLOCK) for P in Ps)
    fresh = [-(-(P + c["T"]) // BLOCK) for P in Ps]           # blocks of the caches that the commit writes
    nb = sum(held) + free + sum(fresh) + 16
    ids = dr.rng.permutation(nb).astype(np.int32)
    table, dst = np.full((B, width), -1, np.int32), np.full((B, width), -1, np.int32)
    at = 0
    for b in range(B):
        table[b, :held[b]] = ids[at:at + held[b]]
        at += held[b]
    free_ids = ids[at:at + free]
    at += free
    for b in range(B):
        dst[b, :fresh[b]] = ids[at:at + fresh[b]]
        at += fresh[b]
    # the prefix in order and an accepted path behind it; the general call gets the first rows in another order
    L_cap = max(Ps) + c["T"]
    idx = np.zeros((B, L_cap), np.int32)
    new = np.zeros(B, np.int32)
    for b, P in enumerate(Ps):
        a = _branch_rows(c)
        nodes = np.concatenate([[0], np.sort(dr.rng.choice(np.arange(1, c["T"]), a - 1, replace=False))]) if a > 1 else np.zeros(1)
        idx[b, :P + a] = np.concatenate([np.arange(P), P + nodes])
        new[b] = P + a
    return {"case": c, "kc": dr.normal((L, nb, c["Hkv"], BLOCK, c["d"]), dt), "vc": dr.normal((L, nb, c["Hkv"], BLOCK, c["d"]), dt),
            "table": _dev(table), "dst": _dev(dst), "free": _dev(free_ids), "prefix_len": _dev(np.asarray(Ps, np.int32)),
            "tail_len": _dev(np.full(B, c["T"], np.int32)), "idx": _dev(idx), "new_len": _dev(new),
            "src_len": _dev(np.asarray([P + c["T"] for P in Ps], np.int32))}


def _run_branch(s):
    c = s["case"]
    r = api.replicate_branches(s["kc"], s["vc"], s["table"], s["prefix_len"], s["tail_len"], c["N"], s["free"])
    src = r["branch_table"][:, c["N"] - 1].contiguous()       # the branch that was accepted
    k = api.commit_path_indices(s["kc"], s["vc"], s["kc"], s["vc"], s["idx"], s["src_len"], s["new_len"], src_table=src,
                                dst_table=s["dst"], fast=c["fast"])
    return {"replicate": r, "commit": k, "dst_table": s["dst"], "k_cache": s["kc"], "v_cache": s["vc"]}


def prepare(case, seed):
    dr = _Draw(seed)
    return {"attn": _prepare_attn, "step": _prepare_step, "head": _prepare_head, "branch": _prepare_branch}[case["kind"]](case, dr)


def run(state):
    return {"attn": _run_attn, "step": _run_step, "head": _run_head, "branch": _run_branch}[state["case"]["kind"]](state)
