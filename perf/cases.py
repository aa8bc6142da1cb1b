"""Performance cases of the decode path: what is timed, on which inputs, and how its outputs are checked.

A case is one call into the library as a decoding program makes it, with the sizes of one layer (or, for
``step``, of a whole stack of layers) in a plain dict:

* ``sparse``  sparse attention of one layer over a token set rho chosen earlier (``binding.sparse_attn``);
  by far the most frequent call of a decode step: all layers but three or four.
* ``full``    full attention of one layer over the whole cache (``binding.full_attn``): the first two layers
  of a step, and every layer of a program that does not select.
* ``select``  a selection layer in one call (``binding.select_layer``): the layer's full attention and rho.
* ``step``    the attention part of one decode step over a stack of layers (``runner.StepRunner.run``).

Sizes: 1 to 64 sequences of 600 to 131 072 cached tokens, 8 to 64 query heads over 8 KV heads, budgets of 256 to
4096 tokens with a quarter of them as the recency window, head-major, token-major and paged caches.  Decoding
has one direction and one data type (bf16 in and out, binary32 inside, int32 indices).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2508_07101_amd import binding as cb
from paper_2508_07101_amd import workloads as wl
from paper_2508_07101_amd.runner import StepRunner

DEVICE = "cuda"
D = 128


def _case(name, kind, batch, heads, seq_len, budget, **more):
    c = dict(name=name, kind=kind, batch=batch, heads=heads, kv_heads=8, seq_len=seq_len, min_len=0, budget=budget,
             window=budget // 4, topk=0, sinks=0, layout="head_major", lowrank=0, planted=0, len_seed=1)
    c.update(more)
    return c


def listed():
    return [
        # a chat turn of a single user: 4 K tokens of context, the smallest call there is
        _case("sparse_small", "sparse", 1, 32, 4096, 1024),
        # one user far into a long reasoning trace: the layer that a step runs 29 times
        _case("sparse_single", "sparse", 1, 32, 32768, 2048),
        # eight equally long traces decoded together, with the largest budget
        _case("sparse_batch", "sparse", 8, 32, 16384, 4096),
        # a serving batch: 64 requests of different lengths in a paged cache
        _case("sparse_serving", "sparse", 64, 32, 32768, 2048, min_len=8192, layout="paged"),
        # the dense layers of the single user's step, and the baseline that sparse layers are compared with
        _case("full_single", "full", 1, 32, 32768, 2048),
        # dense layers of a young serving batch: short and long requests, odd lengths, paged
        _case("full_ragged", "full", 16, 32, 16383, 2048, min_len=601, layout="paged"),
        # selection layers, from the short single context ...
        _case("select_small", "select", 1, 32, 4096, 1024, topk=1024, planted=16),
        _case("select_single", "select", 1, 32, 32768, 2048, planted=64),
        # ... over a batch whose heads agree with each other more or less
        _case("select_batch", "select", 8, 32, 16384, 4096, lowrank=8),
        # ... and the longest context, with eight query heads per KV head
        _case("select_long", "select", 1, 64, 131072, 4096, planted=256),
        # ... to the serving batch, the most work of all
        _case("select_serving", "select", 64, 32, 32768, 2048, min_len=8192, layout="paged"),
        # a whole decode step of a single user: 36 layers, two dense, selection at layers 2 and 12, four sinks
        _case("step_loop", "step", 1, 32, 32512, 2048, sinks=4, planted=64, layers=36, reselect=12),
    ]


def _lengths(c):
    """The cached tokens of every sequence: part of the case, not of the seed."""
    if not c["min_len"]:
        return [c["seq_len"]] * c["batch"]
    rng = np.random.default_rng(c["len_seed"])
    return [int(v) for v in rng.integers(c["min_len"], c["seq_len"] + 1, size=c["batch"])]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["sparse", "sparse", "full", "select", "select", "step"])
    heads = rng.choice([32, 32, 64, 16, 8])
    batch = log(1, 64)
    # no more cached tokens than the serving batch holds
    seq_len = log(700, min(131072, 1300000 // batch))
    budget = min(rng.choice([256, 512, 1024, 2048, 3072, 4096]), 64 * (seq_len // 100))
    layout = rng.choice(["head_major", "token_major", "paged"])
    c = dict(kind=kind, batch=batch, heads=heads, kv_heads=8, seq_len=seq_len, min_len=0, budget=budget,
             window=budget // 4, topk=0, sinks=rng.choice([0, 0, 4]), layout=layout, lowrank=0, planted=0,
             len_seed=rng.randrange(1 << 30))
    if batch > 1 and rng.random() < 0.6:      # ragged; a selection layer's sequences are longer than the budget
        lowest = budget + 1 if kind in ("select", "step") else 600
        c["min_len"] = min(seq_len, max(lowest, seq_len // rng.choice([2, 4, 16])))
    if layout == "head_major":
        c["lowrank"] = rng.choice([0, 8])
        c["planted"] = rng.choice([0, 16, 64])
    if kind == "step":                        # a few layers, the serving batch's tokens shared among them
        c["layers"] = rng.randint(4, 8)
        c["reselect"] = rng.choice([0, 4])
        c["seq_len"] = max(700, min(seq_len, 1300000 // (batch * c["layers"])))
        c["budget"] = min(budget, 64 * (c["seq_len"] // 100))
        c["window"] = c["budget"] // 4
        c["min_len"] = min(c["seq_len"], max(c["min_len"], c["budget"] + 1)) if c["min_len"] else 0
    return c


def _schedule(c):
    kinds = [wl.LAYER_SPARSE] * c["layers"]
    kinds[0] = kinds[1] = wl.LAYER_FULL
    kinds[2] = wl.LAYER_SELECT
    if c["reselect"] and c["reselect"] < c["layers"]:
        kinds[c["reselect"]] = wl.LAYER_SELECT
    return kinds


def _inputs(c, seed):
    """Queries and caches (and the block table) as the workloads draw them, in the case's layout."""
    lens = _lengths(c)
    layers = c.get("layers", 1)
    w = wl.Workload("case", layers, c["batch"], c["heads"], c["kv_heads"], D, max(lens), c["budget"], c["window"],
                    c["topk"], tuple(_schedule(c)) if c["kind"] == "step" else (wl.LAYER_FULL,) * layers,
                    n_planted=c["planted"], lowrank=c["lowrank"], paged=c["layout"] == "paged", seed=seed % (1 << 40),
                    lengths=tuple(lens), n_sink=c["sinks"])
    inp = wl.make_inputs(w, DEVICE)
    if c["layout"] == "token_major":          # [B][L][G][d], the order in which a projection writes the cache
        for layer in inp.layers:
            layer.k = layer.k.transpose(1, 2).contiguous().transpose(1, 2)
            layer.v = layer.v.transpose(1, 2).contiguous().transpose(1, 2)
    return inp


def _draw_rho(c, seed):
    """A token set as an earlier selection layer leaves it: sinks, history, the last `window` positions; ascending."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed % (1 << 40) * 7 + 3)
    idx = torch.zeros((c["batch"], c["budget"]), dtype=torch.int32, device=DEVICE)
    lens = _lengths(c)
    for b, n in enumerate(lens):
        if n <= c["budget"]:
            idx[b, :n] = torch.arange(n, device=DEVICE, dtype=torch.int32)
            continue
        lead, lc = c["sinks"], n - c["window"]
        score = torch.rand(lc, generator=gen, device=DEVICE)
        score[:lead] = 2.0
        hist = score.topk(c["budget"] - c["window"]).indices.sort().values
        idx[b] = torch.cat([hist, torch.arange(lc, n, device=DEVICE)]).to(torch.int32)
    cnt = torch.tensor([min(n, c["budget"]) for n in lens], dtype=torch.int32, device=DEVICE)
    return idx, cnt


def prepare(case, seed):
    c = case
    inp = _inputs(c, seed)
    if c["kind"] == "step":
        return {"kind": "step", "runner": StepRunner(inp), "inp": inp}
    layer = inp.layers[0]
    params = cb.make_params(c["batch"], c["heads"], c["kv_heads"], c["budget"], c["window"], c["topk"], n_sink=c["sinks"])
    bound = max(inp.seq_lens_host)
    state = {"kind": c["kind"], "params": params, "q": layer.q, "inp": inp,
             "kv": cb.KvCache(layer.k, layer.v, inp.seq_lens, bound, inp.block_table),
             "out": torch.empty_like(layer.q), "ws": cb.alloc_workspace(params, bound, DEVICE)}
    if c["kind"] == "sparse":
        state["idx"], state["cnt"] = _draw_rho(c, seed)
    elif c["kind"] == "select":
        state["idx"] = torch.zeros((c["batch"], c["budget"]), dtype=torch.int32, device=DEVICE)
        state["cnt"] = torch.zeros((c["batch"],), dtype=torch.int32, device=DEVICE)
    return state


def run(state):
    s = state
    if s["kind"] == "sparse":
        cb.sparse_attn(s["params"], s["q"], s["kv"], s["idx"], s["cnt"], s["out"], s["ws"])
        return {"out": s["out"]}
    if s["kind"] == "full":
        cb.full_attn(s["params"], s["q"], s["kv"], s["out"], s["ws"])
        return {"out": s["out"]}
    if s["kind"] == "select":
        cb.select_layer(s["params"], s["q"], s["kv"], s["out"], s["idx"], s["cnt"], s["ws"])
        return {"out": s["out"], "idx": s["idx"], "cnt": s["cnt"]}
    r = s["runner"]
    r.run()
    return {"out": r.outs, "idx": r.idx, "cnt": r.cnt}


def work(case):
    """Every K and V row that a layer attends to is read once, q and rho once; outputs are written once.  Two
    products per (head, row): four operations per element."""
    c = case
    kinds = {"sparse": [wl.LAYER_SPARSE], "full": [wl.LAYER_FULL], "select": [wl.LAYER_SELECT]}.get(c["kind"]) or _schedule(c)
    n_bytes = n_flops = 0
    for kind in kinds:
        for n in _lengths(c):
            rows = min(n, c["budget"]) if kind == wl.LAYER_SPARSE else n
            n_bytes += 2 * rows * c["kv_heads"] * D * 2 + 2 * c["heads"] * D * 2
            n_bytes += 4 * min(n, c["budget"]) if kind != wl.LAYER_FULL else 0
            n_flops += 4 * rows * c["heads"] * D
    return {"bytes": n_bytes, "flops": n_flops}


def tolerance(case):
    # bf16 outputs (rounding alone: 2^-9 of a value at most) of softmax sums whose weights enter the product as bf16;
    # indices and counts are whole numbers and the same always
    return {"rel": 1e-2, "max": 4e-2, "differ": 0.0}


# ---- the same in plain torch, in 64 bits

def _rows(c, inp, layer, b, n):
    """K and V of sequence b, [G][n][d]."""
    lay = inp.layers[layer]
    if inp.block_table is None:
        return lay.k[b, :, :n], lay.v[b, :, :n]
    pages = inp.block_table[b, : (n + 15) // 16].long()
    return tuple(x[pages].permute(1, 0, 2, 3).reshape(c["kv_heads"], -1, D)[:, :n] for x in (lay.k, lay.v))


def _attention64(c, q, k, v, rho=None):
    """softmax(q k^T / sqrt d) v of one sequence: q [H][d], k and v [G][n][d]."""
    if rho is not None:
        k, v = k[:, rho], v[:, rho]
    qg = q.double().view(c["kv_heads"], -1, D)
    out = []
    for g in range(c["kv_heads"]):
        p = torch.softmax(qg[g] @ k[g].double().t().contiguous() / math.sqrt(D), dim=-1)
        out.append(p @ v[g].double())
    return torch.cat(out)


def _select_ref(c, q, k, n):
    """rho of one sequence: scores summed left to right in binary32 (the definition's order, so that near-equal
    scores rank alike), every head's best tokens, first occurrence in rank-major order, window and sinks."""
    if n <= c["budget"]:
        return torch.arange(n, device=q.device)
    lc, lead = n - c["window"], c["sinks"]
    want = c["budget"] - c["window"]
    top = min(c["topk"] or want, lc - lead)
    group = c["heads"] // c["kv_heads"]
    qf, picks = q.float(), []
    for g in range(c["kv_heads"]):
        kf = k[g, lead:lc].float().t().contiguous()
        acc = torch.zeros((group, lc - lead), device=q.device)
        for i in range(D):
            acc = acc + qf[g * group: (g + 1) * group, i: i + 1] * kf[i]
        picks.append(acc.sort(dim=-1, descending=True, stable=True).indices[:, :top] + lead)
    flat = torch.cat(picks).t().reshape(-1).cpu().numpy()      # rank-major
    tokens, first = np.unique(flat, return_index=True)
    kept = np.sort(tokens[np.argsort(first)[: want - lead]])
    rho = np.concatenate([np.arange(lead), kept, np.arange(lc, n)])
    return torch.from_numpy(rho).to(q.device)


def exact(case, seed):
    c = case
    inp = _inputs(c, seed)
    lens = _lengths(c)
    kinds = {"sparse": [wl.LAYER_SPARSE], "full": [wl.LAYER_FULL], "select": [wl.LAYER_SELECT]}.get(c["kind"]) or _schedule(c)
    idx, cnt = _draw_rho(c, seed) if c["kind"] == "sparse" else (torch.zeros((c["batch"], c["budget"]), dtype=torch.int32, device=DEVICE), None)
    if cnt is None:
        cnt = torch.tensor([min(n, c["budget"]) for n in lens], dtype=torch.int32, device=DEVICE)
    outs = []
    for layer, kind in enumerate(kinds):
        out = torch.empty((c["batch"], c["heads"], D), dtype=torch.float64, device=DEVICE)
        for b, n in enumerate(lens):
            q = inp.layers[layer].q[b]
            k, v = _rows(c, inp, layer, b, n)
            if kind == wl.LAYER_SELECT:
                rho = _select_ref(c, q, k, n)
                idx[b, : len(rho)] = rho.to(torch.int32)
            out[b] = _attention64(c, q, k, v, idx[b, : cnt[b]].long() if kind == wl.LAYER_SPARSE else None)
        outs.append(out)
    if c["kind"] in ("sparse", "full"):
        return {"out": outs[0]}
    return {"out": outs[0] if c["kind"] == "select" else outs, "idx": idx, "cnt": cnt}
