"""Workloads that this library is timed and compared on, through its public entry points.

A case is a dict of plain values.  Five kinds of work:

    verify   one deterministic verify step: mask, DAG-masked attention, per-node argmax, longest accepted path
    sample   non-deterministic verification: softmax normalisers, acceptance, draw from the residual
    tree     un-merging a token graph into a token tree and verifying the tree (sizes are read back in between)
    commit   moving the accepted rows of a deep K/V cache behind the prefix
    graph    a drafted token tree -> pruned, merged token graph

Sizes of the listed cases are those of workload.CONFIGS and of bench.py's further legs, and generic ones between and
beside them.  All inputs are synthetic and come from the seed alone: Q, K, V ~ N(0, 1); verifier logits ~ N(0, 1) with
+5 on the token of one child of most nodes, so that acceptance is not trivial.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2407_16207_amd as gsd
from paper_2407_16207_amd.workload import merged_tree_dag, random_dag

VERIFY = {"kind": "verify", "dtype": "bf16", "batch": 1, "q_heads": 32, "kv_heads": 32, "head_dim": 128,
          "prefix_min": 1024, "prefix_max": 1024, "shape": "layered", "layers": 8, "width": 8, "parents": 2,
          "vocab": 32000, "plant": 0.7, "buffers": True, "normalisers": False}


def listed():
    return [
        # the smallest call there is: a first try of the library, a unit test of a caller; launches and host work count
        dict(VERIFY, name="verify_f32_tiny", dtype="f32", q_heads=4, kv_heads=4, head_dim=64, prefix_min=128,
             prefix_max=128, layers=4, width=4, vocab=1000),
        # full precision at the size of a 7B model's layer: what a user compares the bf16 path with
        dict(VERIFY, name="verify_f32_7b", dtype="f32"),
        # one user of a 7B-shaped model, short context: latency
        dict(VERIFY, name="verify_7b"),
        # four users of a 13B-shaped model without shared K/V heads: K/V traffic
        dict(VERIFY, name="verify_13b", batch=4, q_heads=40, kv_heads=40, prefix_min=2048, prefix_max=2048, layers=16,
             parents=3, plant=0.75),
        # one user of a 70B-shaped model with grouped heads, a small graph on a long context: few rows, long K/V axis
        dict(VERIFY, name="verify_70b_one", q_heads=64, kv_heads=8, prefix_min=4096, prefix_max=4096),
        # the headline configuration of bench.py
        dict(VERIFY, name="verify_70b", batch=8, q_heads=64, kv_heads=8, prefix_min=4096, prefix_max=4096, layers=32,
             parents=3, plant=0.8),
        # a full server: 32 sequences of very different length, the largest graphs
        dict(VERIFY, name="verify_70b_ragged", batch=32, q_heads=64, kv_heads=8, prefix_min=1024, prefix_max=8192,
             layers=64, parents=4, plant=0.8),
        # nothing round: head_dim 64, three query heads to a K/V head, graphs that are not layered, rows of logits that
        # start on no 16-byte boundary; the short call forms, with log-sum-exp and softmax normalisers asked for
        dict(VERIFY, name="verify_odd", batch=5, q_heads=24, kv_heads=8, head_dim=64, prefix_min=100, prefix_max=1500,
             shape="random", layers=77, width=1, parents=3, vocab=32003, buffers=False, normalisers=True),
        # sampling instead of greedy verification, on the headline configuration's graphs
        {"name": "sample_70b", "kind": "sample", "dtype": "bf16", "batch": 8, "layers": 32, "width": 8, "parents": 3,
         "vocab": 32000},
        # exact verification of token graphs as drafting makes them: trees with a few merged leaves
        {"name": "tree_70b", "kind": "tree", "dtype": "bf16", "batch": 8, "q_heads": 64, "kv_heads": 8, "head_dim": 128,
         "prefix": 4096, "nodes": 256, "merges": 10, "cap": 512, "vocab": 32000},
        # the accepted tokens become context: all layers of the headline configuration's cache
        {"name": "commit_70b", "kind": "commit", "dtype": "bf16", "batch": 8, "kv_heads": 8, "head_dim": 128,
         "prefix": 4096, "layers": 32, "width": 8, "cache_layers": 80},
        # drafting: eight trees of the largest size, pruning off so that all that recurs is merged
        {"name": "graph_512", "kind": "graph", "batch": 8, "nodes": 512, "degree": 4, "alphabet": 40, "tau": 2,
         "theta_prob": 0.0, "theta_sib": 0.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choice(["verify"] * 6 + ["sample"] * 2 + ["tree", "commit", "graph"])
    if kind == "verify":
        f32 = rng.random() < 0.2
        kv_heads, group = rng.choice([(4, 1), (4, 3), (4, 8), (8, 1), (8, 2), (8, 3), (8, 4), (8, 8), (16, 1), (16, 4), (32, 1), (40, 1)])
        width = rng.randint(1, 8)
        prefix = _log_int(rng, 64, 8192)
        return {"kind": "verify", "dtype": "f32" if f32 else "bf16", "batch": _log_int(rng, 1, 32),
                "q_heads": kv_heads * group, "kv_heads": kv_heads, "head_dim": rng.choice([64, 128, 128, 128]),
                "prefix_min": rng.choice([prefix, max(1, prefix // 4)]), "prefix_max": prefix,
                "shape": rng.choice(["layered", "layered", "random"]), "layers": _log_int(rng, 2, 64), "width": width,
                "parents": rng.randint(1, 4), "vocab": _log_int(rng, 1000, 64000), "plant": round(rng.uniform(0.6, 0.9), 2),
                "buffers": rng.random() < 0.6, "normalisers": rng.random() < 0.3}
    if kind == "sample":
        return {"kind": "sample", "dtype": rng.choice(["bf16", "bf16", "f32"]), "batch": _log_int(rng, 1, 16),
                "layers": _log_int(rng, 2, 48), "width": rng.randint(1, 8), "parents": rng.randint(1, 4),
                "vocab": rng.choice([32000, _log_int(rng, 1000, 64000), _log_int(rng, 1000, 64000)])}
    if kind == "tree":
        kv_heads = rng.choice([4, 8, 16])
        return {"kind": "tree", "dtype": "bf16", "batch": _log_int(rng, 1, 16), "q_heads": kv_heads * rng.choice([1, 4, 8]),
                "kv_heads": kv_heads, "head_dim": rng.choice([64, 128, 128]), "prefix": _log_int(rng, 64, 4096),
                "nodes": _log_int(rng, 16, 300), "merges": rng.randint(1, 10), "cap": 512, "vocab": _log_int(rng, 1000, 40000)}
    if kind == "commit":
        return {"kind": "commit", "dtype": rng.choice(["bf16", "bf16", "f32"]), "batch": _log_int(rng, 1, 16),
                "kv_heads": rng.choice([4, 8, 32]), "head_dim": rng.choice([64, 128, 128]), "prefix": _log_int(rng, 64, 4096),
                "layers": _log_int(rng, 2, 64), "width": rng.randint(2, 8), "cache_layers": rng.randint(1, 80)}
    pruned = rng.random() < 0.5
    return {"kind": "graph", "batch": _log_int(rng, 1, 64), "nodes": _log_int(rng, 16, 512), "degree": rng.randint(2, 8),
            "alphabet": _log_int(rng, 16, 2000), "tau": rng.randint(1, 4), "theta_prob": 0.2 if pruned else 0.0,
            "theta_sib": 0.3 if pruned else 0.0}


def draw(rng):
    """One more case from the same ranges; what would cost more than the largest listed one is drawn again."""
    top = {k: max(work(c)[k] for c in listed()) for k in ("bytes", "flops")}
    while True:
        c = _draw_once(rng)
        w = work(c)
        f32_top = 2e10 if c.get("dtype") == "f32" else top["flops"]     # full precision: the small and middle sizes only
        cache = _cache_bytes(c) if c["kind"] == "commit" else 0
        if w["bytes"] <= top["bytes"] and w["flops"] <= f32_top and cache <= 12e9:
            return c


# ------------------------------------------------------------------------------------------------- inputs

def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype, scale=1.0):
    """N(0, scale^2) in `dtype`, drawn in slabs so that the fp32 intermediate stays small."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    slab = 1 << 27
    for lo in range(0, flat.numel(), slab):
        part = flat[lo:lo + slab]
        part.copy_(torch.randn(part.numel(), generator=g, device="cuda", dtype=torch.float32).mul_(scale))
    return out


def _layered(rng, layers, width, max_parents):
    """Parents of a layered graph: layer 0 hangs off the root, the others draw 1..max_parents from the layer above."""
    offsets, parents = [0], []
    for layer in range(layers):
        order = np.argsort(rng.random((width, width)), axis=1)
        counts = np.minimum(rng.integers(1, max_parents + 1, width), width)
        for i in range(width):
            parents += [-1] if layer == 0 else sorted((order[i, :counts[i]] + (layer - 1) * width).tolist())
            offsets.append(len(parents))
    return offsets, parents


def _graphs(rng, case):
    """Packed token graphs: (node_offsets, parent_offsets, parent_idx) of the whole batch, int32 on the host."""
    node_offsets, parent_offsets, parent_idx = [0], [0], []
    for _ in range(case["batch"]):
        if case["kind"] == "tree":
            off, par = merged_tree_dag(rng, case["nodes"], 4, case["merges"])
        elif case.get("shape", "layered") == "layered":
            off, par = _layered(rng, case["layers"], case["width"], case["parents"])
        else:
            off, par = random_dag(rng, case["layers"] * case["width"], case["parents"])
        base = len(parent_idx)
        parent_offsets += [int(x) + base for x in off[1:]]
        parent_idx += [int(p) for p in par]
        node_offsets.append(node_offsets[-1] + len(off) - 1)
    return tuple(np.asarray(x, dtype=np.int32) for x in (node_offsets, parent_offsets, parent_idx))


def _edges(node_offsets, parent_offsets, parent_idx):
    """Per edge: (packed parent row, or -1 - sequence for the root; packed child row)."""
    child = np.repeat(np.arange(len(parent_offsets) - 1), np.diff(parent_offsets))
    seq = np.searchsorted(node_offsets, child, side="right") - 1
    return np.where(parent_idx < 0, -1 - seq, node_offsets[seq] + parent_idx), child


def _one_child_each(rng, parents, children, rows):
    """For every parent row one of its children at random, -1 where it has none."""
    order = rng.permutation(len(parents))
    pick = np.full(rows, -1, dtype=np.int64)
    pick[parents[order]] = children[order]
    return pick


def _planted_logits(g, rng, graphs, tokens, vocab, dtype, plant):
    """Verifier logits [T, vocab] and root_pred [B]: noise, and a bump on one child's token at most nodes."""
    node_offsets, parent_offsets, parent_idx = graphs
    total, batch = len(tokens), len(node_offsets) - 1
    logits = _normal(g, (total, vocab), dtype)
    parents, children = _edges(*graphs)
    inner = parents >= 0
    pick = _one_child_each(rng, parents[inner], children[inner], total)
    pick[rng.random(total) >= plant] = -1
    rows = np.nonzero(pick >= 0)[0]
    at = (_dev(rows), _dev(tokens[pick[rows]].astype(np.int64)))
    logits[at] = (logits[at].float() + 5.0).to(dtype)
    root_pick = _one_child_each(rng, -1 - parents[~inner], children[~inner], batch)
    root_pred = np.where((root_pick >= 0) & (rng.random(batch) < plant), tokens[root_pick], rng.integers(0, vocab, batch))
    return logits, root_pred.astype(np.int32)


def _prepare_verify(case, seed):
    rng, g, dtype = np.random.default_rng(seed), _generator(seed), _dtype(case)
    graphs = _graphs(rng, case)
    node_offsets = graphs[0]
    batch, total, n = case["batch"], int(node_offsets[-1]), int(np.diff(node_offsets).max())
    tokens = rng.integers(0, case["vocab"], total).astype(np.int32)
    prefix = rng.integers(case["prefix_min"], case["prefix_max"] + 1, batch).astype(np.int32)
    rows = prefix.astype(np.int64) + np.diff(node_offsets)
    kv_offsets = np.concatenate([[0], np.cumsum(rows)[:-1]]).astype(np.int64)
    logits, root_pred = _planted_logits(g, rng, graphs, tokens, case["vocab"], dtype, case["plant"])
    s = {"node_offsets": _dev(graphs[0]), "parent_offsets": _dev(graphs[1]), "parent_idx": _dev(graphs[2]),
         "tokens": _dev(tokens), "root_pred": _dev(root_pred), "prefix": _dev(prefix), "kv_offsets": _dev(kv_offsets),
         "q": _normal(g, (total, case["q_heads"], case["head_dim"]), dtype),
         "k": _normal(g, (int(rows.sum()), case["kv_heads"], case["head_dim"]), dtype),
         "v": _normal(g, (int(rows.sum()), case["kv_heads"], case["head_dim"]), dtype),
         "logits": logits, "n": n, "max_prefix": int(prefix.max()), "scale": 1.0 / math.sqrt(case["head_dim"]),
         "normalisers": case["normalisers"], "desc": None}
    if case["buffers"]:      # a serving loop keeps its outputs, its workspace and the descriptor that names them
        s["mask"] = torch.empty((total, (n + 63) // 64), dtype=torch.int64, device="cuda")
        s["out"] = torch.empty_like(s["q"])
        s["pred"] = torch.empty(total, dtype=torch.int32, device="cuda")
        s["accept_len"] = torch.empty(batch, dtype=torch.int32, device="cuda")
        s["accept_path"] = torch.empty((batch, n), dtype=torch.int32, device="cuda")
        s["bonus"] = torch.empty(batch, dtype=torch.int32, device="cuda")
        if case["normalisers"]:
            s["row_max"] = torch.empty(total, dtype=torch.float32, device="cuda")
            s["row_sumexp"] = torch.empty(total, dtype=torch.float32, device="cuda")
        desc = gsd.make_attn_desc(s["q"], s["k"], s["v"], s["kv_offsets"], s["prefix"], s["node_offsets"], s["mask"], n,
                                  s["max_prefix"], s["scale"], out=s["out"])
        need = gsd.gsd_dag_attention_workspace(desc)
        s["workspace"] = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
        desc.workspace, desc.workspace_bytes = s["workspace"].data_ptr(), need
        s["desc"] = desc
    return s


def _prepare_sample(case, seed):
    rng, g, dtype = np.random.default_rng(seed), _generator(seed), _dtype(case)
    graphs = _graphs(rng, case)
    batch, total, vocab = case["batch"], int(graphs[0][-1]), case["vocab"]
    # peaked like a trained model's, and a drafter that agrees with the verifier on most of it
    both = _normal(g, (total + batch, vocab), dtype, 3.0)
    draft = _normal(g, (total + batch, vocab), dtype, 1.5)
    draft.add_(both, alpha=0.8)
    parents, children = _edges(*graphs)
    row_of = np.zeros(total, dtype=np.int64)             # the row whose draft distribution a node's token comes from
    row_of[children[::-1]] = np.where(parents >= 0, parents, total - 1 - parents)[::-1]
    tokens, prob = [], []
    for lo in range(0, total, 1024):
        q = torch.softmax(draft[_dev(row_of[lo:lo + 1024])].float(), dim=1)
        t = torch.multinomial(q, 1, generator=g)
        tokens.append(t[:, 0].to(torch.int32))
        prob.append(q.gather(1, t)[:, 0].clamp_min(1e-6))
    return {"node_offsets": _dev(graphs[0]), "parent_offsets": _dev(graphs[1]), "parent_idx": _dev(graphs[2]),
            "tokens": torch.cat(tokens), "draft_prob": torch.cat(prob), "n": int(np.diff(graphs[0]).max()),
            "logits": both[:total], "root_logits": both[total:], "draft_logits": draft[:total],
            "root_draft_logits": draft[total:], "accept_u": torch.rand(total, generator=g, device="cuda"),
            "resample_u": torch.rand(batch, generator=g, device="cuda")}


def _prepare_tree(case, seed):
    rng, g, dtype = np.random.default_rng(seed), _generator(seed), _dtype(case)
    graphs = _graphs(rng, case)
    batch, total, cap, prefix = case["batch"], int(graphs[0][-1]), case["cap"], case["prefix"]
    tokens = rng.integers(0, case["vocab"], total).astype(np.int32)
    logits, root_pred = _planted_logits(g, rng, graphs, tokens, case["vocab"], dtype, 0.8)
    rows = batch * (prefix + cap)                        # a cache with room for the largest tree of every sequence
    return {"node_offsets": _dev(graphs[0]), "parent_offsets": _dev(graphs[1]), "parent_idx": _dev(graphs[2]),
            "tokens": _dev(tokens), "root_pred": _dev(root_pred), "n": case["nodes"], "cap": cap, "max_prefix": prefix,
            "prefix": _dev(np.full(batch, prefix, dtype=np.int32)),
            "kv_offsets": _dev(np.arange(batch, dtype=np.int64) * (prefix + cap)),
            "q": _normal(g, (total, case["q_heads"], case["head_dim"]), dtype),
            "k": _normal(g, (rows, case["kv_heads"], case["head_dim"]), dtype),
            "v": _normal(g, (rows, case["kv_heads"], case["head_dim"]), dtype),
            "logits": logits, "scale": 1.0 / math.sqrt(case["head_dim"]),
            # outputs at the size of the largest tree; a pass fills as much of them as its trees take
            "mask": torch.zeros(batch * cap * (cap // 64), dtype=torch.int64, device="cuda"),
            "out": torch.zeros((batch * cap, case["q_heads"], case["head_dim"]), dtype=dtype, device="cuda"),
            "accept_path": torch.zeros(batch * cap, dtype=torch.int32, device="cuda")}


def _prepare_commit(case, seed):
    rng, g = np.random.default_rng(seed), _generator(seed)
    batch, n, depth = case["batch"], case["layers"] * case["width"], case["layers"]
    rows = batch * (case["prefix"] + n)
    shape = (case["cache_layers"], rows, case["kv_heads"], case["head_dim"])
    path = np.full((batch, n), -1, dtype=np.int32)
    path[:, :depth] = np.arange(depth) * case["width"] + rng.integers(0, case["width"], (batch, depth))
    length = rng.integers((depth + 1) // 2, depth + 1, batch).astype(np.int32)      # some stop early, none at once
    path[np.arange(n)[None, :] >= length[:, None]] = -1
    return {"k": _normal(g, shape, _dtype(case)), "v": _normal(g, shape, _dtype(case)),
            "kv_offsets": _dev(np.arange(batch, dtype=np.int64) * (case["prefix"] + n)),
            "prefix": _dev(np.full(batch, case["prefix"], dtype=np.int32)), "accept_len": _dev(length),
            "accept_path": _dev(path), "new_prefix": torch.empty(batch, dtype=torch.int32, device="cuda")}


def _prepare_graph(case, seed):
    rng = np.random.default_rng(seed)
    node_offsets, parent, tokens, prob = [0], [], [], []
    for _ in range(case["batch"]):
        here, frontier = 0, [-1]
        while here < case["nodes"]:                      # breadth first; every expanded node has at least one child
            below = []
            for node in frontier:
                kids = min(int(rng.integers(1, case["degree"] + 1)), case["nodes"] - here)
                weights = rng.exponential(size=kids + 1)
                prob += sorted((weights[:kids] / weights.sum()).tolist(), reverse=True)
                parent += [node] * kids
                below += range(here, here + kids)
                here += kids
            frontier = below
        node_offsets.append(len(parent))
    tokens = rng.integers(0, case["alphabet"], len(parent))
    return {"node_offsets": _dev(np.asarray(node_offsets, dtype=np.int32)), "parent": _dev(np.asarray(parent, dtype=np.int32)),
            "tokens": _dev(tokens.astype(np.int32)), "prob": _dev(np.asarray(prob, dtype=np.float32)), "n": case["nodes"],
            # the graph as the next step's launches take it: one array of fixed size, as much of it filled as there is
            "packed": torch.zeros(12 * len(parent) + 1, dtype=torch.int32, device="cuda"),
            "tau": case["tau"], "theta_prob": case["theta_prob"], "theta_sib": case["theta_sib"]}


def prepare(case, seed):
    make = {"verify": _prepare_verify, "sample": _prepare_sample, "tree": _prepare_tree, "commit": _prepare_commit,
            "graph": _prepare_graph}[case["kind"]]
    state = make(case, seed)
    state["kind"] = case["kind"]
    return state


# ------------------------------------------------------------------------------------------------- one pass

def _run_verify(s):
    graph = (s["node_offsets"], s["parent_offsets"], s["parent_idx"])
    if s["desc"] is not None:
        gsd.gsd_build_mask(*graph, s["n"], mask=s["mask"])
        gsd.gsd_dag_attention_desc(s["desc"])
        kept = dict(accept_len=s["accept_len"], accept_path=s["accept_path"], bonus_token=s["bonus"])
        out = [s["mask"], s["out"]]
        if s["normalisers"]:
            gsd.gsd_node_argmax_stats(s["logits"], s["pred"], s["row_max"], s["row_sumexp"])
            out += [s["row_max"], s["row_sumexp"]]
            out += gsd.gsd_accept_longest_path(*graph, s["tokens"], s["root_pred"], s["n"], pred=s["pred"], **kept)
        else:
            out += gsd.gsd_accept_longest_path(*graph, s["tokens"], s["root_pred"], s["n"], logits=s["logits"],
                                               pred=s["pred"], **kept)
        return out
    mask = gsd.gsd_build_mask(*graph, s["n"])
    attention = (s["q"], s["k"], s["v"], s["kv_offsets"], s["prefix"], s["node_offsets"], mask, s["n"], s["max_prefix"],
                 s["scale"])
    if s["normalisers"]:
        out = [mask, *gsd.gsd_dag_attention(*attention, return_lse=True)]
        pred, row_max, row_sumexp = gsd.gsd_node_argmax_stats(s["logits"])
        out += [row_max, row_sumexp]
        out += gsd.gsd_accept_longest_path(*graph, s["tokens"], s["root_pred"], s["n"], pred=pred)
    else:
        out = [mask, gsd.gsd_dag_attention(*attention)]
        out += gsd.gsd_accept_longest_path(*graph, s["tokens"], s["root_pred"], s["n"], logits=s["logits"])
    return out


def _run_sample(s):
    return gsd.gsd_accept_stochastic(s["node_offsets"], s["parent_offsets"], s["parent_idx"], s["tokens"], s["logits"],
                                     s["root_logits"], s["draft_logits"], s["root_draft_logits"], s["draft_prob"],
                                     s["accept_u"], s["resample_u"], s["n"])


def _run_tree(s):
    offsets, parent, parent_offsets, origin, paths = gsd.gsd_unmerge_to_tree(
        s["node_offsets"], s["parent_offsets"], s["parent_idx"], s["n"], s["cap"])
    sizes = np.diff(offsets.cpu().numpy())               # the calls below are sized by the tree
    total, n = int(sizes.sum()), int(sizes.max())
    first = torch.repeat_interleave(s["node_offsets"][:-1], offsets.diff(), output_size=total)
    origin, parent, parent_offsets = origin[:total], parent[:total], parent_offsets[:total + 1]
    source = first + origin                              # packed graph row of every tree node
    q = gsd.gsd_gather_rows(s["q"], source)
    tokens = gsd.gsd_gather_rows(s["tokens"], source)
    pred = gsd.gsd_gather_rows(gsd.gsd_node_argmax(s["logits"]), source)
    words, batch = (n + 63) // 64, len(sizes)
    mask = gsd.gsd_build_mask(offsets, parent_offsets, parent, n, mask=s["mask"][:total * words].view(total, words))
    gsd.gsd_dag_attention(q, s["k"], s["v"], s["kv_offsets"], s["prefix"], offsets, mask, n, s["max_prefix"], s["scale"],
                          out=s["out"][:total])
    length, _, bonus, _ = gsd.gsd_accept_longest_path(offsets, parent_offsets, parent, tokens, s["root_pred"], n, pred=pred,
                                                      accept_path=s["accept_path"][:batch * n].view(batch, n))
    return [offsets, paths, s["mask"], s["out"], length, s["accept_path"], bonus]


def _run_commit(s):
    gsd.gsd_commit_kv(s["k"], s["v"], s["kv_offsets"], s["prefix"], s["accept_len"], s["accept_path"],
                      new_prefix_lens=s["new_prefix"])
    return [s["k"], s["v"], s["new_prefix"]]


def _run_graph(s):
    # only the entries below the counts that come back are written; a caller reads the counts before it uses the rest
    offsets, parent_offsets, parent_idx, origin, flags, counts = gsd.gsd_build_token_graph(
        s["node_offsets"], s["parent"], s["tokens"], s["prob"], s["n"], s["tau"], s["theta_prob"], s["theta_sib"])
    nodes, edges = counts.cpu().sum(0).tolist()
    torch.cat([parent_offsets[:nodes + 1], parent_idx[:edges], origin[:nodes], flags[:nodes]],
              out=s["packed"][:3 * nodes + 1 + edges])
    return [offsets, counts, s["packed"]]


def run(state):
    return {"verify": _run_verify, "sample": _run_sample, "tree": _run_tree, "commit": _run_commit,
            "graph": _run_graph}[state["kind"]](state)


# ------------------------------------------------------------------------------------------------- what it takes

def _cache_bytes(case):
    elt = 4 if case["dtype"] == "f32" else 2
    rows = case["batch"] * (case["prefix"] + case["layers"] * case["width"])
    return 2.0 * case["cache_layers"] * rows * case["kv_heads"] * case["head_dim"] * elt


def work(case):
    """Bytes: every input once, every output once.  Flops: two per multiply-add of the two attention contractions over
    the keys a node sees on average (a layered graph shows a node about half of its sequence, the others a few nodes)."""
    elt = 4 if case.get("dtype") == "f32" else 2
    batch = case["batch"]
    if case["kind"] == "graph":
        nodes = batch * case["nodes"]
        return {"bytes": nodes * (3 * 4 + 4 * 4.0), "flops": 0.0}
    if case["kind"] == "commit":
        moved = batch * 0.75 * case["layers"]            # accepted lengths are uniform over the upper half of the depth
        return {"bytes": 4.0 * case["cache_layers"] * moved * case["kv_heads"] * case["head_dim"] * elt + 8.0 * batch, "flops": 0.0}
    if case["kind"] == "sample":
        total = batch * case["layers"] * case["width"]
        return {"bytes": float((total + 2 * batch) * case["vocab"] * elt + 40 * total), "flops": 0.0}
    n = case["nodes"] if case["kind"] == "tree" else case["layers"] * case["width"]
    prefix = case["prefix"] if case["kind"] == "tree" else (case["prefix_min"] + case["prefix_max"]) / 2
    total, seen = batch * n, n / 2 if case.get("shape") == "layered" else min(n / 2, 16)
    heads = case["q_heads"] * case["head_dim"]
    kv = 2.0 * batch * (prefix + n) * case["kv_heads"] * case["head_dim"]
    return {"bytes": elt * (kv + 2.0 * total * heads + float(total) * case["vocab"]) + total * (n / 8.0 + 24),
            "flops": 4.0 * total * heads * (prefix + seen)}


def tolerance(case):
    """Ids, masks, paths and committed rows are whole values or copies: the same bits.  bf16 attention rounds P and O to
    bf16 (2^-9 each); fp32 attention and the softmax normalisers are fp32 sums."""
    if case["kind"] in ("commit", "graph"):
        return "exact"
    if case["kind"] == "sample" or case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 4e-2}
