"""The native part of the Python binding (csrc/binding.cpp) against the Python it stands in for: the same results, the caller's own
tensors handed back, the same exceptions, and everything that is not a plain tensor left to Python."""
import numpy as np
import pytest
import torch

import paper_2407_16207_amd as gsd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def args():
    g = torch.Generator(device="cuda").manual_seed(1)
    dev = lambda x, t=torch.int32: torch.tensor(x, dtype=t, device="cuda")
    n = 6
    graph = (dev([0, n]), dev([0, 1, 2, 3, 5, 6, 7]), dev([-1, 0, 0, 1, 2, 3, 4]))
    heads, dim, prefix = 4, 64, 40
    a = {"graph": graph, "n": n, "tokens": dev([1, 2, 3, 4, 5, 6]), "root_pred": dev([1]), "prefix": dev([prefix]),
         "kv_offsets": dev([0], torch.int64), "max_prefix": prefix, "mask": gsd.gsd_build_mask(*graph, n)}
    for dtype in (torch.float32, torch.bfloat16):
        r = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(dtype)
        a[dtype] = {"q": r(n, heads, dim), "k": r(prefix + n, 2, dim), "v": r(prefix + n, 2, dim), "logits": r(n, 1000)}
    return a


def both(monkeypatch, call):
    """What `call` returns or raises with the native part and without."""
    assert gsd._short is not None, "the binding's native part has not been built"
    got = []
    for short in (gsd._short, None):
        with monkeypatch.context() as m:
            m.setattr(gsd, "_short", short)
            try:
                got.append(call())
            except Exception as e:        # noqa: BLE001 - compared below
                got.append((type(e), str(e)))
    torch.cuda.synchronize()
    return got


def flat(x):
    return list(x) if isinstance(x, (tuple, list)) else [x]


def same(monkeypatch, call):
    a, b = (flat(x) for x in both(monkeypatch, call))
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert type(x) is torch.Tensor and x.dtype == y.dtype and x.shape == y.shape and x.stride() == y.stride()
        assert x.device == y.device and torch.equal(x, y)


def attention_args(a, dtype):
    t = a[dtype]
    return (t["q"], t["k"], t["v"], a["kv_offsets"], a["prefix"], a["graph"][0], a["mask"], a["n"], a["max_prefix"], 0.125)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_results_are_the_same(args, monkeypatch, dtype):
    a, t = args, args[dtype]
    wide = torch.cat([t["logits"], t["logits"]], 1)[:, 3:1003]                     # rows that are not side by side
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for kw in ({}, {"words_per_row": 3}, {"mask": torch.zeros((a["n"], 1), dtype=torch.int64, device="cuda")},
               {"dag_error_flag": torch.zeros(1, dtype=torch.int32, device="cuda")}, {"stream": side}):
        same(monkeypatch, lambda: gsd.gsd_build_mask(*a["graph"], a["n"], **kw))
    for x in (t["logits"], wide):
        same(monkeypatch, lambda: gsd.gsd_node_argmax(x))
        same(monkeypatch, lambda: gsd.gsd_node_argmax_stats(x))
        same(monkeypatch, lambda: gsd.gsd_accept_longest_path(*a["graph"], a["tokens"], a["root_pred"], a["n"], logits=x))
    pred = gsd.gsd_node_argmax(t["logits"])
    same(monkeypatch, lambda: gsd.gsd_accept_longest_path(*a["graph"], a["tokens"], a["root_pred"], a["n"], pred=pred))
    for kw in ({}, {"return_lse": True}, {"num_splits": 2}, {"out": torch.zeros_like(t["q"])}, {"stream": side},
               {"lse": torch.zeros((a["n"], 4), device="cuda"), "return_lse": True},
               {"workspace": torch.zeros(1 << 16, dtype=torch.uint8, device="cuda"), "num_splits": 2}):
        same(monkeypatch, lambda: gsd.gsd_dag_attention(*attention_args(a, dtype), **kw))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_results_of_the_surrounding_calls_are_the_same(args, monkeypatch, dtype):
    a, t, short = args, args[dtype], gsd._short
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    for kw in ({}, {"dag_error_flag": flag}):
        got = both(monkeypatch, lambda: gsd.gsd_unmerge_to_tree(*a["graph"], a["n"], 32, **kw))
        size = int(got[0][0][-1])
        assert size > a["n"] and [x.shape for x in got[0]] == [x.shape for x in got[1]]
        assert all(torch.equal(x[:k], y[:k]) for x, y, k in zip(*got, (2, size, size + 1, size, 1)))      # what the call writes
    index = torch.tensor([4, 0, 0, 5], dtype=torch.int32, device="cuda")
    for src in (t["q"], a["tokens"], t["logits"], t["logits"][:, 2:], t["q"][:1]):
        i = index.clamp(max=src.shape[0] - 1).to(torch.int32)
        same(monkeypatch, lambda: gsd.gsd_gather_rows(src, i))
        same(monkeypatch, lambda: gsd.gsd_gather_rows(src, i, rows=3))
        same(monkeypatch, lambda: gsd.gsd_gather_rows(src, i, out=torch.zeros((6, *src.shape[1:]), dtype=src.dtype, device="cuda")))
    same(monkeypatch, lambda: gsd.gsd_softmax_stats(t["logits"]))
    same(monkeypatch, lambda: gsd.gsd_softmax_stats(t["logits"][:, 1:]))
    path = torch.tensor([[1, 3, 5, -1, -1, -1]], dtype=torch.int32, device="cuda")
    length = torch.tensor([3], dtype=torch.int32, device="cuda")

    def commit(cut):
        k, v = torch.stack([t["k"]] * 3), torch.stack([t["v"]] * 3)
        k, v = (k, v) if cut is None else (k[0], v[0]) if cut == 3 else (k[:, :, :1], v[:, :, :1])
        return gsd.gsd_commit_kv(k, v, a["kv_offsets"], a["prefix"], length, path), k, v
    for cut in (None, 3, 1):
        same(monkeypatch, lambda: commit(cut))
    n, u = a["n"], torch.linspace(0, 0.9, a["n"], device="cuda")
    for p, q in ((t["logits"], t["logits"].roll(1, 0)), (t["logits"][:, 3:], t["logits"].roll(1, 0)[:, 3:])):
        same(monkeypatch, lambda: gsd.gsd_accept_stochastic(*a["graph"], a["tokens"], p, p[2:3], q, q[2:3], u + 0.05, u, u[:1], n))
    tree = (a["graph"][0], torch.tensor([-1, -1, 0, 0, 1, 2], dtype=torch.int32, device="cuda"),
            torch.tensor([1, 2, 2, 3, 3, 3], dtype=torch.int32, device="cuda"), u)
    for kw in ({}, {"edge_capacity": 20}, {"error_flag": flag}):
        got = both(monkeypatch, lambda: gsd.gsd_build_token_graph(*tree, n, 1, 0.0, 0.0, **kw))
        nodes, edges = got[0][5][0].tolist()
        assert [x.shape for x in got[0]] == [x.shape for x in got[1]]
        assert all(torch.equal(x[:k], y[:k]) for x, y, k in zip(*got, (2, nodes + 1, edges, nodes, nodes, 1)))
    # and all of these are short ways
    assert short.unmerge_to_tree(*a["graph"], n, 32, None, None) is not None and short.gather_rows(t["q"], index, None, None, None) is not None
    assert short.softmax_stats(t["logits"], None, None, None) is not None
    assert short.commit_kv(torch.stack([t["k"]] * 3), torch.stack([t["v"]] * 3), a["kv_offsets"], a["prefix"], length, path, None, None) is not None
    assert short.accept_stochastic(*a["graph"], a["tokens"], *[t["logits"], t["logits"][:1]] * 2, u, u, u[:1], n, None) is not None
    assert short.build_token_graph(*tree, n, 1, 0.0, 0.0, None, None, None) is not None
    torch.cuda.synchronize()


def test_the_callers_tensors_come_back(args, monkeypatch):
    a, t = args, args[torch.bfloat16]
    kept = {name: torch.empty(shape, dtype=torch.int32, device="cuda") for name, shape in
            (("pred", (a["n"],)), ("accept_len", (1,)), ("accept_path", (1, a["n"])), ("bonus_token", (1,)))}
    mask, out, lse = torch.empty_like(a["mask"]), torch.empty_like(t["q"]), torch.empty((a["n"], 4), device="cuda")
    for got in both(monkeypatch, lambda: gsd.gsd_accept_longest_path(*a["graph"], a["tokens"], a["root_pred"], a["n"],
                                                                    logits=t["logits"], **kept)):
        assert all(x is kept[name] for x, name in zip(got, ("accept_len", "accept_path", "bonus_token", "pred")))
    assert all(x is mask for x in both(monkeypatch, lambda: gsd.gsd_build_mask(*a["graph"], a["n"], mask=mask)))
    for got in both(monkeypatch, lambda: gsd.gsd_dag_attention(*attention_args(a, torch.bfloat16), out=out, lse=lse, return_lse=True)):
        assert got[0] is out and got[1] is lse


def test_plain_tensors_take_the_short_way(args):
    a, t = args, args[torch.bfloat16]
    short = gsd._short
    assert short.build_mask(*a["graph"], a["n"], None, None, None, None) is not None
    assert short.node_argmax(t["logits"], None, None) is not None
    assert short.node_argmax_stats(torch.nn.Parameter(t["logits"]), None, None, None, None) is not None
    assert short.accept_longest_path(*a["graph"], a["tokens"], a["root_pred"], a["n"], t["logits"], None, None, None, None, None) is not None
    assert short.dag_attention(*attention_args(a, torch.bfloat16), None, None, 2, 0, True, None) is not None
    torch.cuda.synchronize()


class Subclass(torch.Tensor):
    pass


def test_exceptions_are_the_same(args, monkeypatch):
    a, t = args, args[torch.float32]
    att = attention_args(a, torch.float32)
    half, host, wrong, u = t["q"].half(), a["graph"][0].cpu(), a["graph"][0].long(), torch.ones(a["n"], device="cuda")
    calls = [lambda: gsd.gsd_build_mask(host, *a["graph"][1:], a["n"]), lambda: gsd.gsd_build_mask(wrong, *a["graph"][1:], a["n"]),
             lambda: gsd.gsd_build_mask(*a["graph"], 0), lambda: gsd.gsd_build_mask(*a["graph"], 513), lambda: gsd.gsd_build_mask(*a["graph"], 1 << 40),
             lambda: gsd.gsd_build_mask(*a["graph"], a["n"], mask=a["mask"][:3]), lambda: gsd.gsd_build_mask(*a["graph"], 80, words_per_row=1),
             lambda: gsd.gsd_node_argmax(half.flatten(1)), lambda: gsd.gsd_node_argmax(t["logits"].t()), lambda: gsd.gsd_node_argmax(t["logits"][:0]),
             lambda: gsd.gsd_node_argmax(t["logits"], pred=wrong), lambda: gsd.gsd_node_argmax_stats(t["logits"], row_max=wrong),
             lambda: gsd.gsd_accept_longest_path(*a["graph"], a["tokens"], a["root_pred"], a["n"]),
             lambda: gsd.gsd_accept_longest_path(*a["graph"], a["tokens"], a["root_pred"], a["n"], logits=t["logits"][:3]),
             lambda: gsd.gsd_dag_attention(half, *att[1:]), lambda: gsd.gsd_dag_attention(att[0][:, :3], *att[1:]),
             lambda: gsd.gsd_dag_attention(*att[:2], att[2][:-1], *att[3:]), lambda: gsd.gsd_dag_attention(*att[:-1], -1.0),
             lambda: gsd.gsd_dag_attention(*att[:-1], 1e39), lambda: gsd.gsd_dag_attention(*att, num_splits=-1),
             lambda: gsd.gsd_unmerge_to_tree(*a["graph"], a["n"], 0), lambda: gsd.gsd_unmerge_to_tree(*a["graph"], 513, 8),
             lambda: gsd.gsd_unmerge_to_tree(wrong, *a["graph"][1:], a["n"], 8), lambda: gsd.gsd_gather_rows(t["q"], wrong),
             lambda: gsd.gsd_gather_rows(t["q"], a["tokens"], out=half), lambda: gsd.gsd_gather_rows(t["q"][:0], a["tokens"]),
             lambda: gsd.gsd_gather_rows(half[:, 0, :1], a["tokens"]), lambda: gsd.gsd_softmax_stats(half.flatten(1)),
             lambda: gsd.gsd_softmax_stats(t["logits"][:0]),
             lambda: gsd.gsd_commit_kv(t["k"], t["v"][:3], a["kv_offsets"], a["prefix"], a["root_pred"], a["tokens"][None]),
             lambda: gsd.gsd_commit_kv(t["k"][None], t["v"][None], a["kv_offsets"], a["prefix"], a["root_pred"], a["tokens"][None],
                                       new_prefix_lens=a["prefix"]),
             lambda: gsd.gsd_accept_stochastic(*a["graph"], a["tokens"], t["logits"], t["logits"][:1], t["logits"], t["logits"][:2], u, u,
                                               u[:1], a["n"]),
             lambda: gsd.gsd_accept_stochastic(*a["graph"], a["tokens"], *[t["logits"], t["logits"][:1]] * 2, u, u, u[:1], 513),
             lambda: gsd.gsd_build_token_graph(a["graph"][0], a["tokens"], a["tokens"], u, a["n"], 0, 0.0, 0.0),
             lambda: gsd.gsd_build_token_graph(a["graph"][0], a["tokens"], a["tokens"], u, a["n"], 1, -1.0, 0.0),
             lambda: gsd.gsd_build_token_graph(a["graph"][0], a["tokens"], a["tokens"], u, a["n"], 1, 0.0, 0.0, edge_capacity=0),
             lambda: gsd.gsd_dag_attention(*att, lse=wrong), lambda: gsd.gsd_dag_attention(*att[:6], att[6][:, 0], *att[7:])]
    for k, call in enumerate(calls):
        x, y = both(monkeypatch, call)
        assert isinstance(x, tuple) and isinstance(x[0], type) and x == y, (k, x, y)


def test_outputs_that_a_call_would_write_past_are_refused_either_way(args, monkeypatch):
    """Refused on the host, with nothing launched; a larger buffer is as good as the exact one."""
    a, t = args, args[torch.bfloat16]
    i4 = lambda *shape: torch.full(shape, 7, dtype=torch.int32, device="cuda")
    f4 = lambda *shape: torch.full(shape, 7.0, device="cuda")
    n, q = a["n"], t["q"]
    accept = {"pred": i4(n), "accept_len": i4(1), "accept_path": i4(1, n), "bonus_token": i4(1)}
    cache = torch.stack([t["k"]] * 2)
    calls = [(lambda **kw: gsd.gsd_node_argmax(t["logits"], **kw), {"pred": i4(n)}),
             (lambda **kw: gsd.gsd_node_argmax_stats(t["logits"], **kw), {"pred": i4(n), "row_max": f4(n), "row_sumexp": f4(n)}),
             (lambda **kw: gsd.gsd_softmax_stats(t["logits"], **kw), {"row_max": f4(n), "row_sumexp": f4(n)}),
             (lambda **kw: gsd.gsd_accept_longest_path(*a["graph"], a["tokens"], a["root_pred"], n, logits=t["logits"], **kw), accept),
             (lambda **kw: gsd.gsd_commit_kv(cache, cache.clone(), a["kv_offsets"], a["prefix"], i4(1) * 0, i4(1, n) * 0, **kw),
              {"new_prefix_lens": i4(1)}),
             (lambda **kw: gsd.gsd_dag_attention(*attention_args(a, torch.bfloat16), return_lse=True, **kw),
              {"out": torch.zeros_like(q), "lse": f4(n, 4)})]
    for call, outputs in calls:
        for name, full in outputs.items():
            for wrong in (full[:-1], full[:0]) + ((full[:, :-1].contiguous(),) if full.dim() > 1 else ()):
                x, y = both(monkeypatch, lambda: call(**{**outputs, name: wrong}))
                assert isinstance(x, tuple) and x[0] is ValueError and x == y, (name, x, y)
            longer = torch.full((full.shape[0] + 1, *full.shape[1:]), 7, dtype=full.dtype, device="cuda")
            same(monkeypatch, lambda: call(**{**outputs, name: longer}))
            assert (longer[full.shape[0]:] == 7).all()
    for wrong in (q.float(), torch.zeros(n, 4, 128, dtype=q.dtype, device="cuda")[:, :, ::2], torch.zeros(n, 4, 64, dtype=q.dtype)):
        x, y = both(monkeypatch, lambda: gsd.gsd_dag_attention(*attention_args(a, torch.bfloat16), out=wrong))
        assert isinstance(x, tuple) and x[0] is ValueError and x == y


def test_inputs_that_a_call_would_read_past_are_refused_either_way(args, monkeypatch):
    a, t, short = args, args[torch.float32], lambda x: x[:-1]
    att, n, u = attention_args(a, torch.float32), a["n"], torch.ones(a["n"], device="cuda")
    length, path = a["root_pred"] * 0, a["tokens"][None] * 0
    cache = torch.stack([t["k"]] * 2)
    both_logits = [t["logits"], t["logits"][:1]] * 2
    for call in (lambda: gsd.gsd_dag_attention(*att[:3], short(att[3]), *att[4:]), lambda: gsd.gsd_dag_attention(*att[:5], short(att[5]), *att[6:]),
                 lambda: gsd.gsd_accept_longest_path(*a["graph"], a["tokens"], short(a["root_pred"]), n, logits=t["logits"]),
                 lambda: gsd.gsd_commit_kv(cache, cache, short(a["kv_offsets"]), a["prefix"], length, path),
                 lambda: gsd.gsd_commit_kv(cache, cache, a["kv_offsets"], a["prefix"], short(length), path),
                 lambda: gsd.gsd_commit_kv(cache, cache, a["kv_offsets"], a["prefix"], length, short(path)),
                 lambda: gsd.gsd_gather_rows(t["q"], a["tokens"] - 1, rows=n + 1),
                 lambda: gsd.gsd_accept_stochastic(*a["graph"], a["tokens"], *both_logits, u, u, u[:0], n)):
        x, y = both(monkeypatch, call)
        assert isinstance(x, tuple) and x[0] is ValueError and x == y, (x, y)


def test_other_tensors_go_the_long_way(args):
    """Subclasses, and calls under a torch mode that wants to see them."""
    from torch.utils._python_dispatch import TorchDispatchMode
    a, t = args, args[torch.float32]
    assert gsd._short.node_argmax(t["logits"].as_subclass(Subclass), None, None) is None
    assert gsd._short.node_argmax(t["logits"].cpu(), None, None) is None

    class Seen(TorchDispatchMode):
        names = []

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.names.append(func.name())
            return func(*args, **(kwargs or {}))
    with Seen() as seen:
        assert gsd._short.node_argmax(t["logits"], None, None) is None
        pred = gsd.gsd_node_argmax(t["logits"])
    assert any("empty" in name for name in seen.names)
    assert torch.equal(pred, gsd.gsd_node_argmax(t["logits"]))
    assert torch.equal(gsd.gsd_node_argmax(t["logits"].as_subclass(Subclass)), pred)
    assert torch.equal(gsd.gsd_node_argmax(torch.nn.Parameter(t["logits"])), pred)


def test_an_allocation_that_fails(args, monkeypatch):
    """2^31 - 1 words for each of 2^16 nodes: more than any memory.  The exception of torch.empty, and calls go on after it."""
    nodes, _, parents = args["graph"]
    offsets = torch.zeros((1 << 16) + 1, dtype=torch.int32, device="cuda")
    got = both(monkeypatch, lambda: gsd.gsd_build_mask(nodes, offsets, parents, 6, words_per_row=2**31 - 1))
    assert [x[0] for x in got] == [torch.OutOfMemoryError] * 2
    same(monkeypatch, lambda: gsd.gsd_build_mask(*args["graph"], args["n"]))


def test_steps_from_several_threads(args):
    """Four threads, each with its own stream and its own outputs from the allocator, which the calls ask without the interpreter's
    lock: the results of the same calls one after the other."""
    import threading
    a, t = args, args[torch.bfloat16]

    def step(scale):
        mask = gsd.gsd_build_mask(*a["graph"], a["n"])
        q, k, v, *rest = attention_args(a, torch.bfloat16)
        out, lse = gsd.gsd_dag_attention((q.float() * scale).to(q.dtype), k, v, *rest, num_splits=2, return_lse=True)
        accepted = gsd.gsd_accept_longest_path(*a["graph"], a["tokens"], a["root_pred"], a["n"], logits=t["logits"] * scale)
        return [mask, out, lse, *accepted, *gsd.gsd_node_argmax_stats(t["logits"] * scale), *gsd.gsd_softmax_stats(t["logits"] * scale)]
    scales = [0.5, 1.0, -1.0, 2.0]
    want = [step(scale) for scale in scales]
    torch.cuda.synchronize()
    got, failed = [[] for _ in scales], []

    def run(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(25):
                    got[i].append(step(scales[i]))
                torch.cuda.current_stream().synchronize()
        except Exception as e:        # noqa: BLE001 - reported below
            failed.append(e)
    threads = [threading.Thread(target=run, args=(i,)) for i in range(4)]
    for thread in threads:
        thread.start()
    for thread in threads:
        thread.join()
    assert not failed, failed
    for i in range(4):
        assert len(got[i]) == 25
        assert all(torch.equal(x, y) for results in got[i] for x, y in zip(results, want[i]))


@pytest.mark.parametrize("transform", ["vmap", "grad", "jvp"])
def test_calls_under_a_function_transform(args, monkeypatch, transform):
    """Inside a torch.func transform, on tensors that it has nothing to do with and on one that it has wrapped: what Python does."""
    t, seen = args[torch.float32], []

    def body(x):
        seen.append(both(monkeypatch, lambda: gsd.gsd_node_argmax(t["logits"])))
        seen.append(both(monkeypatch, lambda: gsd.gsd_softmax_stats(x.expand(4, 3) if x.dim() == 1 else x)))
        return x.sum()
    x = torch.ones(4, 3, device="cuda")
    if transform == "vmap":
        torch.func.vmap(body)(x)
    elif transform == "grad":
        torch.func.grad(body)(x)
    else:
        torch.func.jvp(body, (x,), (x,))
    assert len(seen) == 2
    for a, b in seen:
        raised = isinstance(a, tuple) and isinstance(a[0], type)
        assert raised == (isinstance(b, tuple) and isinstance(b[0], type)), (a, b)
        if raised:
            assert a == b
        else:
            assert all(torch.equal(p, q) for p, q in zip(flat(a), flat(b)))
