"""The Python binding on its own, without a GPU: what it hands to the library and what it refuses, with stand-ins for the
library and for torch's allocator."""
import contextlib
import ctypes
import os
import subprocess
import types
import warnings

import pytest
import torch

import paper_2407_16207_amd as gsd


class Allocator:
    """Stands in for torch in the binding: notes which stream every allocation belongs to and who else uses it."""

    def __init__(self):
        self.current, self.blocks = "current", []
        self.cuda = types.SimpleNamespace(stream=self.on_stream)
        self.uint8 = torch.uint8

    @contextlib.contextmanager
    def on_stream(self, stream):
        outer, self.current = self.current, stream
        yield
        self.current = outer

    def empty(self, size, dtype=None, device=None):
        block = types.SimpleNamespace(owner=self.current, users=[], data_ptr=lambda: 0x10000)
        block.record_stream = block.users.append
        self.blocks.append(block)
        return block


class Stream:
    cuda_stream = 7


@pytest.mark.parametrize("own", [True, False])
def test_attention_workspace_lives_as_long_as_its_stream_needs_it(monkeypatch, own):
    """A workspace that the binding allocates is dropped when the call returns, with its kernels still to run: the allocator
    has to know that they run on the call's stream, or the block is handed out again beneath them."""
    stream, seen, allocator = Stream(), [], Allocator()
    lib = types.SimpleNamespace(gsd_dag_attention_workspace=lambda desc: 4096,
                                gsd_dag_attention=lambda desc, ptr: seen.append(ptr) or 0)
    monkeypatch.setattr(gsd, "_lib", lib)
    monkeypatch.setattr(gsd, "torch", allocator)
    monkeypatch.setattr(gsd, "make_attn_desc", lambda *a, **kw: gsd.AttnDesc())
    monkeypatch.setattr(gsd, "_raw_stream", lambda device: 3, raising=False)
    monkeypatch.setattr(gsd, "_device", lambda: 0, raising=False)
    q = types.SimpleNamespace(device="cuda")
    gsd.gsd_dag_attention(q, q, q, None, None, None, None, 1, 1, 1.0, out=q, stream=stream if own else None)
    (block,) = allocator.blocks
    assert seen == [7 if own else 3]
    if own:
        assert block.owner is stream or stream in block.users
    else:
        assert block.owner == "current"


class OnGpu(torch.Tensor):
    """A host tensor that passes for a device tensor: for calls that end before a launch."""
    is_cuda = True


def on_gpu(*shape, dtype=torch.int32):
    return torch.zeros(shape, dtype=dtype).as_subclass(OnGpu)


def graph_tensors():
    return on_gpu(2), on_gpu(5), on_gpu(4)                       # one sequence of four nodes


def attention_tensors(dtype=torch.float32, **other):
    q, k, v = (on_gpu(4, 2, 64, dtype=other.get(name, dtype)) for name in "qkv")
    return q, k, v, on_gpu(1, dtype=torch.int64), on_gpu(1), on_gpu(2), on_gpu(4, 1, dtype=torch.int64)


def test_arguments_are_checked_before_the_library_is_loaded(monkeypatch):
    """A wrong argument is reported as such also where the library has not been built."""
    monkeypatch.setattr(gsd, "_lib", None)
    monkeypatch.setattr(gsd, "LIB_PATH", "/nonexistent/libgsd.so")
    host = torch.zeros(4, dtype=torch.int32)
    rows = torch.zeros(4, 8)
    for call in (lambda: gsd.gsd_build_mask(host, host, host, 4),
                 lambda: gsd.make_attn_desc(rows, rows, rows, host, host, host, host, 4, 4, 1.0),
                 lambda: gsd.gsd_node_argmax(rows), lambda: gsd.gsd_node_argmax_stats(rows), lambda: gsd.gsd_softmax_stats(rows),
                 lambda: gsd.gsd_accept_longest_path(host, host, host, host, host, 4, pred=host),
                 lambda: gsd.gsd_unmerge_to_tree(host, host, host, 4, 8), lambda: gsd.gsd_gather_rows(rows, host),
                 lambda: gsd.gsd_commit_kv(torch.zeros(2, 4, 1, 8), torch.zeros(2, 4, 1, 8), host, host, host, host),
                 lambda: gsd.gsd_accept_stochastic(host, host, host, host, rows, rows, rows, rows, rows, rows, rows, 4),
                 lambda: gsd.gsd_build_token_graph(host, host, host, rows, 4, 2, 0.0, 0.0)):
        with pytest.raises(ValueError):
            call()
    with pytest.raises(RuntimeError, match="no fallback"):
        gsd.gsd_node_argmax(on_gpu(4, 8, dtype=torch.float32), pred=on_gpu(4))


@pytest.mark.parametrize("name", ["q", "k", "v"])
def test_unsupported_dtype_is_a_type_error(name):
    with pytest.raises(TypeError, match="unsupported dtype"):
        gsd.make_attn_desc(*attention_tensors(**{name: torch.float16}), 4, 8, 0.1)


@pytest.mark.parametrize("which", range(4))
def test_unsupported_logits_dtype_is_a_type_error(which):
    logits = [on_gpu(4, 8, dtype=torch.float32), on_gpu(1, 8, dtype=torch.float32), on_gpu(4, 8, dtype=torch.float32),
              on_gpu(1, 8, dtype=torch.float32)]
    logits[which] = logits[which].half()
    with pytest.raises(TypeError, match="unsupported dtype"):
        gsd.gsd_accept_stochastic(*graph_tensors(), on_gpu(4), *logits, on_gpu(4, dtype=torch.float32),
                                  on_gpu(4, dtype=torch.float32), on_gpu(1, dtype=torch.float32), 4)


@pytest.mark.parametrize("max_nodes,max_prefix,scale,splits", [(4, 1 << 31, 0.1, 0), (1 << 31, 8, 0.1, 0), (4, 8, 1e39, 0),
                                                               (4, 8, 0.1, 1 << 31)])
def test_values_beyond_a_descriptor_field_are_refused_by_the_library(max_nodes, max_prefix, scale, splits):
    desc = gsd.make_attn_desc(*attention_tensors(), max_nodes, max_prefix, scale, num_splits=splits)
    with pytest.raises(gsd.GsdError) as e:
        gsd.gsd_dag_attention_workspace(desc)
    assert e.value.status == gsd.GSD_ERR_INVALID_ARG


def test_descriptor_fields():
    q, k, v, kv_offsets, prefix, nodes, mask = attention_tensors()
    out, lse, ws = torch.zeros(4, 2, 64), torch.zeros(4, 2), torch.zeros(40)
    d = gsd.make_attn_desc(q, k, v, kv_offsets, prefix, nodes, mask, 3, 9, 0.25, out=out, lse=lse, num_splits=2, workspace=ws,
                           wg_waves=8)
    want = {"batch": 1, "total_nodes": 4, "max_nodes": 3, "max_prefix": 9, "num_q_heads": 2, "num_kv_heads": 2, "head_dim": 64,
            "dtype": gsd.GSD_F32, "words_per_row": 1, "num_splits": 2, "softmax_scale": 0.25, "wg_waves": 8, "q": q.data_ptr(),
            "o": out.data_ptr(), "lse": lse.data_ptr(), "k": k.data_ptr(), "v": v.data_ptr(), "kv_offsets": kv_offsets.data_ptr(),
            "prefix_lens": prefix.data_ptr(), "node_offsets": nodes.data_ptr(), "mask": mask.data_ptr(), "q_token_stride": 128,
            "q_head_stride": 64, "o_token_stride": 128, "o_head_stride": 64, "kv_token_stride": 128, "kv_head_stride": 64,
            "workspace": ws.data_ptr(), "workspace_bytes": 160}
    assert {name: getattr(d, name) for name, _ in gsd.AttnDesc._fields_} == want


def test_empty_sources_and_caches_are_refused():
    with pytest.raises(IndexError):
        gsd.gsd_gather_rows(on_gpu(0, 8), on_gpu(0))
    with pytest.raises(IndexError):
        gsd.gsd_gather_rows(on_gpu(3, 8), on_gpu(0), out=on_gpu(0, 8))
    for shape in ((0, 4, 1, 8), (2, 0, 1, 8)):
        with pytest.raises(IndexError):
            gsd.gsd_commit_kv(on_gpu(*shape), on_gpu(*shape), on_gpu(1, dtype=torch.int64), on_gpu(1), on_gpu(1), on_gpu(1, 4))


def recording_library(monkeypatch):
    """Stands in for the library: every call is noted and succeeds."""
    class Library:
        calls = []

        def __getattr__(self, name):
            return lambda *args: self.calls.append(name) or 0
    gsd._import_torch()
    monkeypatch.setattr(gsd, "_lib", Library())
    monkeypatch.setattr(gsd, "_raw_stream", lambda device: 3)
    monkeypatch.setattr(gsd, "_device", lambda: 0)
    return Library.calls


def calls_with_outputs():
    """(call, its outputs as keywords, of the size they have to have)"""
    rows = on_gpu(4, 8, dtype=torch.float32)
    f4 = dict(dtype=torch.float32)
    yield (lambda **kw: gsd.gsd_node_argmax(rows, **kw), {"pred": on_gpu(4)})
    yield (lambda **kw: gsd.gsd_node_argmax_stats(rows, **kw), {"pred": on_gpu(4), "row_max": on_gpu(4, **f4), "row_sumexp": on_gpu(4, **f4)})
    yield (lambda **kw: gsd.gsd_softmax_stats(rows, **kw), {"row_max": on_gpu(4, **f4), "row_sumexp": on_gpu(4, **f4)})
    outputs = {"pred": on_gpu(4), "accept_len": on_gpu(1), "accept_path": on_gpu(1, 6), "bonus_token": on_gpu(1)}
    yield (lambda **kw: gsd.gsd_accept_longest_path(*graph_tensors(), on_gpu(4), on_gpu(1), 6, logits=rows, **kw), dict(outputs))
    del outputs["pred"]                                  # an input without logits, of which the nodes there are are read
    yield (lambda **kw: gsd.gsd_accept_longest_path(*graph_tensors(), on_gpu(4), on_gpu(1), 6, pred=on_gpu(3), **kw), outputs)
    cache = on_gpu(2, 9, 1, 8, **f4)
    yield (lambda **kw: gsd.gsd_commit_kv(cache, cache, on_gpu(2, dtype=torch.int64), on_gpu(2), on_gpu(2), on_gpu(2, 4), **kw),
           {"new_prefix_lens": on_gpu(2)})
    yield (lambda **kw: gsd.gsd_dag_attention(*attention_tensors(), 4, 8, 0.1, workspace=on_gpu(16), **kw),
           {"out": on_gpu(4, 2, 64, **f4), "lse": on_gpu(4, 2, **f4)})


def test_outputs_that_a_call_would_write_past_are_refused(monkeypatch):
    """A kernel knows no end of the buffers it is given: one element less than a call writes is refused before the library is
    reached, one more is as good as the exact size."""
    calls = recording_library(monkeypatch)
    for call, outputs in calls_with_outputs():
        call(**outputs)
        for name, t in outputs.items():
            for wrong in ([t[:-1], t[:0]] if t.dim() == 1 else [t[:-1], t[:, :-1].contiguous()]):
                del calls[:]
                with pytest.raises(ValueError, match=name):
                    call(**{**outputs, name: wrong})
                assert not calls
            call(**{**outputs, name: on_gpu(*(size + 1 for size in t.shape), dtype=t.dtype)})
            assert calls


def test_inputs_that_a_call_would_read_past_are_refused(monkeypatch):
    """What there is one of per sequence (or gathered row): two sequences, and one too few of each."""
    calls = recording_library(monkeypatch)
    f4, i8 = dict(dtype=torch.float32), dict(dtype=torch.int64)
    graph, rows, roots = (on_gpu(3), on_gpu(5), on_gpu(4)), on_gpu(4, 8, **f4), on_gpu(2, 8, **f4)
    q, cache = on_gpu(4, 2, 64, **f4), on_gpu(2, 9, 1, 8, **f4)
    cases = [(lambda kv_offsets, node_offsets: gsd.gsd_dag_attention(q, q, q, kv_offsets, on_gpu(2), node_offsets, on_gpu(4, 1, **i8), 4, 8,
                                                                   0.1, out=q, workspace=on_gpu(16)),
              {"kv_offsets": on_gpu(2, **i8), "node_offsets": on_gpu(3)}),
             (lambda root_pred: gsd.gsd_accept_longest_path(*graph, on_gpu(4), root_pred, 4, pred=on_gpu(4), accept_len=on_gpu(2),
                                                            accept_path=on_gpu(2, 4), bonus_token=on_gpu(2)), {"root_pred": on_gpu(2)}),
             (lambda kv_offsets, accept_len, accept_path: gsd.gsd_commit_kv(cache, cache, kv_offsets, on_gpu(2), accept_len, accept_path,
                                                                            new_prefix_lens=on_gpu(2)),
              {"kv_offsets": on_gpu(2, **i8), "accept_len": on_gpu(2), "accept_path": on_gpu(2, 4)}),
             (lambda index: gsd.gsd_gather_rows(rows, index, rows=3, out=on_gpu(3, 8, **f4)), {"index": on_gpu(3)}),
             (lambda resample_u: gsd.gsd_accept_stochastic(*graph, on_gpu(4), rows, roots, rows, roots, on_gpu(4, **f4), on_gpu(4, **f4),
                                                           resample_u, 4), {"resample_u": on_gpu(2, **f4)})]
    for call, inputs in cases:
        call(**inputs)
        assert calls
        for name, t in inputs.items():
            del calls[:]
            with pytest.raises(ValueError, match=name):
                call(**{**inputs, name: t[:-1]})
            assert not calls
            call(**{**inputs, name: on_gpu(t.shape[0] + 1, *t.shape[1:], dtype=t.dtype)})
            assert calls


def test_attention_outputs_of_another_kind_are_refused(monkeypatch):
    """What the descriptor cannot say of `out`: its type, its last stride, and that it is memory of the GPU."""
    calls = recording_library(monkeypatch)
    f4 = dict(dtype=torch.float32)
    for wrong in (on_gpu(4, 2, 64, dtype=torch.bfloat16), on_gpu(4, 2, 64, dtype=torch.float64), on_gpu(4, 2, 128, **f4)[:, :, ::2],
                  on_gpu(4, 2, 32, **f4), on_gpu(8, 64, **f4)):
        with pytest.raises(ValueError, match="out"):
            gsd.gsd_dag_attention(*attention_tensors(), 4, 8, 0.1, workspace=on_gpu(16), out=wrong)
    assert not calls
    gsd.gsd_dag_attention(*attention_tensors(), 4, 8, 0.1, workspace=on_gpu(16), out=on_gpu(4, 2, 96, **f4)[:, :, :64])
    assert calls == ["gsd_dag_attention"]


@pytest.fixture
def reload(monkeypatch):
    """Loads the library again with what stands at `path` for the binding's native part: (library, native part, warnings)."""
    gsd.load_library()

    def load(path):
        monkeypatch.setattr(gsd, "_lib", None)
        monkeypatch.setattr(gsd, "_short", None)
        monkeypatch.setattr(gsd, "BINDING_PATH", str(path))
        with warnings.catch_warnings(record=True) as said:
            warnings.simplefilter("always")
            lib = gsd.load_library()
        return lib, gsd._short, [str(w.message) for w in said if w.category is RuntimeWarning]
    return load


@pytest.mark.parametrize("kind", ["none", "text", "undefined symbol"])
def test_a_native_part_that_does_not_load_is_done_without(reload, tmp_path, kind):
    """As after an upgrade of torch: the calls' way through Python and ctypes is whole, and one warning says that they take it."""
    path = tmp_path / "_binding.so"
    if kind == "text":
        path.write_text("no library")
    elif kind == "undefined symbol":
        (tmp_path / "b.c").write_text("extern int gone_from_torch(void);\nvoid *PyInit__binding(void) { gone_from_torch(); return 0; }\n")
        subprocess.check_call(["gcc", "-shared", "-fPIC", "-o", str(path), str(tmp_path / "b.c")])
    lib, short, said = reload(path)
    assert lib.gsd_version().startswith(b"gsd") and short is None
    assert len(said) == 1 and str(path) in said[0]
    desc = gsd.make_attn_desc(*attention_tensors(), 4, 8, 0.1)
    assert gsd.gsd_dag_attention_workspace(desc) >= 0


def test_the_native_part_that_has_been_built_loads(reload):
    from paper_2407_16207_amd import build
    if not os.path.exists(gsd.BINDING_PATH):
        assert build.build_binding() == gsd.BINDING_PATH
    lib, short, said = reload(gsd.BINDING_PATH)
    assert short is not None and not said
    assert short.node_argmax(torch.zeros(4, 8), None, None) is None        # a host tensor: not for the native part


@pytest.mark.parametrize("other", ["torch", "library"])
def test_a_native_part_built_for_something_else_is_done_without(reload, monkeypatch, other):
    """It loads, but would misread tensors (another torch) or descriptors (another gsd.h)."""
    path = gsd.BINDING_PATH
    if other == "torch":
        monkeypatch.setattr(torch.version, "git_version", "0" * 40)
    elif other == "library":
        monkeypatch.setattr(gsd, "built_for", lambda module, header, right=gsd.built_for: right(module, "0" * len(header)))
    _, short, said = reload(path)
    assert short is None and len(said) == 1 and "built for" in said[0]


def test_names_and_identities_of_the_build():
    """The native part's file is named for the Python it is for; the library says which gsd.h it was built with."""
    import importlib.machinery
    from paper_2407_16207_amd import build
    assert gsd.BINDING_PATH == build.BINDING_PATH and gsd.BINDING_PATH.endswith(importlib.machinery.EXTENSION_SUFFIXES[0])
    identity = gsd.load_library().gsd_header_id
    identity.restype = ctypes.c_char_p
    assert identity().decode() == build.header_id()
