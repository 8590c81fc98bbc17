"""Thin Python binding of libgsd (include/gsd.h): the MI355X verification hot path of Graph-structured
Speculative Decoding.  Argument marshalling only: torch supplies device memory and the stream, every step of
the path runs in the library's HIP kernels.  There is no CPU fallback; a missing library raises.

    gsd_build_mask, gsd_dag_attention, gsd_node_argmax, gsd_accept_longest_path,
    gsd_unmerge_to_tree, gsd_gather_rows, gsd_commit_kv, gsd_softmax_stats, gsd_accept_stochastic,
    gsd_build_token_graph

mirror the C entry points of the same names.
"""
from __future__ import annotations

import ctypes
import importlib.machinery
import importlib.util
import os
import struct
import warnings

_PKG_DIR = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG_DIR, "libgsd.so")
# the way of plain tensors to the library without Python in between, for the Python that its name says
BINDING_PATH = os.path.join(_PKG_DIR, "_binding" + importlib.machinery.EXTENSION_SUFFIXES[0])

GSD_OK = 0
GSD_ERR_INVALID_ARG, GSD_ERR_UNSUPPORTED, GSD_ERR_WORKSPACE, GSD_ERR_HIP = 1, 3, 4, 5
GSD_F32, GSD_BF16 = 0, 1
GSD_MAX_NODES_PER_SEQ = 512
GSD_STATIC_SCRATCH_BYTES = 32 << 20

EXPORTS = ("gsd_status_string", "gsd_last_error", "gsd_version", "gsd_build_mask", "gsd_dag_attention_workspace",
           "gsd_dag_attention_splits", "gsd_dag_attention", "gsd_dag_attention_static", "gsd_node_argmax",
           "gsd_node_argmax_stats", "gsd_accept_longest_path", "gsd_unmerge_to_tree", "gsd_gather_rows", "gsd_commit_kv",
           "gsd_softmax_stats", "gsd_accept_stochastic", "gsd_build_token_graph")


class GsdError(RuntimeError):
    def __init__(self, status: int, detail: str):
        super().__init__(f"libgsd status {status}: {detail}")
        self.status = status


class AttnDesc(ctypes.Structure):
    """Mirror of struct gsd_attn_desc."""
    _fields_ = [
        ("batch", ctypes.c_int32), ("total_nodes", ctypes.c_int32), ("max_nodes", ctypes.c_int32),
        ("max_prefix", ctypes.c_int32), ("num_q_heads", ctypes.c_int32), ("num_kv_heads", ctypes.c_int32),
        ("head_dim", ctypes.c_int32), ("dtype", ctypes.c_int32), ("words_per_row", ctypes.c_int32),
        ("num_splits", ctypes.c_int32), ("softmax_scale", ctypes.c_float), ("wg_waves", ctypes.c_int32),
        ("q", ctypes.c_void_p), ("o", ctypes.c_void_p), ("lse", ctypes.c_void_p), ("k", ctypes.c_void_p),
        ("v", ctypes.c_void_p), ("kv_offsets", ctypes.c_void_p), ("prefix_lens", ctypes.c_void_p),
        ("node_offsets", ctypes.c_void_p), ("mask", ctypes.c_void_p),
        ("q_token_stride", ctypes.c_int64), ("q_head_stride", ctypes.c_int64),
        ("o_token_stride", ctypes.c_int64), ("o_head_stride", ctypes.c_int64),
        ("kv_token_stride", ctypes.c_int64), ("kv_head_stride", ctypes.c_int64),
        ("workspace", ctypes.c_void_p), ("workspace_bytes", ctypes.c_size_t),
    ]


class StochasticDesc(ctypes.Structure):
    """Mirror of struct gsd_stochastic_desc."""
    _fields_ = [
        ("batch", ctypes.c_int32), ("total_nodes", ctypes.c_int32), ("max_nodes", ctypes.c_int32),
        ("vocab", ctypes.c_int32), ("dtype", ctypes.c_int32),
        ("node_offsets", ctypes.c_void_p), ("parent_offsets", ctypes.c_void_p), ("parent_idx", ctypes.c_void_p),
        ("tokens", ctypes.c_void_p), ("logits", ctypes.c_void_p), ("root_logits", ctypes.c_void_p),
        ("draft_logits", ctypes.c_void_p), ("root_draft_logits", ctypes.c_void_p), ("row_stride", ctypes.c_int64),
        ("draft_prob", ctypes.c_void_p), ("accept_u", ctypes.c_void_p), ("resample_u", ctypes.c_void_p),
        ("row_max", ctypes.c_void_p), ("row_sumexp", ctypes.c_void_p), ("accept_len", ctypes.c_void_p),
        ("accept_path", ctypes.c_void_p), ("end_node", ctypes.c_void_p), ("bonus_token", ctypes.c_void_p),
    ]


# the descriptors from all their values at once: filled field by field a ctypes structure takes about 2 us
_ATTN_FORMAT = struct.Struct("@10i f i 9P 6q P N")
_STOCHASTIC_FORMAT = struct.Struct("@5i 8P q 9P")
assert _ATTN_FORMAT.size == ctypes.sizeof(AttnDesc) and _STOCHASTIC_FORMAT.size == ctypes.sizeof(StochasticDesc)


def _packed(kind, layout, *values):
    try:
        return kind.from_buffer_copy(layout.pack(*values))
    except struct.error:         # a number beyond its field: cut off as in C, and refused by the library for what comes of it
        return kind(*values)


_NO_SIZE = ctypes.c_size_t(-1).value
_lib = None
_short = None                # csrc/binding.cpp, where it has been built: takes plain tensors, gives None for everything else
torch = None                 # set by the first call: importing this module does not need it
_raw_stream = _device = None
_DTYPE_CODES = {}


def _import_torch():
    """Every call's first step, so that its arguments are checked whether or not the library has been built."""
    global torch, _raw_stream, _device
    import torch as module
    # the current device and its current stream as plain numbers (torch.cuda.current_stream() builds an object: 3 us)
    _raw_stream, _device = module._C._cuda_getCurrentRawStream, module._C._cuda_getDevice
    _DTYPE_CODES.update({module.float32: GSD_F32, module.bfloat16: GSD_BF16})
    torch = module


def _load_hip_runtime():
    """libgsd.so is linked without a HIP runtime of its own: it must run on the runtime that owns torch's
    device memory and streams.  Make that runtime's symbols globally visible before libgsd is loaded."""
    candidates = [os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"),
                  "/opt/rocm/lib/libamdhip64.so"]
    for path in candidates:
        if os.path.exists(path):
            ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)
            return path
    raise RuntimeError("no HIP runtime (libamdhip64.so) found next to torch or under /opt/rocm")


def built_for(module, header: str) -> str:
    """What csrc/binding.cpp depends on and cannot notice by itself: how the torch in `module` lays out a tensor, and the
    declarations in gsd.h (`header`: their identity)."""
    return f"torch {module.__version__} {module.version.git_version}, gsd.h {header}"


def _load_binding(lib):
    """csrc/binding.cpp, bound to the library; None, with a warning, if it is not there, does not load or was built for another
    torch or another library.  Every call has its way through this module and ctypes as well, which only takes the host longer
    (a verify step 39 us instead of 24)."""
    try:
        spec = importlib.util.spec_from_file_location(__name__ + "._binding", BINDING_PATH)
        binding = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(binding)
        header = getattr(lib, "gsd_header_id", None)
        if header is not None:
            header.restype = ctypes.c_char_p
        wanted = built_for(torch, header().decode() if header is not None else "of another time")
        found = getattr(binding, "built_for", "something unknown")
        if found != wanted:
            raise ImportError(f"built for {found}; here is {wanted}")
        binding.bind(*(ctypes.cast(getattr(lib, name), ctypes.c_void_p).value for name in (
            "gsd_build_mask", "gsd_dag_attention_workspace", "gsd_dag_attention", "gsd_node_argmax",
            "gsd_node_argmax_stats", "gsd_accept_longest_path", "gsd_unmerge_to_tree", "gsd_gather_rows", "gsd_commit_kv",
            "gsd_softmax_stats", "gsd_accept_stochastic", "gsd_build_token_graph")), _device, _raw_stream)
    except (ImportError, OSError) as e:
        warnings.warn(f"calls go without {BINDING_PATH}, which takes them longer: {e}", RuntimeWarning, stacklevel=3)
        return None
    return binding


def load_library() -> ctypes.CDLL:
    """Load libgsd.so (built in-tree by paper_2407_16207_amd.build); raises if it is not there."""
    global _lib, _short
    if _lib is None:
        if torch is None:
            _import_torch()
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with `python -m paper_2407_16207_amd.build` "
                               "(there is no fallback path)")
        _load_hip_runtime()
        lib = ctypes.CDLL(LIB_PATH)
        for name in ("gsd_status_string", "gsd_last_error", "gsd_version"):
            getattr(lib, name).restype = ctypes.c_char_p
        lib.gsd_dag_attention_workspace.restype = ctypes.c_size_t
        lib.gsd_dag_attention_workspace.argtypes = [ctypes.POINTER(AttnDesc)]
        lib.gsd_dag_attention_splits.argtypes = [ctypes.POINTER(AttnDesc)]
        lib.gsd_dag_attention.argtypes = [ctypes.POINTER(AttnDesc), ctypes.c_void_p]
        lib.gsd_dag_attention_static.argtypes = [ctypes.POINTER(AttnDesc), ctypes.c_void_p]
        i32, i64, vp = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p
        lib.gsd_build_mask.argtypes = [i32, i32, i32, vp, vp, vp, vp, vp, vp]
        lib.gsd_node_argmax.argtypes = [i32, i32, ctypes.c_int, vp, i64, vp, vp]
        lib.gsd_node_argmax_stats.argtypes = [i32, i32, ctypes.c_int, vp, i64, vp, vp, vp, vp]
        lib.gsd_accept_longest_path.argtypes = [i32, i32, i32, vp, vp, vp, vp, vp, ctypes.c_int, i32, i64, vp, vp,
                                                vp, vp, vp, vp]
        lib.gsd_unmerge_to_tree.argtypes = [i32, i32, i32, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp]
        lib.gsd_gather_rows.argtypes = [i64, i64, vp, i64, i64, vp, vp, i64, vp]
        lib.gsd_commit_kv.argtypes = [i32, i32, i32, i64, vp, vp, i64, i64, vp, vp, vp, vp, vp, vp]
        lib.gsd_softmax_stats.argtypes = [i64, i32, ctypes.c_int, vp, i64, vp, vp, vp]
        lib.gsd_accept_stochastic.argtypes = [ctypes.POINTER(StochasticDesc), vp]
        lib.gsd_build_token_graph.argtypes = [i32, i32, i32, ctypes.c_float, ctypes.c_float, vp, vp, vp, vp, vp, vp, vp,
                                              vp, i64, vp, vp, vp, vp]
        _short = _load_binding(lib)
        _lib = lib
    return _lib


def _check(status: int):
    if status != GSD_OK:
        lib = load_library()
        detail = lib.gsd_last_error().decode() or lib.gsd_status_string(status).decode()
        raise GsdError(status, detail)


def _result(done):
    """What the short way returned: the call's result, or the status of a refused call."""
    if type(done) is int:
        _check(done)
    return done


def _stream_ptr(stream):
    if stream is not None:
        return stream.cuda_stream
    return _raw_stream(_device())


def _ptr(t):
    return None if t is None else t.data_ptr()


def _dtype_code(t) -> int:
    code = _DTYPE_CODES.get(t.dtype)
    if code is None:
        raise TypeError(f"unsupported dtype {t.dtype}")
    return code


def _require(t, dtype, name, least=0):
    """`least`: elements that a call writes (or, of an input, reads); the kernels know no end of a buffer."""
    if t.is_cuda and t.dtype is dtype and t.is_contiguous() and t.numel() >= least:
        return
    if not t.is_cuda:
        raise ValueError(f"{name} must live on the GPU")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    raise ValueError(f"{name} must hold {least} elements, has {t.numel()}")


def _require_graph(node_offsets, parent_offsets, parent_idx):
    _require(node_offsets, torch.int32, "node_offsets")
    _require(parent_offsets, torch.int32, "parent_offsets")
    _require(parent_idx, torch.int32, "parent_idx")


def _logits_layout(logits, message="logits must be a GPU tensor [rows, vocab] with a contiguous last dim"):
    """(rows, vocab, row stride) of a logits tensor."""
    shape, stride = logits.shape, logits.stride()
    if not logits.is_cuda or len(shape) != 2 or stride[1] != 1:
        raise ValueError(message)
    return shape[0], shape[1], stride[0]


def gsd_build_mask(node_offsets, parent_offsets, parent_idx, max_nodes: int, words_per_row: int | None = None,
                   mask=None, dag_error_flag=None, stream=None):
    """mask[T, W] (int64 storage of the uint64 words) from the packed token graph.  See gsd_build_mask in gsd.h."""
    if _short is not None:
        done = _short.build_mask(node_offsets, parent_offsets, parent_idx, max_nodes, words_per_row, mask, dag_error_flag,
                                 stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    _require_graph(node_offsets, parent_offsets, parent_idx)
    batch = node_offsets.numel() - 1
    total = parent_offsets.numel() - 1
    W = (max_nodes + 63) // 64 if words_per_row is None else int(words_per_row)
    if mask is None:
        mask = torch.empty((total, W), dtype=torch.int64, device=node_offsets.device)
    else:
        _require(mask, torch.int64, "mask")
        if mask.numel() != total * W:
            raise ValueError("mask has the wrong size")
    if dag_error_flag is not None:
        _require(dag_error_flag, torch.int32, "dag_error_flag")
    lib = _lib or load_library()
    _check(lib.gsd_build_mask(batch, max_nodes, W, node_offsets.data_ptr(), parent_offsets.data_ptr(),
                              parent_idx.data_ptr(), mask.data_ptr(), _ptr(dag_error_flag), _stream_ptr(stream)))
    return mask


def make_attn_desc(q, k, v, kv_offsets, prefix_lens, node_offsets, mask, max_nodes: int, max_prefix: int,
                   softmax_scale: float, out=None, lse=None, num_splits: int = 0, workspace=None,
                   wg_waves: int = 0) -> AttnDesc:
    if torch is None:
        _import_torch()
    code = _dtype_code(q)
    q_stride, k_stride = q.stride(), k.stride()
    for t, stride, name in ((q, q_stride, "q"), (k, k_stride, "k"), (v, v.stride(), "v")):
        if not t.is_cuda or len(stride) != 3 or stride[2] != 1 or _dtype_code(t) != code:
            raise ValueError(f"{name} must be a GPU tensor [rows, heads, head_dim] with a contiguous last dim")
    if k_stride != v.stride() or k.shape != v.shape:
        raise ValueError("k and v must share shape and strides")
    _require(kv_offsets, torch.int64, "kv_offsets", prefix_lens.numel())
    _require(prefix_lens, torch.int32, "prefix_lens")
    _require(node_offsets, torch.int32, "node_offsets", prefix_lens.numel() + 1)
    _require(mask, torch.int64, "mask")
    total_nodes, num_q_heads, head_dim = q.shape
    o_stride = out.stride() if out is not None else (0, 0)
    if out is not None and (out.dtype is not q.dtype or len(o_stride) != 3 or o_stride[2] != 1 or
                            any(has < needs for has, needs in zip(out.shape, q.shape))):
        raise ValueError("out must have q's dtype, q's shape or more in every dim, and a contiguous last dim")
    if out is not None and out.device != q.device and not out.is_cuda and not out.is_pinned():
        raise ValueError("out must live on the GPU")
    if lse is not None and lse.numel() < total_nodes * num_q_heads:
        raise ValueError(f"lse must hold {total_nodes * num_q_heads} elements, has {lse.numel()}")
    return _packed(
        AttnDesc, _ATTN_FORMAT,
        prefix_lens.numel(), total_nodes, int(max_nodes), int(max_prefix), num_q_heads, k.shape[1], head_dim, code,
        mask.shape[1], int(num_splits), float(softmax_scale), int(wg_waves),
        q.data_ptr(), out.data_ptr() if out is not None else 0, lse.data_ptr() if lse is not None else 0,
        k.data_ptr(), v.data_ptr(), kv_offsets.data_ptr(), prefix_lens.data_ptr(), node_offsets.data_ptr(), mask.data_ptr(),
        q_stride[0], q_stride[1], o_stride[0], o_stride[1], k_stride[0], k_stride[1],
        workspace.data_ptr() if workspace is not None else 0,
        workspace.numel() * workspace.element_size() if workspace is not None else 0)


def gsd_dag_attention_workspace(desc: AttnDesc) -> int:
    n = (_lib or load_library()).gsd_dag_attention_workspace(ctypes.byref(desc))
    if n == _NO_SIZE:
        _check(GSD_ERR_INVALID_ARG)
    return n


def gsd_dag_attention_splits(desc: AttnDesc) -> int:
    return (_lib or load_library()).gsd_dag_attention_splits(ctypes.byref(desc))


def gsd_dag_attention(q, k, v, kv_offsets, prefix_lens, node_offsets, mask, max_nodes: int, max_prefix: int,
                      softmax_scale: float, out=None, lse=None, num_splits: int = 0, workspace=None, stream=None,
                      return_lse: bool = False, wg_waves: int = 0):
    """DAG-masked attention of every packed node; returns out (same dtype/shape as q).  See gsd.h."""
    if _short is not None and workspace is None:
        done = _short.dag_attention(q, k, v, kv_offsets, prefix_lens, node_offsets, mask, max_nodes, max_prefix,
                                    softmax_scale, out, lse, num_splits, wg_waves, return_lse, stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    if out is None:
        out = torch.empty_like(q, memory_format=torch.contiguous_format)
    if return_lse and lse is None:
        lse = torch.empty((q.shape[0], q.shape[1]), dtype=torch.float32, device=q.device)
    if lse is not None:
        _require(lse, torch.float32, "lse")
    desc = make_attn_desc(q, k, v, kv_offsets, prefix_lens, node_offsets, mask, max_nodes, max_prefix, softmax_scale,
                          out=out, lse=lse, num_splits=num_splits, workspace=workspace, wg_waves=wg_waves)
    if workspace is None:
        need = gsd_dag_attention_workspace(desc)
        if need:
            if stream is None:
                workspace = torch.empty(need, dtype=torch.uint8, device=q.device)
            else:        # dropped below with the kernels still to run: it has to go back to the pool of the stream they run on
                with torch.cuda.stream(stream):
                    workspace = torch.empty(need, dtype=torch.uint8, device=q.device)
            desc.workspace, desc.workspace_bytes = workspace.data_ptr(), need
    lib = _lib or load_library()
    _check(lib.gsd_dag_attention(ctypes.byref(desc), _stream_ptr(stream)))
    return (out, lse) if return_lse else out


def gsd_dag_attention_desc(desc: AttnDesc, stream=None):
    """Launch from a prepared descriptor (no allocation, for timing loops)."""
    _check((_lib or load_library()).gsd_dag_attention(ctypes.byref(desc), _stream_ptr(stream)))


def gsd_dag_attention_static(desc: AttnDesc, stream=None):
    """gsd_dag_attention_static of gsd.h: launch from a prepared descriptor, split partials in the library's static
    scratch array (the descriptor's workspace fields are ignored).  Allocates nothing."""
    _check((_lib or load_library()).gsd_dag_attention_static(ctypes.byref(desc), _stream_ptr(stream)))


def gsd_node_argmax(logits, pred=None, stream=None):
    """pred[r] = lowest index of the row maximum of logits[r].  See gsd_node_argmax in gsd.h."""
    if _short is not None:
        done = _short.node_argmax(logits, pred, stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    rows, vocab, row_stride = _logits_layout(logits)
    if pred is None:
        pred = torch.empty(rows, dtype=torch.int32, device=logits.device)
    _require(pred, torch.int32, "pred", rows)
    lib = _lib or load_library()
    _check(lib.gsd_node_argmax(rows, vocab, _dtype_code(logits), logits.data_ptr(), row_stride, pred.data_ptr(),
                               _stream_ptr(stream)))
    return pred


def gsd_node_argmax_stats(logits, pred=None, row_max=None, row_sumexp=None, stream=None):
    """One pass over the logits: (pred, row_max, row_sumexp) as gsd_node_argmax and gsd_softmax_stats give them.
    See gsd_node_argmax_stats in gsd.h."""
    if _short is not None:
        done = _short.node_argmax_stats(logits, pred, row_max, row_sumexp, stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    rows, vocab, row_stride = _logits_layout(logits)
    pred = torch.empty(rows, dtype=torch.int32, device=logits.device) if pred is None else pred
    row_max = torch.empty(rows, dtype=torch.float32, device=logits.device) if row_max is None else row_max
    row_sumexp = torch.empty(rows, dtype=torch.float32, device=logits.device) if row_sumexp is None else row_sumexp
    _require(pred, torch.int32, "pred", rows)
    _require(row_max, torch.float32, "row_max", rows)
    _require(row_sumexp, torch.float32, "row_sumexp", rows)
    lib = _lib or load_library()
    _check(lib.gsd_node_argmax_stats(rows, vocab, _dtype_code(logits), logits.data_ptr(), row_stride, pred.data_ptr(),
                                     row_max.data_ptr(), row_sumexp.data_ptr(), _stream_ptr(stream)))
    return pred, row_max, row_sumexp


def gsd_accept_longest_path(node_offsets, parent_offsets, parent_idx, tokens, root_pred, max_nodes: int,
                            logits=None, pred=None, accept_len=None, accept_path=None, bonus_token=None,
                            stream=None):
    """Longest accepted root path per sequence; returns (accept_len[B], accept_path[B, max_nodes], bonus[B], pred).
    With `logits` the per-node argmax runs first on the same stream.  See gsd_accept_longest_path in gsd.h."""
    if _short is not None:
        done = _short.accept_longest_path(node_offsets, parent_offsets, parent_idx, tokens, root_pred, max_nodes, logits,
                                          pred, accept_len, accept_path, bonus_token, stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    _require_graph(node_offsets, parent_offsets, parent_idx)
    batch = node_offsets.numel() - 1
    _require(tokens, torch.int32, "tokens")
    _require(root_pred, torch.int32, "root_pred", batch)
    total = tokens.numel()
    dev = tokens.device
    if pred is None:
        if logits is None:
            raise ValueError("give logits or pred")
        pred = torch.empty(total, dtype=torch.int32, device=dev)
    _require(pred, torch.int32, "pred", total if logits is not None else 0)
    accept_len = torch.empty(batch, dtype=torch.int32, device=dev) if accept_len is None else accept_len
    accept_path = torch.empty((batch, max_nodes), dtype=torch.int32, device=dev) if accept_path is None else accept_path
    bonus_token = torch.empty(batch, dtype=torch.int32, device=dev) if bonus_token is None else bonus_token
    _require(accept_len, torch.int32, "accept_len", batch)
    _require(accept_path, torch.int32, "accept_path", batch * max_nodes)
    _require(bonus_token, torch.int32, "bonus_token", batch)
    if logits is not None:
        message = "logits must be a GPU tensor [T, vocab] with a contiguous last dim"
        rows, vocab, row_stride = _logits_layout(logits, message)
        if rows != total:
            raise ValueError(message)
        dtype = _dtype_code(logits)
    else:
        dtype, vocab, row_stride = GSD_F32, 0, 0
    lib = _lib or load_library()
    _check(lib.gsd_accept_longest_path(batch, total, max_nodes, node_offsets.data_ptr(), parent_offsets.data_ptr(),
                                       parent_idx.data_ptr(), tokens.data_ptr(), _ptr(logits), dtype, vocab, row_stride,
                                       pred.data_ptr(), root_pred.data_ptr(), accept_len.data_ptr(),
                                       accept_path.data_ptr(), bonus_token.data_ptr(), _stream_ptr(stream)))
    return accept_len, accept_path, bonus_token, pred


def gsd_unmerge_to_tree(node_offsets, parent_offsets, parent_idx, max_nodes: int, max_tree_nodes: int,
                        dag_error_flag=None, stream=None):
    """Token graph -> token tree with replicated successors.  Returns (tree_node_offsets[B+1], tree_parent,
    tree_parent_offsets, tree_origin, path_count[B]); the three per-node arrays are allocated at their bound
    B*max_tree_nodes (+1) and only their first tree_node_offsets[B] (+1) entries are written.  See gsd.h."""
    if _short is not None:
        done = _short.unmerge_to_tree(node_offsets, parent_offsets, parent_idx, max_nodes, max_tree_nodes, dag_error_flag,
                                      stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    _require_graph(node_offsets, parent_offsets, parent_idx)
    batch = node_offsets.numel() - 1
    dev = node_offsets.device
    bound = batch * int(max_tree_nodes)
    tree_node_offsets = torch.empty(batch + 1, dtype=torch.int32, device=dev)
    tree_parent = torch.empty(bound, dtype=torch.int32, device=dev)
    tree_parent_offsets = torch.empty(bound + 1, dtype=torch.int32, device=dev)
    tree_origin = torch.empty(bound, dtype=torch.int32, device=dev)
    path_count = torch.empty(batch, dtype=torch.int64, device=dev)
    if dag_error_flag is not None:
        _require(dag_error_flag, torch.int32, "dag_error_flag")
    lib = _lib or load_library()
    _check(lib.gsd_unmerge_to_tree(batch, max_nodes, max_tree_nodes, node_offsets.data_ptr(), parent_offsets.data_ptr(),
                                   parent_idx.data_ptr(), tree_node_offsets.data_ptr(), tree_parent.data_ptr(),
                                   tree_parent_offsets.data_ptr(), tree_origin.data_ptr(), path_count.data_ptr(),
                                   _ptr(dag_error_flag), _stream_ptr(stream)))
    return tree_node_offsets, tree_parent, tree_parent_offsets, tree_origin, path_count


def _rows_contiguous(t) -> bool:
    """Whether every dim 0 slice is contiguous, decided without building one where that is possible; IndexError if none."""
    return t.numel() > 0 and t.is_contiguous() or t[0].is_contiguous()


def gsd_gather_rows(src, index, out=None, rows: int | None = None, stream=None):
    """out[r] = src[index[r]] along dim 0 (rows of any trailing shape, contiguous within a row).  See gsd.h."""
    if _short is not None:
        done = _short.gather_rows(src, index, out, rows, stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    _require(index, torch.int32, "index")
    if not src.is_cuda or src.dim() < 1 or not _rows_contiguous(src):
        raise ValueError("src must be a GPU tensor whose rows (dim 0 slices) are contiguous")
    rows = index.numel() if rows is None else int(rows)
    if out is None:
        out = torch.empty((rows,) + tuple(src.shape[1:]), dtype=src.dtype, device=src.device)
    elif out.dtype != src.dtype or tuple(out.shape[1:]) != tuple(src.shape[1:]) or out.shape[0] < rows or \
            not _rows_contiguous(out):
        raise ValueError("out must match src's dtype and row shape and hold `rows` rows")
    if rows == 0:
        return out
    _require(index, torch.int32, "index", rows)
    es = src.element_size()
    row_elems = 1
    for d in src.shape[1:]:
        row_elems *= d
    src_stride = src.stride(0) if src.shape[0] > 1 else row_elems
    out_stride = out.stride(0) if out.shape[0] > 1 else row_elems
    lib = _lib or load_library()
    _check(lib.gsd_gather_rows(rows, row_elems * es, src.data_ptr(), src.shape[0], src_stride * es, index.data_ptr(),
                               out.data_ptr(), out_stride * es, _stream_ptr(stream)))
    return out


def gsd_commit_kv(k, v, kv_offsets, prefix_lens, accept_len, accept_path, new_prefix_lens=None, stream=None):
    """In-place KV-cache commit of the accepted path.  k, v: [L, R, Hkv, D] (or [R, Hkv, D] for one layer) with
    contiguous rows; returns new_prefix_lens[B].  See gsd_commit_kv in gsd.h."""
    if _short is not None:
        done = _short.commit_kv(k, v, kv_offsets, prefix_lens, accept_len, accept_path, new_prefix_lens, stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    if k.dim() == 3:
        k, v = k.unsqueeze(0), v.unsqueeze(0)
    if k.dim() != 4 or k.shape != v.shape or k.stride() != v.stride() or not k.is_cuda or \
            not (k.numel() and k.is_contiguous() or k[0, 0].is_contiguous()):
        raise ValueError("k and v must be GPU tensors [layers, rows, kv_heads, head_dim] with contiguous rows")
    batch = prefix_lens.numel()
    _require(kv_offsets, torch.int64, "kv_offsets", batch)
    _require(prefix_lens, torch.int32, "prefix_lens")
    _require(accept_len, torch.int32, "accept_len", batch)
    _require(accept_path, torch.int32, "accept_path")
    max_nodes = accept_path.shape[1]
    _require(accept_path, torch.int32, "accept_path", batch * max_nodes)
    if new_prefix_lens is None:
        new_prefix_lens = torch.empty(batch, dtype=torch.int32, device=k.device)
    _require(new_prefix_lens, torch.int32, "new_prefix_lens", batch)
    es = k.element_size()
    layers, _, heads, head_dim = k.shape
    layer_stride, token_stride = k.stride()[:2]
    lib = _lib or load_library()
    _check(lib.gsd_commit_kv(batch, max_nodes, layers, heads * head_dim * es, k.data_ptr(), v.data_ptr(),
                             token_stride * es, layer_stride * es, kv_offsets.data_ptr(), prefix_lens.data_ptr(),
                             accept_len.data_ptr(), accept_path.data_ptr(), new_prefix_lens.data_ptr(),
                             _stream_ptr(stream)))
    return new_prefix_lens


def gsd_softmax_stats(logits, row_max=None, row_sumexp=None, stream=None):
    """(row_max[r], row_sumexp[r]) of every logits row.  See gsd_softmax_stats in gsd.h."""
    if _short is not None:
        done = _short.softmax_stats(logits, row_max, row_sumexp, stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    rows, vocab, row_stride = _logits_layout(logits)
    row_max = torch.empty(rows, dtype=torch.float32, device=logits.device) if row_max is None else row_max
    row_sumexp = torch.empty(rows, dtype=torch.float32, device=logits.device) if row_sumexp is None else row_sumexp
    _require(row_max, torch.float32, "row_max", rows)
    _require(row_sumexp, torch.float32, "row_sumexp", rows)
    lib = _lib or load_library()
    _check(lib.gsd_softmax_stats(rows, vocab, _dtype_code(logits), logits.data_ptr(), row_stride, row_max.data_ptr(),
                                 row_sumexp.data_ptr(), _stream_ptr(stream)))
    return row_max, row_sumexp


def gsd_accept_stochastic(node_offsets, parent_offsets, parent_idx, tokens, logits, root_logits, draft_logits,
                          root_draft_logits, draft_prob, accept_u, resample_u, max_nodes: int, stream=None):
    """Non-deterministic verification; returns (accept_len[B], accept_path[B, max_nodes], end_node[B], bonus_token[B],
    row_max[T+B], row_sumexp[T+B]).  See gsd_accept_stochastic in gsd.h."""
    if _short is not None:
        done = _short.accept_stochastic(node_offsets, parent_offsets, parent_idx, tokens, logits, root_logits, draft_logits,
                                        root_draft_logits, draft_prob, accept_u, resample_u, max_nodes, stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    _require_graph(node_offsets, parent_offsets, parent_idx)
    _require(tokens, torch.int32, "tokens")
    _require(draft_prob, torch.float32, "draft_prob")
    _require(accept_u, torch.float32, "accept_u")
    _require(resample_u, torch.float32, "resample_u", node_offsets.numel() - 1)
    code = _dtype_code(logits)
    (T, V), row_stride = logits.shape, logits.stride(0)
    B = node_offsets.numel() - 1
    for t, name, rows in ((logits, "logits", T), (root_logits, "root_logits", B), (draft_logits, "draft_logits", T),
                          (root_draft_logits, "root_draft_logits", B)):
        stride = t.stride()
        if not t.is_cuda or len(stride) != 2 or t.shape != (rows, V) or stride[1] != 1 or \
                _dtype_code(t) != code or (rows > 1 and stride[0] != row_stride):
            raise ValueError(f"{name} must be a GPU tensor [{rows}, {V}] of the same dtype and row stride as logits")
    dev = logits.device
    row_max = torch.empty(T + B, dtype=torch.float32, device=dev)
    row_sumexp = torch.empty(T + B, dtype=torch.float32, device=dev)
    accept_len = torch.empty(B, dtype=torch.int32, device=dev)
    accept_path = torch.empty((B, max_nodes), dtype=torch.int32, device=dev)
    end_node = torch.empty(B, dtype=torch.int32, device=dev)
    bonus_token = torch.empty(B, dtype=torch.int32, device=dev)
    d = _packed(
        StochasticDesc, _STOCHASTIC_FORMAT,
        B, T, int(max_nodes), V, code, node_offsets.data_ptr(), parent_offsets.data_ptr(), parent_idx.data_ptr(),
        tokens.data_ptr(), logits.data_ptr(), root_logits.data_ptr(), draft_logits.data_ptr(),
        root_draft_logits.data_ptr(), row_stride, draft_prob.data_ptr(), accept_u.data_ptr(), resample_u.data_ptr(),
        row_max.data_ptr(), row_sumexp.data_ptr(), accept_len.data_ptr(), accept_path.data_ptr(), end_node.data_ptr(),
        bonus_token.data_ptr())
    lib = _lib or load_library()
    _check(lib.gsd_accept_stochastic(ctypes.byref(d), _stream_ptr(stream)))
    return accept_len, accept_path, end_node, bonus_token, row_max, row_sumexp


def gsd_build_token_graph(node_offsets, tree_parent, tokens, draft_prob, max_nodes: int, tau: int, theta_prob: float,
                          theta_sib: float, edge_capacity: int | None = None, error_flag=None, stream=None):
    """Drafted token trees -> pruned, merged token graphs.  Returns (graph_node_offsets[B+1], parent_offsets[T+1],
    parent_idx[edge_capacity], origin[T], flags[T], counts[B, 2]); only the first T' (+1) / E entries are written.
    See gsd_build_token_graph in gsd.h."""
    if _short is not None:
        done = _short.build_token_graph(node_offsets, tree_parent, tokens, draft_prob, max_nodes, tau, theta_prob, theta_sib,
                                        edge_capacity, error_flag, stream)
        if done is not None:
            return _result(done)
    if torch is None:
        _import_torch()
    _require(node_offsets, torch.int32, "node_offsets")
    _require(tree_parent, torch.int32, "tree_parent")
    _require(tokens, torch.int32, "tokens")
    _require(draft_prob, torch.float32, "draft_prob")
    B, T = node_offsets.numel() - 1, tokens.numel()
    dev = tokens.device
    cap = int(edge_capacity) if edge_capacity is not None else 8 * T
    counts = torch.empty((B, 2), dtype=torch.int32, device=dev)
    g_off = torch.empty(B + 1, dtype=torch.int32, device=dev)
    p_off = torch.empty(T + 1, dtype=torch.int32, device=dev)
    p_idx = torch.empty(cap, dtype=torch.int32, device=dev)
    origin = torch.empty(T, dtype=torch.int32, device=dev)
    flags = torch.empty(T, dtype=torch.int32, device=dev)
    if error_flag is not None:
        _require(error_flag, torch.int32, "error_flag")
    lib = _lib or load_library()
    _check(lib.gsd_build_token_graph(B, max_nodes, tau, theta_prob, theta_sib, node_offsets.data_ptr(),
                                     tree_parent.data_ptr(), tokens.data_ptr(), draft_prob.data_ptr(), counts.data_ptr(),
                                     g_off.data_ptr(), p_off.data_ptr(), p_idx.data_ptr(), cap, origin.data_ptr(),
                                     flags.data_ptr(), _ptr(error_flag), _stream_ptr(stream)))
    return g_off, p_off, p_idx, origin, flags, counts
