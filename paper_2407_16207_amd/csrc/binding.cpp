// The short way through the Python binding, from plain tensors to the library's entry points.
//
// A function here takes what its namesake in __init__.py takes, all arguments in their order, and
//   returns the call's result                        if every argument is what it should be,
//   returns the library's status, a number           if the library refuses the call,
//   returns None, with nothing done                  otherwise: the caller then goes the long way, which has the messages.
// "Plain" is a torch.Tensor or Parameter (no subclass) with ordinary memory on a GPU, of the right type and contiguous, while no
// torch mode is active that would want to see the allocations.
// What a call costs the host is then mostly its launches, 3.1-3.7 us each: mask 5.5 -> 3.8 us, argmax and acceptance 10.5 -> 7.7, a whole
// verify step in the short call forms, which allocate nine outputs, 37-40 -> 23.6; building eight token graphs and reading them back
// 58.6 -> 53 us, of which the kernels take half.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cfloat>
#include <climits>
#include <cmath>
#include <type_traits>
#include <vector>

#include "gsd.h"

namespace {

// The library is loaded by ctypes; its entry points come from there (bind below).
decltype(&gsd_build_mask) build_mask_fn;
decltype(&gsd_dag_attention_workspace) attention_workspace_fn;
decltype(&gsd_dag_attention) attention_fn;
decltype(&gsd_node_argmax) argmax_fn;
decltype(&gsd_node_argmax_stats) argmax_stats_fn;
decltype(&gsd_accept_longest_path) accept_fn;
decltype(&gsd_unmerge_to_tree) unmerge_fn;
decltype(&gsd_gather_rows) gather_fn;
decltype(&gsd_commit_kv) commit_fn;
decltype(&gsd_softmax_stats) softmax_stats_fn;
decltype(&gsd_accept_stochastic) accept_stochastic_fn;
decltype(&gsd_build_token_graph) build_graph_fn;
PyObject *device_fn, *raw_stream_fn;         // the current device, and its current stream, as numbers

bool modes_active() {
    return c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::PythonTorchFunctionTLS::stack_len() > 0;
}

// the tensor behind a plain object, or NULL; of any layout
const at::Tensor *tensor(PyObject *o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda()) return nullptr;
    const c10::DispatchKeySet keys = t.key_set() - c10::autograd_dispatch_keyset_with_ADInplaceOrView - c10::autocast_dispatch_keyset;
    return keys == c10::DispatchKeySet(c10::DispatchKey::CUDA) ? &t : nullptr;
}

const at::Tensor *tensor(PyObject *o, at::ScalarType type, int64_t least = 0) {
    const at::Tensor *t = tensor(o);
    return t && t->scalar_type() == type && t->is_contiguous() && t->numel() >= least ? t : nullptr;
}

bool number(PyObject *o, int32_t &x) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v < INT32_MIN || v > INT32_MAX) return false;
    x = int32_t(v);
    return true;
}

bool dtype_code(const at::Tensor &t, int &code) {
    if (t.scalar_type() == at::kFloat) code = GSD_F32;
    else if (t.scalar_type() == at::kBFloat16) code = GSD_BF16;
    else return false;
    return true;
}

bool logits_layout(const at::Tensor &t) { return t.dim() == 2 && t.stride(1) == 1 && t.size(0) <= INT32_MAX && t.size(1) <= INT32_MAX; }

// An output: the caller's tensor, which has to be of the type, contiguous and large enough, or a new one.
struct Output {
    PyObject *given = nullptr;
    at::Tensor t;
    bool take(PyObject *o, at::ScalarType type, int64_t least = 0) {
        if (o == Py_None) return true;
        const at::Tensor *x = tensor(o, type, least);
        if (!x) return false;
        given = o;
        t = *x;
        return true;
    }
    void make(at::IntArrayRef sizes, at::ScalarType type, c10::Device device) {
        if (!given) t = at::empty(sizes, at::TensorOptions().dtype(type).device(device));
    }
    PyObject *object() const {
        if (!given) return THPVariable_Wrap(t);
        Py_INCREF(given);
        return given;
    }
};

PyObject *no_short_way() { Py_RETURN_NONE; }

// The outputs' allocations and the library's call, without the interpreter's lock, as torch.empty and ctypes do them: another thread
// may need it before the allocator or the device lets this one go on.  What is thrown leaves with the lock taken again.
template <typename F>
int call(F &&f) {
    struct Unlocked {
        PyThreadState *state = PyEval_SaveThread();
        ~Unlocked() { PyEval_RestoreThread(state); }
    } unlocked;
    return f();
}

struct Graph {
    const at::Tensor *nodes, *offsets, *parents;
    int32_t batch, total;
    bool take(PyObject *const *args) {
        nodes = tensor(args[0], at::kInt);
        offsets = tensor(args[1], at::kInt);
        parents = tensor(args[2], at::kInt);
        if (!nodes || !offsets || !parents) return false;
        const int64_t b = nodes->numel() - 1, t = offsets->numel() - 1;
        batch = int32_t(b);
        total = int32_t(t);
        return b >= 1 && b <= INT32_MAX && t >= 0 && t <= INT32_MAX;
    }
    const int32_t *node_offsets() const { return static_cast<const int32_t *>(nodes->data_ptr()); }
    const int32_t *parent_offsets() const { return static_cast<const int32_t *>(offsets->data_ptr()); }
    const int32_t *parent_idx() const { return static_cast<const int32_t *>(parents->data_ptr()); }
};

// the stream of a call, asked for when everything else is in order: the caller's, or the current one
bool stream_of(PyObject *o, void *&stream) {
    PyObject *value;
    if (o == Py_None) {
        PyObject *device = PyObject_CallNoArgs(device_fn);
        value = device ? PyObject_CallOneArg(raw_stream_fn, device) : nullptr;
        Py_XDECREF(device);
    } else {
        value = PyObject_GetAttrString(o, "cuda_stream");
    }
    const bool number = value && PyLong_CheckExact(value);
    if (number) stream = PyLong_AsVoidPtr(value);
    Py_XDECREF(value);
    if (!PyErr_Occurred()) return number;
    PyErr_Clear();
    return false;
}

// node_offsets, parent_offsets, parent_idx, max_nodes, words_per_row, mask, dag_error_flag, stream
PyObject *build_mask(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    Graph g;
    int32_t max_nodes, words;
    Output mask, flag;
    void *stream;
    if (count != 8 || modes_active() || !g.take(args) || !number(args[3], max_nodes) || max_nodes < 1 || !mask.take(args[5], at::kLong) ||
        !flag.take(args[6], at::kInt) || !stream_of(args[7], stream))
        return no_short_way();
    if (args[4] == Py_None) words = (max_nodes - 1) / 64 + 1;
    else if (!number(args[4], words) || words < 1) return no_short_way();
    if (mask.given && mask.t.numel() != int64_t(g.total) * words) return no_short_way();
    const int status = call([&] {
        mask.make({g.total, words}, at::kLong, g.nodes->device());
        return build_mask_fn(g.batch, max_nodes, words, g.node_offsets(), g.parent_offsets(), g.parent_idx(),
                             static_cast<uint64_t *>(mask.t.data_ptr()), flag.given ? static_cast<int32_t *>(flag.t.data_ptr()) : nullptr, stream);
    });
    return status ? PyLong_FromLong(status) : mask.object();
    END_HANDLE_TH_ERRORS
}

// logits, pred, row_max, row_sumexp, stream; without the two in the middle: gsd_node_argmax
PyObject *argmax(PyObject *const *args, bool stats) {
    const at::Tensor *logits = modes_active() ? nullptr : tensor(args[0]);
    int code;
    Output pred, row_max, row_sumexp;
    void *stream;
    if (!logits || !logits_layout(*logits) || !dtype_code(*logits, code) || !pred.take(args[1], at::kInt, logits->size(0)) ||
        (stats && (!row_max.take(args[2], at::kFloat, logits->size(0)) || !row_sumexp.take(args[3], at::kFloat, logits->size(0)))) ||
        !stream_of(args[stats ? 4 : 2], stream))
        return no_short_way();
    const int32_t rows = int32_t(logits->size(0)), vocab = int32_t(logits->size(1));
    const int status = call([&] {
        pred.make({rows}, at::kInt, logits->device());
        if (stats) {
            row_max.make({rows}, at::kFloat, logits->device());
            row_sumexp.make({rows}, at::kFloat, logits->device());
        }
        int32_t *to = static_cast<int32_t *>(pred.t.data_ptr());
        if (!stats) return argmax_fn(rows, vocab, code, logits->data_ptr(), logits->stride(0), to, stream);
        return argmax_stats_fn(rows, vocab, code, logits->data_ptr(), logits->stride(0), to, static_cast<float *>(row_max.t.data_ptr()),
                               static_cast<float *>(row_sumexp.t.data_ptr()), stream);
    });
    if (status) return PyLong_FromLong(status);
    return stats ? Py_BuildValue("(NNN)", pred.object(), row_max.object(), row_sumexp.object()) : pred.object();
}

PyObject *node_argmax(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    return count == 3 ? argmax(args, false) : no_short_way();
    END_HANDLE_TH_ERRORS
}

PyObject *node_argmax_stats(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    return count == 5 ? argmax(args, true) : no_short_way();
    END_HANDLE_TH_ERRORS
}

// node_offsets, parent_offsets, parent_idx, tokens, root_pred, max_nodes, logits, pred, accept_len, accept_path, bonus_token, stream
PyObject *accept_longest_path(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    Graph g;
    int32_t max_nodes;
    Output pred, length, path, bonus;
    void *stream;
    if (count != 12 || modes_active() || !g.take(args)) return no_short_way();
    const at::Tensor *tokens = tensor(args[3], at::kInt), *root_pred = tensor(args[4], at::kInt, g.batch);
    if (!tokens || !root_pred || tokens->numel() > INT32_MAX || !number(args[5], max_nodes) || max_nodes < 1 ||
        !pred.take(args[7], at::kInt, args[6] == Py_None ? 0 : tokens->numel()) || !length.take(args[8], at::kInt, g.batch) ||
        !path.take(args[9], at::kInt, int64_t(g.batch) * max_nodes) || !bonus.take(args[10], at::kInt, g.batch) || !stream_of(args[11], stream))
        return no_short_way();
    const int32_t total = int32_t(tokens->numel());
    const at::Tensor *logits = nullptr;
    int code = GSD_F32;
    if (args[6] != Py_None) {
        logits = tensor(args[6]);
        if (!logits || !logits_layout(*logits) || logits->size(0) != total || !dtype_code(*logits, code)) return no_short_way();
    } else if (!pred.given) {
        return no_short_way();
    }
    const c10::Device device = tokens->device();
    const int status = call([&] {
        pred.make({total}, at::kInt, device);
        length.make({g.batch}, at::kInt, device);
        path.make({g.batch, max_nodes}, at::kInt, device);
        bonus.make({g.batch}, at::kInt, device);
        auto ints = [](const at::Tensor &t) { return static_cast<int32_t *>(t.data_ptr()); };
        return accept_fn(g.batch, total, max_nodes, g.node_offsets(), g.parent_offsets(), g.parent_idx(), ints(*tokens),
                         logits ? logits->data_ptr() : nullptr, code, logits ? int32_t(logits->size(1)) : 0, logits ? logits->stride(0) : 0,
                         ints(pred.t), ints(*root_pred), ints(length.t), ints(path.t), ints(bonus.t), stream);
    });
    if (status) return PyLong_FromLong(status);
    return Py_BuildValue("(NNNN)", length.object(), path.object(), bonus.object(), pred.object());
    END_HANDLE_TH_ERRORS
}

// q, k, v, kv_offsets, prefix_lens, node_offsets, mask, max_nodes, max_prefix, softmax_scale, out, lse, num_splits, wg_waves, return_lse,
// stream: only where no stream is given, so that a workspace allocated here belongs to the stream of the call
PyObject *dag_attention(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    if (count != 16 || args[15] != Py_None || modes_active()) return no_short_way();
    const at::Tensor *q = tensor(args[0]), *k = tensor(args[1]), *v = tensor(args[2]);
    const at::Tensor *kv_offsets = tensor(args[3], at::kLong), *prefix = tensor(args[4], at::kInt), *nodes = tensor(args[5], at::kInt);
    const at::Tensor *mask = tensor(args[6], at::kLong);
    if (!q || !k || !v || !kv_offsets || !prefix || !nodes || !mask || mask->dim() < 2 || kv_offsets->numel() < prefix->numel() ||
        nodes->numel() <= prefix->numel())
        return no_short_way();
    gsd_attn_desc d = {};
    int code, code_k, code_v;
    if (q->dim() != 3 || k->dim() != 3 || v->dim() != 3 || q->stride(2) != 1 || k->stride(2) != 1 || v->stride(2) != 1 || !dtype_code(*q, code) ||
        !dtype_code(*k, code_k) || !dtype_code(*v, code_v) || code != code_k || code != code_v || k->strides() != v->strides() ||
        k->sizes() != v->sizes())
        return no_short_way();
    Output lse;
    void *stream;
    if (!number(args[7], d.max_nodes) || !number(args[8], d.max_prefix) || !PyFloat_CheckExact(args[9]) ||
        !lse.take(args[11], at::kFloat, q->size(0) * q->size(1)) ||
        !number(args[12], d.num_splits) || !number(args[13], d.wg_waves) || !PyBool_Check(args[14]) || !stream_of(args[15], stream))
        return no_short_way();
    const double scale = PyFloat_AS_DOUBLE(args[9]);
    if (!(std::fabs(scale) <= FLT_MAX)) return no_short_way();
    for (int64_t x : {prefix->numel(), q->size(0), q->size(1), q->size(2), k->size(1), mask->size(1)})
        if (x > INT32_MAX) return no_short_way();
    const at::Tensor *given = args[10] == Py_None ? nullptr : tensor(args[10]);
    if (args[10] != Py_None && (!given || given->dim() != 3 || given->scalar_type() != q->scalar_type() || given->stride(2) != 1 ||
                                given->size(0) < q->size(0) || given->size(1) < q->size(1) || given->size(2) < q->size(2)))
        return no_short_way();
    const bool return_lse = args[14] == Py_True;
    at::Tensor out, workspace;
    d.batch = int32_t(prefix->numel());
    d.total_nodes = int32_t(q->size(0));
    d.num_q_heads = int32_t(q->size(1));
    d.num_kv_heads = int32_t(k->size(1));
    d.head_dim = int32_t(q->size(2));
    d.dtype = code;
    d.words_per_row = int32_t(mask->size(1));
    d.softmax_scale = float(scale);
    d.q = q->data_ptr();
    d.k = k->data_ptr();
    d.v = v->data_ptr();
    d.kv_offsets = static_cast<const int64_t *>(kv_offsets->data_ptr());
    d.prefix_lens = static_cast<const int32_t *>(prefix->data_ptr());
    d.node_offsets = static_cast<const int32_t *>(nodes->data_ptr());
    d.mask = static_cast<const uint64_t *>(mask->data_ptr());
    d.q_token_stride = q->stride(0);
    d.q_head_stride = q->stride(1);
    d.kv_token_stride = k->stride(0);
    d.kv_head_stride = k->stride(1);
    bool sized = false;
    const int status = call([&] {
        out = given ? *given : at::empty(q->sizes(), at::TensorOptions().dtype(q->scalar_type()).device(q->device()));
        if (return_lse) lse.make({q->size(0), q->size(1)}, at::kFloat, q->device());
        d.o = out.data_ptr();
        d.o_token_stride = out.stride(0);
        d.o_head_stride = out.stride(1);
        d.lse = lse.t.defined() ? static_cast<float *>(lse.t.data_ptr()) : nullptr;
        const size_t need = attention_workspace_fn(&d);
        sized = need != size_t(-1);
        if (!sized) return 0;
        if (need > 0) {
            workspace = at::empty({int64_t(need)}, at::TensorOptions().dtype(at::kByte).device(q->device()));
            d.workspace = workspace.data_ptr();
            d.workspace_bytes = need;
        }
        return attention_fn(&d, stream);
    });
    if (!sized) return no_short_way();
    if (status) return PyLong_FromLong(status);
    PyObject *result = args[10];
    if (given) Py_INCREF(result);
    else result = THPVariable_Wrap(out);
    return return_lse ? Py_BuildValue("(NN)", result, lse.object()) : result;
    END_HANDLE_TH_ERRORS
}

template <typename T>
T *to(const at::Tensor &t) { return static_cast<T *>(t.data_ptr()); }

at::Tensor ints(at::IntArrayRef sizes, c10::Device device) { return at::empty(sizes, at::TensorOptions().dtype(at::kInt).device(device)); }
at::Tensor floats(at::IntArrayRef sizes, c10::Device device) { return at::empty(sizes, at::TensorOptions().dtype(at::kFloat).device(device)); }

// node_offsets, parent_offsets, parent_idx, max_nodes, max_tree_nodes, dag_error_flag, stream
PyObject *unmerge_to_tree(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    Graph g;
    int32_t max_nodes, cap;
    Output flag;
    void *stream;
    if (count != 7 || modes_active() || !g.take(args) || !number(args[3], max_nodes) || !number(args[4], cap) || cap < 1 ||
        int64_t(g.batch) * cap >= INT32_MAX || !flag.take(args[5], at::kInt) || !stream_of(args[6], stream))
        return no_short_way();
    const c10::Device device = g.nodes->device();
    const int64_t bound = int64_t(g.batch) * cap;
    at::Tensor offsets, parent, parent_offsets, origin, paths;
    const int status = call([&] {
        offsets = ints({g.batch + 1}, device), parent = ints({bound}, device), parent_offsets = ints({bound + 1}, device);
        origin = ints({bound}, device), paths = at::empty({g.batch}, at::TensorOptions().dtype(at::kLong).device(device));
        return unmerge_fn(g.batch, max_nodes, cap, g.node_offsets(), g.parent_offsets(), g.parent_idx(), to<int32_t>(offsets), to<int32_t>(parent),
                          to<int32_t>(parent_offsets), to<int32_t>(origin), to<int64_t>(paths), flag.given ? to<int32_t>(flag.t) : nullptr, stream);
    });
    if (status) return PyLong_FromLong(status);
    return Py_BuildValue("(NNNNN)", THPVariable_Wrap(offsets), THPVariable_Wrap(parent), THPVariable_Wrap(parent_offsets),
                         THPVariable_Wrap(origin), THPVariable_Wrap(paths));
    END_HANDLE_TH_ERRORS
}

// src, index, out, rows, stream
PyObject *gather_rows(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    if (count != 5 || modes_active()) return no_short_way();
    const at::Tensor *src = tensor(args[0]), *index = tensor(args[1], at::kInt);
    if (!src || !index || src->dim() < 1 || src->numel() == 0 || !src->is_contiguous()) return no_short_way();
    int64_t rows = index->numel();
    int32_t given_rows;
    if (args[3] != Py_None) {
        if (!number(args[3], given_rows)) return no_short_way();
        rows = given_rows;
    }
    if (rows < 1 || rows > index->numel()) return no_short_way();
    const at::Tensor *given = args[2] == Py_None ? nullptr : tensor(args[2]);
    if (args[2] != Py_None && (!given || given->scalar_type() != src->scalar_type() || given->dim() != src->dim() ||
                               given->sizes().slice(1) != src->sizes().slice(1) || given->size(0) < rows || given->numel() == 0 ||
                               !given->is_contiguous()))
        return no_short_way();
    void *stream;
    if (!stream_of(args[4], stream)) return no_short_way();
    const int64_t row_bytes = src->numel() / src->size(0) * int64_t(src->element_size());
    at::Tensor out;
    const int status = call([&] {
        if (given) {
            out = *given;
        } else {
            std::vector<int64_t> sizes = src->sizes().vec();
            sizes[0] = rows;
            out = at::empty(sizes, at::TensorOptions().dtype(src->scalar_type()).device(src->device()));
        }
        return gather_fn(rows, row_bytes, src->data_ptr(), src->size(0), row_bytes, to<int32_t>(*index), out.data_ptr(), row_bytes, stream);
    });
    if (status) return PyLong_FromLong(status);
    if (!given) return THPVariable_Wrap(out);
    Py_INCREF(args[2]);
    return args[2];
    END_HANDLE_TH_ERRORS
}

// k, v, kv_offsets, prefix_lens, accept_len, accept_path, new_prefix_lens, stream; caches of several layers, whole
PyObject *commit_kv(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    if (count != 8 || modes_active()) return no_short_way();
    const at::Tensor *k = tensor(args[0]), *v = tensor(args[1]), *kv_offsets = tensor(args[2], at::kLong), *prefix = tensor(args[3], at::kInt);
    const at::Tensor *length = tensor(args[4], at::kInt), *path = tensor(args[5], at::kInt);
    Output new_prefix;
    void *stream;
    if (!k || !v || !kv_offsets || !prefix || !length || !path || k->dim() != 4 || k->numel() == 0 || !k->is_contiguous() ||
        k->sizes() != v->sizes() || k->strides() != v->strides() || path->dim() < 2 || path->size(1) > INT32_MAX || prefix->numel() > INT32_MAX ||
        kv_offsets->numel() < prefix->numel() || length->numel() < prefix->numel() || path->numel() < prefix->numel() * path->size(1) ||
        k->size(0) > INT32_MAX || !new_prefix.take(args[6], at::kInt, prefix->numel()) || !stream_of(args[7], stream))
        return no_short_way();
    const int64_t element = int64_t(k->element_size());
    const int status = call([&] {
        new_prefix.make({prefix->numel()}, at::kInt, k->device());
        return commit_fn(int32_t(prefix->numel()), int32_t(path->size(1)), int32_t(k->size(0)), k->size(2) * k->size(3) * element, k->data_ptr(),
                         v->data_ptr(), k->stride(1) * element, k->stride(0) * element, to<int64_t>(*kv_offsets), to<int32_t>(*prefix),
                         to<int32_t>(*length), to<int32_t>(*path), to<int32_t>(new_prefix.t), stream);
    });
    return status ? PyLong_FromLong(status) : new_prefix.object();
    END_HANDLE_TH_ERRORS
}

// logits, row_max, row_sumexp, stream
PyObject *softmax_stats(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    const at::Tensor *logits = count != 4 || modes_active() ? nullptr : tensor(args[0]);
    int code;
    Output row_max, row_sumexp;
    void *stream;
    if (!logits || !logits_layout(*logits) || !dtype_code(*logits, code) || !row_max.take(args[1], at::kFloat, logits->size(0)) ||
        !row_sumexp.take(args[2], at::kFloat, logits->size(0)) || !stream_of(args[3], stream))
        return no_short_way();
    const int status = call([&] {
        row_max.make({logits->size(0)}, at::kFloat, logits->device());
        row_sumexp.make({logits->size(0)}, at::kFloat, logits->device());
        return softmax_stats_fn(logits->size(0), int32_t(logits->size(1)), code, logits->data_ptr(), logits->stride(0), to<float>(row_max.t),
                                to<float>(row_sumexp.t), stream);
    });
    if (status) return PyLong_FromLong(status);
    return Py_BuildValue("(NN)", row_max.object(), row_sumexp.object());
    END_HANDLE_TH_ERRORS
}

// node_offsets, parent_offsets, parent_idx, tokens, logits, root_logits, draft_logits, root_draft_logits, draft_prob, accept_u, resample_u,
// max_nodes, stream
PyObject *accept_stochastic(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    Graph g;
    int32_t max_nodes;
    int code;
    void *stream;
    if (count != 13 || modes_active() || !g.take(args)) return no_short_way();
    const at::Tensor *tokens = tensor(args[3], at::kInt), *prob = tensor(args[8], at::kFloat), *accept_u = tensor(args[9], at::kFloat),
                     *resample_u = tensor(args[10], at::kFloat, g.batch), *logits = tensor(args[4]);
    if (!tokens || !prob || !accept_u || !resample_u || !logits || !logits_layout(*logits) || !dtype_code(*logits, code) ||
        !number(args[11], max_nodes) || max_nodes < 1)
        return no_short_way();
    const int64_t total = logits->size(0), vocab = logits->size(1), row_stride = logits->stride(0);
    const at::Tensor *rows[4];
    for (int x = 0; x < 4; ++x) {
        const at::Tensor *t = rows[x] = tensor(args[4 + x]);
        const int64_t want = x % 2 ? g.batch : total;
        int other;
        if (!t || t->dim() != 2 || t->size(0) != want || t->size(1) != vocab || t->stride(1) != 1 || !dtype_code(*t, other) || other != code ||
            (want > 1 && t->stride(0) != row_stride))
            return no_short_way();
    }
    if (!stream_of(args[12], stream)) return no_short_way();
    const c10::Device device = logits->device();
    at::Tensor row_max, row_sumexp, length, path, end, bonus;
    gsd_stochastic_desc d = {};
    d.batch = g.batch;
    d.total_nodes = int32_t(total);
    d.max_nodes = max_nodes;
    d.vocab = int32_t(vocab);
    d.dtype = code;
    d.node_offsets = g.node_offsets();
    d.parent_offsets = g.parent_offsets();
    d.parent_idx = g.parent_idx();
    d.tokens = to<int32_t>(*tokens);
    d.logits = rows[0]->data_ptr();
    d.root_logits = rows[1]->data_ptr();
    d.draft_logits = rows[2]->data_ptr();
    d.root_draft_logits = rows[3]->data_ptr();
    d.row_stride = row_stride;
    d.draft_prob = to<float>(*prob);
    d.accept_u = to<float>(*accept_u);
    d.resample_u = to<float>(*resample_u);
    const int status = call([&] {
        row_max = floats({total + g.batch}, device), row_sumexp = floats({total + g.batch}, device), length = ints({g.batch}, device);
        path = ints({g.batch, max_nodes}, device), end = ints({g.batch}, device), bonus = ints({g.batch}, device);
        d.row_max = to<float>(row_max);
        d.row_sumexp = to<float>(row_sumexp);
        d.accept_len = to<int32_t>(length);
        d.accept_path = to<int32_t>(path);
        d.end_node = to<int32_t>(end);
        d.bonus_token = to<int32_t>(bonus);
        return accept_stochastic_fn(&d, stream);
    });
    if (status) return PyLong_FromLong(status);
    return Py_BuildValue("(NNNNNN)", THPVariable_Wrap(length), THPVariable_Wrap(path), THPVariable_Wrap(end), THPVariable_Wrap(bonus),
                         THPVariable_Wrap(row_max), THPVariable_Wrap(row_sumexp));
    END_HANDLE_TH_ERRORS
}

// node_offsets, tree_parent, tokens, draft_prob, max_nodes, tau, theta_prob, theta_sib, edge_capacity, error_flag, stream
PyObject *build_token_graph(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    if (count != 11 || modes_active()) return no_short_way();
    const at::Tensor *nodes = tensor(args[0], at::kInt), *parent = tensor(args[1], at::kInt), *tokens = tensor(args[2], at::kInt),
                     *prob = tensor(args[3], at::kFloat);
    int32_t max_nodes, tau, given_capacity;
    Output flag;
    void *stream;
    if (!nodes || !parent || !tokens || !prob || !number(args[4], max_nodes) || !number(args[5], tau) || !PyFloat_CheckExact(args[6]) ||
        !PyFloat_CheckExact(args[7]) || !flag.take(args[9], at::kInt))
        return no_short_way();
    const double theta_prob = PyFloat_AS_DOUBLE(args[6]), theta_sib = PyFloat_AS_DOUBLE(args[7]);
    const int64_t batch = nodes->numel() - 1, total = tokens->numel();
    int64_t capacity = 8 * total;
    if (args[8] != Py_None) {
        if (!number(args[8], given_capacity)) return no_short_way();
        capacity = given_capacity;
    }
    if (batch < 1 || batch >= INT32_MAX || capacity < 0 || !(std::fabs(theta_prob) <= FLT_MAX) || !(std::fabs(theta_sib) <= FLT_MAX) ||
        !stream_of(args[10], stream))
        return no_short_way();
    const c10::Device device = tokens->device();
    at::Tensor counts, offsets, parent_offsets, parent_idx, origin, flags;
    const int status = call([&] {
        counts = ints({batch, 2}, device), offsets = ints({batch + 1}, device), parent_offsets = ints({total + 1}, device);
        parent_idx = ints({capacity}, device), origin = ints({total}, device), flags = ints({total}, device);
        return build_graph_fn(int32_t(batch), max_nodes, tau, float(theta_prob), float(theta_sib), to<int32_t>(*nodes), to<int32_t>(*parent),
                              to<int32_t>(*tokens), to<float>(*prob), to<int32_t>(counts), to<int32_t>(offsets), to<int32_t>(parent_offsets),
                              to<int32_t>(parent_idx), capacity, to<int32_t>(origin), to<int32_t>(flags), flag.given ? to<int32_t>(flag.t) : nullptr,
                              stream);
    });
    if (status) return PyLong_FromLong(status);
    return Py_BuildValue("(NNNNNN)", THPVariable_Wrap(offsets), THPVariable_Wrap(parent_offsets), THPVariable_Wrap(parent_idx),
                         THPVariable_Wrap(origin), THPVariable_Wrap(flags), THPVariable_Wrap(counts));
    END_HANDLE_TH_ERRORS
}

// the addresses of the library's entry points, in the order of the list at the top, and what tells the current device and stream
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t count) {
    constexpr int kEntries = 12;
    void *at[kEntries];
    if (count != kEntries + 2) {
        PyErr_SetString(PyExc_TypeError, "twelve addresses and two functions");
        return nullptr;
    }
    for (int x = 0; x < kEntries; ++x) {
        at[x] = PyLong_AsVoidPtr(args[x]);
        if (PyErr_Occurred()) return nullptr;
    }
    int next = 0;
    auto entry = [&](auto &fn) { fn = reinterpret_cast<std::remove_reference_t<decltype(fn)>>(at[next++]); };
    entry(build_mask_fn);
    entry(attention_workspace_fn);
    entry(attention_fn);
    entry(argmax_fn);
    entry(argmax_stats_fn);
    entry(accept_fn);
    entry(unmerge_fn);
    entry(gather_fn);
    entry(commit_fn);
    entry(softmax_stats_fn);
    entry(accept_stochastic_fn);
    entry(build_graph_fn);
    Py_INCREF(args[kEntries]);
    Py_INCREF(args[kEntries + 1]);
    device_fn = args[kEntries];                   // kept for good, like the library
    raw_stream_fn = args[kEntries + 1];
    Py_RETURN_NONE;
}

#define GSD_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {GSD_METHOD(bind), GSD_METHOD(build_mask), GSD_METHOD(node_argmax), GSD_METHOD(node_argmax_stats),
                         GSD_METHOD(accept_longest_path), GSD_METHOD(dag_attention), GSD_METHOD(unmerge_to_tree), GSD_METHOD(gather_rows),
                         GSD_METHOD(commit_kv), GSD_METHOD(softmax_stats), GSD_METHOD(accept_stochastic), GSD_METHOD(build_token_graph),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// GSD_BUILT_FOR: the torch and the gsd.h this was compiled with, which is compared before anything here is called
PyMODINIT_FUNC PyInit__binding() {
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", GSD_BUILT_FOR) < 0) Py_CLEAR(m);
    return m;
}
