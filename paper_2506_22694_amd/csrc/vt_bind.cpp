// The way from Python into the draft step, for plain calls: argument checks and marshalling of binding.py's hottest functions in
// native code.  A step of a small head is over on the GPU sooner than Python has described it: d = 256, k = 1024 takes the GPU 8.0 us,
// and took the host 9.9, of which the two launches are 5 (through here 6.1; the step 9.6 -> 8.2 us, a draft round of three levels
// on a head of 5000 rows 57.4 -> 53.2).
//
// Every function here returns the status of the library's call, or -1 for a call that is not plain -- a tensor subclass or a
// wrapped tensor (vmap, functionalisation, lazy negation), a host tensor, a stride, a type or a shape that does not fit, an argument
// that is no tensor: binding.py then goes its own way, which has the checks and the messages.  Nothing is kept between calls but
// the addresses of the library's functions.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <c10/core/DispatchKeySet.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <limits>

#include "vocabtrim.h"

namespace {

decltype(&vt_draft_head_step) g_step = nullptr;
decltype(&vt_draft_head_step_static) g_step_static = nullptr;
decltype(&vt_draft_tree_level) g_level = nullptr;
decltype(&vt_tree_rerank) g_rerank = nullptr;
decltype(&vt_count_tokens) g_count = nullptr;
PyObject *g_raw_stream = nullptr;      // torch's: device index -> handle of its current stream

struct NotPlain {};

// What makes a tensor more than its memory: the pointer of such a one is not what Python would be given.
bool wrapped(const at::Tensor &t) {
    constexpr c10::DispatchKeySet special({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                           c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                           c10::DispatchKey::Conjugate, c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
    return t.unsafeGetTensorImpl()->key_set().has_any(special);
}
const at::Tensor &tensor(PyObject *o) {
    if (!THPVariable_CheckExact(o)) throw NotPlain();
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != c10::kStrided || !t.has_storage() || wrapped(t)) throw NotPlain();
    return t;
}
// a tensor of the device, contiguous
const at::Tensor &operand(PyObject *o) {
    const at::Tensor &t = tensor(o);
    if (!t.is_cuda() || !t.is_contiguous()) throw NotPlain();
    return t;
}
int32_t int32(int64_t v) {
    if (v < 0 || v > std::numeric_limits<int32_t>::max()) throw NotPlain();
    return (int32_t)v;
}
int32_t int32(PyObject *o) {
    if (!PyLong_CheckExact(o)) throw NotPlain();
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow != 0) throw NotPlain();
    return int32((int64_t)v);
}
int element(const at::Tensor &t) {
    if (t.scalar_type() == at::kBFloat16) return VT_BF16;
    if (t.scalar_type() == at::kFloat) return VT_F32;
    throw NotPlain();
}
void *stream_of(const at::Tensor &t) {
    const auto index = t.device().index();
    if (index < 0 || g_raw_stream == nullptr) throw NotPlain();
    PyObject *i = PyLong_FromLong(index);
    if (i == nullptr) throw NotPlain();
    PyObject *r = PyObject_CallOneArg(g_raw_stream, i);
    Py_DECREF(i);
    if (r == nullptr) throw NotPlain();
    void *p = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    if (PyErr_Occurred()) throw NotPlain();
    return p;
}

// h, W_trim, map of a step, checked against one another
struct Head {
    const void *h, *W;
    const int32_t *map;
    int h_type, w_type;
    int32_t n, k, d, m;
    void *stream;
    Head(PyObject *h_, PyObject *W_, PyObject *map_, PyObject *m_) {
        if (at::impl::torch_function_mode_enabled()) throw NotPlain();
        const at::Tensor &th = operand(h_), &tW = operand(W_), &tmap = operand(map_);
        if (th.dim() != 2 || tW.dim() != 2) throw NotPlain();
        n = int32(th.size(0));
        d = int32(th.size(1));
        k = int32(tW.size(0));
        m = int32(m_);
        if (tW.size(1) != d || tmap.numel() != k || tmap.scalar_type() != at::kInt) throw NotPlain();
        h_type = element(th);
        w_type = element(tW);
        stream = stream_of(th);
        h = th.data_ptr();
        W = tW.data_ptr();
        map = static_cast<const int32_t *>(tmap.data_ptr());
    }
};

template <typename T>
T *pointer(PyObject *o) {
    return static_cast<T *>(tensor(o).data_ptr());
}

// Runs call() without the interpreter's lock; -1 where the arguments were not plain.
template <typename F>
PyObject *status_of(F &&prepare) {
    int status = -1;
    try {
        auto call = prepare();
        Py_BEGIN_ALLOW_THREADS status = call();
        Py_END_ALLOW_THREADS
    } catch (const NotPlain &) {
        PyErr_Clear();
    } catch (const std::exception &) {
        PyErr_Clear();      // (what torch refuses here it refuses there, with its own message)
    }
    return PyLong_FromLong(status);
}

// step(h, W_trim, map, m, workspace, out_ids, out_logp)
PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
    return status_of([&] {
        if (n_args != 7 || g_step == nullptr) throw NotPlain();
        const Head x(a[0], a[1], a[2], a[3]);
        const at::Tensor &ws = tensor(a[4]);
        void *const wsp = ws.data_ptr();
        const size_t ws_bytes = (size_t)ws.numel();
        int32_t *const ids = pointer<int32_t>(a[5]);
        float *const logp = pointer<float>(a[6]);
        return [=] {
            return g_step(x.h, x.h_type, x.n, x.W, x.w_type, x.k, x.d, x.map, x.m, ids, logp, nullptr, nullptr, wsp, ws_bytes, x.stream);
        };
    });
}

// step_static(h, W_trim, map, m, out_ids, out_logp)
PyObject *step_static(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
    return status_of([&] {
        if (n_args != 6 || g_step_static == nullptr) throw NotPlain();
        const Head x(a[0], a[1], a[2], a[3]);
        const at::Tensor &ids = operand(a[4]), &logp = operand(a[5]);
        const int64_t items = (int64_t)x.n * x.m;
        if (ids.scalar_type() != at::kInt || logp.scalar_type() != at::kFloat || ids.numel() != items || logp.numel() != items) throw NotPlain();
        int32_t *const pi = static_cast<int32_t *>(ids.data_ptr());
        float *const pl = static_cast<float *>(logp.data_ptr());
        return [=] { return g_step_static(x.h, x.h_type, x.n, x.W, x.w_type, x.k, x.d, x.map, x.m, pi, pl, nullptr, nullptr, x.stream); };
    });
}

// level(h, W_trim, map, m, parent_cum, K, workspace, parent, token, cum, out_ids, out_logp)
PyObject *level(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
    return status_of([&] {
        if (n_args != 12 || g_level == nullptr) throw NotPlain();
        const Head x(a[0], a[1], a[2], a[3]);
        const at::Tensor &from = operand(a[4]);
        if (from.scalar_type() != at::kFloat || from.numel() != x.n) throw NotPlain();
        const float *const cum = static_cast<const float *>(from.data_ptr());
        const int32_t K = int32(a[5]);
        const at::Tensor &ws = tensor(a[6]);
        void *const wsp = ws.data_ptr();
        const size_t ws_bytes = (size_t)ws.numel();
        int32_t *const parent = pointer<int32_t>(a[7]), *const token = pointer<int32_t>(a[8]), *const ids = pointer<int32_t>(a[10]);
        float *const score = pointer<float>(a[9]), *const logp = pointer<float>(a[11]);
        return [=] {
            return g_level(x.h, x.h_type, x.n, x.W, x.w_type, x.k, x.d, x.map, x.m, cum, K, parent, token, score, ids, logp, wsp, ws_bytes,
                           x.stream);
        };
    });
}

// rerank(cum, T, out)
PyObject *rerank(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
    return status_of([&] {
        if (n_args != 3 || g_rerank == nullptr || at::impl::torch_function_mode_enabled()) throw NotPlain();
        const at::Tensor &cum = operand(a[0]), &out = tensor(a[2]);
        const int32_t T = int32(a[1]), N = int32(cum.numel());
        if (cum.scalar_type() != at::kFloat || cum.dim() != 1 || !out.is_cuda() || out.scalar_type() != at::kInt || out.numel() < T) throw NotPlain();
        const float *const pc = static_cast<const float *>(cum.data_ptr());
        int32_t *const po = static_cast<int32_t *>(out.data_ptr());
        void *const stream = stream_of(cum);
        return [=] { return g_rerank(pc, N, T, po, stream); };
    });
}

// count(ids, V, counts, workspace)
PyObject *count(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
    return status_of([&] {
        if (n_args != 4 || g_count == nullptr || at::impl::torch_function_mode_enabled()) throw NotPlain();
        const at::Tensor &ids = operand(a[0]), &counts = operand(a[2]), &ws = operand(a[3]);
        const int type = ids.scalar_type() == at::kInt ? VT_I32 : ids.scalar_type() == at::kLong ? VT_I64 : -1;
        if (type < 0) throw NotPlain();
        const int32_t V = int32(a[1]);
        const int64_t n = ids.numel();
        const void *const p = n != 0 ? ids.data_ptr() : nullptr;
        int64_t *const pc = static_cast<int64_t *>(counts.data_ptr());
        void *const wsp = ws.data_ptr(), *const stream = stream_of(ids);
        const size_t ws_bytes = (size_t)ws.numel();
        return [=] { return g_count(p, type, n, V, pc, nullptr, wsp, ws_bytes, stream); };
    });
}

// connect(raw_stream, step, step_static, level, rerank, count): torch's stream query and the addresses of the library's functions
PyObject *connect(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
    if (n_args != 6) {
        PyErr_SetString(PyExc_TypeError, "connect takes six arguments");
        return nullptr;
    }
    void *p[5];
    for (int i = 0; i < 5; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i + 1]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_INCREF(a[0]);
    Py_XDECREF(g_raw_stream);
    g_raw_stream = a[0];
    g_step = reinterpret_cast<decltype(g_step)>(p[0]);
    g_step_static = reinterpret_cast<decltype(g_step_static)>(p[1]);
    g_level = reinterpret_cast<decltype(g_level)>(p[2]);
    g_rerank = reinterpret_cast<decltype(g_rerank)>(p[3]);
    g_count = reinterpret_cast<decltype(g_count)>(p[4]);
    Py_RETURN_NONE;
}

template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyCFunction fast() {
    return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F));
}
PyMethodDef methods[] = {{"connect", fast<connect>(), METH_FASTCALL, nullptr},
                         {"step", fast<step>(), METH_FASTCALL, nullptr},
                         {"step_static", fast<step_static>(), METH_FASTCALL, nullptr},
                         {"level", fast<level>(), METH_FASTCALL, nullptr},
                         {"rerank", fast<rerank>(), METH_FASTCALL, nullptr},
                         {"count", fast<count>(), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_vt_bind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch and the interpreter whose headers this was compiled with (binding.py compares them with its own)
PyMODINIT_FUNC PyInit__vt_bind(void) {
    PyObject *m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "built_for", VT_BUILT_FOR) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
