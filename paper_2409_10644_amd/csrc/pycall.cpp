// CPython marshalling of the entry points that a decoding loop calls per layer, per level or per step: tensors to
// addresses, the current stream to its handle, then the call with the interpreter's lock released, as ctypes does.
// Host time per call, on the same machine: 7.5 us through ctypes and torch.cuda.current_stream(), of which the library
// call itself (validation, plan, kernel launch) is 2.5; see the binding for who calls what.
//
// Nothing of the library is linked: the binding hands over the addresses of the entry points it has loaded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include <initializer_list>

#include "mcsd.h"

namespace {

enum Fn { ATTN, ATTN_ROWS, ATTN_GQA, ATTN_FP8, ATTN_STATIC, VERIFY, VERIFY_SAMPLING, COMMIT, STOP_DIST, STOP_HIDDEN, SLICE, N_FN };
const char *const FN_NAME[N_FN] = {"mcsd_tree_attention", "mcsd_tree_attention_rows", "mcsd_tree_attention_gqa", "mcsd_tree_attention_fp8kv",
                                   "mcsd_tree_attention_static", "mcsd_verify_tree", "mcsd_verify_tree_sampling", "mcsd_commit_path",
                                   "mcsd_early_stop_distribution", "mcsd_early_stop_hidden", "mcsd_slice_mask"};
void *g_fn[N_FN];
// torch.Tensor and its methods, torch's raw stream and device getters, and what raises on a status
PyObject *g_tensor, *g_data_ptr, *g_numel, *g_element_size, *g_raw_stream, *g_device, *g_raise;
// the binding's structures, and ctypes' error for an argument that is another one
PyObject *g_mask_view, *g_mlp, *g_argument_error;
PyObject *g_str_data_ptr, *g_str_cuda_stream, *g_str_numel, *g_str_element_size;

int64_t call_int(PyObject *method, PyObject *name, PyObject *self)
{
    PyObject *r = Py_TYPE(self) == (PyTypeObject *)g_tensor ? PyObject_CallOneArg(method, self) : PyObject_CallMethodNoArgs(self, name);
    if (!r) return 0;
    const int64_t v = (int64_t)PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    return v;
}

// Reads the arguments of one call in order; the first one that does not fit sets a Python error and ok = false.
struct Args {
    PyObject *const *a;
    Py_ssize_t n, i = 0;
    bool ok = true;
    Args(PyObject *const *args, Py_ssize_t nargs, Py_ssize_t want) : a(args), n(nargs)
    {
        if (nargs != want) {
            PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, nargs);
            ok = false;
        }
    }
    PyObject *next() { return a[i++]; }
    int64_t integer()
    {
        if (!ok) return 0;
        PyObject *o = next();
        int64_t v;
        if (PyLong_Check(o)) {
            v = (int64_t)PyLong_AsUnsignedLongLongMask(o);
        } else {
            PyObject *x = PyNumber_Index(o);
            if (!x) { ok = false; return 0; }
            v = (int64_t)PyLong_AsUnsignedLongLongMask(x);
            Py_DECREF(x);
        }
        if (v == -1 && PyErr_Occurred()) ok = false;
        return v;
    }
    int32_t i32() { return (int32_t)integer(); }
    float f32()
    {
        if (!ok) return 0.f;
        const double v = PyFloat_AsDouble(next());
        if (v == -1.0 && PyErr_Occurred()) ok = false;
        return (float)v;
    }
    void *address(PyObject *o)
    {
        if (!ok || o == Py_None) return nullptr;
        void *p = (void *)(uintptr_t)call_int(g_data_ptr, g_str_data_ptr, o);
        if (!p && PyErr_Occurred()) ok = false;
        return p;
    }
    void *tensor() { return ok ? address(next()) : nullptr; }
    // a tensor and its size in bytes
    void *workspace(size_t &bytes)
    {
        bytes = 0;
        if (!ok) return nullptr;
        PyObject *o = next();
        void *p = address(o);
        if (ok && o != Py_None) {
            bytes = (size_t)(call_int(g_numel, g_str_numel, o) * call_int(g_element_size, g_str_element_size, o));
            if (PyErr_Occurred()) ok = false;
        }
        return p;
    }
    // the memory of a ctypes structure of the given class, which the caller's argument keeps alive
    void *structure(PyObject *cls)
    {
        if (!ok) return nullptr;
        PyObject *o = next();
        if (!PyObject_TypeCheck(o, (PyTypeObject *)cls)) {
            PyErr_Format(g_argument_error, "argument %zd: expected %s, got %s", i, ((PyTypeObject *)cls)->tp_name, Py_TYPE(o)->tp_name);
            ok = false;
            return nullptr;
        }
        Py_buffer b;
        if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) { ok = false; return nullptr; }
        void *p = b.buf;
        PyBuffer_Release(&b);
        return p;
    }
    // the addresses of a sequence of tensors
    int32_t tensors(void **out, int32_t most)
    {
        if (!ok) return 0;
        PyObject *o = next();
        PyObject *f = PySequence_Fast(o, "expected a sequence of tensors");
        if (!f) { ok = false; return 0; }
        const Py_ssize_t len = PySequence_Fast_GET_SIZE(f);
        for (Py_ssize_t k = 0; ok && k < len && k < most; ++k) {
            PyObject *t = PySequence_Fast_GET_ITEM(f, k);
            if (t == Py_None) {
                PyErr_SetString(PyExc_TypeError, "expected a tensor");
                ok = false;
            } else {
                out[k] = address(t);
            }
        }
        Py_DECREF(f);
        return (int32_t)len;
    }
    void *stream()
    {
        if (!ok) return nullptr;
        PyObject *o = next(), *r;
        if (o == Py_None) {                   // the current stream of the current device
            PyObject *d = PyObject_CallNoArgs(g_device);
            r = d ? PyObject_CallOneArg(g_raw_stream, d) : nullptr;
            Py_XDECREF(d);
        } else {
            r = PyObject_GetAttr(o, g_str_cuda_stream);
        }
        if (!r) { ok = false; return nullptr; }
        void *p = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(r);
        Py_DECREF(r);
        if (PyErr_Occurred()) ok = false;
        return p;
    }
};

PyObject *done(int status, Fn fn)
{
    if (status == MCSD_OK) Py_RETURN_NONE;
    PyObject *r = PyObject_CallFunction(g_raise, "is", status, FN_NAME[fn]);
    Py_XDECREF(r);
    return nullptr;                           // (g_raise raises)
}

#define MCSD_UNLOCKED(TYPE, FN, ...)                                                 \
    if (!a.ok) return nullptr;                                                       \
    int status;                                                                      \
    Py_BEGIN_ALLOW_THREADS                                                           \
    status = ((decltype(&TYPE))g_fn[FN])(__VA_ARGS__);                               \
    Py_END_ALLOW_THREADS                                                             \
    return done(status, FN)

// tree_attention and, with a first row, tree_attention_rows; with H_kv and a first row, tree_attention_gqa
template <Fn FN>
PyObject *py_attention(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a(args, nargs, FN == ATTN ? 19 : (FN == ATTN_ROWS ? 20 : (FN == ATTN_GQA ? 21 : 18)));
    auto view = (const mcsd_mask_view_t *)a.structure(g_mask_view);
    const auto dtype = (mcsd_dtype_t)a.i32();
    const int32_t B = a.i32(), H = a.i32();
    const int32_t Hkv = FN == ATTN_GQA ? a.i32() : 0;
    const int32_t d = a.i32();
    const int32_t row = FN == ATTN_ROWS || FN == ATTN_GQA ? a.i32() : 0;
    void *q = a.tensor(), *kt = a.tensor(), *vt = a.tensor();
    const int64_t node_stride = a.integer();
    void *kp = a.tensor(), *vp = a.tensor();
    auto base = (const int64_t *)a.tensor();
    auto lens = (const int32_t *)a.tensor();
    const int64_t head_stride = a.integer();
    const int32_t max_prefix = a.i32();
    const float scale = a.f32();
    void *out = a.tensor();
    size_t ws_bytes = 0;
    void *ws = FN == ATTN_STATIC ? nullptr : a.workspace(ws_bytes);
    void *st = a.stream();
    if constexpr (FN == ATTN) {
        MCSD_UNLOCKED(mcsd_tree_attention, FN, view, dtype, B, H, d, q, kt, vt, node_stride, kp, vp, base, lens, head_stride, max_prefix, scale, out, ws, ws_bytes, st);
    } else if constexpr (FN == ATTN_ROWS) {
        MCSD_UNLOCKED(mcsd_tree_attention_rows, FN, view, dtype, B, H, d, row, q, kt, vt, node_stride, kp, vp, base, lens, head_stride, max_prefix, scale, out, ws, ws_bytes, st);
    } else if constexpr (FN == ATTN_GQA) {
        MCSD_UNLOCKED(mcsd_tree_attention_gqa, FN, view, dtype, B, H, Hkv, d, row, q, kt, vt, node_stride, kp, vp, base, lens, head_stride, max_prefix, scale, out, ws, ws_bytes, st);
    } else {
        MCSD_UNLOCKED(mcsd_tree_attention_static, FN, view, dtype, B, H, d, q, kt, vt, node_stride, kp, vp, base, lens, head_stride, max_prefix, scale, out, st);
    }
}

PyObject *py_attention_fp8(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a(args, nargs, 21);
    auto view = (const mcsd_mask_view_t *)a.structure(g_mask_view);
    const int32_t B = a.i32(), H = a.i32(), Hkv = a.i32(), row = a.i32();
    void *q = a.tensor(), *kt = a.tensor(), *vt = a.tensor();
    const int64_t node_stride = a.integer();
    void *kp = a.tensor(), *vp = a.tensor();
    const float ks = a.f32(), vs = a.f32();
    auto base = (const int64_t *)a.tensor();
    auto lens = (const int32_t *)a.tensor();
    const int64_t head_stride = a.integer();
    const int32_t max_prefix = a.i32();
    const float scale = a.f32();
    void *out = a.tensor();
    size_t ws_bytes;
    void *ws = a.workspace(ws_bytes);
    void *st = a.stream();
    MCSD_UNLOCKED(mcsd_tree_attention_fp8kv, ATTN_FP8, view, B, H, Hkv, row, q, kt, vt, node_stride, kp, vp, ks, vs, base, lens, head_stride, max_prefix, scale, out, ws, ws_bytes, st);
}

template <Fn FN>
PyObject *py_verify(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a(args, nargs, FN == VERIFY ? 17 : 18);
    auto view = (const mcsd_mask_view_t *)a.structure(g_mask_view);
    const auto mode = (mcsd_mode_t)a.i32();
    const auto sampling = FN == VERIFY ? MCSD_WITH_REPLACEMENT : (mcsd_sampling_t)a.i32();
    const int32_t B = a.i32(), V = a.i32();
    auto tokens = (const int32_t *)a.tensor();
    auto p = (const float *)a.tensor(), q = (const float *)a.tensor();
    const int64_t ps = a.integer(), qs = a.integer();
    auto ua = (const float *)a.tensor(), us = (const float *)a.tensor();
    const int32_t n_new = a.i32();
    auto path = (int32_t *)a.tensor(), len = (int32_t *)a.tensor(), fresh = (int32_t *)a.tensor();
    size_t ws_bytes;
    void *ws = a.workspace(ws_bytes);
    void *st = a.stream();
    if constexpr (FN == VERIFY) {
        MCSD_UNLOCKED(mcsd_verify_tree, FN, view, mode, B, V, tokens, p, q, ps, qs, ua, us, n_new, path, len, fresh, ws, ws_bytes, st);
    } else {
        MCSD_UNLOCKED(mcsd_verify_tree_sampling, FN, view, mode, sampling, B, V, tokens, p, q, ps, qs, ua, us, n_new, path, len, fresh, ws, ws_bytes, st);
    }
}

PyObject *py_commit(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a(args, nargs, 24);
    auto view = (const mcsd_mask_view_t *)a.structure(g_mask_view);
    const auto dtype = (mcsd_dtype_t)a.i32();
    const int32_t B = a.i32(), H = a.i32(), d = a.i32();
    constexpr int32_t MOST = MCSD_COMMIT_MAX_LAYERS;
    void *kt[MOST], *vt[MOST], *kp[MOST], *vp[MOST];
    const int32_t n_layers = a.tensors(kt, MOST), n2 = a.tensors(vt, MOST);
    const int64_t node_stride = a.integer();
    const int32_t n3 = a.tensors(kp, MOST), n4 = a.tensors(vp, MOST);
    auto base = (const int64_t *)a.tensor();
    const int64_t head_stride = a.integer();
    const int32_t max_prefix = a.i32(), capacity = a.i32();
    auto path = (const int32_t *)a.tensor(), len = (const int32_t *)a.tensor(), tokens = (const int32_t *)a.tensor(), fresh = (const int32_t *)a.tensor();
    const int32_t n_new = a.i32(), n_append = a.i32();
    auto lens = (int32_t *)a.tensor(), ids = (int32_t *)a.tensor(), n_ids = (int32_t *)a.tensor();
    void *st = a.stream();
    if (a.ok && (n2 != n_layers || n3 != n_layers || n4 != n_layers)) {
        PyErr_SetString(PyExc_AssertionError, "as many tensors per list as layers");
        return nullptr;
    }
    // (more layers than the arrays hold: the entry point answers before it reads them)
    MCSD_UNLOCKED(mcsd_commit_path, COMMIT, view, dtype, B, H, d, n_layers, kt, vt, node_stride, kp, vp, base, head_stride, max_prefix, capacity, path, len, tokens, fresh,
                  n_new, n_append, lens, ids, n_ids, st);
}

PyObject *py_stop_distribution(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a(args, nargs, 13);
    auto mlp = (const mcsd_mlp_t *)a.structure(g_mlp);
    const int32_t B = a.i32(), W = a.i32(), V = a.i32(), k = a.i32();
    auto rows = (const float *)a.tensor();
    const int64_t bs = a.integer(), rs = a.integer();
    const float beta = a.f32();
    auto features = (float *)a.tensor(), prob = (float *)a.tensor();
    auto stop = (int32_t *)a.tensor();
    void *st = a.stream();
    MCSD_UNLOCKED(mcsd_early_stop_distribution, STOP_DIST, mlp, B, W, V, k, rows, bs, rs, beta, features, prob, stop, st);
}

PyObject *py_stop_hidden(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a(args, nargs, 10);
    auto mlp = (const mcsd_mlp_t *)a.structure(g_mlp);
    const int32_t B = a.i32(), W = a.i32();
    auto hidden = (const float *)a.tensor();
    const int64_t bs = a.integer(), rs = a.integer();
    const float beta = a.f32();
    auto prob = (float *)a.tensor();
    auto stop = (int32_t *)a.tensor();
    void *st = a.stream();
    MCSD_UNLOCKED(mcsd_early_stop_hidden, STOP_HIDDEN, mlp, B, W, hidden, bs, rs, beta, prob, stop, st);
}

// slice_mask(handle, gamma, view): fills the view
PyObject *py_slice(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    Args a(args, nargs, 3);
    auto mask = nargs == 3 && args[0] == Py_None ? (a.i++, nullptr) : (const mcsd_mask_t *)(uintptr_t)a.integer();
    const int32_t gamma = a.i32();
    auto view = (mcsd_mask_view_t *)a.structure(g_mask_view);
    if (!a.ok) return nullptr;
    return done(((decltype(&mcsd_slice_mask))g_fn[SLICE])(mask, gamma, view), SLICE);
}

// setup(addresses of the entry points in the order of Fn, torch.Tensor, raw_stream, device, raise, MaskView, Mlp, ctypes.ArgumentError)
PyObject *py_setup(PyObject *, PyObject *args)
{
    PyObject *addr;
    if (!PyArg_ParseTuple(args, "O!OOOOO!O!O", &PyTuple_Type, &addr, &g_tensor, &g_raw_stream, &g_device, &g_raise, &PyType_Type, &g_mask_view,
                          &PyType_Type, &g_mlp, &g_argument_error)) return nullptr;
    if (PyTuple_GET_SIZE(addr) != N_FN) {
        PyErr_SetString(PyExc_ValueError, "one address per entry point");
        return nullptr;
    }
    for (int i = 0; i < N_FN; ++i) g_fn[i] = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(PyTuple_GET_ITEM(addr, i));
    for (PyObject *o : {g_tensor, g_raw_stream, g_device, g_raise, g_mask_view, g_mlp, g_argument_error}) Py_INCREF(o);       // held for the life of the process
    g_data_ptr = PyObject_GetAttr(g_tensor, g_str_data_ptr);
    g_numel = PyObject_GetAttr(g_tensor, g_str_numel);
    g_element_size = PyObject_GetAttr(g_tensor, g_str_element_size);
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

PyObject *py_names(PyObject *, PyObject *)
{
    PyObject *t = PyTuple_New(N_FN);
    for (int i = 0; t && i < N_FN; ++i) PyTuple_SET_ITEM(t, i, PyUnicode_FromString(FN_NAME[i]));
    return t;
}

#define FAST(name, f) {name, (PyCFunction)(void (*)(void))(f), METH_FASTCALL, nullptr}
PyMethodDef METHODS[] = {
    {"setup", py_setup, METH_VARARGS, nullptr},
    {"names", py_names, METH_NOARGS, nullptr},
    FAST("tree_attention", (py_attention<ATTN>)),
    FAST("tree_attention_rows", (py_attention<ATTN_ROWS>)),
    FAST("tree_attention_gqa", (py_attention<ATTN_GQA>)),
    FAST("tree_attention_static", (py_attention<ATTN_STATIC>)),
    FAST("tree_attention_fp8kv", py_attention_fp8),
    FAST("verify_tree", (py_verify<VERIFY>)),
    FAST("verify_tree_sampling", (py_verify<VERIFY_SAMPLING>)),
    FAST("commit_path", py_commit),
    FAST("early_stop_distribution", py_stop_distribution),
    FAST("early_stop_hidden", py_stop_hidden),
    FAST("slice_mask", py_slice),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef MODULE = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, METHODS, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void)
{
    g_str_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_str_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    g_str_numel = PyUnicode_InternFromString("numel");
    g_str_element_size = PyUnicode_InternFromString("element_size");
    return PyModule_Create(&MODULE);
}
