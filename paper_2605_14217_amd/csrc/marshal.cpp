// Marshalling of the calls of a serving loop: the arguments of a schedule or apply call, as torch tensors, to the C ABI.
//
// A ctypes call of 21 arguments, with every property of ten tensors asked for from Python, takes 4 to 7 us beside the 3 us of
// the launch itself; a launch of 6 us waits for it.  Here the same takes below 1 us, also with the slot manager's pools (binding.PoolRef) and with
// numbers of any type.  Anything else -- a tensor subclass, another table, a check that fails, an exception of torch -- answers None, and the
// caller goes through binding.py's own path, which makes the same checks and raises what they raise.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/preft.h"

namespace {

decltype(&preft_schedule) g_schedule;
decltype(&preft_lora_apply) g_lora;
decltype(&preft_lora_apply_packed) g_packed;
decltype(&preft_direft_apply) g_direft;
decltype(&preft_loreft_apply) g_loreft;
decltype(&preft_direft_apply_layers) g_layers;

const at::Tensor *tensor(PyObject *o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

struct Matrix { void *p; int64_t ld; int32_t rows, cols; at::ScalarType type; };

bool as_matrix(PyObject *o, Matrix &m)
{
    const at::Tensor *t = tensor(o);
    if (!t || t->dim() != 2 || !t->is_cuda() || t->stride(1) != 1) return false;
    if (t->size(0) > INT32_MAX || t->size(1) > INT32_MAX) return false;
    m = {t->data_ptr(), t->stride(0), (int32_t)t->size(0), (int32_t)t->size(1), t->scalar_type()};
    return m.type == at::kBFloat16 || m.type == at::kFloat;
}

// a contiguous device table of n entries
template <typename T>
bool as_table(PyObject *o, int64_t n, T *&p)
{
    const at::Tensor *t = tensor(o);
    if (!t || t->scalar_type() != (sizeof(T) == 4 ? at::kInt : at::kLong) || t->numel() != n || !t->is_cuda() || !t->is_contiguous()) return false;
    p = static_cast<T *>(t->data_ptr());
    return true;
}

struct Segments { int32_t *start, *adapter, *prefill, S; };

bool as_segments(PyObject *const *o, Segments &s)
{
    const at::Tensor *t = tensor(o[1]);
    if (!t || t->numel() >= INT32_MAX) return false;
    s.S = (int32_t)t->numel();
    return as_table(o[0], (int64_t)s.S + 1, s.start) && as_table(o[1], s.S, s.adapter) && as_table(o[2], s.S, s.prefill);
}

PyObject *g_pool_ref, *g_address, *g_length;                  // binding.PoolRef, and the names of what it holds

bool as_pool_ref(PyObject *o, int64_t &n, const void *const *&p)
{
    if ((PyObject *)Py_TYPE(o) != g_pool_ref) return false;
    PyObject *address = PyObject_GetAttr(o, g_address), *length = address ? PyObject_GetAttr(o, g_length) : nullptr;
    bool ok = length && PyLong_CheckExact(address) && PyLong_CheckExact(length);
    if (ok) {
        void *at = PyLong_AsVoidPtr(address);
        const long long count = PyLong_AsLongLong(length);
        ok = !PyErr_Occurred() && count >= 0 && count <= INT32_MAX && (n < 0 || count == n);
        if (ok) { p = static_cast<const void *const *>(at); n = count; }
    }
    Py_XDECREF(address);
    Py_XDECREF(length);
    return ok;
}

bool as_pool(PyObject *o, int64_t &n, const void *const *&p)      // n < 0: any length
{
    if (as_pool_ref(o, n, p)) return true;
    const at::Tensor *t = tensor(o);
    if (!t || t->scalar_type() != at::kLong || (n >= 0 && t->numel() != n) || t->numel() > INT32_MAX) return false;
    n = t->numel();
    p = static_cast<const void *const *>(t->data_ptr());
    return true;
}

bool as_int(PyObject *o, int32_t &v)
{
    int overflow = 0;
    long long x;
    if (PyLong_CheckExact(o)) {
        x = PyLong_AsLongLongAndOverflow(o, &overflow);
    } else {                                                  // whole numbers of other types: NumPy's, truth values
        PyObject *i = PyIndex_Check(o) ? PyNumber_Index(o) : nullptr;
        if (!i) return false;
        x = PyLong_AsLongLongAndOverflow(i, &overflow);
        Py_DECREF(i);
    }
    if (overflow || x < INT32_MIN || x > INT32_MAX) return false;
    v = (int32_t)x;
    return true;
}

// what every apply call ends with: rank, scale, mode, workspace, stream, further mode bits
struct Rest { int32_t rank, mode, extra; float scale; void *workspace, *stream; size_t bytes; };

bool as_workspace(PyObject *o, void *&p, size_t &bytes)
{
    const at::Tensor *t = tensor(o);
    if (!t) return false;
    p = t->data_ptr();
    bytes = (size_t)t->numel() * t->element_size();
    return true;
}

bool as_stream(PyObject *o, void *&p)
{
    if (!PyLong_CheckExact(o)) return false;
    p = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}

bool as_rest(PyObject *const *o, Rest &r)
{
    if (!as_int(o[0], r.rank) || !as_int(o[2], r.mode) || !as_int(o[5], r.extra)) return false;
    const double scale = PyFloat_AsDouble(o[1]);              // whole numbers and NumPy's too
    if (scale == -1.0 && PyErr_Occurred()) return false;
    r.scale = (float)scale;
    r.mode |= r.extra;
    return as_workspace(o[3], r.workspace, r.bytes) && as_stream(o[4], r.stream);
}

int dtype_of(at::ScalarType t) { return t == at::kBFloat16 ? PREFT_BF16 : PREFT_F32; }

template <typename F>
PyObject *answer(F call)
{
    try {
        int rc = 0;
        if (call(rc)) return PyLong_FromLong(rc);
    } catch (...) {                                           // the caller's own path says what is wrong
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}

template <typename F>
int without_gil(F launch)
{
    PyThreadState *state = PyEval_SaveThread();
    const int rc = launch();
    PyEval_RestoreThread(state);
    return rc;
}

// (workspace, seg_start, seg_adapter, seg_prefill_len, T, N, mode, stream)
PyObject *schedule(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    return answer([&](int &rc) {
        Segments s;
        void *ws, *stream;
        size_t bytes;
        int32_t T, N, mode;
        if (n != 8 || !g_schedule || !as_workspace(o[0], ws, bytes) || !as_segments(o + 1, s) || !as_int(o[4], T) || !as_int(o[5], N) ||
            !as_int(o[6], mode) || !as_stream(o[7], stream)) return false;
        rc = without_gil([&] { return g_schedule(ws, bytes, s.start, s.adapter, s.prefill, s.S, T, N, mode, stream); });
        return true;
    });
}

// (y, x, seg_start, seg_adapter, seg_prefill_len, A_pool, B_pool, rest ...)
PyObject *lora(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    return answer([&](int &rc) {
        Matrix y, x;
        Segments s;
        Rest r;
        int64_t N = -1;
        const void *const *A, *const *B;
        if (n != 13 || !g_lora || !as_matrix(o[0], y) || !as_matrix(o[1], x) || y.rows != x.rows || y.type != x.type || !as_segments(o + 2, s) ||
            !as_pool(o[5], N, A) || !as_pool(o[6], N, B) || !as_rest(o + 7, r)) return false;
        rc = without_gil([&] {
            return g_lora(y.p, y.ld, x.p, x.ld, y.rows, x.cols, y.cols, s.start, s.adapter, s.prefill, s.S, A, B, (int32_t)N, r.rank, r.scale,
                          dtype_of(y.type), r.mode, r.workspace, r.bytes, r.stream);
        });
        return true;
    });
}

// (ys, x, seg_start, seg_adapter, seg_prefill_len, A_pools, B_pools, rest ...); ys and the pools lists or tuples
PyObject *lora_packed(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    return answer([&](int &rc) {
        auto sequence = [](PyObject *v) { return PyList_CheckExact(v) || PyTuple_CheckExact(v); };
        if (n != 13 || !g_packed || !sequence(o[0]) || !sequence(o[5]) || !sequence(o[6])) return false;
        const Py_ssize_t k = PySequence_Fast_GET_SIZE(o[0]);
        if (k < 1 || k > PREFT_MAX_PACKED || PySequence_Fast_GET_SIZE(o[5]) != k || PySequence_Fast_GET_SIZE(o[6]) != k) return false;
        Matrix x, y;
        Segments s;
        Rest r;
        int64_t N = -1, ld[PREFT_MAX_PACKED];
        void *yp[PREFT_MAX_PACKED];
        int32_t d_out[PREFT_MAX_PACKED];
        const void *const *A[PREFT_MAX_PACKED], *const *B[PREFT_MAX_PACKED];
        if (!as_matrix(o[1], x) || !as_segments(o + 2, s) || !as_rest(o + 7, r)) return false;
        for (Py_ssize_t i = 0; i < k; ++i) {
            if (!as_matrix(PySequence_Fast_GET_ITEM(o[0], i), y) || y.rows != x.rows || y.type != x.type ||
                !as_pool(PySequence_Fast_GET_ITEM(o[5], i), N, A[i]) || !as_pool(PySequence_Fast_GET_ITEM(o[6], i), N, B[i])) return false;
            yp[i] = y.p; ld[i] = y.ld; d_out[i] = y.cols;
        }
        rc = without_gil([&] {
            return g_packed((int32_t)k, yp, ld, d_out, x.p, x.ld, x.rows, x.cols, s.start, s.adapter, s.prefill, s.S, A, B, (int32_t)N, r.rank,
                            r.scale, dtype_of(x.type), r.mode, r.workspace, r.bytes, r.stream);
        });
        return true;
    });
}

// (loreft, h, seg_start, seg_adapter, seg_prefill_len, W1_pool, W2t_pool, b_pool or None, rest ...)
PyObject *reft(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    return answer([&](int &rc) {
        Matrix h;
        Segments s;
        Rest r;
        int64_t N = -1;
        const void *const *W1, *const *W2t, *const *b = nullptr;
        if (n != 14 || !g_direft || !g_loreft || !as_matrix(o[1], h) || !as_segments(o + 2, s) || !as_pool(o[5], N, W1) || !as_pool(o[6], N, W2t) ||
            (o[7] != Py_None && !as_pool(o[7], N, b)) || !as_rest(o + 8, r)) return false;
        const auto entry = o[0] == Py_True ? g_loreft : g_direft;
        rc = without_gil([&] {
            return entry(h.p, h.ld, h.rows, h.cols, s.start, s.adapter, s.prefill, s.S, W1, W2t, b, (int32_t)N, r.rank, r.scale, dtype_of(h.type),
                         r.mode, r.workspace, r.bytes, r.stream);
        });
        return true;
    });
}

// (hs, h_layers, seg_start, seg_adapter, seg_prefill_len, W1_pools, W2t_pools, b_pools or None, N, rest ...); hs a list or tuple
PyObject *reft_layers(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    return answer([&](int &rc) {
        if (n != 15 || !g_layers || !(PyList_CheckExact(o[0]) || PyTuple_CheckExact(o[0]))) return false;
        const Py_ssize_t L = PySequence_Fast_GET_SIZE(o[0]);
        if (L < 1 || L > PREFT_MAX_LAYERS) return false;
        Matrix h, first;
        for (Py_ssize_t i = 0; i < L; ++i) {
            if (!as_matrix(PySequence_Fast_GET_ITEM(o[0], i), h)) return false;
            if (i == 0) first = h;
            if (h.ld != first.ld || h.rows != first.rows || h.cols != first.cols || h.type != first.type) return false;
        }
        Segments s;
        Rest r;
        int32_t N;
        int64_t *table, *W1, *W2t, *b = nullptr;
        if (!as_table(o[1], L, table) || !as_segments(o + 2, s) || !as_table(o[5], L, W1) || !as_table(o[6], L, W2t) ||
            (o[7] != Py_None && !as_table(o[7], L, b)) || !as_int(o[8], N) || !as_rest(o + 9, r)) return false;
        using Pools = const void *const *const *;
        rc = without_gil([&] {
            return g_layers(reinterpret_cast<void *const *>(table), h.ld, (int32_t)L, h.rows, h.cols, s.start, s.adapter, s.prefill, s.S,
                            reinterpret_cast<Pools>(W1), reinterpret_cast<Pools>(W2t), reinterpret_cast<Pools>(b), N, r.rank, r.scale,
                            dtype_of(h.type), r.mode, r.workspace, r.bytes, r.stream);
        });
        return true;
    });
}

// binding.PoolRef, and the addresses of the loaded library's entry points in the order below
PyObject *bind(PyObject *, PyObject *const *o, Py_ssize_t n)
{
    void *p[6];
    if (n != 7) { PyErr_SetString(PyExc_TypeError, "a class and six addresses"); return nullptr; }
    PyObject *const pool_ref = *o++;
    for (int i = 0; i < 6; ++i) {
        p[i] = PyLong_AsVoidPtr(o[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    g_schedule = reinterpret_cast<decltype(g_schedule)>(p[0]);
    g_lora = reinterpret_cast<decltype(g_lora)>(p[1]);
    g_packed = reinterpret_cast<decltype(g_packed)>(p[2]);
    g_direft = reinterpret_cast<decltype(g_direft)>(p[3]);
    g_loreft = reinterpret_cast<decltype(g_loreft)>(p[4]);
    g_layers = reinterpret_cast<decltype(g_layers)>(p[5]);
    if (!g_address) g_address = PyUnicode_InternFromString("_address");
    if (!g_length) g_length = PyUnicode_InternFromString("_n");
    if (!g_address || !g_length) return nullptr;
    Py_INCREF(pool_ref);
    Py_XDECREF(g_pool_ref);
    g_pool_ref = pool_ref;
    Py_RETURN_NONE;
}

// What it was compiled against (build.py): sizes, strides and addresses are read at that torch's and Python's offsets
PyObject *built_for(PyObject *, PyObject *) { return PyUnicode_FromString(PREFT_BUILT_FOR); }

PyMethodDef methods[] = {
    {"built_for", built_for, METH_NOARGS, nullptr},
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(bind)), METH_FASTCALL, nullptr},
    {"schedule", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(schedule)), METH_FASTCALL, nullptr},
    {"lora", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(lora)), METH_FASTCALL, nullptr},
    {"lora_packed", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(lora_packed)), METH_FASTCALL, nullptr},
    {"reft", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(reft)), METH_FASTCALL, nullptr},
    {"reft_layers", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(reft_layers)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
