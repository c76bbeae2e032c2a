// Native argument marshalling for the entry points of a decode step.
//
// A decode step of a small batch is two launches of 5-15 us each.  Through ctypes (a property, a method call
// and a c_void_p object per tensor, and torch.cuda.current_stream()) the host took 8.0 us per call of chunk_score,
// launch included, and 24.5 us for the two calls of the fp32 4K step (three launches then), so the host, not the
// GPU, set the pace of such a step.  Here a tensor costs one type check and three field reads: 4.0 us per
// chunk_score, 9.0 us per step (two launches).
//
// Every function takes the arguments of the C entry point of the same name (include/leoam.h) in its
// order, tensors or None for device pointers, the stream as whatever binding._stream takes (it is called
// last, after every tensor has been looked at), and returns the status.  Nothing is kept from one call for
// the next: every tensor is looked at on every call.  Only plain torch.Tensor objects are read here; anything
// else (subclasses, other objects with the same methods, tensors whose fields raise) goes through the checker
// that binding.py registers, which raises what it always raised.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/leoam.h"

namespace {

PyObject* g_shape_type = nullptr;      // binding.Shape
PyObject* g_pointer_of = nullptr;      // binding._p: tensor -> ctypes.c_void_p or None, raises ValueError

PyObject* g_stream_of = nullptr;       // binding._stream: stream object, integer or None -> handle

// the entry points of the library that binding.py loaded (addresses handed over by setup, so this
// module depends on no second copy of it)
struct {
    decltype(&::chunk_score) chunk_score;
    decltype(&::chunk_score_pin) chunk_score_pin;
    decltype(&::kv_chunk_abstract_append) kv_chunk_abstract_append;
    decltype(&::chunk_topk_select) chunk_topk_select;
    decltype(&::sparse_chunk_attention_decode) sparse_chunk_attention_decode;
    decltype(&::chunk_select_attention_decode) chunk_select_attention_decode;
} g_lib;
constexpr int kEntryPoints = 6;
static_assert(sizeof(g_lib) == kEntryPoints * sizeof(void*), "one address each");

// device pointer of a tensor (or None); false with a Python error set
bool pointer_arg(PyObject* o, void** out) {
    *out = nullptr;
    if (o == Py_None) return true;
    if (THPVariable_CheckExact(o)) {
        try {
            const at::Tensor& t = THPVariable_Unpack(o);
            if (t.is_cuda() && t.is_contiguous()) {
                *out = t.data_ptr();
                return true;
            }
        } catch (const std::exception&) {
            // (the checker below raises it as the Python error it is)
        }
    }
    PyObject* p = PyObject_CallOneArg(g_pointer_of, o);
    if (!p) return false;
    PyObject* v = p == Py_None ? Py_NewRef(Py_None) : PyObject_GetAttrString(p, "value");
    Py_DECREF(p);
    if (!v) return false;
    if (v != Py_None) *out = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    return !PyErr_Occurred();
}

// 32-bit integers wrap as ctypes lets them
bool int_arg(PyObject* o, int32_t* out) {
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) return false;
    *out = (int32_t)(uint32_t)v;
    return true;
}

// The arguments of one call, read in order; `ok` turns false (with a Python error set) at the first bad one.
struct Args {
    PyObject* const* a;
    Py_ssize_t n, i = 0;
    bool ok = true;
    leoam_shape shape;

    Args(PyObject* const* args, Py_ssize_t nargs, Py_ssize_t wanted) : a(args), n(nargs) {
        if (nargs != wanted) {
            PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", wanted, nargs);
            ok = false;
            return;
        }
        const int is = PyObject_IsInstance(a[0], g_shape_type);
        if (is < 0) {
            ok = false;
            return;
        }
        if (is == 0) {
            PyErr_SetString(PyExc_TypeError, "expected a Shape");
            ok = false;
            return;
        }
        Py_buffer view;
        if (PyObject_GetBuffer(a[0], &view, PyBUF_SIMPLE) != 0) {
            ok = false;
            return;
        }
        ok = view.len == (Py_ssize_t)sizeof(leoam_shape);
        if (ok) memcpy(&shape, view.buf, sizeof(leoam_shape));
        else PyErr_SetString(PyExc_TypeError, "Shape has another layout");
        PyBuffer_Release(&view);
        i = 1;
    }
    template <typename P = void> P* ptr() {
        void* p = nullptr;
        if (ok) ok = pointer_arg(a[i++], &p);
        return static_cast<P*>(p);
    }
    int32_t i32() {
        int32_t v = 0;
        if (ok) ok = int_arg(a[i++], &v);
        return v;
    }
    float f32() {
        double v = 0.0;
        if (ok) {
            v = PyFloat_AsDouble(a[i++]);
            ok = !(v == -1.0 && PyErr_Occurred());
        }
        return (float)v;
    }
    size_t bytes() {
        size_t v = 0;
        if (ok) {
            v = PyLong_AsSize_t(a[i++]);
            ok = !(v == (size_t)-1 && PyErr_Occurred());
        }
        return v;
    }
    void* stream() {
        void* v = nullptr;
        if (ok) {
            PyObject* s = PyObject_CallOneArg(g_stream_of, a[i++]);
            if (s) v = PyLong_AsVoidPtr(s);
            Py_XDECREF(s);
            ok = !PyErr_Occurred();
        }
        return v;
    }
};

// the call runs without the interpreter lock (a launch can wait for room in the queue)
template <typename F> PyObject* status_of(const Args& args, F&& call) {
    if (!args.ok) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyObject* py_setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 3 + kEntryPoints) {
        PyErr_SetString(PyExc_TypeError, "setup(shape_type, pointer_of, stream_of, addresses in the order of g_lib)");
        return nullptr;
    }
    void* at[kEntryPoints];
    for (int i = 0; i < kEntryPoints; ++i) {
        at[i] = PyLong_AsVoidPtr(a[3 + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    memcpy(&g_lib, at, sizeof(g_lib));
    Py_XDECREF(g_shape_type);
    Py_XDECREF(g_pointer_of);
    Py_XDECREF(g_stream_of);
    g_shape_type = Py_NewRef(a[0]);
    g_pointer_of = Py_NewRef(a[1]);
    g_stream_of = Py_NewRef(a[2]);
    Py_RETURN_NONE;
}

PyObject* py_chunk_score(PyObject*, PyObject* const* a, Py_ssize_t n) {
    Args r(a, n, 7);
    const void* q = r.ptr();
    const void* abstract = r.ptr();
    const int32_t* n_chunks = r.ptr<int32_t>();
    float* ub = r.ptr<float>();
    float* lb = r.ptr<float>();
    void* st = r.stream();
    return status_of(r, [&] { return g_lib.chunk_score(&r.shape, q, abstract, n_chunks, ub, lb, st); });
}

PyObject* py_chunk_score_pin(PyObject*, PyObject* const* a, Py_ssize_t n) {
    Args r(a, n, 6);
    const int32_t* n_chunks = r.ptr<int32_t>();
    const int32_t sink = r.i32(), tail = r.i32();
    float* ub = r.ptr<float>();
    void* st = r.stream();
    return status_of(r, [&] { return g_lib.chunk_score_pin(&r.shape, n_chunks, sink, tail, ub, st); });
}

PyObject* py_abstract_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
    Args r(a, n, 8);
    const void* K = r.ptr();
    int32_t* off = r.ptr<int32_t>();
    int32_t* n_chunks = r.ptr<int32_t>();
    const int32_t chunk_size = r.i32();
    void* abstract = r.ptr();
    int32_t* status = r.ptr<int32_t>();
    void* st = r.stream();
    return status_of(r, [&] { return g_lib.kv_chunk_abstract_append(&r.shape, K, off, n_chunks, chunk_size, abstract, status, st); });
}

PyObject* py_topk_select(PyObject*, PyObject* const* a, Py_ssize_t n) {
    Args r(a, n, 12);
    const float* ub = r.ptr<float>();
    const int32_t* off = r.ptr<int32_t>();
    const int32_t* n_chunks = r.ptr<int32_t>();
    const int32_t max_chunks = r.i32(), budget = r.i32();
    int32_t* idx = r.ptr<int32_t>();
    int32_t* count = r.ptr<int32_t>();
    int32_t* tokens = r.ptr<int32_t>();
    void* ws = r.ptr();
    const size_t ws_bytes = r.bytes();
    void* st = r.stream();
    return status_of(r, [&] {
        return g_lib.chunk_topk_select(&r.shape, ub, off, n_chunks, max_chunks, budget, idx, count, tokens, ws, ws_bytes, st);
    });
}

PyObject* py_sparse_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
    Args r(a, n, 15);
    const void* q = r.ptr();
    const void* K = r.ptr();
    const void* V = r.ptr();
    const void* qmeta = r.ptr();
    const int32_t* off = r.ptr<int32_t>();
    const int32_t* n_chunks = r.ptr<int32_t>();
    const int32_t* idx = r.ptr<int32_t>();
    const int32_t* count = r.ptr<int32_t>();
    const float scale = r.f32();
    float* out = r.ptr<float>();
    float* lse = r.ptr<float>();
    void* ws = r.ptr();
    const size_t ws_bytes = r.bytes();
    void* st = r.stream();
    return status_of(r, [&] {
        return g_lib.sparse_chunk_attention_decode(&r.shape, q, K, V, qmeta, off, n_chunks, idx, count, scale, out, lse, ws, ws_bytes, st);
    });
}

PyObject* py_select_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
    Args r(a, n, 19);
    const float* ub = r.ptr<float>();
    const void* q = r.ptr();
    const void* K = r.ptr();
    const void* V = r.ptr();
    const void* qmeta = r.ptr();
    const int32_t* off = r.ptr<int32_t>();
    const int32_t* n_chunks = r.ptr<int32_t>();
    const int32_t max_chunks = r.i32(), budget = r.i32();
    const float scale = r.f32();
    int32_t* idx = r.ptr<int32_t>();
    int32_t* count = r.ptr<int32_t>();
    int32_t* tokens = r.ptr<int32_t>();
    float* out = r.ptr<float>();
    float* lse = r.ptr<float>();
    void* ws = r.ptr();
    const size_t ws_bytes = r.bytes();
    void* st = r.stream();
    return status_of(r, [&] {
        return g_lib.chunk_select_attention_decode(&r.shape, ub, q, K, V, qmeta, off, n_chunks, max_chunks, budget, scale, idx, count,
                                             tokens, out, lse, ws, ws_bytes, st);
    });
}

#define LEOAM_METHOD(name, fn) {name, (PyCFunction)(void (*)(void))fn, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {LEOAM_METHOD("setup", py_setup),
                           LEOAM_METHOD("chunk_score", py_chunk_score),
                           LEOAM_METHOD("chunk_score_pin", py_chunk_score_pin),
                           LEOAM_METHOD("kv_chunk_abstract_append", py_abstract_append),
                           LEOAM_METHOD("chunk_topk_select", py_topk_select),
                           LEOAM_METHOD("sparse_chunk_attention_decode", py_sparse_attention),
                           LEOAM_METHOD("chunk_select_attention_decode", py_select_attention),
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_bind", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind() { return PyModule_Create(&g_module); }
