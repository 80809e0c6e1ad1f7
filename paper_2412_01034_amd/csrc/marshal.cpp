// The marshalling of binding.py's smallest calls without the interpreter in between: it asks each tensor for its size, place,
// layout and address in C++ and calls the library's C function.  4096 x 4096 at M = 1 takes 4.5 us on the GPU, and asking from
// Python took longer than that.
//
// A function returns the library's status, or None for everything that is not the plain case (another type than torch.Tensor, a
// torch function mode, a tensor that is too small, on the host or not contiguous, numbers that do not fit): binding.py then goes its
// own way, with its own errors.  Nothing is kept between calls but the addresses of the library's functions.
//
// Layouts of torch, Python and qail.h are compiled in, so the module says what it was built for (`built_for`) and binding.py uses it with
// nothing else.
#define PY_SSIZE_T_CLEAN
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "qail.h"

namespace {

decltype(&qail_w4a16_linear) g_linear = nullptr;
decltype(&qail_w4a16_linear_batch) g_linear_batch = nullptr;
decltype(&qail_w4a4_conv_batch) g_conv_batch = nullptr;

bool number(PyObject* o, int32_t& v) {   // an int of at least 0 that fits 32 bits
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long long l = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || l < 0 || l > INT_MAX) return false;
    v = (int32_t)l;
    return true;
}

// The address of a plain contiguous tensor on the GPU of at least `need` bytes.
template <typename T>
bool tensor(PyObject* o, int64_t need, T*& p, size_t* nbytes = nullptr) {
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous() || (int64_t)t.nbytes() < need) return false;
    p = static_cast<T*>(t.data_ptr());
    if (nbytes) *nbytes = t.nbytes();
    return true;
}

// The array a ctypes object holds.
struct Items {
    Py_buffer view{};
    explicit Items(PyObject* o) {
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            view.buf = nullptr;
        }
    }
    ~Items() {
        if (view.buf) PyBuffer_Release(&view);
    }
};

template <typename F>
PyObject* call(F f) {
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// Runs f, which returns nullptr where the call is not a plain one; whatever torch throws is left to the other way too.
template <typename F>
PyObject* plainly(F f) {
    PyObject* r = nullptr;
    try {
        if (!at::impl::torch_function_mode_enabled()) r = f();
    } catch (...) {
        PyErr_Clear();
    }
    if (r) return r;
    Py_RETURN_NONE;
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// (N, K, group_size, qweight, scales, zeros, x, y, M, workspace)
PyObject* w4a16_linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return plainly([&]() -> PyObject* {
        int32_t N, K, g, M;
        if (n != 10 || !g_linear || !number(a[0], N) || !number(a[1], K) || !number(a[2], g) || !number(a[8], M) || g == 0) return nullptr;
        const int64_t G = K / g;
        const uint32_t *q, *z;
        const uint16_t *s, *x;
        uint16_t* y;
        void* ws = nullptr;
        size_t ws_bytes = 0;
        if (!tensor(a[3], (int64_t)N * K / 2, q) || !tensor(a[4], N * G * 2, s) || !tensor(a[5], N * ((G + 7) / 8) * 4, z) ||
            !tensor(a[6], (int64_t)M * K * 2, x) || !tensor(a[7], (int64_t)M * N * 2, y) ||
            (a[9] != Py_None && !tensor(a[9], 0, ws, &ws_bytes)))
            return nullptr;
        const qail_wdesc d = {N, K, g, QAIL_W4_ASYM_GROUP};
        void* const st = stream();
        return call([&] { return g_linear(&d, q, s, z, x, y, M, ws, ws_bytes, st); });
    });
}

// (items, count, M, workspace)
PyObject* w4a16_linear_batch(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return plainly([&]() -> PyObject* {
        int32_t count, M;
        void* ws = nullptr;
        size_t ws_bytes = 0;
        if (n != 4 || !g_linear_batch || !number(a[1], count) || !number(a[2], M) || (a[3] != Py_None && !tensor(a[3], 0, ws, &ws_bytes)))
            return nullptr;
        const Items items(a[0]);
        if (!items.view.buf) return nullptr;
        void* const st = stream();
        return call([&] { return g_linear_batch(static_cast<const qail_w4a16_item*>(items.view.buf), count, M, ws, ws_bytes, st); });
    });
}

// (items, count)
PyObject* w4a4_conv_batch(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return plainly([&]() -> PyObject* {
        int32_t count;
        if (n != 2 || !g_conv_batch || !number(a[1], count)) return nullptr;
        const Items items(a[0]);
        if (!items.view.buf) return nullptr;
        void* const st = stream();
        return call([&] { return g_conv_batch(static_cast<const qail_conv_item*>(items.view.buf), count, st); });
    });
}

// Addresses of qail_w4a16_linear, qail_w4a16_linear_batch and qail_w4a4_conv_batch.
PyObject* use(PyObject*, PyObject* args) {
    unsigned long long l, b, c;
    if (!PyArg_ParseTuple(args, "KKK", &l, &b, &c)) return nullptr;
    g_linear = reinterpret_cast<decltype(g_linear)>(l);
    g_linear_batch = reinterpret_cast<decltype(g_linear_batch)>(b);
    g_conv_batch = reinterpret_cast<decltype(g_conv_batch)>(c);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"use", use, METH_VARARGS, nullptr},
    {"w4a16_linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(w4a16_linear)), METH_FASTCALL, nullptr},
    {"w4a16_linear_batch", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(w4a16_linear_batch)), METH_FASTCALL, nullptr},
    {"w4a4_conv_batch", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(w4a4_conv_batch)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    PyObject* m = PyModule_Create(&module);
    PyObject* built_for = m ? Py_BuildValue("(lsnnn)", (long)(PY_VERSION_HEX >> 16), QAIL_TORCH, (Py_ssize_t)sizeof(qail_wdesc),
                                            (Py_ssize_t)sizeof(qail_w4a16_item), (Py_ssize_t)sizeof(qail_conv_item))
                            : nullptr;
    if (!built_for || PyModule_AddObject(m, "built_for", built_for) < 0) {   // (takes the reference where it succeeds)
        Py_XDECREF(built_for);
        Py_XDECREF(m);
        return nullptr;
    }
    return m;
}
