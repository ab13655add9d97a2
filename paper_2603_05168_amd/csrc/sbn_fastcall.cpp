// The Python side of one call, in C++: shapes, types, pointers and the current stream are read from the tensors without the
// interpreter, and the C ABI is called.  A direct call of the layer costs the host 2.1 us less its launch in Python and 0.6 here (the
// kernel of one token through 2560 x 2560 takes 3.4 us), so without this the host and not the device sets the pace of single calls.
// Marshalling only: whatever is not a plain tensor of the expected kind (an integer address, a subclass, another type or rank, a
// tensor without storage) is answered with None, and the Python code beside it does the call or raises its own error.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <exception>
#include <new>

namespace {

using linear_fn = int (*)(const void *, int64_t, int64_t, int64_t, int, int, const void *, const float *, const float *, float *, int8_t *, float *,
                          int32_t *, int, void *, size_t, void *);
using grouped_fn = int (*)(int, const void *const *, const int64_t *, const int64_t *, const int64_t *, int, int, const void *const *,
                           const float *const *, float *const *, int, void *, size_t, void *);
linear_fn g_linear = nullptr;
grouped_fn g_grouped = nullptr;

const at::Tensor *plain(PyObject *o)
{
    return Py_TYPE(o) == reinterpret_cast<PyTypeObject *>(THPVariableClass) ? &THPVariable_Unpack(o) : nullptr;
}

// address of a plain tensor, null for None; false for anything else
bool address(PyObject *o, void *&p)
{
    p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor *t = plain(o);
    if (!t) return false;
    p = t->data_ptr();
    return true;
}

bool small_int(PyObject *o, int &v)
{
    if (!PyLong_CheckExact(o)) return false;
    const long l = PyLong_AsLong(o);
    if ((l == -1 && PyErr_Occurred()) || l < INT32_MIN || l > INT32_MAX) {
        PyErr_Clear();
        return false;
    }
    v = (int)l;
    return true;
}

// The call itself, without the interpreter's lock: -> status, or null with a Python error where it throws (the lock is held again by
// then; the call has begun, so the Python code must not do it once more)
template <class Call> PyObject *released(Call &&call)
{
    struct Unlocked {
        PyThreadState *state = PyEval_SaveThread();
        ~Unlocked() { PyEval_RestoreThread(state); }
    };
    try {
        int status;
        {
            Unlocked unlocked;
            status = call();
        }
        return PyLong_FromLong(status);
    } catch (const std::bad_alloc &) {
        return PyErr_NoMemory();
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "exception of an unknown kind");
    }
    return nullptr;
}

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// (X, packed, gamma, Y, N, M, workspace, bias, xq_out, sx_out, acc_out, path) -> status, or None
PyObject *linear(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 12 || !g_linear) Py_RETURN_NONE;
    try {
        const at::Tensor *Y = plain(a[3]), *ws = plain(a[6]), *rows = plain(a[0] != Py_None ? a[0] : a[8]);
        if (!Y || !ws || !rows || !Y->is_cuda() || Y->dim() < 2 || rows->dim() != 2 || Y->scalar_type() != at::kFloat) Py_RETURN_NONE;
        if (a[0] != Py_None && rows->scalar_type() != at::kBFloat16) Py_RETURN_NONE;
        void *x, *packed, *gamma, *bias, *xq, *sx, *acc;
        int N, M, path;
        if (!address(a[0], x) || !address(a[1], packed) || !address(a[2], gamma) || !address(a[7], bias) || !address(a[8], xq) || !address(a[9], sx) ||
            !address(a[10], acc) || !small_int(a[4], N) || !small_int(a[5], M) || !small_int(a[11], path))
            Py_RETURN_NONE;
        const int64_t tokens = rows->size(0), d_in = rows->size(1), d_out = Y->size(1);
        void *y = Y->data_ptr(), *w = ws->data_ptr(), *stream = current_stream();
        const size_t bytes = ws->nbytes();
        return released([&] {
            return g_linear(x, tokens, d_in, d_out, N, M, packed, static_cast<const float *>(gamma), static_cast<const float *>(bias), static_cast<float *>(y),
                            static_cast<int8_t *>(xq), static_cast<float *>(sx), static_cast<int32_t *>(acc), path, w, bytes, stream);
        });
    } catch (...) {
        Py_RETURN_NONE;   // a tensor without storage, no device: the Python code raises its own error
    }
}

// A ctypes array of at least `count` pointers or 64-bit integers, held while its address is in use; anything else is not held.
struct Array {
    Py_buffer view{};
    bool held;
    enum Kind { POINTERS, INTEGERS };
    Array(PyObject *o, int count, Kind kind)
    {
        held = PyObject_GetBuffer(o, &view, PyBUF_ND | PyBUF_FORMAT) == 0;
        if (!held) {
            PyErr_Clear();
            return;
        }
        // the formats of ctypes, which names the byte order; a ctypes pointer has no dimension
        const auto is = [&](const char *format) { return !strcmp(view.format, format); };
        if (view.ndim != 1 || view.itemsize != 8 || view.shape[0] < count || !(kind == POINTERS ? is("<P") : is("<q") || is("<l"))) release();
    }
    ~Array() { release(); }
    Array(const Array &) = delete;
    void release()
    {
        if (held) PyBuffer_Release(&view);
        held = false;
    }
    template <class T> T as() const { return reinterpret_cast<T>(view.buf); }
};

// (count, X, tokens, d_in, d_out, N, M, packed, gamma, Y, path, workspace): the arrays as they are at this call -> status, or None
PyObject *grouped(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 12 || !g_grouped) Py_RETURN_NONE;
    try {
        const at::Tensor *ws = plain(a[11]);
        int count, N, M, path;
        if (!ws || !ws->is_cuda() || !small_int(a[0], count) || count < 0 || !small_int(a[5], N) || !small_int(a[6], M) || !small_int(a[10], path))
            Py_RETURN_NONE;
        const Array X(a[1], count, Array::POINTERS), tokens(a[2], count, Array::INTEGERS), d_in(a[3], count, Array::INTEGERS),
            d_out(a[4], count, Array::INTEGERS), packed(a[7], count, Array::POINTERS), gamma(a[8], count, Array::POINTERS), Y(a[9], count, Array::POINTERS);
        if (!X.held || !tokens.held || !d_in.held || !d_out.held || !packed.held || !gamma.held || !Y.held) Py_RETURN_NONE;
        void *w = ws->data_ptr(), *stream = current_stream();
        const size_t bytes = ws->nbytes();
        return released([&] {
            return g_grouped(count, X.as<const void *const *>(), tokens.as<const int64_t *>(), d_in.as<const int64_t *>(), d_out.as<const int64_t *>(), N, M,
                             packed.as<const void *const *>(), gamma.as<const float *const *>(), Y.as<float *const *>(), path, w, bytes, stream);
        });
    } catch (...) {
        Py_RETURN_NONE;
    }
}

// (object, count): whether the grouped call takes the object as an array
template <Array::Kind KIND> PyObject *takes_array(PyObject *, PyObject *args)
{
    PyObject *o;
    int count;
    if (!PyArg_ParseTuple(args, "Oi", &o, &count)) return nullptr;
    return PyBool_FromLong(Array(o, count, KIND).held);
}

PyObject *stream(PyObject *, PyObject *) { return PyLong_FromVoidPtr(current_stream()); }

// (address of a C function without arguments): called as the library's functions are
PyObject *call(PyObject *, PyObject *args)
{
    unsigned long long f;
    if (!PyArg_ParseTuple(args, "K", &f)) return nullptr;
    return released(reinterpret_cast<int (*)()>(f));
}

// addresses of the C ABI's functions in the library that the binding has loaded
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long l, g;
    if (!PyArg_ParseTuple(args, "KK", &l, &g)) return nullptr;
    g_linear = reinterpret_cast<linear_fn>(l);
    g_grouped = reinterpret_cast<grouped_fn>(g);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(linear)), METH_FASTCALL, nullptr},
    {"grouped", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(grouped)), METH_FASTCALL, nullptr},
    {"array_of_pointers", takes_array<Array::POINTERS>, METH_VARARGS, nullptr},
    {"array_of_integers", takes_array<Array::INTEGERS>, METH_VARARGS, nullptr},
    {"call", call, METH_VARARGS, nullptr},
    {"stream", stream, METH_NOARGS, nullptr},
    {"bind", bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall()
{
    PyObject *m = PyModule_Create(&module);
    // tensors are read by the layout of this version's headers, so the binding compares it with the torch that runs
    if (m && PyModule_AddStringConstant(m, "torch_version", SBN_TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
