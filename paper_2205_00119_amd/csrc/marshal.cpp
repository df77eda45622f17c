// Argument marshalling of the Python binding: tensor sequences -> pointer tables, segment tuples ->
// mics_segment arrays.  Per-element Python code for this (three calls into the interpreter for each
// of 64 gradient buffers) took twice as long as the kernel of an 8 MB reduction.
//
// No state.  Everything is called with the GIL held; nothing outlives the call.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>

namespace {

// Device address of a tensor, a raw integer address, or None (NULL).  False: a Python error is set.
bool address_of(PyObject* x, uint64_t* out)
{
    if (x == Py_None) {
        *out = 0;
        return true;
    }
    if (PyLong_Check(x)) {
        *out = PyLong_AsUnsignedLongLongMask(x);
        return !(*out == (uint64_t)-1 && PyErr_Occurred());
    }
    if (THPVariable_CheckExact(x)) {
        const at::Tensor& t = THPVariable_Unpack(x);
        if (!t.is_contiguous()) {
            PyErr_SetString(PyExc_ValueError, "tensor must be contiguous");
            return false;
        }
        *out = (uint64_t)(uintptr_t)t.data_ptr();
        return true;
    }
    // subclasses and tensor-like objects answer for themselves
    PyObject* flag = PyObject_CallMethod(x, "is_contiguous", nullptr);
    if (!flag) return false;
    const int contiguous = PyObject_IsTrue(flag);
    Py_DECREF(flag);
    if (contiguous < 0) return false;
    if (!contiguous) {
        PyErr_SetString(PyExc_ValueError, "tensor must be contiguous");
        return false;
    }
    PyObject* ptr = PyObject_CallMethod(x, "data_ptr", nullptr);
    if (!ptr) return false;
    *out = PyLong_AsUnsignedLongLongMask(ptr);
    Py_DECREF(ptr);
    return !(*out == (uint64_t)-1 && PyErr_Occurred());
}

// C++ exceptions become the Python ones that the tensor's own methods raise (type, and text without
// the C++ stack).
template <typename F>
PyObject* guarded(F&& f)
{
    try {
        return f();
    } catch (const std::exception&) {
        torch::translate_exception_to_python(std::current_exception());
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
    }
    return nullptr;
}

// address(x) -> int, or None for None
PyObject* address(PyObject*, PyObject* x)
{
    return guarded([&]() -> PyObject* {
        uint64_t a = 0;
        if (x == Py_None) Py_RETURN_NONE;
        if (!address_of(x, &a)) return nullptr;
        return PyLong_FromUnsignedLongLong(a);
    });
}

// The writable buffer `args[0]` and the sequence `args[1]`, whose length has to fill it.
struct Target {
    Py_buffer buf{};
    PyObject* seq = nullptr;
    ~Target()
    {
        Py_XDECREF(seq);
        if (buf.obj) PyBuffer_Release(&buf);
    }
    bool open(PyObject* const* args, Py_ssize_t n, size_t item_bytes)
    {
        if (n != 2) {
            PyErr_SetString(PyExc_TypeError, "expected (array, sequence)");
            return false;
        }
        if (PyObject_GetBuffer(args[0], &buf, PyBUF_WRITABLE) < 0) return false;
        seq = PySequence_Fast(args[1], "expected a sequence");
        if (!seq) return false;
        if ((size_t)buf.len != (size_t)PySequence_Fast_GET_SIZE(seq) * item_bytes) {
            PyErr_SetString(PyExc_ValueError, "array and sequence differ in length");
            return false;
        }
        return true;
    }
};

// addresses(array of c_void_p, sequence)
PyObject* addresses(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    return guarded([&]() -> PyObject* {
        Target t;
        if (!t.open(args, nargs, sizeof(uint64_t))) return nullptr;
        uint64_t* out = (uint64_t*)t.buf.buf;
        const Py_ssize_t n = t.buf.len / (Py_ssize_t)sizeof(uint64_t);
        for (Py_ssize_t i = 0; i < n; ++i) {
            // a tensor-like object may run Python code: look the sequence up again each time
            if (i >= PySequence_Fast_GET_SIZE(t.seq)) {
                PyErr_SetString(PyExc_RuntimeError, "sequence changed its length");
                return nullptr;
            }
            PyObject* x = PySequence_Fast_GET_ITEM(t.seq, i);
            Py_INCREF(x);
            const bool ok = address_of(x, out + i);
            Py_DECREF(x);
            if (!ok) return nullptr;
        }
        Py_RETURN_NONE;
    });
}

// segments(array of mics_segment, sequence of up to 4 numbers each): what is left out is 0
PyObject* segments(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    constexpr Py_ssize_t kFields = 4;
    return guarded([&]() -> PyObject* {
        Target t;
        if (!t.open(args, nargs, kFields * sizeof(uint64_t))) return nullptr;
        uint64_t* out = (uint64_t*)t.buf.buf;
        const Py_ssize_t n = t.buf.len / (Py_ssize_t)(kFields * sizeof(uint64_t));
        for (Py_ssize_t i = 0; i < n; ++i) {
            if (i >= PySequence_Fast_GET_SIZE(t.seq)) {
                PyErr_SetString(PyExc_RuntimeError, "sequence changed its length");
                return nullptr;
            }
            // a tuple of its own: what its numbers' __int__ does cannot change it.  The item's __iter__ may
            // drop the list's reference to it.
            PyObject* item = PySequence_Fast_GET_ITEM(t.seq, i);
            Py_INCREF(item);
            PyObject* sg = PySequence_Tuple(item);
            Py_DECREF(item);
            if (!sg) return nullptr;
            const Py_ssize_t m = PyTuple_GET_SIZE(sg);
            bool ok = m <= kFields;
            if (!ok) PyErr_SetString(PyExc_TypeError, "too many initializers");
            for (Py_ssize_t f = 0; ok && f < m; ++f) {
                PyObject* v = PyNumber_Long(PyTuple_GET_ITEM(sg, f));
                ok = v != nullptr;
                if (!ok) break;
                out[i * kFields + f] = PyLong_AsUnsignedLongLongMask(v);
                Py_DECREF(v);
            }
            Py_DECREF(sg);
            if (!ok) return nullptr;
        }
        Py_RETURN_NONE;
    });
}

PyMethodDef methods[] = {
    {"address", address, METH_O, "Device address of a contiguous tensor, an integer, or None."},
    {"addresses", (PyCFunction)(void (*)())addresses, METH_FASTCALL, "Fills an array of pointers from a sequence."},
    {"segments", (PyCFunction)(void (*)())segments, METH_FASTCALL, "Fills an array of mics_segment from a sequence."},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
