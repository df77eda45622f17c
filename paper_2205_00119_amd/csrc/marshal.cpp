// Argument marshalling of the Python binding: tensor sequences -> pointer tables, segment tuples ->
// mics_segment arrays.  Per-element Python code for this (three calls into the interpreter for each
// of 64 gradient buffers) took twice as long as the kernel of an 8 MB reduction.
//
// Whole calls as well: the functions from `gather` on take the arguments of a Python entry point that are of the plain
// kinds (tensors, numbers, torch streams, lists and tuples of them, ctypes arrays of segments), make the tables on the
// stack and call the library without ctypes: us per call from Python, ctypes / so: gather 1 MB 5.4 / 4.6, reduction of 64
// buffers, 8 MB 5.7 / 4.9, of 76 segments 8.0 / 6.1, Adam 5.9 / 5.1; the launch itself is 2.5 to 4 of them.
// Whatever they do not know they leave alone and return None; the entry point then goes through ctypes.
//
// No state but what bind() and bind_segment() set at import.  Everything is called with the GIL held, which is given up
// while the library works; nothing outlives the call.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <exception>

#include "../../include/mics.h"

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

// The library's entry points, and torch's two that name the current stream.
struct {
    decltype(&mics_hier_gather_reorder) hier_gather_reorder;
    decltype(&mics_hier_gather_reorder_coalesced) hier_gather_reorder_coalesced;
    decltype(&mics_reduce_scatter_accum) reduce_scatter_accum;
    decltype(&mics_reduce_scatter_accum_typed) reduce_scatter_accum_typed;
    decltype(&mics_reduce_scatter_accum_coalesced) reduce_scatter_accum_coalesced;
    decltype(&mics_reduce_scatter_accum_coalesced_typed) reduce_scatter_accum_coalesced_typed;
    decltype(&mics_replica_average) replica_average;
    decltype(&mics_adam_shard) adam_shard;
    decltype(&mics_adam_shard_typed) adam_shard_typed;
    decltype(&mics_replica_average_adam_shard) replica_average_adam_shard;
    decltype(&mics_replica_average_adam_shard_typed) replica_average_adam_shard_typed;
} lib;
constexpr Py_ssize_t kEntries = sizeof lib / sizeof(void*);
PyObject *device_of_thread, *raw_stream, *segment_type;
PyObject *stream_attr, *item_attr;                 // "cuda_stream", "_type_"

// bind(addresses in the order above, current device, raw stream of a device)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != 3 || !PyTuple_CheckExact(args[0]) || PyTuple_GET_SIZE(args[0]) != kEntries) {
        PyErr_SetString(PyExc_TypeError, "expected (tuple of addresses, callable, callable)");
        return nullptr;
    }
    void* at[kEntries];
    for (Py_ssize_t i = 0; i < kEntries; ++i) {
        at[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(args[0], i));
        if (!at[i] && PyErr_Occurred()) return nullptr;
    }
    if (!stream_attr) stream_attr = PyUnicode_InternFromString("cuda_stream");
    if (!item_attr) item_attr = PyUnicode_InternFromString("_type_");
    if (!stream_attr || !item_attr) return nullptr;
    std::memcpy((void*)&lib, at, sizeof at);
    Py_INCREF(args[1]);
    Py_INCREF(args[2]);
    Py_XSETREF(device_of_thread, args[1]);
    Py_XSETREF(raw_stream, args[2]);
    Py_RETURN_NONE;
}

// bind_segment(mics_segment, the ctypes structure)
PyObject* bind_segment(PyObject*, PyObject* type)
{
    Py_INCREF(type);
    Py_XSETREF(segment_type, type);
    Py_RETURN_NONE;
}

// The arguments of one call.  `plain` turns false at the first that is not of a plain kind; no Python code of an
// argument runs before the stream's, so the lists cannot change meanwhile.
class Call {
  public:
    // kinds: a letter for each argument (of_kind).  They are looked at before any table is made, because a call that goes
    // through ctypes after all has this in front of it (us without it / tables first / so: 64 buffers, a count of numpy's
    // 2.3 / 3.0 / 2.45).  What programs pass in earnest is taken as it is: through ctypes, with that in front / past it, a
    // torch stream 3.0 / 0.8, a weight decay of 0 2.7 / 0.85, segments in a ctypes array 3.2 / 0.85.
    Call(PyObject* const* args, Py_ssize_t n, const char* kinds) : a(args), plain(n == (Py_ssize_t)std::strlen(kinds))
    {
        for (Py_ssize_t i = 0; plain && i < n; ++i) plain = of_kind(args[i], kinds[i]);
    }

    void* ptr(int i) { return plain ? address(a[i]) : nullptr; }
    size_t size(int i) { return plain ? PyLong_AsUnsignedLongLongMask(a[i]) : 0; }
    int num(int i) { return (int)size(i); }
    int flag(int i) { return plain && PyObject_IsTrue(a[i]); }
    float real(int i)
    {
        if (!plain) return 0;
        if (PyFloat_Check(a[i])) return (float)PyFloat_AS_DOUBLE(a[i]);
        const double v = PyLong_AsDouble(a[i]);
        if (v == -1 && PyErr_Occurred()) {                 // too large
            PyErr_Clear();
            plain = false;
        }
        return (float)v;
    }
    template <typename T>
    const T* const* table(int i)
    {
        if (!plain) return nullptr;
        entries = (int)PySequence_Fast_GET_SIZE(a[i]);
        for (int q = 0; plain && q < entries; ++q) pointers[q] = address(PySequence_Fast_GET_ITEM(a[i], q));
        return (const T* const*)pointers;
    }
    const mics_segment* segments(int i)
    {
        if (!plain) return nullptr;
        if (!sequence(a[i])) {                             // a ctypes array of them
            Py_buffer buf;
            plain = PyObject_GetBuffer(a[i], &buf, PyBUF_SIMPLE) == 0;
            if (!plain) {
                PyErr_Clear();
                return nullptr;
            }
            const void* at = buf.buf;
            n_segments = (int)(buf.len / (Py_ssize_t)sizeof(mics_segment));
            PyBuffer_Release(&buf);                        // the array stays where it is
            return (const mics_segment*)at;
        }
        n_segments = (int)PySequence_Fast_GET_SIZE(a[i]);
        for (int t = 0; t < n_segments; ++t) {
            PyObject* sg = PySequence_Fast_GET_ITEM(a[i], t);
            plain = segment(sg);
            if (!plain) return nullptr;
            size_t f[4] = {0, 0, 0, 0};
            for (Py_ssize_t k = 0; k < PySequence_Fast_GET_SIZE(sg); ++k)
                f[k] = PyLong_AsUnsignedLongLongMask(PySequence_Fast_GET_ITEM(sg, k));
            segs[t] = mics_segment{f[0], f[1], f[2], f[3]};
        }
        return segs;
    }
    // An integer, a torch stream, or None: the current stream of the current device.  After everything else: this runs
    // Python code, whose exceptions (an interrupt may arrive in it) are the call's.
    void* stream(int i)
    {
        if (!plain) return nullptr;
        PyObject* raw = nullptr;
        if (PyLong_Check(a[i])) {
            raw = a[i];
            Py_INCREF(raw);
        } else if (a[i] != Py_None) {
            raw = PyObject_GetAttr(a[i], stream_attr);
            raised = !raw;
        } else if (device_of_thread) {
            PyObject* dev = PyObject_CallNoArgs(device_of_thread);
            raw = dev ? PyObject_CallOneArg(raw_stream, dev) : nullptr;
            raised = !raw;
            Py_XDECREF(dev);
        }
        plain = raw && PyLong_CheckExact(raw);
        void* const got = plain ? (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(raw) : nullptr;
        Py_XDECREF(raw);
        return got;
    }
    template <typename F>
    PyObject* run(F&& f)
    {
        if (raised) return nullptr;
        if (!plain) Py_RETURN_NONE;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = f();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    }
    // The table's number of entries, which argument i has to state exactly (num() would cut it to 32 bits).
    int entries_as(int i)
    {
        int overflow;                                      // the value is -1 then
        plain = plain && PyLong_AsLongAndOverflow(a[i], &overflow) == entries;
        return entries;
    }
    int entries = 0, n_segments = 0;

  private:
    static constexpr int kMaxSegments = 128;
    PyObject* const* a;
    bool plain, raised = false;
    void* pointers[MICS_MAX_GROUP];
    mics_segment segs[kMaxSegments];

    static bool sequence(PyObject* x) { return PyList_CheckExact(x) || PyTuple_CheckExact(x); }
    static bool segment(PyObject* x)
    {
        if (!sequence(x) || PySequence_Fast_GET_SIZE(x) > 4) return false;
        for (Py_ssize_t k = 0; k < PySequence_Fast_GET_SIZE(x); ++k)
            if (!PyLong_CheckExact(PySequence_Fast_GET_ITEM(x, k))) return false;
        return true;
    }
    static bool segment_list(PyObject* x)                  // as far as its first item
    {
        if (sequence(x)) {
            const Py_ssize_t m = PySequence_Fast_GET_SIZE(x);
            return m <= kMaxSegments && (!m || segment(PySequence_Fast_GET_ITEM(x, 0)));
        }
        PyObject* const names = Py_TYPE(x)->tp_dict;       // of a ctypes array's type: _type_ is its items' type
        return names && segment_type && PyDict_GetItem(names, item_attr) == segment_type;
    }
    // p pointer, t table of them, g segments, i integer, b flag, f number, s stream
    static bool of_kind(PyObject* x, char kind)
    {
        switch (kind) {
            case 'p': return x == Py_None || PyLong_CheckExact(x) || THPVariable_CheckExact(x);
            case 't': return sequence(x) && PySequence_Fast_GET_SIZE(x) <= MICS_MAX_GROUP;
            case 'g': return segment_list(x);
            case 'i': return PyLong_CheckExact(x);
            case 'b': return PyBool_Check(x) || PyLong_CheckExact(x);
            case 'f': return PyFloat_Check(x) || PyLong_CheckExact(x);
            default: return true;
        }
    }
    void* address(PyObject* x)
    {
        if (x == Py_None) return nullptr;
        if (PyLong_CheckExact(x)) return (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(x);
        plain = THPVariable_CheckExact(x);
        if (!plain) return nullptr;
        try {
            const at::Tensor& t = THPVariable_Unpack(x);
            plain = t.is_contiguous();
            return plain ? t.data_ptr() : nullptr;
        } catch (...) {                                    // the tensor's own methods say what is wrong
            plain = false;
            return nullptr;
        }
    }
};

#define MICS_CALL(name) PyObject* name(PyObject*, PyObject* const* args, Py_ssize_t n)

MICS_CALL(gather)
{
    Call c(args, n, "ptiiiiis");
    void* dst = c.ptr(0);
    const auto bufs = c.table<void>(1);
    const size_t n_valid = c.size(2), shard = c.size(3);
    const int p = c.num(4), k = c.entries_as(5), eb = c.num(6);
    void* st = c.stream(7);
    return c.run([&] { return lib.hier_gather_reorder(dst, bufs, n_valid, shard, p, k, eb, st); });
}

MICS_CALL(gather_coalesced)
{
    Call c(args, n, "ptgiiis");
    void* dst = c.ptr(0);
    const auto bufs = c.table<void>(1);
    const auto segs = c.segments(2);
    const int p = c.num(3), k = c.entries_as(4), eb = c.num(5);
    void* st = c.stream(6);
    return c.run([&] { return lib.hier_gather_reorder_coalesced(dst, bufs, segs, c.n_segments, p, k, eb, st); });
}

MICS_CALL(reduce)
{
    Call c(args, n, "ptiibs");
    float* acc = (float*)c.ptr(0);
    const auto g = c.table<uint16_t>(1);
    const size_t offset = c.size(2), count = c.size(3);
    const int accumulate = c.flag(4);
    void* st = c.stream(5);
    return c.run([&] { return lib.reduce_scatter_accum(acc, g, offset, count, c.entries, accumulate, st); });
}

MICS_CALL(reduce_typed)
{
    Call c(args, n, "ptiibis");
    float* acc = (float*)c.ptr(0);
    const auto g = c.table<void>(1);
    const size_t offset = c.size(2), count = c.size(3);
    const int accumulate = c.flag(4), dtype = c.num(5);
    void* st = c.stream(6);
    return c.run([&] { return lib.reduce_scatter_accum_typed(acc, g, offset, count, c.entries, accumulate, dtype, st); });
}

MICS_CALL(reduce_coalesced)
{
    Call c(args, n, "ptgbs");
    float* acc = (float*)c.ptr(0);
    const auto g = c.table<uint16_t>(1);
    const auto segs = c.segments(2);
    const int accumulate = c.flag(3);
    void* st = c.stream(4);
    return c.run([&] { return lib.reduce_scatter_accum_coalesced(acc, g, segs, c.n_segments, c.entries, accumulate, st); });
}

MICS_CALL(reduce_coalesced_typed)
{
    Call c(args, n, "ptgbis");
    float* acc = (float*)c.ptr(0);
    const auto g = c.table<void>(1);
    const auto segs = c.segments(2);
    const int accumulate = c.flag(3), dtype = c.num(4);
    void* st = c.stream(5);
    return c.run([&] {
        return lib.reduce_scatter_accum_coalesced_typed(acc, g, segs, c.n_segments, c.entries, accumulate, dtype, st);
    });
}

MICS_CALL(average)
{
    Call c(args, n, "ptifs");
    float* out = (float*)c.ptr(0);
    const auto copies = c.table<float>(1);
    const size_t count = c.size(2);
    const float scale = c.real(3);
    void* st = c.stream(4);
    return c.run([&] { return lib.replica_average(out, copies, count, c.entries, scale, st); });
}

struct Hyper {
    float lr, beta1, beta2, eps, weight_decay;
    int step;
    Hyper(Call& c, int i)
        : lr(c.real(i)), beta1(c.real(i + 1)), beta2(c.real(i + 2)), eps(c.real(i + 3)), weight_decay(c.real(i + 4)), step(c.num(i + 5))
    {
    }
};
struct States {
    float *master, *exp_avg, *exp_avg_sq;
    void* param;
    explicit States(Call& c) : master((float*)c.ptr(0)), exp_avg((float*)c.ptr(1)), exp_avg_sq((float*)c.ptr(2)), param(c.ptr(3)) {}
};

MICS_CALL(adam)
{
    Call c(args, n, "pppppifffffis");
    const States s(c);
    const float* grad = (const float*)c.ptr(4);
    const size_t count = c.size(5);
    const Hyper h(c, 6);
    void* st = c.stream(12);
    return c.run([&] {
        return lib.adam_shard(s.master, s.exp_avg, s.exp_avg_sq, (uint16_t*)s.param, grad, count, h.lr, h.beta1, h.beta2, h.eps,
                              h.weight_decay, h.step, st);
    });
}

MICS_CALL(adam_typed)
{
    Call c(args, n, "ppppipifffffis");
    const States s(c);
    const int dtype = c.num(4);
    const float* grad = (const float*)c.ptr(5);
    const size_t count = c.size(6);
    const Hyper h(c, 7);
    void* st = c.stream(13);
    return c.run([&] {
        return lib.adam_shard_typed(s.master, s.exp_avg, s.exp_avg_sq, s.param, dtype, grad, count, h.lr, h.beta1, h.beta2, h.eps,
                                    h.weight_decay, h.step, st);
    });
}

MICS_CALL(update)
{
    Call c(args, n, "pppptiffffffis");
    const States s(c);
    const auto copies = c.table<float>(4);
    const size_t count = c.size(5);
    const float scale = c.real(6);
    const Hyper h(c, 7);
    void* st = c.stream(13);
    return c.run([&] {
        return lib.replica_average_adam_shard(s.master, s.exp_avg, s.exp_avg_sq, (uint16_t*)s.param, copies, count, c.entries, scale,
                                              h.lr, h.beta1, h.beta2, h.eps, h.weight_decay, h.step, st);
    });
}

MICS_CALL(update_typed)
{
    Call c(args, n, "ppppitiffffffis");
    const States s(c);
    const int dtype = c.num(4);
    const auto copies = c.table<float>(5);
    const size_t count = c.size(6);
    const float scale = c.real(7);
    const Hyper h(c, 8);
    void* st = c.stream(14);
    return c.run([&] {
        return lib.replica_average_adam_shard_typed(s.master, s.exp_avg, s.exp_avg_sq, s.param, dtype, copies, count, c.entries, scale,
                                                    h.lr, h.beta1, h.beta2, h.eps, h.weight_decay, h.step, st);
    });
}

#define MICS_METHOD(name) {#name, (PyCFunction)(void (*)())name, METH_FASTCALL, "A whole call; None if an argument is not plain."}

PyMethodDef methods[] = {
    {"address", address, METH_O, "Device address of a contiguous tensor, an integer, or None."},
    {"addresses", (PyCFunction)(void (*)())addresses, METH_FASTCALL, "Fills an array of pointers from a sequence."},
    {"segments", (PyCFunction)(void (*)())segments, METH_FASTCALL, "Fills an array of mics_segment from a sequence."},
    {"bind", (PyCFunction)(void (*)())bind, METH_FASTCALL, "Sets the library's entry points."},
    {"bind_segment", bind_segment, METH_O, "Sets the type whose ctypes arrays are tables of segments."},
    MICS_METHOD(gather), MICS_METHOD(gather_coalesced), MICS_METHOD(reduce), MICS_METHOD(reduce_typed),
    MICS_METHOD(reduce_coalesced), MICS_METHOD(reduce_coalesced_typed), MICS_METHOD(average), MICS_METHOD(adam),
    MICS_METHOD(adam_typed), MICS_METHOD(update), MICS_METHOD(update_typed),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
