// The calls of the library from Python: arguments read off Python objects, the C function called, its status returned.
//
// A call is a few microseconds of launches, and through ctypes as much again: the checks and addresses attribute by attribute in Python, a
// conversion per argument; for a segmented call half a microsecond per tensor on top (128 tensors of 1024 to 8192 values, compress and
// decompress: 140 us, of which 23 were the kernels').  Here it is some ten nanoseconds per argument and tensor.  us of the host per call, arrays read here and the rest in
// Python / all here: 128 small tensors compressed 9.7 / 5.9, decompressed 8.0 / 5.6, one tensor compressed 13.5 / 10.1, one message decompressed 5.3 / 4.2.  Compress and
// decompress of the 128, 15 to 18 / 11.8; of twelve bf16 tensors and a message each 75 / 63.
//
// Each function returns None for anything but the plain case (a tensor subclass, an exotic number, a buffer that is too small, a tensor that
// the library would refuse); the caller then goes through it in Python, which accepts what can be
// accepted and raises the error that fits.
#include <torch/csrc/autograd/python_variable.h>

#include <Python.h>

#include <stdint.h>

#include <vector>

#include "adatopk.h"

namespace {

struct Fast {  // borrowed items of a list or tuple
    PyObject *seq;
    Py_ssize_t n;
    bool ok;
    explicit Fast(PyObject *s) : seq(s), n(0), ok(PyList_CheckExact(s) || PyTuple_CheckExact(s)) {
        if (ok) n = PySequence_Fast_GET_SIZE(s);
    }
    PyObject *at(Py_ssize_t i) const { return PySequence_Fast_GET_ITEM(seq, i); }
};

// tensors(seq) -> (addresses, lengths, first tensor's dtype) for contiguous device tensors of one dtype: bytes objects
// that hold one pointer / one int64 per tensor.
PyObject *tensors(PyObject *, PyObject *arg) {
    const Fast f(arg);
    if (!f.ok || f.n == 0) Py_RETURN_NONE;
    PyObject *addr = PyBytes_FromStringAndSize(nullptr, f.n * static_cast<Py_ssize_t>(sizeof(void *)));
    PyObject *len = PyBytes_FromStringAndSize(nullptr, f.n * static_cast<Py_ssize_t>(sizeof(int64_t)));
    PyObject *result = nullptr;
    bool plain = addr != nullptr && len != nullptr;
    if (!plain) PyErr_Clear();
    try {
        void **a = plain ? reinterpret_cast<void **>(PyBytes_AS_STRING(addr)) : nullptr;
        int64_t *l = plain ? reinterpret_cast<int64_t *>(PyBytes_AS_STRING(len)) : nullptr;
        at::ScalarType dtype = at::ScalarType::Undefined;
        for (Py_ssize_t i = 0; plain && i < f.n; ++i) {
            if (!THPVariable_CheckExact(f.at(i))) {
                plain = false;
                break;
            }
            const at::Tensor &t = THPVariable_Unpack(f.at(i));
            if (i == 0) dtype = t.scalar_type();
            plain = t.scalar_type() == dtype && t.is_cuda() && t.is_contiguous();
            if (plain) {
                a[i] = t.mutable_data_ptr();
                l[i] = t.numel();
            }
        }
        if (plain) {
            PyObject *dt = PyObject_GetAttrString(f.at(0), "dtype");
            if (dt != nullptr) result = PyTuple_Pack(3, addr, len, dt);
            Py_XDECREF(dt);
        }
    } catch (...) {  // no address to be had (a wrapper of functorch, a tensor without storage): Python says why
        result = nullptr;
    }
    Py_XDECREF(addr);
    Py_XDECREF(len);
    if (result == nullptr) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return result;
}

// int64s(seq, count) -> (bytes of `count` int64, their sum), or None unless seq holds exactly so many plain ints.
PyObject *int64s(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    if (nargs != 2) {
        PyErr_SetString(PyExc_TypeError, "int64s(seq, count)");
        return nullptr;
    }
    const Fast f(args[0]);
    const Py_ssize_t count = PyLong_AsSsize_t(args[1]);
    if (count < 0 && PyErr_Occurred()) return nullptr;
    if (!f.ok || f.n != count) Py_RETURN_NONE;
    PyObject *out = PyBytes_FromStringAndSize(nullptr, f.n * static_cast<Py_ssize_t>(sizeof(int64_t)));
    if (out == nullptr) return nullptr;
    int64_t *p = reinterpret_cast<int64_t *>(PyBytes_AS_STRING(out));
    int64_t sum = 0;
    bool plain = true;
    for (Py_ssize_t i = 0; plain && i < f.n; ++i) {
        int overflow = 0;
        plain = PyLong_CheckExact(f.at(i));
        if (!plain) break;
        p[i] = PyLong_AsLongLongAndOverflow(f.at(i), &overflow);
        plain = overflow == 0 && !__builtin_add_overflow(sum, p[i], &sum);
    }
    PyObject *result = plain ? Py_BuildValue("(OL)", out, static_cast<long long>(sum)) : nullptr;
    Py_DECREF(out);
    if (plain) return result;
    Py_RETURN_NONE;
}

// ---- the calls
PyObject *g_current_device = nullptr, *g_raw_stream = nullptr;  // torch's functions, set once by streams()

// streams(current_device, raw_stream): how the stream of a call is found.
PyObject *streams(PyObject *, PyObject *const *args, Py_ssize_t nargs) {
    if (nargs != 2) {
        PyErr_SetString(PyExc_TypeError, "streams(current_device, raw_stream)");
        return nullptr;
    }
    Py_XSETREF(g_current_device, Py_NewRef(args[0]));
    Py_XSETREF(g_raw_stream, Py_NewRef(args[1]));
    Py_RETURN_NONE;
}

struct Call {
    bool plain = true;    // so far
    bool raised = false;  // Python code that was called has raised an exception

    // Whether an object is true.
    int truth(PyObject *o) {
        const int is = plain ? PyObject_IsTrue(o) : 0;
        raised = raised || is < 0;
        plain = plain && is >= 0;
        return is;
    }
    // A plain tensor in contiguous device memory, or nullptr.
    const at::Tensor *tensor(PyObject *o) {
        if (!plain || !THPVariable_CheckExact(o)) {
            plain = false;
            return nullptr;
        }
        const at::Tensor &t = THPVariable_Unpack(o);
        plain = t.is_cuda() && t.is_contiguous();
        return plain ? &t : nullptr;
    }
    void *address(const at::Tensor *t) { return plain && t != nullptr ? t->mutable_data_ptr() : nullptr; }
    // ... with at least `count` entries of a type
    void *buffer(PyObject *o, at::ScalarType type, int64_t count) {
        const at::Tensor *t = tensor(o);
        if (t != nullptr) plain = t->scalar_type() == type && t->numel() >= count;
        return address(t);
    }
    void *error_norms(PyObject *o, int64_t count) { return o == Py_None ? nullptr : buffer(o, at::ScalarType::Float, count); }
    int64_t number(PyObject *o) {
        int overflow = 0;
        plain = plain && PyLong_CheckExact(o);
        const int64_t v = plain ? PyLong_AsLongLongAndOverflow(o, &overflow) : 0;
        plain = plain && overflow == 0;
        return v;
    }
    adatopk_dtype dtype(at::ScalarType t) {
        plain = plain && (t == at::ScalarType::Float || t == at::ScalarType::BFloat16 || t == at::ScalarType::Half);
        return t == at::ScalarType::Float ? ADATOPK_F32 : (t == at::ScalarType::BFloat16 ? ADATOPK_BF16 : ADATOPK_F16);
    }
    // `count` numbers of a list or tuple, or as many as there are (count < 0)
    bool numbers(PyObject *o, Py_ssize_t count, std::vector<int64_t> &out) {
        const Fast f(o);
        plain = plain && f.ok && (count < 0 || f.n == count);
        if (!plain) return false;
        out.resize(static_cast<size_t>(f.n));
        for (Py_ssize_t i = 0; plain && i < f.n; ++i) out[static_cast<size_t>(i)] = number(f.at(i));
        return plain;
    }
    // contiguous device tensors of one type
    bool tensors(PyObject *o, std::vector<void *> &at, std::vector<int64_t> &n, at::ScalarType &type) {
        const Fast f(o);
        plain = plain && f.ok && f.n != 0;
        if (!plain) return false;
        at.resize(static_cast<size_t>(f.n));
        n.resize(static_cast<size_t>(f.n));
        for (Py_ssize_t i = 0; plain && i < f.n; ++i) {
            const at::Tensor *t = tensor(f.at(i));
            if (t == nullptr) break;
            if (i == 0) type = t->scalar_type();
            plain = t->scalar_type() == type;
            at[static_cast<size_t>(i)] = address(t);
            n[static_cast<size_t>(i)] = t->numel();
        }
        return plain;
    }
    void *stream() {
        if (!plain) return nullptr;
        if (g_raw_stream == nullptr) {
            plain = false;
            return nullptr;
        }
        PyObject *device = PyObject_CallNoArgs(g_current_device);
        PyObject *raw = device != nullptr ? PyObject_CallOneArg(g_raw_stream, device) : nullptr;
        void *handle = raw != nullptr ? PyLong_AsVoidPtr(raw) : nullptr;
        raised = raw == nullptr;
        plain = raw != nullptr && !PyErr_Occurred();
        Py_XDECREF(device);
        Py_XDECREF(raw);
        return handle;
    }
};

// The body of a call: `f` reads the arguments and returns the status; what it throws (a wrapper of functorch, a tensor without storage)
// and what is not plain is left to Python.  An exception out of Python code, that of a signal among them (an interrupt while the stream is asked for),
// is the call's: nothing has been enqueued.
template <typename F> PyObject *call(Py_ssize_t nargs, Py_ssize_t expected, F &&f) {
    if (nargs != expected) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        Call c;
        const long status = f(c);
        if (c.raised) return nullptr;
        if (c.plain && !PyErr_Occurred()) return PyLong_FromLong(status);
    } catch (...) {
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}
// Calls the library at address `fn` without holding the interpreter, as ctypes does.
template <typename Fn, typename... Args> long without_gil(Call &c, PyObject *fn, Args... args) {
    const Fn f = c.plain ? reinterpret_cast<Fn>(PyLong_AsVoidPtr(fn)) : nullptr;
    if (f == nullptr) {
        c.plain = false;
        return 0;
    }
    long status;
    Py_BEGIN_ALLOW_THREADS
    status = static_cast<long>(f(args...));
    Py_END_ALLOW_THREADS
    return status;
}

// (fn, dense, k, idx, val, err or None, workspace)
PyObject *compress(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    return call(nargs, 7, [&](Call &c) -> long {
        const at::Tensor *x = c.tensor(a[1]);
        if (x == nullptr) return 0;
        const int64_t k = c.number(a[2]);
        const adatopk_dtype dt = c.dtype(x->scalar_type());
        void *idx = c.buffer(a[3], at::ScalarType::Int, k), *val = c.buffer(a[4], x->scalar_type(), k), *err = c.error_norms(a[5], 1);
        const at::Tensor *ws = c.tensor(a[6]);
        void *stream = c.stream();
        if (!c.plain) return 0;
        return without_gil<decltype(&adatopk_compress)>(c, a[0], c.address(x), x->numel(), dt, k, static_cast<int32_t *>(idx), val,
                                                        static_cast<float *>(err), c.address(ws), static_cast<size_t>(ws->numel()), stream);
    });
}

// (fn, idx, val, k, dense): the three ways to decompress pairs
PyObject *decompress(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    return call(nargs, 5, [&](Call &c) -> long {
        const at::Tensor *y = c.tensor(a[4]);
        if (y == nullptr) return 0;
        const int64_t k = c.number(a[3]);
        const adatopk_dtype dt = c.dtype(y->scalar_type());
        void *idx = c.buffer(a[1], at::ScalarType::Int, k), *val = c.buffer(a[2], y->scalar_type(), k), *stream = c.stream();
        if (!c.plain) return 0;
        return without_gil<decltype(&adatopk_decompress)>(c, a[0], static_cast<const int32_t *>(idx), static_cast<const void *>(val), k, dt, c.address(y),
                                                          y->numel(), stream);
    });
}

// (fn, wire, wire_bytes, index_bytes, dense, accumulate)
PyObject *decompress_wire(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    return call(nargs, 6, [&](Call &c) -> long {
        const at::Tensor *wire = c.tensor(a[1]), *y = c.tensor(a[4]);
        if (wire == nullptr || y == nullptr) return 0;
        const int64_t bytes = c.number(a[2]), ib = c.number(a[3]);
        const adatopk_dtype dt = c.dtype(y->scalar_type());
        c.plain = c.plain && bytes >= 0 && (ib == 4 || ib == 8);
        const int accumulate = c.truth(a[5]);
        void *stream = c.stream();
        if (!c.plain) return 0;
        return without_gil<decltype(&adatopk_decompress_wire)>(c, a[0], static_cast<const void *>(c.address(wire)), static_cast<size_t>(bytes), dt,
                                                               static_cast<int32_t>(ib), y->numel(), accumulate, c.address(y), stream);
    });
}

// (fn, dense, k, index_bytes, ratio, wire_out, workspace)
PyObject *compress_wire(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    return call(nargs, 7, [&](Call &c) -> long {
        const at::Tensor *x = c.tensor(a[1]), *wire = c.tensor(a[5]), *ws = c.tensor(a[6]);
        if (x == nullptr || wire == nullptr || ws == nullptr) return 0;
        const int64_t k = c.number(a[2]), ib = c.number(a[3]);
        const adatopk_dtype dt = c.dtype(x->scalar_type());
        c.plain = c.plain && PyFloat_CheckExact(a[4]) && (ib == 4 || ib == 8);
        void *stream = c.stream();
        if (!c.plain) return 0;
        return without_gil<decltype(&adatopk_compress_wire)>(c, a[0], static_cast<const void *>(c.address(x)), x->numel(), dt, k, static_cast<int32_t>(ib),
                                                             PyFloat_AS_DOUBLE(a[4]), c.address(wire), static_cast<size_t>(wire->nbytes()),
                                                             c.address(ws), static_cast<size_t>(ws->numel()), stream);
    });
}

// (fn, tensors, ks, idx, val, offsets, err or None, workspace)
PyObject *compress_segmented(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    return call(nargs, 8, [&](Call &c) -> long {
        std::vector<void *> xs;
        std::vector<int64_t> ns, ks, off;
        at::ScalarType type = at::ScalarType::Undefined;
        if (!c.tensors(a[1], xs, ns, type)) return 0;
        const Py_ssize_t S = static_cast<Py_ssize_t>(xs.size());
        const adatopk_dtype dt = c.dtype(type);
        if (!c.numbers(a[2], S, ks) || !c.numbers(a[5], S + 1, off)) return 0;
        int64_t total = 0;
        for (const int64_t k : ks) c.plain = c.plain && !__builtin_add_overflow(total, k, &total);
        void *idx = c.buffer(a[3], at::ScalarType::Int, total), *val = c.buffer(a[4], type, total), *err = c.error_norms(a[6], S);
        const at::Tensor *ws = c.tensor(a[7]);
        void *stream = c.stream();
        if (!c.plain) return 0;
        return without_gil<decltype(&adatopk_compress_segmented)>(c, a[0], static_cast<const void *const *>(xs.data()), static_cast<const int64_t *>(ns.data()),
                                                                  static_cast<const int64_t *>(ks.data()), static_cast<int32_t>(S), dt,
                                                                  static_cast<int32_t *>(idx), val, static_cast<const int64_t *>(off.data()),
                                                                  static_cast<float *>(err), c.address(ws), static_cast<size_t>(ws->numel()), stream);
    });
}

// (fn, idx, val, offsets, tensors)
PyObject *decompress_segmented(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    return call(nargs, 5, [&](Call &c) -> long {
        std::vector<void *> ys;
        std::vector<int64_t> ns, off;
        at::ScalarType type = at::ScalarType::Undefined;
        if (!c.tensors(a[4], ys, ns, type)) return 0;
        const Py_ssize_t S = static_cast<Py_ssize_t>(ys.size());
        const adatopk_dtype dt = c.dtype(type);
        if (!c.numbers(a[3], S + 1, off)) return 0;
        void *idx = c.buffer(a[1], at::ScalarType::Int, off.back()), *val = c.buffer(a[2], type, off.back()), *stream = c.stream();
        if (!c.plain) return 0;
        return without_gil<decltype(&adatopk_decompress_segmented)>(c, a[0], static_cast<const int32_t *>(idx), static_cast<const void *>(val),
                                                                    static_cast<const int64_t *>(off.data()), static_cast<int32_t>(S), dt,
                                                                    static_cast<void *const *>(ys.data()), static_cast<const int64_t *>(ns.data()), stream);
    });
}

// (fn, tensors, ks, index_bytes, ratios or None, wire_out, offsets, workspace)
PyObject *compress_wire_segmented(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    return call(nargs, 8, [&](Call &c) -> long {
        std::vector<void *> xs;
        std::vector<int64_t> ns, ks, off;
        std::vector<double> ratios;
        at::ScalarType type = at::ScalarType::Undefined;
        if (!c.tensors(a[1], xs, ns, type)) return 0;
        const Py_ssize_t S = static_cast<Py_ssize_t>(xs.size());
        const adatopk_dtype dt = c.dtype(type);
        const int64_t ib = c.number(a[3]);
        if (!c.numbers(a[2], S, ks) || !c.numbers(a[6], S, off) || (ib != 4 && ib != 8)) return c.plain = false;
        if (a[4] != Py_None) {
            const Fast f(a[4]);
            c.plain = f.ok && f.n == S;
            for (Py_ssize_t i = 0; c.plain && i < S; ++i) {
                c.plain = PyFloat_CheckExact(f.at(i));
                if (c.plain) ratios.push_back(PyFloat_AS_DOUBLE(f.at(i)));
            }
        }
        const at::Tensor *wire = c.tensor(a[5]), *ws = c.tensor(a[7]);
        void *stream = c.stream();
        if (!c.plain) return 0;
        return without_gil<decltype(&adatopk_compress_wire_segmented)>(
            c, a[0], static_cast<const void *const *>(xs.data()), static_cast<const int64_t *>(ns.data()), static_cast<const int64_t *>(ks.data()),
            static_cast<int32_t>(S), dt, static_cast<int32_t>(ib), a[4] != Py_None ? static_cast<const double *>(ratios.data()) : nullptr, c.address(wire),
            static_cast<const int64_t *>(off.data()), static_cast<size_t>(wire->nbytes()), c.address(ws), static_cast<size_t>(ws->numel()), stream);
    });
}

template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)> constexpr PyMethodDef fast(const char *name, const char *doc) {
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(F)), METH_FASTCALL, doc};
}
PyMethodDef methods[] = {
    {"tensors", tensors, METH_O, "(addresses, lengths, dtype) of contiguous device tensors of one dtype, or None"},
    fast<int64s>("int64s", "(int64 array, sum) of a sequence of `count` ints, or None"),
    fast<streams>("streams", "how the stream of a call is found: torch's current_device and raw stream functions"),
    fast<compress>("compress", "status of the call at an address, or None"),
    fast<decompress>("decompress", "status of the call at an address, or None"),
    fast<compress_wire>("compress_wire", "status of the call at an address, or None"),
    fast<decompress_wire>("decompress_wire", "status of the call at an address, or None"),
    fast<compress_segmented>("compress_segmented", "status of the call at an address, or None"),
    fast<decompress_segmented>("decompress_segmented", "status of the call at an address, or None"),
    fast<compress_wire_segmented>("compress_wire_segmented", "status of the call at an address, or None"),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "The calls of the library, their arguments read in C.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
