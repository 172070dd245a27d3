// The host arrays of a segmented call, read off Python sequences in one go.
//
// A segmented call takes, per tensor, its address, its length and a few numbers.  Collected attribute by
// attribute in Python that is about half a microsecond per tensor and call, more than the kernels need for a
// batch of small messages (128 tensors of 1024 to 8192 values, compress and decompress: 140 us, of which 23 were
// the kernels').  Here it is some ten nanoseconds per tensor.
//
// Each function returns None for anything but the plain case (a tensor subclass, an exotic number, a tensor that
// the library would refuse); the caller then goes through it in Python, which accepts what can be
// accepted and raises the error that fits.
#include <torch/csrc/autograd/python_variable.h>

#include <Python.h>

#include <stdint.h>

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

PyMethodDef methods[] = {
    {"tensors", tensors, METH_O, "(addresses, lengths, dtype) of contiguous device tensors of one dtype, or None"},
    {"int64s", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(int64s)), METH_FASTCALL,
     "(int64 array, sum) of a sequence of `count` ints, or None"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "Host arrays of the segmented calls.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
