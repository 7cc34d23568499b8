// Argument marshalling of the package's entry points in native code: tensors to pointers, numbers to C numbers, the current stream, one call.
// A call through ctypes costs 2.8 us of host time beside the launch itself, which is more than the smallest kernels take; this costs 0.5 us.
//
// A function here either makes the C call and returns its status, or returns None and has done nothing: an argument is not what the usual call
// has (a tensor on the host, of another type or strides, a subclass, a number that is none).  The Python functions then look at the arguments themselves and raise what
// is to be raised.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <exception>
#include <type_traits>
#include <utility>

#include "wk.h"

namespace {

union Arg {
    void *p;
    int64_t i;
    float f;
};

template <typename P>
P as(const Arg &a) {
    if constexpr (std::is_pointer_v<P>) return reinterpret_cast<P>(a.p);
    else if constexpr (std::is_floating_point_v<P>) return a.f;
    else return static_cast<P>(a.i);
}

template <typename... P, size_t... I>
int call(void *fn, const Arg *a, wk_status (*)(P...), std::index_sequence<I...>) {
    return reinterpret_cast<wk_status (*)(P...)>(fn)(as<P>(a[I])...);
}

template <typename... P>
int invoke_as(void *fn, const Arg *a, wk_status (*type)(P...)) {
    return call(fn, a, type, std::index_sequence_for<P...>{});
}

template <auto F>
int invoke(void *fn, const Arg *a) { return invoke_as(fn, a, F); }

// What the C parameters are made of, in their order:
//   a Python argument each: b a tensor, t a tensor of the first one's type, i, f, d a tensor of int32, float32, float64 (all these or None);
//     5 a list or tuple of five floats; r a ctypes structure of the type that was bound; n a whole number; x a float;
//     w a workspace tensor or None, which is two parameters, its address and its bytes; v a whole number, or None for what m is
//   none: h, q, e the first tensor's three sizes, y its type; m the second tensor's size(1), k the same or 0 for None; o the address of n_out, which is
//     returned (negative) where the call succeeds; s the current stream, behind all others
struct Entry {
    const char *name, *signature;
    int (*invoke)(void *, const Arg *);
    void *fn;              // of the library that is loaded
    PyTypeObject *type;    // of r
};

Entry entries[] = {
    {"wk_score_chunks", "fn5nnidis", invoke<&wk_score_chunks>},
    {"wk_compress_chunk", "rbbbibbows", invoke<&wk_compress_chunk>},
    {"wk_gather_window", "riinbbnbbnis", invoke<&wk_gather_window>},
    {"wk_attention", "btttfhqvemyxiws", invoke<&wk_attention>},
    {"wk_attention_in_place", "bbbnkriinbfqxs", invoke<&wk_attention_in_place>},
    {"wk_chunk_lse", "rbqxfs", invoke<&wk_chunk_lse>},
    {"wk_window_update", "riinninbbniiwns", invoke<&wk_window_update>},
};
constexpr int kEntries = sizeof(entries) / sizeof(entries[0]);
constexpr int kMaxArgs = 24;

// The tensors of a call, as far as they came.
struct Tensors {
    const at::Tensor *first = nullptr, *second = nullptr;
    int n = 0;

    // pointer of a tensor kernels can address (type: its scalar type, -1: any), null for None; false: not the usual one
    bool take(PyObject *o, Arg &a, int type, const at::Tensor **out = nullptr) {
        a.p = nullptr;
        ++n;
        if (o == Py_None) return true;
        if (!THPVariable_CheckExact(o)) return false;
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous() || (type >= 0 && (int)t.scalar_type() != type)) return false;
        a.p = t.data_ptr();
        if (n == 1) first = &t;
        if (n == 2) second = &t;
        if (out) *out = &t;
        return true;
    }
    bool size(int of, Arg &a) const {   // of the first one, which has three
        if (!first || first->dim() != 3) return false;
        a.i = first->size(of);
        return true;
    }
    bool stride(Arg &a, bool needed) const {
        if (second ? second->dim() < 2 : needed) return false;
        a.i = second ? second->size(1) : 0;
        return true;
    }
};

bool whole(PyObject *o, Arg &a) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    a.i = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

PyObject *run(const Entry &e, PyObject *const *args, Py_ssize_t n) try {
    Arg a[kMaxArgs];
    float five[5];
    int32_t n_out = 0;
    int count = 0;
    Py_ssize_t at = 0;
    Tensors seen;
    bool usual = e.fn != nullptr, returns_count = false;
    for (const char *s = e.signature; *s && usual; ++s) {
        Arg &x = a[count++];
        x.p = nullptr;   // (all of it)
        switch (*s) {   // those without an argument
        case 'h': usual = seen.size(0, x); continue;
        case 'q': usual = seen.size(1, x); continue;
        case 'e': usual = seen.size(2, x); continue;
        case 'k': usual = seen.stride(x, false); continue;
        case 'm': usual = seen.stride(x, true); continue;
        case 'y':
            usual = seen.first && (seen.first->scalar_type() == at::kFloat || seen.first->scalar_type() == at::kBFloat16);
            x.i = usual && seen.first->scalar_type() == at::kBFloat16 ? WK_BF16 : WK_F32;
            continue;
        case 'o':
            x.p = &n_out;
            returns_count = true;
            continue;
        case 's':
            x.p = c10::hip::getCurrentHIPStream().stream();   // (a tensor on it has shown that the device is in use)
            usual = seen.first != nullptr;
            continue;
        }
        if (at >= n) return PyErr_Format(PyExc_TypeError, "%s: too few arguments", e.name);
        PyObject *o = args[at++];
        switch (*s) {
        case 'b': usual = seen.take(o, x, -1); break;
        case 't': usual = seen.first && seen.take(o, x, (int)seen.first->scalar_type()); break;
        case 'i': usual = seen.take(o, x, (int)at::kInt); break;
        case 'f': usual = seen.take(o, x, (int)at::kFloat); break;
        case 'd': usual = seen.take(o, x, (int)at::kDouble); break;
        case 'w': {
            const at::Tensor *t = nullptr;
            usual = seen.take(o, x, -1, &t);
            a[count++].i = t ? (int64_t)t->nbytes() : 0;
            break;
        }
        case 'n': usual = whole(o, x); break;
        case 'v': usual = o == Py_None ? seen.stride(x, true) : whole(o, x); break;
        case 'x':
            usual = PyFloat_CheckExact(o);
            if (usual) x.f = (float)PyFloat_AS_DOUBLE(o);
            break;
        case '5':
            usual = (PyList_CheckExact(o) || PyTuple_CheckExact(o)) && PySequence_Fast_GET_SIZE(o) == 5;
            for (int k = 0; k < 5 && usual; ++k) {
                PyObject *v = PySequence_Fast_GET_ITEM(o, k);
                usual = PyFloat_CheckExact(v);
                if (usual) five[k] = (float)PyFloat_AS_DOUBLE(v);
            }
            x.p = five;
            break;
        case 'r': {
            Py_buffer view;   // (the caller holds the structure, whose memory does not move)
            usual = Py_TYPE(o) == e.type && PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) == 0;
            if (usual) {
                x.p = view.buf;
                PyBuffer_Release(&view);
            }
            break;
        }
        default: usual = false;
        }
    }
    if (PyErr_Occurred()) PyErr_Clear();
    if (!usual) Py_RETURN_NONE;
    int status = 0;
    Py_BEGIN_ALLOW_THREADS
    status = e.invoke(e.fn, a);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(returns_count && status == WK_OK ? -(long)n_out : status);
} catch (const std::exception &) {   // a tensor without storage: the Python functions say so
    Py_RETURN_NONE;
}

template <int K>
PyObject *method(PyObject *, PyObject *const *args, Py_ssize_t n) { return run(entries[K], args, n); }

// bind(name, address, type): the function of the library that is loaded, and the type of its structure (or None)
PyObject *bind(PyObject *, PyObject *args) {
    const char *name;
    unsigned long long address;
    PyObject *type;
    if (!PyArg_ParseTuple(args, "sKO", &name, &address, &type)) return nullptr;
    for (Entry &e : entries)
        if (!std::strcmp(e.name, name)) {
            e.fn = reinterpret_cast<void *>(address);
            Py_INCREF(type);   // (classes of the package: for good)
            e.type = reinterpret_cast<PyTypeObject *>(type);
            Py_RETURN_NONE;
        }
    return PyErr_Format(PyExc_KeyError, "%s", name);
}

// interface(): of the wk.h this was compiled with, and so of the signatures that it calls
PyObject *interface(PyObject *, PyObject *) { return PyLong_FromUnsignedLongLong(WK_INTERFACE); }

PyMethodDef methods[kEntries + 3];

template <int... K>
void fill(std::integer_sequence<int, K...>) {
    ((methods[K] = PyMethodDef{entries[K].name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&method<K>)), METH_FASTCALL, nullptr}), ...);
    methods[kEntries] = PyMethodDef{"bind", &bind, METH_VARARGS, nullptr};
    methods[kEntries + 1] = PyMethodDef{"interface", &interface, METH_NOARGS, nullptr};
    methods[kEntries + 2] = PyMethodDef{nullptr, nullptr, 0, nullptr};
}

PyModuleDef module = {PyModuleDef_HEAD_INIT, "wk_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_wk_binding() {
    fill(std::make_integer_sequence<int, kEntries>{});
    return PyModule_Create(&module);
}
