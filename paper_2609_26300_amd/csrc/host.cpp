// host.cpp -- the call path of the Python binding in native code (_host, a CPython extension): checks the
// tensors of a call and enters the C ABI. A decode step checks sixteen tensors; in Python that and ctypes took
// about as long as the step's kernels at 4K tokens (37 us a step against 20 us of GPU time).
//
// call(kind, entry, args, specs): `entry` is the address of a C ABI function and `kind` says which one (its
// place in the table below, which holds its prototype); `args` is a tuple and `specs` a tuple of the same
// length that says what each argument has to be:
//   None                      an int or a float, passed as it is;
//   (dtype, shape, nullable)  a contiguous CUDA tensor of that dtype and shape, passed as its address (None: a
//                             null pointer, where nullable);
//   True                      any contiguous CUDA tensor, passed as its address and its size in bytes.
// Returns the call's status; or None, nothing having been called, when an argument is anything else: the caller
// then makes the checks in Python, which name what is wrong or accept what only they accept (pinned host memory).
#include "compkv.h"

#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/Dtype.h>

#include <cstdint>
#include <type_traits>
#include <utility>

namespace {

constexpr Py_ssize_t kMostArgs = 20;

struct Word {
    uint64_t u = 0;
    double f = 0.0;
};

template <typename T>
T as(const Word& w) {
    if constexpr (std::is_floating_point_v<T>)
        return static_cast<T>(w.f);
    else if constexpr (std::is_pointer_v<T>)
        return reinterpret_cast<T>(w.u);
    else
        return static_cast<T>(w.u);
}

// the C ABI functions, in the order of the binding's kinds; -1: not this many arguments
template <typename... A, size_t... I>
int enter(int (*f)(A...), const Word* w, std::index_sequence<I...>) {
    return f(as<A>(w[I])...);
}
template <typename... A>
bool dispatch_one(int (*f)(A...), const Word* w, Py_ssize_t n, int* status) {
    if (n != static_cast<Py_ssize_t>(sizeof...(A))) return false;
    *status = enter(f, w, std::index_sequence_for<A...>{});
    return true;
}
#define COMPKV_ENTRY(name) dispatch_one(reinterpret_cast<decltype(&name)>(entry), w, n, status)
bool dispatch(long kind, uint64_t entry, const Word* w, Py_ssize_t n, int* status) {
    switch (kind) {
        case 0: return COMPKV_ENTRY(compkv_build_stats);
        case 1: return COMPKV_ENTRY(compkv_append_stats);
        case 2: return COMPKV_ENTRY(compkv_score_select);
        case 3: return COMPKV_ENTRY(compkv_sparse_decode);
        case 4: return COMPKV_ENTRY(compkv_dense_decode);
        case 5: return COMPKV_ENTRY(compkv_decode_step);
        case 6: return COMPKV_ENTRY(compkv_decode_step_noalloc);
        default: return false;
    }
}
#undef COMPKV_ENTRY

// address of tensor `o` if it is what `spec` asks for; false otherwise
bool tensor_word(PyObject* o, PyObject* spec, uint64_t* word) {
    if (!PyTuple_CheckExact(spec) || PyTuple_GET_SIZE(spec) != 3) return false;
    if (o == Py_None) {
        *word = 0;
        return PyTuple_GET_ITEM(spec, 2) == Py_True;
    }
    if (!THPVariable_Check(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    PyObject* dtype = PyTuple_GET_ITEM(spec, 0);
    PyObject* shape = PyTuple_GET_ITEM(spec, 1);
    if (!THPDtype_Check(dtype) || !PyTuple_CheckExact(shape)) return false;
    if (!t.is_cuda() || t.scalar_type() != reinterpret_cast<THPDtype*>(dtype)->scalar_type || !t.is_contiguous())
        return false;
    const Py_ssize_t n = PyTuple_GET_SIZE(shape);
    if (t.dim() != n) return false;
    for (Py_ssize_t i = 0; i < n; ++i) {
        const long long want = PyLong_AsLongLong(PyTuple_GET_ITEM(shape, i));
        if (want == -1 && PyErr_Occurred()) {
            PyErr_Clear();
            return false;
        }
        if (t.size(i) != want) return false;
    }
    *word = reinterpret_cast<uint64_t>(t.data_ptr());
    return true;
}

PyObject* call(PyObject*, PyObject* const* in, Py_ssize_t count) {
    if (count != 4 || !PyLong_Check(in[0]) || !PyLong_Check(in[1]) || !PyTuple_CheckExact(in[2]) ||
        !PyTuple_CheckExact(in[3]) || PyTuple_GET_SIZE(in[2]) != PyTuple_GET_SIZE(in[3])) {
        PyErr_SetString(PyExc_TypeError, "call(kind, entry, args, specs), args and specs tuples of one length");
        return nullptr;
    }
    const long kind = PyLong_AsLong(in[0]);
    const uint64_t entry = PyLong_AsUnsignedLongLong(in[1]);
    if (PyErr_Occurred()) return nullptr;
    Word w[kMostArgs];
    Py_ssize_t n = 0;
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(in[2]); ++i) {
        PyObject* a = PyTuple_GET_ITEM(in[2], i);
        PyObject* s = PyTuple_GET_ITEM(in[3], i);
        if (n + 2 > kMostArgs && !(n + 1 == kMostArgs && s != Py_True)) {
            PyErr_SetString(PyExc_TypeError, "too many arguments");
            return nullptr;
        }
        try {
            if (s == Py_None && PyFloat_Check(a)) {
                w[n++].f = PyFloat_AS_DOUBLE(a);
            } else if (s == Py_None) {
                if (!PyLong_Check(a)) Py_RETURN_NONE;
                w[n++].u = PyLong_AsUnsignedLongLongMask(a);
            } else if (s == Py_True) {
                if (!THPVariable_Check(a)) Py_RETURN_NONE;
                const at::Tensor& t = THPVariable_Unpack(a);
                if (!t.is_cuda() || !t.is_contiguous()) Py_RETURN_NONE;
                w[n++].u = reinterpret_cast<uint64_t>(t.data_ptr());
                w[n++].u = static_cast<uint64_t>(t.nbytes());
            } else if (!tensor_word(a, s, &w[n++].u)) {
                Py_RETURN_NONE;
            }
        } catch (...) {  // (a tensor without storage: the checks in Python say so)
            Py_RETURN_NONE;
        }
    }
    int status = 0;
    bool known;
    Py_BEGIN_ALLOW_THREADS
    known = dispatch(kind, entry, w, n, &status);
    Py_END_ALLOW_THREADS
    if (!known) {
        PyErr_SetString(PyExc_TypeError, "no such function with this many arguments");
        return nullptr;
    }
    return PyLong_FromLong(status);
}

PyMethodDef methods[] = {{"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(call)), METH_FASTCALL,
                          "call(kind, entry, args, specs) -> status or None"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host(void) { return PyModule_Create(&module); }
