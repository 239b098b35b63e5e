// What a checked call costs the host beyond its launch, in native code: the checks of a tensor argument (dev) and the call
// of a C-ABI entry point with converted arguments (one function per entry point).  binding.py builds the argument tuples.
//
// A tensor that passes every check gives its address; anything else gives None and binding.py repeats the checks in Python,
// which raises the error with the argument's name.  In Python a tensor's checks take 0.6 us and the conversion of the
// step's 19 arguments by ctypes 1.7 us; here 0.1 us and 0.2 us.
#include <Python.h>

#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "ragged.h"

namespace {

// dtype: None, a torch.dtype or a tuple of them
bool dtype_is(PyObject* want, at::ScalarType have) {
    if (THPDtype_Check(want)) return reinterpret_cast<THPDtype*>(want)->scalar_type == have;
    if (!PyTuple_Check(want)) return false;
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(want); ++i) {
        PyObject* one = PyTuple_GET_ITEM(want, i);
        if (THPDtype_Check(one) && reinterpret_cast<THPDtype*>(one)->scalar_type == have) return true;
    }
    return false;
}

// shape: None or a tuple of integers
bool shape_is(PyObject* want, c10::IntArrayRef have) {
    if (!PyTuple_Check(want) || PyTuple_GET_SIZE(want) != static_cast<Py_ssize_t>(have.size())) return false;
    for (size_t i = 0; i < have.size(); ++i) {
        PyObject* one = PyTuple_GET_ITEM(want, i);
        if (!PyLong_CheckExact(one)) return false;
        int overflow = 0;
        if (PyLong_AsLongLongAndOverflow(one, &overflow) != have[i] || overflow != 0) return false;
    }
    return true;
}

// dev(tensor, dtype, shape) -> address of a contiguous GPU tensor of that type and shape, or None.  Only plain tensors: a
// subclass may have its own idea of its attributes.
PyObject* dev(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 3) {
        PyErr_SetString(PyExc_TypeError, "dev takes a tensor, a dtype and a shape");
        return nullptr;
    }
    if (!THPVariable_CheckExact(args[0])) Py_RETURN_NONE;
    try {
        const at::Tensor& t = THPVariable_Unpack(args[0]);
        if (!t.is_cuda() || !t.is_contiguous()) Py_RETURN_NONE;
        if (args[1] != Py_None && !dtype_is(args[1], t.scalar_type())) Py_RETURN_NONE;
        if (args[2] != Py_None && !shape_is(args[2], t.sizes())) Py_RETURN_NONE;
        return PyLong_FromVoidPtr(t.data_ptr());
    } catch (...) {                                            // a tensor without storage of its own (tracing, vmap)
        Py_RETURN_NONE;
    }
}

template <typename T>
bool convert(PyObject* o, T& out) {
    if constexpr (std::is_pointer_v<T>) {
        if (o == Py_None) { out = nullptr; return true; }
        out = reinterpret_cast<T>(PyLong_AsVoidPtr(o));
    } else if constexpr (std::is_floating_point_v<T>) {
        out = static_cast<T>(PyFloat_AsDouble(o));
    } else {
        if (!PyLong_Check(o)) { PyErr_SetString(PyExc_TypeError, "an integer is required"); return false; }
        out = static_cast<T>(PyLong_AsUnsignedLongLongMask(o));
    }
    return !PyErr_Occurred();
}

template <typename... A, size_t... I>
PyObject* invoke(int (*fn)(A...), PyObject* const* args, std::index_sequence<I...>) {
    std::tuple<A...> v;
    if (!(convert(args[I], std::get<I>(v)) && ...)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = fn(std::get<I>(v)...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}
template <typename... A>
PyObject* invoke(int (*fn)(A...), PyObject* const* args, Py_ssize_t n) {
    if (n != static_cast<Py_ssize_t>(sizeof...(A))) {
        PyErr_Format(PyExc_TypeError, "%zd arguments given, %zd expected", n, static_cast<Py_ssize_t>(sizeof...(A)));
        return nullptr;
    }
    return invoke(fn, args, std::make_index_sequence<sizeof...(A)>{});
}
template <auto Fn>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) { return invoke(Fn, args, n); }

#define ENTRY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<&name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"dev", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&dev)), METH_FASTCALL, nullptr},
    ENTRY(ragged_pack), ENTRY(ragged_attn), ENTRY(ragged_attn_strided), ENTRY(ragged_attn_checked), ENTRY(ragged_attn_padded),
    ENTRY(ragged_unpack), ENTRY(ragged_repack), ENTRY(ragged_cls_extract), ENTRY(ragged_pack_attn_unpack), ENTRY(ragged_linear),
    ENTRY(ragged_layernorm), ENTRY(ragged_token_scores_l2), ENTRY(ragged_keep_topk), ENTRY(ragged_noop),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ragged_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ragged_marshal() { return PyModule_Create(&module); }
