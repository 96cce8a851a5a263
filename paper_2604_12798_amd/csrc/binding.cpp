// CPython module `_native`: the C ABI of libvfa.so (vfa.h) as Python functions with the same names and the same arguments in the
// same order, returning the status code.  Pointers are integers or None.  It checks no tensors (the package's __init__.py does).
// Converting the twenty arguments of a call that is refused at once takes 2.6 us through ctypes, one object at a time, and 0.2 us
// here (measured on the host; a step of two calls got 6.4 us shorter).  The conversions follow from the declared argument types, so
// a signature that changes in vfa.h changes here by itself.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstddef>
#include <cstdint>
#include <tuple>
#include <type_traits>
#include <utility>

#include "vfa.h"

namespace {

// Whole numbers (and what has __index__): the low bits of the C type, as ctypes takes them; the entry point judges the range.
template <typename T, std::enable_if_t<std::is_integral_v<T>, int> = 0>
bool convert(PyObject* o, T& v) {
    v = (T)PyLong_AsUnsignedLongLongMask(o);
    return !(v == (T)-1 && PyErr_Occurred());
}
bool convert(PyObject* o, float& v) {
    v = (float)PyFloat_AsDouble(o);
    return !(v == -1.f && PyErr_Occurred());
}
template <typename T>
bool convert(PyObject* o, T*& v) {
    v = nullptr;
    if (o == Py_None) return true;
    if (!PyLong_Check(o)) {
        PyErr_SetString(PyExc_TypeError, "a pointer is an integer or None");
        return false;
    }
    v = reinterpret_cast<T*>((uintptr_t)PyLong_AsUnsignedLongLongMask(o));
    return true;
}

template <typename R, typename... A, size_t... I>
PyObject* call(R (*f)(A...), PyObject* const* args, Py_ssize_t n, std::index_sequence<I...>) {
    if (n != (Py_ssize_t)sizeof...(A)) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", (Py_ssize_t)sizeof...(A), n);
        return nullptr;
    }
    std::tuple<A...> v{};
    const bool ok = (convert(args[I], std::get<I>(v)) && ...);
    if (!ok) return nullptr;
    R r;
    Py_BEGIN_ALLOW_THREADS  // (as ctypes does: other threads run while the launches are enqueued)
    r = f(std::get<I>(v)...);
    Py_END_ALLOW_THREADS
    return std::is_unsigned_v<R> ? PyLong_FromUnsignedLongLong((unsigned long long)r) : PyLong_FromLongLong((long long)r);
}
template <auto F>
struct Wrap;
template <typename R, typename... A, R (*F)(A...)>
struct Wrap<F> {
    static PyObject* run(PyObject*, PyObject* const* args, Py_ssize_t n) { return call(F, args, n, std::index_sequence_for<A...>{}); }
};

#define VFA_METHOD(name) {#name, (PyCFunction)(void (*)(void)) & Wrap<&name>::run, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    VFA_METHOD(vfa_workspace_bytes), VFA_METHOD(vfa_kblock_summary), VFA_METHOD(vfa_kblock_summary_mode),
    VFA_METHOD(fa_baseline_fwd), VFA_METHOD(fa_lazy_rescale_fwd), VFA_METHOD(fa_lazy_rescale_softexp_fwd),
    VFA_METHOD(vfa_attn_fwd), VFA_METHOD(vsa_attn_fwd), VFA_METHOD(vfa_variant_fwd),
    VFA_METHOD(vfa_kblock_summary_append), VFA_METHOD(vfa_kblock_summary_append_varlen),
    VFA_METHOD(vfa_decode_workspace_bytes), VFA_METHOD(vfa_decode_fwd), VFA_METHOD(vfa_decode_noalloc_fwd), VFA_METHOD(vfa_decode_varlen_fwd),
    VFA_METHOD(vfa_fp8_quantize), VFA_METHOD(vfa_fp8_v_bytes), VFA_METHOD(vfa_fp8_pack_v), VFA_METHOD(vfa_fp8_attn_fwd), VFA_METHOD(vfa_fp8_attn_noexp_fwd),
    VFA_METHOD(vfa_mxfp4_quantize), VFA_METHOD(vfa_mxfp4_workspace_bytes), VFA_METHOD(vfa_mxfp4_attn_fwd), VFA_METHOD(vfa_mxfp4_attn_noexp_fwd),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "The C ABI of libvfa.so.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
