// CPython module `_native`: the C ABI of libvfa.so (vfa.h) as Python functions with the same names and the same arguments in the
// same order, returning the status code.  Pointers are integers or None.  A call through ctypes spends 4 to 5 us on converting
// twenty arguments one object at a time, more than the two kernel launches behind it; this takes 0.6 us.  The conversions follow
// from the declared argument types, so a signature that changes in vfa.h changes here by itself.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <climits>
#include <cstddef>
#include <tuple>
#include <utility>

#include "vfa.h"

namespace {

bool convert(PyObject* o, int& v) {
    const long x = PyLong_AsLong(o);
    if (x == -1 && PyErr_Occurred()) return false;
    if (x < INT_MIN || x > INT_MAX) {
        PyErr_SetString(PyExc_OverflowError, "argument does not fit a C int");
        return false;
    }
    v = (int)x;
    return true;
}
bool convert(PyObject* o, long long& v) {
    v = PyLong_AsLongLong(o);
    return !(v == -1 && PyErr_Occurred());
}
bool convert(PyObject* o, size_t& v) {
    v = PyLong_AsSize_t(o);
    return !(v == (size_t)-1 && PyErr_Occurred());
}
bool convert(PyObject* o, float& v) {
    v = (float)PyFloat_AsDouble(o);
    return !(v == -1.f && PyErr_Occurred());
}
template <typename T>
bool convert(PyObject* o, T*& v) {
    v = o == Py_None ? nullptr : static_cast<T*>(PyLong_AsVoidPtr(o));
    return !(v == nullptr && PyErr_Occurred());
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
    return PyLong_FromLongLong((long long)r);
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
