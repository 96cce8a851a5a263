// CPython module `_native`: the C ABI of libvfa.so (vfa.h) as Python functions with the same names and the same arguments in the
// same order, returning the status code.  Pointers are integers or None.  It checks no tensors (the package's __init__.py does).
// Converting the twenty arguments of a call that is refused at once takes 2.6 us through ctypes, one object at a time, and 0.2 us
// here (measured on the host; a step of two calls got 6.4 us shorter).  The conversions follow from the declared argument types, so
// a signature that changes in vfa.h changes here by itself.
//
// What the wrappers of __init__.py look up on every call, is_cuda, dtype, is_contiguous(), shape and data_ptr() of up to seven objects,
// is looked up here too (check_qkv, check_cache, bytes_of): the same attributes in the same order, so that whatever has them works as
// before, without an interpreter step for each.  Host time of a call, launches included, before / after in us: vfa_attn_fwd 7.1 / 5.3,
// an append and a decode step 12.4 / 10.2.
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

// Attribute and method names, made once when the module is loaded.
struct Names {
    PyObject *data_ptr, *is_cuda, *dtype, *is_contiguous, *dim, *shape, *numel, *element_size;
    bool make() {
        return (data_ptr = PyUnicode_InternFromString("data_ptr")) && (is_cuda = PyUnicode_InternFromString("is_cuda")) &&
               (dtype = PyUnicode_InternFromString("dtype")) && (is_contiguous = PyUnicode_InternFromString("is_contiguous")) &&
               (dim = PyUnicode_InternFromString("dim")) && (shape = PyUnicode_InternFromString("shape")) &&
               (numel = PyUnicode_InternFromString("numel")) && (element_size = PyUnicode_InternFromString("element_size"));
    }
} names;

// A new reference that is given back at the end of the scope.
struct Ref {
    PyObject* o;
    explicit Ref(PyObject* x) : o(x) {}
    ~Ref() { Py_XDECREF(o); }
    Ref(const Ref&) = delete;
    Ref& operator=(const Ref&) = delete;
};
Ref attribute(PyObject* o, PyObject* name) { return Ref(PyObject_GetAttr(o, name)); }
Ref method(PyObject* o, PyObject* name) { return Ref(PyObject_CallMethodNoArgs(o, name)); }
// 1 = true, 0 = false, -1 = an error is set
int truth(const Ref& r) { return r.o ? PyObject_IsTrue(r.o) : -1; }

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
template <typename T>
bool convert_tensor(PyObject* o, T& v) {
    if constexpr (std::is_pointer_v<T>) {
        if (o == Py_None) return convert(o, v);
        const Ref p = method(o, names.data_ptr);
        return p.o && convert(p.o, v);
    } else {
        return convert(o, v);
    }
}

template <bool TENSORS, typename R, typename... A, size_t... I>
PyObject* call(R (*f)(A...), PyObject* const* args, Py_ssize_t n, std::index_sequence<I...>) {
    if (n != (Py_ssize_t)sizeof...(A)) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", (Py_ssize_t)sizeof...(A), n);
        return nullptr;
    }
    std::tuple<A...> v{};
    const bool ok = ((TENSORS && I + 1 < sizeof...(A) ? convert_tensor(args[I], std::get<I>(v)) : convert(args[I], std::get<I>(v))) && ...);
    if (!ok) return nullptr;
    R r;
    Py_BEGIN_ALLOW_THREADS  // (as ctypes does: other threads run while the launches are enqueued)
    r = f(std::get<I>(v)...);
    Py_END_ALLOW_THREADS
    return std::is_unsigned_v<R> ? PyLong_FromUnsignedLongLong((unsigned long long)r) : PyLong_FromLongLong((long long)r);
}
template <bool TENSORS, auto F>
struct Wrap;
template <bool TENSORS, typename R, typename... A, R (*F)(A...)>
struct Wrap<TENSORS, F> {
    static PyObject* run(PyObject*, PyObject* const* args, Py_ssize_t n) { return call<TENSORS>(F, args, n, std::index_sequence_for<A...>{}); }
};

// is_cuda, dtype, is_contiguous() and, unless dims < 0, dim() of a tensor are as they have to be: 1, 0, or -1 with an error set
int is_as_wanted(PyObject* t, PyObject* dtype, long dims) {
    int ok = truth(attribute(t, names.is_cuda));
    if (ok != 1) return ok;
    {
        const Ref d = attribute(t, names.dtype);
        ok = d.o ? PyObject_RichCompareBool(d.o, dtype, Py_EQ) : -1;
        if (ok != 1) return ok;
    }
    ok = truth(method(t, names.is_contiguous));
    if (ok != 1 || dims < 0) return ok;
    const Ref d = method(t, names.dim);
    if (!d.o) return -1;
    const long n = PyLong_AsLong(d.o);
    return n == -1 && PyErr_Occurred() ? -1 : n == dims;
}

// entries [0, n) of a shape
bool entries(const Ref& shape, Py_ssize_t n, bool all, long long* v) {
    if (!shape.o) return false;
    const Ref fast(PySequence_Fast(shape.o, "a shape is a sequence"));
    if (!fast.o) return false;
    const Py_ssize_t have = PySequence_Fast_GET_SIZE(fast.o);
    if (have < n || (all && have != n)) {
        PyErr_Format(PyExc_ValueError, "a shape of %zd entries was expected, not of %zd", n, have);
        return false;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        v[i] = PyLong_AsLongLong(PySequence_Fast_GET_ITEM(fast.o, i));
        if (v[i] == -1 && PyErr_Occurred()) return false;
    }
    return true;
}

// check_qkv(Q, K, V, bfloat16) -> (B, Hq, Hkv, N, d)
PyObject* check_qkv(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 4) return PyErr_Format(PyExc_TypeError, "expected 4 arguments, got %zd", n);
    for (int i = 0; i < 3; ++i) {
        const int ok = is_as_wanted(args[i], args[3], 4);
        if (ok < 0) return nullptr;
        if (!ok) return PyErr_Format(PyExc_ValueError, "Q, K, V must be contiguous 4-d bf16 tensors on the GPU");
    }
    const Ref qs = attribute(args[0], names.shape), ks = attribute(args[1], names.shape), vs = attribute(args[2], names.shape);
    long long q[4], k[4];
    if (!entries(qs, 4, true, q) || !entries(ks, 4, true, k) || !vs.o) return nullptr;
    const int differ = PyObject_RichCompareBool(ks.o, vs.o, Py_NE);
    if (differ < 0) return nullptr;
    if (differ || k[0] != q[0] || k[2] != q[2] || k[3] != q[3])
        return PyErr_Format(PyExc_ValueError, "K, V must be [B, Hkv, N, d] matching Q [B, Hq, N, d]");
    return Py_BuildValue("(LLLLL)", q[0], q[1], k[1], q[2], q[3]);
}

// check_cache(q, K, V, bfloat16 or None) -> (B, Hq, d, Hkv, n_cap); None: the tensors' types are not looked at
PyObject* check_cache(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 4) return PyErr_Format(PyExc_TypeError, "expected 4 arguments, got %zd", n);
    long long q[3], k[3];
    if (!entries(attribute(args[0], names.shape), 3, true, q) || !entries(attribute(args[1], names.shape), 3, false, k)) return nullptr;
    for (int i = 0; i < 3 && args[3] != Py_None; ++i) {
        const int ok = is_as_wanted(args[i], args[3], -1);
        if (ok < 0) return nullptr;
        if (!ok) return PyErr_Format(PyExc_ValueError, "q, K, V must be contiguous bf16 tensors on the GPU");
    }
    return Py_BuildValue("(LLLLL)", q[0], q[1], q[2], k[1], k[2]);
}

// bytes_of(t): numel() * element_size()
PyObject* bytes_of(PyObject*, PyObject* t) {
    const Ref n = method(t, names.numel);
    if (!n.o) return nullptr;
    const Ref e = method(t, names.element_size);
    return e.o ? PyNumber_Multiply(n.o, e.o) : nullptr;
}

#define VFA_FUNCTION(f) (PyCFunction)(void (*)(void)) & f, METH_FASTCALL, nullptr
#define VFA_METHOD(name) {#name, VFA_FUNCTION((Wrap<false, &name>::run))}
#define VFA_METHODS(name) VFA_METHOD(name), {#name "_t", VFA_FUNCTION((Wrap<true, &name>::run))}
PyMethodDef methods[] = {
    VFA_METHOD(vfa_workspace_bytes), VFA_METHODS(vfa_kblock_summary), VFA_METHODS(vfa_kblock_summary_mode),
    VFA_METHODS(fa_baseline_fwd), VFA_METHODS(fa_lazy_rescale_fwd), VFA_METHODS(fa_lazy_rescale_softexp_fwd),
    VFA_METHODS(vfa_attn_fwd), VFA_METHODS(vsa_attn_fwd), VFA_METHODS(vfa_variant_fwd),
    VFA_METHODS(vfa_kblock_summary_append), VFA_METHODS(vfa_kblock_summary_append_varlen),
    VFA_METHOD(vfa_decode_workspace_bytes), VFA_METHODS(vfa_decode_fwd), VFA_METHODS(vfa_decode_noalloc_fwd), VFA_METHODS(vfa_decode_varlen_fwd),
    VFA_METHODS(vfa_fp8_quantize), VFA_METHOD(vfa_fp8_v_bytes), VFA_METHODS(vfa_fp8_pack_v), VFA_METHODS(vfa_fp8_attn_fwd), VFA_METHODS(vfa_fp8_attn_noexp_fwd),
    VFA_METHODS(vfa_mxfp4_quantize), VFA_METHOD(vfa_mxfp4_workspace_bytes), VFA_METHODS(vfa_mxfp4_attn_fwd), VFA_METHODS(vfa_mxfp4_attn_noexp_fwd),
    {"check_qkv", VFA_FUNCTION(check_qkv)}, {"check_cache", VFA_FUNCTION(check_cache)},
    {"bytes_of", &bytes_of, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "The C ABI of libvfa.so.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return names.make() ? PyModule_Create(&module) : nullptr; }
