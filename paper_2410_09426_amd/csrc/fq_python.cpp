// CPython calls of the launching entry points of libflatquant (include/flatquant.h): argument marshalling only, the work of
// binding.py's other functions in native code.  What bounds a decode step is the host: 2.6 us per launch in the HIP runtime, and
// on top of it, for a product with tensors and a stream, 2.6 us through a Python function and ctypes; from here 0.5 us.
//
// Nothing of the library is linked here: binding.py hands over the addresses of the entry points when it loads libflatquant.so, so
// both halves of the binding always talk to the same one, and importing this module loads nothing.
//
// A pointer argument is None, an address, or an object with data_ptr(); a stream is None, a handle, or an object with
// cuda_stream.  Numbers go through int() / float() as they did there, and into the C types like ctypes does it (low bits of an
// integer).  The interpreter lock is released around the call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "../../include/flatquant.h"

namespace {

enum Entry { TRANSFORM, MX, MX_TILED, WEIGHT, W4A4, MX_GEMM, KV, KV_BITS, HEAD, COUNT };
void* g_entry[COUNT];                 // addresses in the loaded library; null until then
PyObject* g_error = nullptr;          // binding.FlatQuantError(status, where)
PyObject* g_load = nullptr;           // binding.lib: loads the library and binds its addresses, or raises
PyObject *g_data_ptr, *g_cuda_stream; // attribute names

struct Reader {                       // reads arguments in order; after a failure everything reads as 0
    PyObject* const* v;
    int i = 0;
    bool ok = true;
    uint64_t bits(PyObject* n) {      // steals n
        if (!n) {
            ok = false;
            return 0;
        }
        const uint64_t r = PyLong_AsUnsignedLongLongMask(n);
        Py_DECREF(n);
        if (r == (uint64_t)-1 && PyErr_Occurred()) ok = false;
        return r;
    }
    void* ptr() {
        PyObject* o = v[i++];
        if (!ok || o == Py_None) return nullptr;
        if (PyLong_Check(o)) return (void*)(uintptr_t)bits(Py_NewRef(o));
        PyObject* a = PyObject_CallMethodNoArgs(o, g_data_ptr);
        if (!a) return (void*)(uintptr_t)bits(nullptr);
        PyObject* n = PyNumber_Long(a);
        Py_DECREF(a);
        return (void*)(uintptr_t)bits(n);
    }
    void* stream() {
        PyObject* o = v[i++];
        if (!ok || !o || o == Py_None) return nullptr;
        if (PyLong_Check(o)) return (void*)(uintptr_t)bits(Py_NewRef(o));
        PyObject* a = PyObject_GetAttr(o, g_cuda_stream);
        if (!a) return (void*)(uintptr_t)bits(nullptr);
        PyObject* n = PyNumber_Long(a);
        Py_DECREF(a);
        return (void*)(uintptr_t)bits(n);
    }
    int64_t i64() {
        PyObject* o = v[i++];
        return ok ? (int64_t)bits(PyNumber_Long(o)) : 0;
    }
    int i32() { return (int)i64(); }
    float f32() {
        PyObject* o = v[i++];
        if (!ok) return 0.0f;
        PyObject* n = PyNumber_Float(o);
        if (!n) {
            ok = false;
            return 0.0f;
        }
        const double d = PyFloat_AS_DOUBLE(n);
        Py_DECREF(n);
        return (float)d;
    }
};

constexpr int kMaxArgs = 16;

// Positional and keyword arguments into out[0 .. n - 1] by the names of a signature whose last two are optional: stream, check.
struct Signature {
    Entry entry;
    const char* name;
    const char* names[kMaxArgs];
    int n = 0;
    PyObject* keys[kMaxArgs] = {};
};

// The entry point's address: on the first call the library is loaded.
template <typename Fn>
bool entry(Entry e, Fn& fn) {
    if (!g_entry[e]) {
        PyObject* r = g_load ? PyObject_CallNoArgs(g_load) : nullptr;
        if (!r && g_load) return false;
        Py_XDECREF(r);
        if (!g_entry[e]) {
            PyErr_SetString(PyExc_RuntimeError, "libflatquant is not bound");
            return false;
        }
    }
    fn = reinterpret_cast<Fn>(g_entry[e]);
    return true;
}

bool collect(const Signature& s, PyObject* const* args, Py_ssize_t nargs, PyObject* kw, PyObject** out) {
    if (nargs > s.n) {
        PyErr_Format(PyExc_TypeError, "%s() takes at most %d positional arguments but %zd were given", s.name, s.n, nargs);
        return false;
    }
    for (int i = 0; i < s.n; ++i) out[i] = i < nargs ? args[i] : nullptr;
    const Py_ssize_t nkw = kw ? PyTuple_GET_SIZE(kw) : 0;
    for (Py_ssize_t k = 0; k < nkw; ++k) {
        PyObject* key = PyTuple_GET_ITEM(kw, k);
        int i = s.n - 1;              // the optional ones are what is mostly named
        while (i >= 0 && s.keys[i] != key) --i;
        if (i < 0) {
            i = s.n - 1;
            while (i >= 0 && PyUnicode_Compare(s.keys[i], key) != 0) --i;
        }
        if (i < 0) {
            PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", s.name, key);
            return false;
        }
        if (out[i]) {
            PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", s.name, key);
            return false;
        }
        out[i] = args[nargs + k];
    }
    for (int i = 0; i < s.n - 2; ++i)
        if (!out[i]) {
            PyErr_Format(PyExc_TypeError, "%s() missing required argument '%s'", s.name, s.names[i]);
            return false;
        }
    return true;
}

PyObject* finish(const Signature& s, fq_status st, PyObject* check) {
    if (st != FQ_OK) {
        const int raise = check ? PyObject_IsTrue(check) : 1;
        if (raise < 0) return nullptr;
        if (raise) {
            PyObject* e = PyObject_CallFunction(g_error, "is", (int)st, s.name);
            if (e) {
                PyErr_SetObject((PyObject*)Py_TYPE(e), e);
                Py_DECREF(e);
            }
            return nullptr;
        }
    }
    return PyLong_FromLong((long)st);
}

// activation and weight transforms: the same arguments, but for the type of the scales
template <typename Scales, typename Fn>
PyObject* transform(const Signature& s, PyObject* const* args, Py_ssize_t nargs, PyObject* kw) {
    PyObject* v[kMaxArgs];
    Fn fn;
    if (!collect(s, args, nargs, kw, v)) return nullptr;
    Reader r{v};
    const void *x = r.ptr(), *P1 = r.ptr(), *P2 = r.ptr(), *clip = r.ptr();
    const int mode = r.i32();
    const int64_t T = r.i64();
    const int n1 = r.i32(), n2 = r.i32();
    const int64_t stride = r.i64();
    void *codes = r.ptr(), *scales = r.ptr(), *stream = r.stream();
    if (!r.ok || !entry(s.entry, fn)) return nullptr;
    fq_status st;
    Py_BEGIN_ALLOW_THREADS
    st = fn(x, P1, P2, (const float*)clip, mode, T, n1, n2, stride, (uint8_t*)codes, (Scales*)scales, stream);
    Py_END_ALLOW_THREADS
    return finish(s, st, v[s.n - 1]);
}

// matrix products
template <typename Scales, typename Fn>
PyObject* product(const Signature& s, PyObject* const* args, Py_ssize_t nargs, PyObject* kw) {
    PyObject* v[kMaxArgs];
    Fn fn;
    if (!collect(s, args, nargs, kw, v)) return nullptr;
    Reader r{v};
    const void *xc = r.ptr(), *xs = r.ptr(), *wc = r.ptr(), *ws = r.ptr();
    const int64_t T = r.i64();
    const int m = r.i32(), n = r.i32();
    void* out = r.ptr();
    const int64_t stride = r.i64();
    void* stream = r.stream();
    if (!r.ok || !entry(s.entry, fn)) return nullptr;
    fq_status st;
    Py_BEGIN_ALLOW_THREADS
    st = fn((const uint8_t*)xc, (const Scales*)xs, (const uint8_t*)wc, (const Scales*)ws, T, m, n, out, stride, stream);
    Py_END_ALLOW_THREADS
    return finish(s, st, v[s.n - 1]);
}

#define ACT() "x", "P1", "P2", "clip", "clip_mode", "T", "n1", "n2", "x_stride", "out_codes", "out_scales", "stream", "check"
Signature kTransform{TRANSFORM, "flatquant_transform_quant", {ACT()}};
Signature kMx{MX, "flatquant_transform_mxfp4", {ACT()}};
Signature kMxTiled{MX_TILED, "flatquant_transform_mxfp4_tiled", {ACT()}};
Signature kWeight{WEIGHT, "flatquant_weight_transform_quant", {"w", "A1", "A2", "clip", "clip_mode", "m", "n1", "n2", "w_stride", "out_codes", "out_scales", "stream", "check"}};
#define GEMM() "x_codes", "x_scales", "w_codes", "w_scales", "T", "m", "n", "out", "out_stride", "stream", "check"
Signature kW4a4{W4A4, "flatquant_w4a4_gemm", {GEMM()}};
Signature kMxGemm{MX_GEMM, "flatquant_mxfp4_gemm", {GEMM()}};
Signature kKv{KV, "flatquant_kv_transform_quant", {"kv", "P", "Hp", "clip", "T", "H", "D", "out_codes", "out_scales", "out_zeros", "stream", "check"}};
Signature kKvBits{KV_BITS, "flatquant_kv_transform_quant_bits", {"kv", "P", "Hp", "clip", "bits", "T", "H", "D", "out_codes", "out_scales", "out_zeros", "stream", "check"}};
Signature kHead{HEAD, "flatquant_head_transform", {"x", "P", "Hp", "T", "H", "D", "out", "stream", "check"}};
Signature* const kAll[COUNT] = {&kTransform, &kMx, &kMxTiled, &kWeight, &kW4a4, &kMxGemm, &kKv, &kKvBits, &kHead};

#define ARGS PyObject*, PyObject *const *a, Py_ssize_t n, PyObject *kw
#define TYPE(entry) decltype(&entry)
PyObject* py_transform(ARGS) { return transform<void, TYPE(flatquant_transform_quant)>(kTransform, a, n, kw); }
PyObject* py_mx(ARGS) { return transform<uint8_t, TYPE(flatquant_transform_mxfp4)>(kMx, a, n, kw); }
PyObject* py_mx_tiled(ARGS) { return transform<uint8_t, TYPE(flatquant_transform_mxfp4_tiled)>(kMxTiled, a, n, kw); }
PyObject* py_weight(ARGS) { return transform<void, TYPE(flatquant_weight_transform_quant)>(kWeight, a, n, kw); }
PyObject* py_w4a4(ARGS) { return product<void, TYPE(flatquant_w4a4_gemm)>(kW4a4, a, n, kw); }
PyObject* py_mx_gemm(ARGS) { return product<uint8_t, TYPE(flatquant_mxfp4_gemm)>(kMxGemm, a, n, kw); }
// KV cache; the code width is an argument of one of the two
template <bool BITS>
PyObject* kv(const Signature& s, PyObject* const* args, Py_ssize_t nargs, PyObject* kw) {
    PyObject* v[kMaxArgs];
    TYPE(flatquant_kv_transform_quant) fn4;
    TYPE(flatquant_kv_transform_quant_bits) fn;
    if (!collect(s, args, nargs, kw, v)) return nullptr;
    Reader r{v};
    const void *x = r.ptr(), *P = r.ptr();
    const int Hp = r.i32();
    const float clip = r.f32();
    const int bits = BITS ? r.i32() : 0;
    const int64_t T = r.i64();
    const int H = r.i32(), D = r.i32();
    void *codes = r.ptr(), *scales = r.ptr(), *zeros = r.ptr(), *stream = r.stream();
    if (!r.ok || !(BITS ? entry(s.entry, fn) : entry(s.entry, fn4))) return nullptr;
    fq_status st;
    Py_BEGIN_ALLOW_THREADS
    st = BITS ? fn(x, P, Hp, clip, bits, T, H, D, (uint8_t*)codes, scales, zeros, stream) : fn4(x, P, Hp, clip, T, H, D, (uint8_t*)codes, scales, zeros, stream);
    Py_END_ALLOW_THREADS
    return finish(s, st, v[s.n - 1]);
}
PyObject* py_kv(ARGS) { return kv<false>(kKv, a, n, kw); }
PyObject* py_kv_bits(ARGS) { return kv<true>(kKvBits, a, n, kw); }
PyObject* py_head(ARGS) {
    PyObject* v[kMaxArgs];
    TYPE(flatquant_head_transform) fn;
    if (!collect(kHead, a, n, kw, v)) return nullptr;
    Reader r{v};
    const void *x = r.ptr(), *P = r.ptr();
    const int Hp = r.i32();
    const int64_t T = r.i64();
    const int H = r.i32(), D = r.i32();
    void *out = r.ptr(), *stream = r.stream();
    if (!r.ok || !entry(kHead.entry, fn)) return nullptr;
    fq_status st;
    Py_BEGIN_ALLOW_THREADS
    st = fn(x, P, Hp, T, H, D, out, stream);
    Py_END_ALLOW_THREADS
    return finish(kHead, st, v[kHead.n - 1]);
}
// connect(load, error): `load` is called when an entry point is needed whose address is not known; `error` is what is raised
PyObject* py_connect(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "connect(load, error)");
        return nullptr;
    }
    Py_XSETREF(g_load, Py_NewRef(a[0]));
    Py_XSETREF(g_error, Py_NewRef(a[1]));
    for (void*& e : g_entry) e = nullptr;
    Py_RETURN_NONE;
}
// bind({name: address}): the entry points of the library just loaded
PyObject* py_bind(PyObject*, PyObject* addresses) {
    void* found[COUNT];
    for (Signature* s : kAll) {
        PyObject* o = PyMapping_GetItemString(addresses, s->name);
        if (!o) return nullptr;
        found[s->entry] = PyLong_AsVoidPtr(o);
        Py_DECREF(o);
        if (PyErr_Occurred()) return nullptr;
    }
    for (int e = 0; e < COUNT; ++e) g_entry[e] = found[e];
    Py_RETURN_NONE;
}

#define FN(name, fn, sig) {name, (PyCFunction)(void (*)(void))fn, METH_FASTCALL | METH_KEYWORDS, name sig "\n--\n\nSee include/flatquant.h; returns the status, raises FlatQuantError if check."}
#define ACT_SIG "(x, P1, P2, clip, clip_mode, T, n1, n2, x_stride, out_codes, out_scales, stream=None, check=True)"
#define GEMM_SIG "(x_codes, x_scales, w_codes, w_scales, T, m, n, out, out_stride, stream=None, check=True)"
PyMethodDef kMethods[] = {
    FN("flatquant_transform_quant", py_transform, ACT_SIG),
    FN("flatquant_transform_mxfp4", py_mx, ACT_SIG),
    FN("flatquant_transform_mxfp4_tiled", py_mx_tiled, ACT_SIG),
    FN("flatquant_weight_transform_quant", py_weight, "(w, A1, A2, clip, clip_mode, m, n1, n2, w_stride, out_codes, out_scales, stream=None, check=True)"),
    FN("flatquant_w4a4_gemm", py_w4a4, GEMM_SIG),
    FN("flatquant_mxfp4_gemm", py_mx_gemm, GEMM_SIG),
    FN("flatquant_kv_transform_quant", py_kv, "(kv, P, Hp, clip, T, H, D, out_codes, out_scales, out_zeros, stream=None, check=True)"),
    FN("flatquant_kv_transform_quant_bits", py_kv_bits, "(kv, P, Hp, clip, bits, T, H, D, out_codes, out_scales, out_zeros, stream=None, check=True)"),
    FN("flatquant_head_transform", py_head, "(x, P, Hp, T, H, D, out, stream=None, check=True)"),
    {"connect", (PyCFunction)(void (*)(void))py_connect, METH_FASTCALL, nullptr},
    {"bind", py_bind, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fqcall", "Native calls of libflatquant's launching entry points (see binding.py).", -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fqcall(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!g_data_ptr || !g_cuda_stream) return nullptr;
    for (Signature* s : kAll)
        for (s->n = 0; s->n < kMaxArgs && s->names[s->n]; ++s->n)
            if (!(s->keys[s->n] = PyUnicode_InternFromString(s->names[s->n]))) return nullptr;
    g_error = Py_NewRef(PyExc_RuntimeError);
    return PyModule_Create(&kModule);
}
