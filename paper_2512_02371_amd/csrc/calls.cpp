// The usual call of each entry point, marshalled natively: exact torch.Tensor objects in, the library's C function out.
//
// On the host a small call costs its launch (3.4 us) and the marshalling: a tensor's strides, sizes, type and address asked for
// through Python, and ctypes, which converts ten arguments in 1.1 us, take 2 us more: hb_fir1d of 256 x 256, 8 taps, call after
// call 5.7 -> 4.0 us, other short kernels 5.6 .. 6.0 -> 3.9 .. 4.2; kernels of 6 us and more leave the host the time anyway.  hb.py comes here first.  A call that is
// anything but usual (another type of tensor, a mode that watches tensor functions, an array of another layout, a wrong shape) is
// not taken: the function returns False before it has done anything, and hb.py marshals it, with the checks and errors it has.
#include <pthread.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>

#include <cstring>
#include <exception>

#include "hb.h"

namespace {

PyObject* g_error = nullptr;                  // hb.HbError
PyTypeObject* g_ndarray = nullptr;
bool g_forked = false;                        // a child of fork() cannot use its parent's device: hb.py lets torch say so

#define HB_CALLS(X) X(hb_fir1d) X(hb_conv2d) X(hb_down2) X(hb_up2) X(hb_sepblur) X(hb_sat2d) X(hb_conv3x3) X(hb_pyr_level) X(hb_resize) X(hb_iir2) X(hb_dct_denoise)
struct Library {
#define HB_POINTER(f) decltype(&::f) f = nullptr;
    HB_CALLS(HB_POINTER)
#undef HB_POINTER
} g_lib;

constexpr int64_t kMostInt = 0x7fffffff;

// A tensor that is its own device memory: no subclass, no wrapper of a transform, no lazy negation.
const at::Tensor* plain(PyObject* o) {
    static const uint64_t usual = c10::DispatchKeySet({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::ADInplaceOrView,
                                                       c10::DispatchKey::AutocastCUDA}).raw_repr();
    if (Py_TYPE(o) != reinterpret_cast<PyTypeObject*>(THPVariableClass)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || (t.key_set().raw_repr() & ~usual) || !t.is_cuda() || t.unsafeGetTensorImpl()->has_symbolic_sizes_strides()) return nullptr;
    return &t;
}

struct Image {
    void* p;
    int planes, h, w;
    int64_t pitch, plane;
};
// Rows of adjacent elements, `dims` dimensions (2, or 3 for planes).
bool image(PyObject* o, at::ScalarType type, int dims, Image& r) {
    const at::Tensor* t = plain(o);
    if (!t || t->dim() != dims || t->scalar_type() != type) return false;
    const auto n = t->sizes(), s = t->strides();
    for (int64_t v : n)
        if (v > kMostInt) return false;
    if (s[dims - 1] != 1) return false;
    r = {t->data_ptr(), dims == 3 ? (int)n[0] : 1, (int)n[dims - 2], (int)n[dims - 1], s[dims - 2], dims == 3 ? s[0] : 0};
    return true;
}

bool bytes(PyObject* o, bool any_type, void*& p, size_t& n) {
    const at::Tensor* t = plain(o);
    if (!t || !t->is_contiguous() || (!any_type && t->scalar_type() != at::kByte)) return false;
    p = t->data_ptr();
    n = t->numel() * t->element_size();
    return true;
}

bool integer(PyObject* o, int& v) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long long x = PyLong_AsLongLongAndOverflow(o, &over);
    if (over || x > kMostInt || x < -kMostInt) return false;
    v = (int)x;
    return true;
}

bool real(PyObject* o, float& v) {
    if (!PyFloat_CheckExact(o)) return false;
    v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}

// A C-ordered numpy array of fp16 values or their bits, copied: another thread may change it once the interpreter is released.
struct Taps {
    hb_half v[HB_MAX_TAPS_CONV2D * HB_MAX_TAPS_CONV2D];
    int n, rows, cols;
};
bool taps(PyObject* o, int dims, Taps& r) {           // dims 0: any
    if (Py_TYPE(o) != g_ndarray) return false;
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) != 0) {
        PyErr_Clear();
        return false;
    }
    const bool ok = b.itemsize == 2 && b.format && (!strcmp(b.format, "H") || !strcmp(b.format, "e")) && b.len <= (Py_ssize_t)sizeof r.v &&
                    (dims == 0 || b.ndim == dims);
    if (ok) {
        memcpy(r.v, b.buf, b.len);
        r.n = (int)(b.len / 2);
        r.rows = b.ndim > 0 ? (int)b.shape[0] : 1;
        r.cols = b.ndim > 1 ? (int)b.shape[1] : 1;
    }
    PyBuffer_Release(&b);
    return ok;
}

struct Banded {
    const int32_t* start;
    const hb_half* coef;
    int band;
};
bool banded(PyObject* s, PyObject* c, int n, Banded& r) {
    const at::Tensor *ts = plain(s), *tc = plain(c);
    if (!ts || !tc || ts->scalar_type() != at::kInt || ts->dim() != 1 || ts->size(0) != n || !ts->is_contiguous() ||
        tc->scalar_type() != at::kHalf || tc->dim() != 2 || tc->size(0) != n || !tc->is_contiguous() || tc->size(1) > kMostInt) return false;
    r = {static_cast<const int32_t*>(ts->data_ptr()), static_cast<const hb_half*>(tc->data_ptr()), (int)tc->size(1)};
    return true;
}

bool usual_state() { return !g_forked && g_error && !at::impl::torch_function_mode_enabled() && !torch::jit::tracer::isTracing(); }

// The call itself, on torch's current stream, without the interpreter's lock (as ctypes makes it).
template <class F>
PyObject* made(const char* name, F call) {
    const hb_stream st = c10::hip::getCurrentHIPStream().stream();
    hb_status s = HB_OK;
    Py_BEGIN_ALLOW_THREADS
    [&]() noexcept { s = call(st); }();
    Py_END_ALLOW_THREADS
    if (s == HB_OK) Py_RETURN_TRUE;
    PyObject* e = PyObject_CallFunction(g_error, "si", name, (int)s);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

// What torch throws while a tensor is asked (memory that may not be had, for one) hb.py meets again, as an error of its own.
// Nothing but exceptions is caught: a daemon thread that wants the interpreter's lock back after the interpreter has ended is unwound
// through here, and the process aborts if that unwinding is stopped.
template <int N, class F>
PyObject* guarded(Py_ssize_t n, F f) {
    if (n != N) Py_RETURN_FALSE;
    try {
        if (usual_state()) return f();
    } catch (const std::exception&) {
    }
    Py_RETURN_FALSE;
}

hb_half* h(void* p) { return static_cast<hb_half*>(p); }
float* f(void* p) { return static_cast<float*>(p); }

PyObject* fir1d(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded<4>(n, [&]() -> PyObject* {
        Image i, o;
        Taps t;
        int anchor;
        if (!image(a[0], at::kHalf, 2, i) || !image(a[1], at::kFloat, 2, o) || i.h != o.h || i.w != o.w || !taps(a[2], 0, t) || !integer(a[3], anchor)) Py_RETURN_FALSE;
        return made("hb_fir1d", [&](hb_stream st) { return g_lib.hb_fir1d(h(i.p), f(o.p), i.h, i.w, i.pitch, o.pitch, t.v, t.n, anchor, st); });
    });
}

// The 2-D filters: hb_conv2d, hb_down2 (every second sample), hb_up2 (twice as many).
template <class Fn, class Shape>
PyObject* filter2d(const char* name, Fn fn, PyObject* const* a, Py_ssize_t n, Shape shape) {
    return guarded<5>(n, [&]() -> PyObject* {
        Image i, o;
        Taps t;
        int ay, ax;
        if (!image(a[0], at::kHalf, 2, i) || !image(a[1], at::kFloat, 2, o) || shape((int64_t)i.h) != o.h || shape((int64_t)i.w) != o.w ||
            !taps(a[2], 2, t) || !integer(a[3], ay) || !integer(a[4], ax)) Py_RETURN_FALSE;
        return made(name, [&](hb_stream st) { return fn(h(i.p), f(o.p), i.h, i.w, i.pitch, o.pitch, t.v, t.rows, t.cols, ay, ax, st); });
    });
}
PyObject* conv2d(PyObject*, PyObject* const* a, Py_ssize_t n) { return filter2d("hb_conv2d", g_lib.hb_conv2d, a, n, [](int64_t v) { return v; }); }
PyObject* down2(PyObject*, PyObject* const* a, Py_ssize_t n) { return filter2d("hb_down2", g_lib.hb_down2, a, n, [](int64_t v) { return (v + 1) / 2; }); }
PyObject* up2(PyObject*, PyObject* const* a, Py_ssize_t n) { return filter2d("hb_up2", g_lib.hb_up2, a, n, [](int64_t v) { return 2 * v; }); }

PyObject* sepblur(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded<6>(n, [&]() -> PyObject* {
        Image i, o;
        Taps x, y;
        int ax, ay;
        if (!image(a[0], at::kHalf, 2, i) || !image(a[1], at::kFloat, 2, o) || i.h != o.h || i.w != o.w || !taps(a[2], 0, x) || !integer(a[3], ax) ||
            !taps(a[4], 0, y) || !integer(a[5], ay)) Py_RETURN_FALSE;
        return made("hb_sepblur", [&](hb_stream st) { return g_lib.hb_sepblur(h(i.p), f(o.p), i.h, i.w, i.pitch, o.pitch, x.v, x.n, ax, y.v, y.n, ay, st); });
    });
}

PyObject* sat2d(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded<3>(n, [&]() -> PyObject* {
        Image i, o;
        void* ws;
        size_t size;
        if (!image(a[0], at::kHalf, 2, i) || !image(a[1], at::kFloat, 2, o) || i.h != o.h || i.w != o.w || !bytes(a[2], true, ws, size)) Py_RETURN_FALSE;
        return made("hb_sat2d", [&](hb_stream st) { return g_lib.hb_sat2d(h(i.p), f(o.p), i.h, i.w, i.pitch, o.pitch, ws, size, st); });
    });
}

PyObject* conv3x3(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded<3>(n, [&]() -> PyObject* {
        const at::Tensor* t[3];
        for (int i = 0; i < 3; ++i) {
            t[i] = plain(a[i]);
            if (!t[i] || t[i]->scalar_type() != at::kHalf || !t[i]->is_contiguous() || t[i]->dim() != 4) Py_RETURN_FALSE;
            for (int64_t v : t[i]->sizes())
                if (v > kMostInt) Py_RETURN_FALSE;
        }
        const auto x = t[0]->sizes(), w = t[1]->sizes(), o = t[2]->sizes();
        if (w[0] != 3 || w[1] != 3 || w[2] != x[3] || o[0] != x[0] || o[1] != x[1] || o[2] != x[2] || o[3] != w[3]) Py_RETURN_FALSE;
        void *px = t[0]->data_ptr(), *pw = t[1]->data_ptr(), *po = t[2]->data_ptr();
        const int N = (int)x[0], H = (int)x[1], W = (int)x[2], ci = (int)x[3], co = (int)w[3];
        return made("hb_conv3x3", [&](hb_stream st) { return g_lib.hb_conv3x3(h(px), h(pw), h(po), N, H, W, ci, co, st); });
    });
}

PyObject* pyr_level(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded<3>(n, [&]() -> PyObject* {
        Image i, r, d{};
        if (!image(a[0], at::kHalf, 2, i) || !image(a[1], at::kFloat, 2, r) || i.h != r.h || i.w != r.w) Py_RETURN_FALSE;
        if (a[2] != Py_None && (!image(a[2], at::kHalf, 2, d) || d.h != i.h / 2 || d.w != i.w / 2)) Py_RETURN_FALSE;
        return made("hb_pyr_level", [&](hb_stream st) { return g_lib.hb_pyr_level(h(i.p), f(r.p), h(d.p), i.h, i.w, i.pitch, r.pitch, d.pitch, st); });
    });
}

PyObject* resize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded<7>(n, [&]() -> PyObject* {
        Image i, o;
        Banded y, x;
        void* ws;
        size_t size;
        if (!image(a[0], at::kHalf, 3, i) || !image(a[1], at::kFloat, 3, o) || i.planes != o.planes || !bytes(a[2], false, ws, size) ||
            !banded(a[3], a[4], o.h, y) || !banded(a[5], a[6], o.w, x)) Py_RETURN_FALSE;
        return made("hb_resize", [&](hb_stream st) {
            return g_lib.hb_resize(h(i.p), f(o.p), ws, size, i.planes, i.h, i.w, o.h, o.w, i.pitch, i.plane, o.pitch, o.plane,
                                   y.start, y.coef, y.band, x.start, x.coef, x.band, st);
        });
    });
}

PyObject* iir2(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded<5>(n, [&]() -> PyObject* {
        const at::Tensor *i = plain(a[0]), *o = plain(a[1]);              // rows of any length: no image
        float alpha, beta;
        void* ws;
        size_t size;
        if (!i || !o || i->dim() != 2 || o->dim() != 2 || i->scalar_type() != at::kHalf || o->scalar_type() != at::kFloat || i->sizes() != o->sizes() ||
            i->stride(1) != 1 || o->stride(1) != 1 || i->size(0) > kMostInt || !real(a[2], alpha) || !real(a[3], beta) || !bytes(a[4], false, ws, size)) Py_RETURN_FALSE;
        void *pi = i->data_ptr(), *po = o->data_ptr();
        const int C = (int)i->size(0);
        const int64_t T = i->size(1), ip = i->stride(0), op = o->stride(0);
        return made("hb_iir2", [&](hb_stream st) { return g_lib.hb_iir2(h(pi), f(po), C, T, ip, op, alpha, beta, ws, size, st); });
    });
}

PyObject* dct_denoise(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded<4>(n, [&]() -> PyObject* {
        Image i, o;
        float threshold;
        void* ws;
        size_t size;
        if (!image(a[0], at::kHalf, 3, i) || !image(a[1], at::kFloat, 3, o) || i.planes != o.planes || i.h != o.h || i.w != o.w || !real(a[2], threshold) ||
            !bytes(a[3], false, ws, size)) Py_RETURN_FALSE;
        return made("hb_dct_denoise", [&](hb_stream st) {
            return g_lib.hb_dct_denoise(h(i.p), f(o.p), i.planes, i.h, i.w, i.pitch, i.plane, o.pitch, o.plane, threshold, ws, size, st);
        });
    });
}

// bind({entry point: address}, error class): what load() found.
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 2 || !PyDict_Check(a[0])) {
        PyErr_SetString(PyExc_TypeError, "bind(addresses, error)");
        return nullptr;
    }
    Library lib;
#define HB_BIND(name)                                                                                                   \
    {                                                                                                                   \
        PyObject* v = PyDict_GetItemString(a[0], #name);                                                                \
        void* p = v ? PyLong_AsVoidPtr(v) : nullptr;                                                                    \
        if (!p) {                                                                                                       \
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name);                                              \
            return nullptr;                                                                                             \
        }                                                                                                               \
        lib.name = reinterpret_cast<decltype(lib.name)>(p);                                                             \
    }
    HB_CALLS(HB_BIND)
#undef HB_BIND
    g_lib = lib;
    Py_INCREF(a[1]);
    g_error = a[1];
    Py_RETURN_NONE;
}

#define HB_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HB_METHOD(bind), HB_METHOD(fir1d), HB_METHOD(conv2d), HB_METHOD(down2), HB_METHOD(up2), HB_METHOD(sepblur), HB_METHOD(sat2d),
                         HB_METHOD(conv3x3), HB_METHOD(pyr_level), HB_METHOD(resize), HB_METHOD(iir2), HB_METHOD(dct_denoise), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
    // the objects that it looks into are those of the torch it was built with
    PyObject* torch = PyImport_ImportModule("torch.version");
    PyObject* version = torch ? PyObject_GetAttrString(torch, "__version__") : nullptr;
    const char* v = version ? PyUnicode_AsUTF8(version) : nullptr;
    if (!v) return nullptr;
    if (strcmp(v, HB_TORCH_VERSION) != 0) {
        PyErr_Format(PyExc_ImportError, "built with torch " HB_TORCH_VERSION ", this is %s", v);
        return nullptr;
    }
    PyObject* numpy = PyImport_ImportModule("numpy");
    PyObject* type = numpy ? PyObject_GetAttrString(numpy, "ndarray") : nullptr;
    if (!type) return nullptr;
    g_ndarray = reinterpret_cast<PyTypeObject*>(type);
    pthread_atfork(nullptr, nullptr, [] { g_forked = true; });
    return PyModule_Create(&module);
}
