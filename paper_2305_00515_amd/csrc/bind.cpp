// CPython binding of the calls that cost less on the GPU than in the
// interpreter: uint8 images one at a time (fixed, two-directional and run-time
// kernels) and one-shot batches of magnitudes.  A 512x512 magnitude takes the
// GPU 3.0 us and took its caller 10.4 us through ctypes: about 4 in checking
// the arguments and allocating the output, 2 in asking torch for its stream,
// 4 in ctypes and the launch; here the whole call takes 4.6.  (3x3 pair of
// 2160x3840: 10.6 -> 5.0; run-time kernels: 12.9 -> 5.7; 16 crops of 64..640 in
// one batch: 94 -> 19.)
//
// Each function of a call handles exact torch tensors in exactly the forms that the
// C entry points take.  For everything else -- another type, a wrong shape, a
// tensor subclass, a function mode, an allocation that fails -- it returns None
// before anything is launched and the caller takes its general path, which
// decides and words the error.  Nothing is kept between these calls.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/Functions.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include <cstdint>
#include <vector>

#define NPY_NO_DEPRECATED_API NPY_1_22_API_VERSION
#define NPY_TARGET_VERSION NPY_1_22_API_VERSION
#include "../../include/sobel4x5.h"
#include "host_arrays.hpp"

// The torch that this is built against: another one's C++ interface may differ.
#ifndef SOBEL4X5_TORCH
#define SOBEL4X5_TORCH "unknown"
#endif

namespace {

using U8 = int (*)(const uint8_t *, int32_t, int32_t, int64_t, int32_t, const sobel4x5_outputs *, void *);
using U8Op = int (*)(const uint8_t *, int32_t, int32_t, int64_t, int32_t, int32_t, const sobel4x5_outputs *, void *);
using U8Weighted = int (*)(const uint8_t *, int32_t, int32_t, int64_t, int32_t, const int32_t *,
                           const sobel4x5_outputs *, void *);
using Batched = int (*)(const sobel4x5_image *, int32_t, int32_t, void *);

// The library's entry points and torch's current-stream query, given once by init.
U8 g_u8;
U8Op g_u8_op;
U8Weighted g_weighted;
Batched g_batched;
PyObject *g_raw_stream;

// An int of the interpreter that fits int32 (no bool, no subclass).
bool small_int(PyObject *o, int32_t *v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(o, &over);
    if (over || x < INT32_MIN || x > INT32_MAX) return false;
    *v = static_cast<int32_t>(x);
    return true;
}

struct Rows {
    void *p;
    int64_t h, w, pitch;
};

// A GPU tensor of rows: 2-D, of this type, unit column stride, not empty.
bool rows_of(PyObject *o, at::ScalarType type, Rows *r, c10::Device *dev = nullptr)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || t.dim() != 2) return false;
    const auto n = t.sizes(), s = t.strides();
    if (n[0] < 1 || n[1] < 1 || n[0] > INT32_MAX || n[1] > INT32_MAX || (n[1] > 1 && s[1] != 1)) return false;
    *r = {t.data_ptr(), n[0], n[1], s[0] * static_cast<int64_t>(t.element_size())};
    if (dev) *dev = t.device();
    return true;
}

bool stream_of(const c10::Device &dev, void **st)
{
    PyObject *i = PyLong_FromLong(dev.index());
    if (!i) return false;
    PyObject *s = PyObject_CallOneArg(g_raw_stream, i);
    Py_DECREF(i);
    if (!s) return false;
    *st = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    return !PyErr_Occurred();
}

PyObject *new_rows(int64_t h, int64_t w, at::ScalarType type, const c10::Device &dev, Rows *r)
{
    at::Tensor t = at::empty({h, w}, at::TensorOptions().dtype(type).device(dev));
    *r = {t.data_ptr(), h, w, w * static_cast<int64_t>(t.element_size())};
    return THPVariable_Wrap(std::move(t));
}

// 100 int32 weights out of a C-contiguous int32 or int64 buffer.
bool weights_of(PyObject *o, int32_t *w)
{
    Py_buffer b;
    if (!PyObject_CheckBuffer(o)) return false;
    if (PyObject_GetBuffer(o, &b, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT)) return false;
    const char f = b.format && b.format[0] && !b.format[1] ? b.format[0] : 0;
    bool ok = false;
    if (b.itemsize == 4 && f == 'i' && b.len == 400) {
        ok = true;
        for (int i = 0; i < 100; ++i) {
            w[i] = static_cast<const int32_t *>(b.buf)[i];
            ok &= w[i] != INT32_MIN;
        }
    } else if (b.itemsize == 8 && f == 'l' && b.len == 800) {
        ok = true;
        for (int i = 0; i < 100; ++i) {
            const int64_t v = static_cast<const int64_t *>(b.buf)[i];
            ok &= v > INT32_MIN && v <= INT32_MAX;
            w[i] = static_cast<int32_t>(v);
        }
    }
    PyBuffer_Release(&b);
    return ok;
}

// Owns a reference.
struct Ref {
    PyObject *o = nullptr;
    Ref() = default;
    explicit Ref(PyObject *p) : o(p) {}
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
    ~Ref() { Py_XDECREF(o); }
    PyObject *take()
    {
        PyObject *p = o;
        o = nullptr;
        return p;
    }
};

// The interpreter's lock given up while the library runs, as ctypes does.
struct Unlocked {
    PyThreadState *s = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(s); }
};

bool out_size(const Rows &src, int32_t border, int r, int64_t *h, int64_t *w)
{
    const int64_t cut = border == SOBEL4X5_BORDER_VALID ? 2 * r : 0;
    *h = src.h - cut;
    *w = src.w - cut;
    return *h >= 1 && *w >= 1;
}

// (src, op or None, border, mag, want_mag, dir_type, dirs, weights or None)
// -> (mag, planes), a status, or None.
PyObject *u8_call(PyObject *const *a)
{
    PyObject *mag = a[3], *dirs = a[6];
    int32_t op = SOBEL4X5_OP_4DIR_5X5, border, dir_type, weights[100];
    if ((a[1] != Py_None && !small_int(a[1], &op)) || op < 0 || op > 2 || !small_int(a[2], &border) ||
        !small_int(a[5], &dir_type) || dir_type < 0 || dir_type > 2 || (a[4] != Py_True && a[4] != Py_False))
        return nullptr;
    if (a[7] != Py_None && !weights_of(a[7], weights)) return nullptr;
    Rows src, r;
    c10::Device dev(c10::kCPU);
    if (!rows_of(a[0], at::kByte, &src, &dev)) return nullptr;
    int64_t ho, wo;
    if (!out_size(src, border, op == SOBEL4X5_OP_2DIR_3X3 ? 1 : 2, &ho, &wo)) return nullptr;

    sobel4x5_outputs out{};
    Ref new_mag, new_dirs;
    if (mag != Py_None) {
        if (!rows_of(mag, at::kByte, &r) || r.h != ho || r.w != wo) return nullptr;
    } else if (a[4] == Py_True) {
        if (!(new_mag.o = new_rows(ho, wo, at::kByte, dev, &r))) return nullptr;
        mag = new_mag.o;
    }
    if (mag != Py_None) {
        out.mag = static_cast<uint8_t *>(r.p);
        out.mag_pitch = r.pitch;
    }
    if (dir_type != SOBEL4X5_DIR_NONE) {
        const at::ScalarType type = dir_type == SOBEL4X5_DIR_S16 ? at::kShort : at::kInt;
        const int n = op == SOBEL4X5_OP_4DIR_5X5 ? 4 : 2;
        if (dirs == Py_None) {
            if (!(new_dirs.o = PyList_New(n))) return nullptr;
            dirs = new_dirs.o;
            for (int i = 0; i < n; ++i) {
                PyObject *t = new_rows(ho, wo, type, dev, &r);
                if (!t) return nullptr;
                PyList_SET_ITEM(dirs, i, t);
                out.dir[i * (4 / n)] = r.p;
            }
            out.dir_pitch = r.pitch;
        } else {
            if (!PyList_CheckExact(dirs) && !PyTuple_CheckExact(dirs)) return nullptr;
            if (PySequence_Fast_GET_SIZE(dirs) != n) return nullptr;
            for (int i = 0; i < n; ++i) {
                if (!rows_of(PySequence_Fast_GET_ITEM(dirs, i), type, &r) || r.h != ho || r.w != wo) return nullptr;
                if (i && r.pitch != out.dir_pitch) return nullptr;
                out.dir[i * (4 / n)] = r.p;
                out.dir_pitch = r.pitch;
            }
        }
    } else {
        dirs = Py_None;
    }
    out.dir_type = dir_type;
    Ref res(PyTuple_Pack(2, mag, dirs));
    void *st;
    if (!res.o || !stream_of(dev, &st)) return nullptr;

    int rc;
    {
        Unlocked u;
        const uint8_t *p = static_cast<const uint8_t *>(src.p);
        const int32_t w = static_cast<int32_t>(src.w), h = static_cast<int32_t>(src.h);
        if (a[7] != Py_None)
            rc = g_weighted(p, w, h, src.pitch, border, weights, &out, st);
        else if (a[1] != Py_None)
            rc = g_u8_op(p, w, h, src.pitch, op, border, &out, st);
        else
            rc = g_u8(p, w, h, src.pitch, border, &out, st);
    }
    return rc == SOBEL4X5_OK ? res.take() : PyLong_FromLong(rc);
}

// (srcs, mags or None, border) -> (mags,), a status, or None.
PyObject *batched_call(PyObject *const *a)
{
    PyObject *mags = a[1];
    int32_t border;
    if ((!PyList_CheckExact(a[0]) && !PyTuple_CheckExact(a[0])) || !small_int(a[2], &border)) return nullptr;
    // Tuples of their own: an allocation below may run a finalizer, and that
    // any code, on the caller's lists.
    Ref srcs(PySequence_Tuple(a[0])), made, given;
    if (!srcs.o) return nullptr;
    const Py_ssize_t n = PyTuple_GET_SIZE(srcs.o);
    if (n < 1 || n > INT32_MAX) return nullptr;
    if (mags == Py_None) {
        if (!(made.o = PyList_New(n))) return nullptr;
        mags = made.o;
    } else {
        if (!PyList_CheckExact(mags) && !PyTuple_CheckExact(mags)) return nullptr;
        if (!(given.o = PySequence_Tuple(mags)) || PyTuple_GET_SIZE(given.o) != n) return nullptr;
    }
    std::vector<sobel4x5_image> imgs(static_cast<size_t>(n));
    c10::Device first(c10::kCPU);
    for (Py_ssize_t i = 0; i < n; ++i) {
        Rows s, m;
        c10::Device dev(c10::kCPU);
        int64_t ho, wo;
        if (!rows_of(PyTuple_GET_ITEM(srcs.o, i), at::kByte, &s, &dev)) return nullptr;
        if (!out_size(s, border, 2, &ho, &wo)) return nullptr;
        if (i == 0) first = dev;
        if (made.o) {
            PyObject *t = new_rows(ho, wo, at::kByte, dev, &m);
            if (!t) return nullptr;
            PyList_SET_ITEM(mags, i, t);
        } else if (!rows_of(PyTuple_GET_ITEM(given.o, i), at::kByte, &m) || m.h != ho || m.w != wo) {
            return nullptr;
        }
        imgs[i] = {static_cast<const uint8_t *>(s.p), static_cast<uint8_t *>(m.p), static_cast<int32_t>(s.w),
                   static_cast<int32_t>(s.h), s.pitch, m.pitch};
    }
    Ref res(PyTuple_Pack(1, mags));
    void *st;
    if (!res.o || !stream_of(first, &st)) return nullptr;
    int rc;
    {
        Unlocked u;
        rc = g_batched(imgs.data(), static_cast<int32_t>(n), border, st);
    }
    return rc == SOBEL4X5_OK ? res.take() : PyLong_FromLong(rc);
}

template <int N, PyObject *(*CALL)(PyObject *const *)>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    PyObject *r = nullptr;
    if (g_raw_stream && !at::impl::torch_function_mode_enabled()) {
        try {
            r = CALL(args);
        } catch (...) {   // an allocation, a tensor without storage: the general path words it
        }
    }
    if (r) return r;
    PyErr_Clear();
    Py_RETURN_NONE;
}

// (sobel4x5_u8, sobel4x5_u8_op, sobel4x5_u8_weighted, sobel4x5_batched as
// addresses, torch's raw current-stream query)
PyObject *init(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "expected 5 arguments");
        return nullptr;
    }
    void *p[4];
    for (int i = 0; i < 4; ++i)
        if (!(p[i] = PyLong_AsVoidPtr(args[i]))) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no address");
            return nullptr;
        }
    g_u8 = reinterpret_cast<U8>(p[0]);
    g_u8_op = reinterpret_cast<U8Op>(p[1]);
    g_weighted = reinterpret_cast<U8Weighted>(p[2]);
    g_batched = reinterpret_cast<Batched>(p[3]);
    Py_INCREF(args[4]);
    Py_XSETREF(g_raw_stream, args[4]);
    Py_RETURN_NONE;
}

template <class F>
PyCFunction fast(F f)
{
    return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f));
}

PyMethodDef methods[] = {
    {"init", fast(init), METH_FASTCALL, nullptr},
    {"u8", fast(entry<8, u8_call>), METH_FASTCALL, nullptr},
    {"batched", fast(entry<3, batched_call>), METH_FASTCALL, nullptr},
    {"host_pool", host_pool, METH_NOARGS, nullptr},
    {"host_array", fast(host_array), METH_FASTCALL, nullptr},
    {"host_bytes", host_bytes, METH_O, nullptr},
    {"host_close", host_close, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind()
{
    if (PyArray_ImportNumPyAPI() < 0) return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddObject(m, "built_for",
                                PyUnicode_FromFormat("torch %s, Python %d.%d", SOBEL4X5_TORCH, PY_MAJOR_VERSION,
                                                     PY_MINOR_VERSION)) < 0)
        Py_CLEAR(m);
    return m;
}
