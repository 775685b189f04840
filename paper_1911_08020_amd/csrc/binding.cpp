// The per-token calls of the Python package, marshalled in native code: the products, the
// encode and the conversions take 3 to 7 us on the GPU, and checking the tensors, fetching
// the current stream and the foreign-function call took 9.7 us of Python per call (4.2 us
// now, of which the launch is about 3).
//
// Each function does its method's own checks on plain tensors and makes the call.  For
// whatever it does not take as it is (a tensor subclass, a wrong type, shape or device, a
// missing buffer that is not simply allocated) it returns None and has done nothing; the
// method's Python code then takes the call, or raises the error that names what is wrong.
// A failing library call raises through the package's own check.  Nothing is kept between
// calls.
#include <Python.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <new>

#include "darb.h"

namespace {

struct PlanRef {
    darb_plan *plan;
    int64_t M, N, nnz, words;
};

const char kPlanName[] = "darb_plan";
PyObject *g_check = nullptr;             // the package's _check(code, where)
PyObject *g_stream_attr = nullptr;       // "cuda_stream"

void free_ref(PyObject *cap) {
    delete static_cast<PlanRef *>(PyCapsule_GetPointer(cap, kPlanName));
}

const PlanRef *plan_of(PyObject *o) {
    return static_cast<const PlanRef *>(PyCapsule_GetPointer(o, kPlanName));
}

// A plain device tensor with memory of its own, or null.
const at::Tensor *tensor(PyObject *o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage()) return nullptr;
    return &t;
}

// A flat buffer of at least n elements of the given type.
const at::Tensor *buffer(PyObject *o, int64_t n, at::ScalarType type) {
    const at::Tensor *t = tensor(o);
    return t && t->scalar_type() == type && t->is_contiguous() && t->numel() >= n ? t : nullptr;
}

bool float_code(const at::Tensor &t, int *code) {
    if (t.scalar_type() == at::kFloat) *code = DARB_F32;
    else if (t.scalar_type() == at::kHalf) *code = DARB_F16;
    else return false;
    return true;
}

const at::Tensor *values_of(PyObject *o, int64_t nnz, int *code) {
    const at::Tensor *t = tensor(o);
    return t && float_code(*t, code) && t->is_contiguous() && t->numel() >= nnz ? t : nullptr;
}

// A [rows, cols] matrix of unit column stride: its leading dimension, or -1.
int64_t leading(const at::Tensor &t, int64_t rows, int64_t cols) {
    if (t.dim() != 2 || t.size(0) != rows || t.size(1) != cols || t.stride(1) != 1) return -1;
    return rows > 1 ? t.stride(0) : (cols > t.stride(0) ? cols : t.stride(0));
}

// The stream's handle: the current one of the current device for None.
bool stream_of(PyObject *o, void **s) {
    if (o == Py_None) {
        *s = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    PyObject *v = PyObject_GetAttr(o, g_stream_attr);
    if (v && PyLong_Check(v)) *s = PyLong_AsVoidPtr(v);
    const bool ok = v && PyLong_Check(v) && !PyErr_Occurred();
    Py_XDECREF(v);
    if (!ok) PyErr_Clear();
    return ok;
}

void *ptr(const at::Tensor &t) { return t.data_ptr(); }

PyObject *none() { Py_RETURN_NONE; }

// The call with the interpreter lock released (as a foreign-function call does), then the
// result, or the package's error.
template <typename F> PyObject *finish(PyObject *result, const char *where, F &&call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    if (rc == DARB_OK) return result;
    Py_DECREF(result);
    PyObject *r = PyObject_CallFunction(g_check, "is", rc, where);
    Py_XDECREF(r);
    if (r) PyErr_SetString(PyExc_RuntimeError, where);
    return nullptr;
}

// Any C++ exception (a tensor without memory, an allocation that fails): the Python code
// takes the call and reports it.
template <typename F> PyObject *guarded(F &&f) {
    try {
        return f();
    } catch (...) {
        if (PyErr_Occurred()) PyErr_Clear();
        return none();
    }
}

// y [M] as given, or a new one on x's device.
PyObject *vector_out(PyObject *o, const PlanRef &p, const at::Tensor &x, at::Tensor *out) {
    if (o == Py_None) {
        *out = at::empty({p.M}, x.options().dtype(at::kFloat));
        return THPVariable_Wrap(*out);
    }
    const at::Tensor *y = buffer(o, p.M, at::kFloat);
    if (!y) return nullptr;
    *out = *y;
    Py_INCREF(o);
    return o;
}

PyObject *matrix_out(PyObject *o, const PlanRef &p, const at::Tensor &X, at::Tensor *out,
                     int64_t *ldy) {
    const int64_t B = X.size(1);
    if (o == Py_None) {
        *out = at::empty({p.M, B}, X.options().dtype(at::kFloat));
        *ldy = leading(*out, p.M, B);
        return THPVariable_Wrap(*out);
    }
    const at::Tensor *Y = tensor(o);
    if (!Y || Y->scalar_type() != at::kFloat) return nullptr;
    *ldy = leading(*Y, p.M, B);
    if (*ldy < 0) return nullptr;
    *out = *Y;
    Py_INCREF(o);
    return o;
}

// What a product multiplies by: values, or codes and scales; byte offsets, or packed words.
struct Format {
    const at::Tensor *values = nullptr, *scales = nullptr;
    const uint8_t *offsets = nullptr;
    const uint32_t *packed = nullptr;
    int code = 0;
};

bool offsets_of(PyObject *o, const PlanRef &p, Format *f) {
    const at::Tensor *t = buffer(o, p.nnz, at::kByte);
    if (t) f->offsets = static_cast<const uint8_t *>(ptr(*t));
    return t != nullptr;
}

bool packed_of(PyObject *o, const PlanRef &p, Format *f) {
    const at::Tensor *t = buffer(o, p.words, at::kInt);
    if (t) f->packed = static_cast<const uint32_t *>(ptr(*t));
    return t != nullptr;
}

template <typename F>
PyObject *vector_product(const PlanRef &p, PyObject *xo, PyObject *yo, PyObject *so,
                         const char *where, F &&call) {
    const at::Tensor *x = tensor(xo);
    int xcode;
    void *s;
    if (!x || !float_code(*x, &xcode) || x->dim() != 1 || x->size(0) != p.N ||
        !x->is_contiguous() || !stream_of(so, &s))
        return none();
    at::Tensor y;
    PyObject *res = vector_out(yo, p, *x, &y);
    if (!res) return none();
    const void *xp = ptr(*x);
    float *yp = static_cast<float *>(ptr(y));
    return finish(res, where, [&] { return call(xcode, xp, yp, s); });
}

template <typename F>
PyObject *matrix_product(const PlanRef &p, PyObject *xo, PyObject *yo, PyObject *so,
                         const char *where, F &&call) {
    const at::Tensor *X = tensor(xo);
    int xcode;
    void *s;
    if (!X || !float_code(*X, &xcode) || X->dim() != 2 || !stream_of(so, &s)) return none();
    const int64_t B = X->size(1), ldx = leading(*X, p.N, B);
    if (ldx < 0) return none();
    at::Tensor Y;
    int64_t ldy;
    PyObject *res = matrix_out(yo, p, *X, &Y, &ldy);
    if (!res) return none();
    const void *xp = ptr(*X);
    float *yp = static_cast<float *>(ptr(Y));
    return finish(res, where, [&] { return call(xcode, B, xp, ldx, yp, ldy, s); });
}

#define DARB_ARGS(N)                                                                        \
    if (n != (N)) return none();                                                            \
    const PlanRef *p = plan_of(a[0]);                                                       \
    if (!p) {                                                                               \
        PyErr_Clear();                                                                      \
        return none();                                                                      \
    }

// (plan, values, offsets, x, y, stream)
PyObject *spmv(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        DARB_ARGS(6)
        Format f;
        if (!(f.values = values_of(a[1], p->nnz, &f.code)) || !offsets_of(a[2], *p, &f)) return none();
        const void *v = ptr(*f.values);
        return vector_product(*p, a[3], a[4], a[5], "darb_spmv",
                              [&](int xc, const void *x, float *y, void *s) {
                                  return darb_spmv(p->plan, f.code, v, f.offsets, xc, x, y, s);
                              });
    });
}

PyObject *spmv_packed(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        DARB_ARGS(6)
        Format f;
        if (!(f.values = values_of(a[1], p->nnz, &f.code)) || !packed_of(a[2], *p, &f)) return none();
        const void *v = ptr(*f.values);
        return vector_product(*p, a[3], a[4], a[5], "darb_spmv_packed",
                              [&](int xc, const void *x, float *y, void *s) {
                                  return darb_spmv_packed(p->plan, f.code, v, f.packed, xc, x, y, s);
                              });
    });
}

// (plan, values, offsets, X, Y, stream)
PyObject *spmm(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        DARB_ARGS(6)
        Format f;
        if (!(f.values = values_of(a[1], p->nnz, &f.code)) || !offsets_of(a[2], *p, &f)) return none();
        const void *v = ptr(*f.values);
        return matrix_product(
            *p, a[3], a[4], a[5], "darb_spmm",
            [&](int xc, int64_t B, const void *X, int64_t ldx, float *Y, int64_t ldy, void *s) {
                return darb_spmm(p->plan, f.code, v, f.offsets, xc, B, X, ldx, Y, ldy, s);
            });
    });
}

PyObject *spmm_packed(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        DARB_ARGS(6)
        Format f;
        if (!(f.values = values_of(a[1], p->nnz, &f.code)) || !packed_of(a[2], *p, &f)) return none();
        const void *v = ptr(*f.values);
        return matrix_product(
            *p, a[3], a[4], a[5], "darb_spmm_packed",
            [&](int xc, int64_t B, const void *X, int64_t ldx, float *Y, int64_t ldy, void *s) {
                return darb_spmm_packed(p->plan, f.code, v, f.packed, xc, B, X, ldx, Y, ldy, s);
            });
    });
}

bool i8_format(PyObject *codes, PyObject *scales, PyObject *offsets, PyObject *packed,
               const PlanRef &p, Format *f) {
    f->values = buffer(codes, p.nnz, at::kChar);
    f->scales = buffer(scales, p.M, at::kFloat);
    if (!f->values || !f->scales || (offsets == Py_None) == (packed == Py_None)) return false;
    return offsets != Py_None ? offsets_of(offsets, p, f) : packed_of(packed, p, f);
}

// (plan, codes, scales, x, offsets, packed, y, stream)
PyObject *spmv_i8(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        DARB_ARGS(8)
        Format f;
        if (!i8_format(a[1], a[2], a[4], a[5], *p, &f)) return none();
        const int8_t *q = static_cast<const int8_t *>(ptr(*f.values));
        const float *sc = static_cast<const float *>(ptr(*f.scales));
        return vector_product(*p, a[3], a[6], a[7], "darb_spmv_i8",
                              [&](int xc, const void *x, float *y, void *s) {
                                  return darb_spmv_i8(p->plan, q, sc, f.offsets, f.packed, xc, x,
                                                      y, s);
                              });
    });
}

PyObject *spmm_i8(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        DARB_ARGS(8)
        Format f;
        if (!i8_format(a[1], a[2], a[4], a[5], *p, &f)) return none();
        const int8_t *q = static_cast<const int8_t *>(ptr(*f.values));
        const float *sc = static_cast<const float *>(ptr(*f.scales));
        return matrix_product(
            *p, a[3], a[6], a[7], "darb_spmm_i8",
            [&](int xc, int64_t B, const void *X, int64_t ldx, float *Y, int64_t ldy, void *s) {
                return darb_spmm_i8(p->plan, q, sc, f.offsets, f.packed, xc, B, X, ldx, Y, ldy, s);
            });
    });
}

// (plan, W, values, offsets, stream)
PyObject *encode(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        DARB_ARGS(5)
        const at::Tensor *W = tensor(a[1]);
        int wcode, vcode;
        void *s;
        if (!W || !float_code(*W, &wcode) || !stream_of(a[4], &s)) return none();
        const int64_t ldw = leading(*W, p->M, p->N);
        const at::Tensor *v = values_of(a[2], p->nnz, &vcode);
        const at::Tensor *o = buffer(a[3], p->nnz, at::kByte);
        if (ldw < 0 || !v || !o || vcode != wcode) return none();
        const void *wp = ptr(*W);
        void *vp = ptr(*v);
        uint8_t *op = static_cast<uint8_t *>(ptr(*o));
        PyObject *res = PyTuple_Pack(2, a[2], a[3]);
        if (!res) return nullptr;
        return finish(res, "darb_encode",
                      [&] { return darb_encode(p->plan, wcode, wp, ldw, vp, op, s); });
    });
}

// (handle, M, N, nnz, packed words): what the functions above take as the plan
PyObject *plan_ref(PyObject *, PyObject *args) {
    unsigned long long h;
    long long M, N, nnz, words;
    if (!PyArg_ParseTuple(args, "KLLLL", &h, &M, &N, &nnz, &words)) return nullptr;
    PlanRef *p = new (std::nothrow)
        PlanRef{reinterpret_cast<darb_plan *>(uintptr_t(h)), M, N, nnz, words};
    if (!p) return PyErr_NoMemory();
    PyObject *cap = PyCapsule_New(p, kPlanName, free_ref);
    if (!cap) delete p;
    return cap;
}

// The current stream of the current device.
PyObject *current_stream(PyObject *, PyObject *) {
    return guarded([]() -> PyObject * {
        return PyLong_FromVoidPtr(c10::hip::getCurrentHIPStream().stream());
    });
}

// The package's function that raises for an error code.
PyObject *set_check(PyObject *, PyObject *f) {
    Py_INCREF(f);
    Py_XSETREF(g_check, f);
    Py_RETURN_NONE;
}

#define DARB_FAST(F) {#F, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(F)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    DARB_FAST(spmv), DARB_FAST(spmv_packed), DARB_FAST(spmv_i8),
    DARB_FAST(spmm), DARB_FAST(spmm_packed), DARB_FAST(spmm_i8),
    DARB_FAST(encode),
    {"plan_ref", plan_ref, METH_VARARGS, nullptr},
    {"current_stream", current_stream, METH_NOARGS, nullptr},
    {"set_check", set_check, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_darbcall", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__darbcall() {
    g_stream_attr = PyUnicode_InternFromString("cuda_stream");
    return g_stream_attr ? PyModule_Create(&module) : nullptr;
}
