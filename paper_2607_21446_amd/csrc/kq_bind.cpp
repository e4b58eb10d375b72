// Native argument marshalling of the Python binding for the calls a serving or
// calibration loop repeats.  Each function takes the Python call's arguments and
// either makes the library call and returns its result, or returns None when an
// argument is not of the plain form checked here (another type, device, layout,
// size or stream object, a tensor without storage) or the library refuses the call:
// binding.py then runs its own checks and raises what they say.  A call that fails
// after that (KQ_ERROR_HIP) may have been enqueued, so it is not made again: its
// error is raised here.  A small call's time is the host's: 9.5 us through Python
// checks and ctypes for a kernel of 2.8.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>

#include "kroquant.h"

namespace {

constexpr int64_t kPackBytes = KQ_PACK_BYTES_PER_FACTOR;

// A plain torch.Tensor (or Parameter), not a subclass; null otherwise.
const at::Tensor* tensor(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

bool dense(const at::Tensor* t, at::ScalarType dtype) {
    return t && t->scalar_type() == dtype && t->is_cuda() && t->is_contiguous();
}
bool matrix(const at::Tensor* t, at::ScalarType dtype) { return dense(t, dtype) && t->dim() == 2; }
// A contiguous tensor of exactly n elements on dev.
bool buffer(const at::Tensor* t, at::ScalarType dtype, int64_t n, at::Device dev) {
    return dense(t, dtype) && t->numel() == n && t->device() == dev;
}

bool stream_of(PyObject* o, void** st) {
    if (o == Py_None) {
        *st = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    if (!PyLong_CheckExact(o)) return false;
    *st = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

bool flag(PyObject* o, bool* v) {
    if (!PyBool_Check(o)) return false;
    *v = o == Py_True;
    return true;
}

at::Tensor empty(at::IntArrayRef shape, at::ScalarType dtype, at::Device dev) {
    return at::empty(shape, at::TensorOptions().dtype(dtype).device(dev));
}

// An output: the caller's buffer, a new one, or (optional and not wanted) none.
struct Out {
    PyObject* given = nullptr;  // borrowed
    at::Tensor made;
    void* ptr = nullptr;
    PyObject* take() {  // new reference
        if (given) {
            Py_INCREF(given);
            return given;
        }
        if (made.defined()) return THPVariable_Wrap(std::move(made));
        Py_RETURN_NONE;
    }
};

bool output(PyObject* o, bool want, at::IntArrayRef shape, at::ScalarType dtype, int64_t n, at::Device dev, Out& out) {
    if (o != Py_None) {
        const at::Tensor* t = tensor(o);
        if (!buffer(t, dtype, n, dev)) return false;
        out.given = o;
        out.ptr = t->data_ptr();
    } else if (want) {
        out.made = empty(shape, dtype, dev);
        out.ptr = out.made.data_ptr();
    }
    return true;
}

// A call that the HIP runtime reported an error of.
struct Failed {
    kq_status status;
    const char* name;
};

// True if the call was made, false if the library refused its arguments.
template <class F>
bool call(const char* name, F f) {
    kq_status st;
    Py_BEGIN_ALLOW_THREADS;
    st = f();
    Py_END_ALLOW_THREADS;
    if (st == KQ_ERROR_HIP) throw Failed{st, name};
    return st == KQ_SUCCESS;
}

// Sets the binding's KQError.
PyObject* raise(const Failed& e) {
    PyObject* const m = PyImport_ImportModule("paper_2607_21446_amd.binding");
    PyObject* const cls = m ? PyObject_GetAttrString(m, "KQError") : nullptr;
    PyObject* const err = cls ? PyObject_CallFunction(cls, "iss", (int)e.status, kq_last_error_detail(), e.name) : nullptr;
    if (err) PyErr_SetObject(cls, err);
    Py_XDECREF(err);
    Py_XDECREF(cls);
    Py_XDECREF(m);
    return nullptr;
}

// Everything a function does runs in here: an exception of a tensor call means an
// argument that Python shall deal with.
template <class F>
PyObject* guarded(F f) {
    try {
        PyObject* r = f();
        if (r) return r;
    } catch (const Failed& e) {
        return raise(e);
    } catch (...) {
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}

struct Quant {
    const at::Tensor* X;
    int64_t M, d;
    Out codes, scales, y;
    void* stream;
    // X, and the outputs' and stream arguments
    bool parse(PyObject* x, PyObject* c, PyObject* s, PyObject* yo, PyObject* want_y, PyObject* st) {
        X = tensor(x);
        if (!matrix(X, at::kBFloat16)) return false;
        M = X->size(0);
        d = X->size(1);
        const at::Device dev = X->device();
        bool want = false;
        if (want_y && !flag(want_y, &want)) return false;
        return stream_of(st, &stream) && output(c, true, {M, d / 2}, at::kByte, M * (d / 2), dev, codes) &&
               output(s, true, {M, d / 32}, at::kByte, M * (d / 32), dev, scales) &&
               (!yo || output(yo, want, {M, d}, at::kFloat, M * d, dev, y));
    }
    const uint16_t* x() const { return static_cast<const uint16_t*>(X->data_ptr()); }
    uint8_t* c() const { return static_cast<uint8_t*>(codes.ptr); }
    uint8_t* s() const { return static_cast<uint8_t*>(scales.ptr); }
    float* yp() const { return static_cast<float*>(y.ptr); }
    PyObject* result(bool with_y, Out* more = nullptr) {
        const int n = 2 + (with_y ? 1 : 0) + (more ? 1 : 0);
        PyObject* t = PyTuple_New(n);
        if (!t) return nullptr;
        PyTuple_SET_ITEM(t, 0, codes.take());
        PyTuple_SET_ITEM(t, 1, scales.take());
        if (with_y) PyTuple_SET_ITEM(t, 2, y.take());
        if (more) PyTuple_SET_ITEM(t, n - 1, more->take());
        return t;
    }
};

struct Pairs {
    const float *A, *B;
    int64_t a, b, nfac;
    bool parse(PyObject* pa, PyObject* pb, at::Device dev) {
        const at::Tensor *ta = tensor(pa), *tb = tensor(pb);
        if (!dense(ta, at::kFloat) || !dense(tb, at::kFloat) || ta->device() != dev || tb->device() != dev) return false;
        if (ta->dim() < 2 || tb->dim() < 2) return false;
        a = ta->size(-1);
        b = tb->size(-1);
        if (ta->size(-2) != a || tb->size(-2) != b || a < 1 || a > 32 || b < 1 || b > 32) return false;
        nfac = ta->numel() / (a * a);
        A = static_cast<const float*>(ta->data_ptr());
        B = static_cast<const float*>(tb->data_ptr());
        return tb->numel() == nfac * b * b;
    }
};

// (X, A, B, codes, scales, y, want_y, stream)
template <class F>
PyObject* kron(const char* name, PyObject* const* v, Py_ssize_t n, F f) {
    if (n != 8) Py_RETURN_NONE;
    return guarded([&]() -> PyObject* {
        Quant q;
        Pairs p;
        if (!q.parse(v[0], v[3], v[4], v[5], v[6], v[7]) || !p.parse(v[1], v[2], q.X->device())) return nullptr;
        if (!call(name, [&] {
                return f(q.x(), q.M, q.d, p.A, p.B, (int)p.a, (int)p.b, p.nfac, q.c(), q.s(), q.yp(), q.stream);
            }))
            return nullptr;
        return q.result(true);
    });
}

PyObject* quantize(PyObject*, PyObject* const* v, Py_ssize_t n) { return kron("kq_quantize", v, n, kq_quantize); }
PyObject* quantize_exact(PyObject*, PyObject* const* v, Py_ssize_t n) { return kron("kq_quantize_exact", v, n, kq_quantize_exact); }

// (X, A, B, kpack, codes, scales, y, want_y, stream)
PyObject* quantize_packed(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (n != 9) Py_RETURN_NONE;
    return guarded([&]() -> PyObject* {
        Quant q;
        Pairs p;
        if (!q.parse(v[0], v[4], v[5], v[6], v[7], v[8]) || !p.parse(v[1], v[2], q.X->device())) return nullptr;
        const at::Tensor* k = tensor(v[3]);
        if (!buffer(k, at::kByte, p.nfac * kPackBytes, q.X->device())) return nullptr;
        if (!call("kq_quantize_packed", [&] {
                return kq_quantize_packed(q.x(), q.M, q.d, p.A, p.B, (int)p.a, (int)p.b, p.nfac, k->data_ptr(), q.c(),
                                          q.s(), q.yp(), q.stream);
            }))
            return nullptr;
        return q.result(true);
    });
}

// (X, lu, a, codes, scales, y, y16, want_y, want_y16, stream)
PyObject* quantize_lu(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (n != 10) Py_RETURN_NONE;
    return guarded([&]() -> PyObject* {
        Quant q;
        Out y16;
        bool want16 = false;
        if (!q.parse(v[0], v[3], v[4], v[5], v[7], v[9]) || !flag(v[8], &want16) || !PyLong_CheckExact(v[2])) return nullptr;
        const long a = PyLong_AsLong(v[2]);
        const at::Tensor* lu = tensor(v[1]);
        if (a < 1 || a > 32 || !dense(lu, at::kFloat) || lu->device() != q.X->device()) return nullptr;
        if (lu->numel() == 0 || lu->numel() % 15) return nullptr;
        if (!output(v[6], want16, {q.M, q.d}, at::kBFloat16, q.M * q.d, q.X->device(), y16)) return nullptr;
        if (!call("kq_quantize_lu", [&] {
                return kq_quantize_lu(q.x(), q.M, q.d, static_cast<const float*>(lu->data_ptr()), (int)a,
                                      lu->numel() / 15, q.c(), q.s(), q.yp(), static_cast<uint16_t*>(y16.ptr), q.stream);
            }))
            return nullptr;
        return q.result(true, &y16);
    });
}

// (X, mult, codes, scales, y, want_y, stream)
PyObject* smoothquant(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (n != 7) Py_RETURN_NONE;
    return guarded([&]() -> PyObject* {
        Quant q;
        if (!q.parse(v[0], v[2], v[3], v[4], v[5], v[6])) return nullptr;
        const at::Tensor* m = tensor(v[1]);
        if (!buffer(m, at::kFloat, q.d, q.X->device())) return nullptr;
        if (!call("kq_smoothquant_quantize", [&] {
                return kq_smoothquant_quantize(q.x(), q.M, q.d, static_cast<const float*>(m->data_ptr()), q.c(), q.s(),
                                               q.yp(), q.stream);
            }))
            return nullptr;
        return q.result(true);
    });
}

// (X, codes, scales, y, want_y, stream)
template <class F>
PyObject* plain(const char* name, PyObject* const* v, Py_ssize_t n, F f) {
    if (n != 6) Py_RETURN_NONE;
    return guarded([&]() -> PyObject* {
        Quant q;
        if (!q.parse(v[0], v[1], v[2], v[3], v[4], v[5])) return nullptr;
        if (!call(name, [&] { return f(q.x(), q.M, q.d, q.c(), q.s(), q.yp(), q.stream); })) return nullptr;
        return q.result(true);
    });
}

PyObject* hadamard32(PyObject*, PyObject* const* v, Py_ssize_t n) { return plain("kq_hadamard32_quantize", v, n, kq_hadamard32_quantize); }
PyObject* fwht(PyObject*, PyObject* const* v, Py_ssize_t n) { return plain("kq_fwht_quantize", v, n, kq_fwht_quantize); }

// (X, codes, scales, stream)
PyObject* mxfp4(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (n != 4) Py_RETURN_NONE;
    return guarded([&]() -> PyObject* {
        Quant q;
        if (!q.parse(v[0], v[1], v[2], nullptr, nullptr, v[3])) return nullptr;
        if (!call("kq_mxfp4_quantize", [&] { return kq_mxfp4_quantize(q.x(), q.M, q.d, q.c(), q.s(), q.stream); })) return nullptr;
        return q.result(false);
    });
}

// (a_codes, a_scales, b_codes, b_scales, C, accumulate, stream, out_dtype)
PyObject* mxfp4_gemm(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (n != 8) Py_RETURN_NONE;
    return guarded([&]() -> PyObject* {
        const at::Tensor* t[4];
        for (int i = 0; i < 4; ++i) {
            t[i] = tensor(v[i]);
            if (!matrix(t[i], at::kByte) || t[i]->device() != t[0]->device()) return nullptr;
        }
        const int64_t M = t[0]->size(0), N = t[2]->size(0), K = 2 * t[0]->size(1);
        if (2 * t[2]->size(1) != K || t[1]->size(0) != M || t[1]->size(1) != K / 32 || t[3]->size(0) != N ||
            t[3]->size(1) != K / 32)
            return nullptr;
        bool accumulate = false;
        void* st = nullptr;
        if (!flag(v[5], &accumulate) || !stream_of(v[6], &st)) return nullptr;
        at::ScalarType dtype = at::kFloat;
        Out C;
        if (v[4] != Py_None) {
            const at::Tensor* c = tensor(v[4]);
            if (!c || c->dim() != 2 || c->size(0) != M || c->size(1) != N) return nullptr;
            dtype = c->scalar_type();
        } else if (v[7] != Py_None) {
            if (!THPDtype_Check(v[7])) return nullptr;
            dtype = reinterpret_cast<THPDtype*>(v[7])->scalar_type;
        }
        if ((dtype != at::kFloat && dtype != at::kBFloat16) || (dtype == at::kBFloat16 && accumulate)) return nullptr;
        if (!output(v[4], true, {M, N}, dtype, M * N, t[0]->device(), C)) return nullptr;
        const int64_t ldc = (C.given ? *tensor(v[4]) : C.made).stride(0);
        const uint8_t* p[4];
        for (int i = 0; i < 4; ++i) p[i] = static_cast<const uint8_t*>(t[i]->data_ptr());
        if (!call(dtype == at::kFloat ? "kq_mxfp4_gemm" : "kq_mxfp4_gemm_bf16", [&] {
                return dtype == at::kFloat
                           ? kq_mxfp4_gemm(p[0], p[1], M, p[2], p[3], N, K, static_cast<float*>(C.ptr), ldc, accumulate, st)
                           : kq_mxfp4_gemm_bf16(p[0], p[1], M, p[2], p[3], N, K, static_cast<uint16_t*>(C.ptr), ldc, st);
            }))
            return nullptr;
        return C.take();
    });
}

// (X, W, Yneg, lu, lambdas, a, workspace, adam, grad, losses, stream); adam None only
PyObject* calib_step(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (n != 11) Py_RETURN_NONE;
    return guarded([&]() -> PyObject* {
        const at::Tensor *X = tensor(v[0]), *W = tensor(v[1]), *Y = tensor(v[2]), *lu = tensor(v[3]), *lam = tensor(v[4]),
                         *ws = tensor(v[6]);
        if (!matrix(X, at::kBFloat16) || !matrix(W, at::kBFloat16) || W->device() != X->device()) return nullptr;
        const int64_t R = X->size(0), d = X->size(1), o = W->size(0);
        const at::Device dev = X->device();
        if (W->size(1) != d || !buffer(Y, at::kFloat, R * o, dev) || !dense(lu, at::kFloat) || lu->device() != dev ||
            lu->numel() == 0 || lu->numel() % 15 || !buffer(lam, at::kFloat, 2, dev) || !dense(ws, at::kByte) ||
            v[7] != Py_None || !PyLong_CheckExact(v[5]))
            return nullptr;
        const long a = PyLong_AsLong(v[5]);
        const int64_t nfac = lu->numel() / 15;
        Out grad, losses;
        void* st = nullptr;
        if (a < 1 || a > 32 || !stream_of(v[10], &st) || !output(v[8], true, {nfac, 5, 3}, at::kFloat, nfac * 15, dev, grad) ||
            !output(v[9], true, {4}, at::kDouble, 4, dev, losses))
            return nullptr;
        if (!call("kq_calib_step", [&] {
                return kq_calib_step(static_cast<const uint16_t*>(X->data_ptr()), R, d,
                                     static_cast<const uint16_t*>(W->data_ptr()), o, static_cast<const float*>(Y->data_ptr()),
                                     static_cast<float*>(lu->data_ptr()), (int)a, nfac,
                                     static_cast<const float*>(lam->data_ptr()), static_cast<float*>(grad.ptr),
                                     static_cast<double*>(losses.ptr), nullptr, nullptr, 0, 0.0f, ws->data_ptr(),
                                     (size_t)ws->numel(), st);
            }))
            return nullptr;
        PyObject* r = PyTuple_New(2);
        if (!r) return nullptr;
        PyTuple_SET_ITEM(r, 0, losses.take());
        PyTuple_SET_ITEM(r, 1, grad.take());
        return r;
    });
}

#define KQ_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {KQ_METHOD(quantize),    KQ_METHOD(quantize_exact), KQ_METHOD(quantize_packed),
                          KQ_METHOD(quantize_lu), KQ_METHOD(smoothquant),    KQ_METHOD(hadamard32),
                          KQ_METHOD(fwht),        KQ_METHOD(mxfp4),          KQ_METHOD(mxfp4_gemm),
                          KQ_METHOD(calib_step),  {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_kqbind", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__kqbind() { return PyModule_Create(&kModule); }
