// Native marshalling for binding.py: the checks, output allocations and C-ABI calls of the tensor helpers in
// one Python call each.  A small layer is bound by what the host does per launch: through ctypes and a dozen tensor
// attributes quant_act took 11.1 us, a GEMM call 11.6, quant_weight with its copy 14.8; here 5.3, 4.3 and 6.9.
//
// Every function returns None when a call is not of the plain form (exact torch tensors on one GPU, of the expected
// dtype, layout and shapes, outputs included; `out` absent or complete): binding.py then takes its Python path, which words
// the error or handles the unusual form.  Only calls that that path would accept are answered here, with the same results.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>

#include "../../include/jet.h"

namespace {

PyObject* g_error = nullptr;   // binding.JetError
PyObject* g_oom = nullptr;     // torch.OutOfMemoryError

constexpr int64_t kGroup = 128;

// nullptr unless obj is a torch.Tensor or Parameter itself on the GPU with dtype
const at::Tensor* plain(PyObject* obj, at::ScalarType dtype) {
    if (!THPVariable_CheckExact(obj)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(obj);
    return (t.is_cuda() && t.scalar_type() == dtype) ? &t : nullptr;
}
const at::Tensor* plain2d(PyObject* obj, at::ScalarType dtype) {
    const at::Tensor* t = plain(obj, dtype);
    return (t && t->dim() == 2 && t->is_contiguous()) ? t : nullptr;
}
// t may hold [rows, cols] densely from its start (binding.py's _need_rows): on like's device, contiguous, of the element
// size, with room, and with rows of `cols` unless it is flat
enum Kind { kCodes, kScales };
bool holds(const at::Tensor& t, Kind kind, int64_t rows, int64_t cols, const at::Tensor& like) {
    cols = std::max<int64_t>(cols, 1);
    return t.is_cuda() && t.device() == like.device() && t.is_contiguous() &&
           (kind == kCodes ? t.element_size() == 1 : t.scalar_type() == at::kFloat) && t.numel() >= rows * cols &&
           (t.dim() == 1 || (t.dim() > 1 && t.size(-1) == cols));
}
bool modes_active() { return at::impl::torch_function_mode_enabled(); }
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }
at::Tensor make(int64_t rows, int64_t cols, at::ScalarType dtype, const at::Tensor& like) {
    return at::empty({rows, cols}, at::TensorOptions().dtype(dtype).device(like.device()));
}
template <class T = uint8_t>
const T* in(const at::Tensor& t) { return static_cast<const T*>(t.const_data_ptr()); }
template <class T = uint8_t>
T* outp(const at::Tensor& t) { return static_cast<T*>(t.data_ptr()); }

// nullptr with JetError set when st is an error, else the new reference `result`
PyObject* finish(jet_status st, const char* where, PyObject* result) {
    if (st == JET_OK) return result;
    Py_XDECREF(result);
    PyObject* e = PyObject_CallFunction(g_error, "is", (int)st, where);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}
// C++ exceptions of the allocator and of torch do not cross into Python as such
template <class F>
PyObject* guarded(F&& f) {
    try {
        return f();
    } catch (const python_error&) {
        return nullptr;       // already set
    } catch (const c10::OutOfMemoryError& e) {
        PyErr_SetString(g_oom, e.what_without_backtrace());
    } catch (const c10::Error& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}
bool set_item(PyObject* d, const char* key, const at::Tensor& t) {
    PyObject* o = THPVariable_Wrap(t);
    if (!o) return false;
    const int r = PyDict_SetItemString(d, key, o);
    Py_DECREF(o);
    return r == 0;
}
// a pair of result tensors of a quantizer: new ones, or those of the caller's dict
struct Pair {
    at::Tensor q, s;
};
// codes [rows, cols] with scales [rows, cols / 128]; false: not of the plain form
bool take_pair(PyObject* out, const char* qk, const char* sk, int64_t rows, int64_t cols, const at::Tensor& like, Pair& p) {
    PyObject *q = PyDict_GetItemString(out, qk), *s = PyDict_GetItemString(out, sk);
    if (!q || !s || !THPVariable_CheckExact(q) || !THPVariable_CheckExact(s)) return false;
    p.q = THPVariable_Unpack(q);
    p.s = THPVariable_Unpack(s);
    return holds(p.q, kCodes, rows, cols, like) && holds(p.s, kScales, rows, cols / kGroup, like);
}
PyObject* dict_of(const Pair* row, const Pair* col) {
    PyObject* d = PyDict_New();
    if (!d) return nullptr;
    if ((row && !(set_item(d, "q_row", row->q) && set_item(d, "s_row", row->s))) ||
        (col && !(set_item(d, "q_colT", col->q) && set_item(d, "s_colT", col->s)))) {
        Py_DECREF(d);
        return nullptr;
    }
    return d;
}
PyObject* same_or(PyObject* out, const Pair* row, const Pair* col) {
    if (out == Py_None) return dict_of(row, col);
    Py_INCREF(out);
    return out;
}
bool args(Py_ssize_t have, Py_ssize_t want) {
    if (have == want) return true;
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return false;
}

// quant_act(x, x_scales | None, row, col, out | None)
PyObject* quant_act(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!args(n, 5)) return nullptr;
    return guarded([&]() -> PyObject* {
        const bool fp8 = a[1] != Py_None;
        const int row = PyObject_IsTrue(a[2]), col = PyObject_IsTrue(a[3]);
        if (row < 0 || col < 0) return nullptr;
        PyObject* out = a[4];
        const at::Tensor* x = plain2d(a[0], fp8 ? at::kByte : at::kBFloat16);
        const at::Tensor* xs_t = fp8 ? plain(a[1], at::kFloat) : nullptr;
        if (!x || (fp8 && !xs_t) || (out != Py_None && !PyDict_CheckExact(out)) || modes_active()) Py_RETURN_NONE;
        const int64_t M = x->size(0), K = x->size(1);
        if (fp8 && !holds(*xs_t, kScales, M, K / kGroup, *x)) Py_RETURN_NONE;
        Pair r, c;
        if (out != Py_None) {
            if ((row && !take_pair(out, "q_row", "s_row", M, K, *x, r)) || (col && !take_pair(out, "q_colT", "s_colT", K, M, *x, c)))
                Py_RETURN_NONE;
        } else {
            if (row) r = {make(M, K, at::kByte, *x), make(M, std::max<int64_t>(K / kGroup, 1), at::kFloat, *x)};
            if (col) c = {make(K, M, at::kByte, *x), make(K, std::max<int64_t>(M / kGroup, 1), at::kFloat, *x)};
        }
        const float* xs = fp8 ? in<float>(*xs_t) : nullptr;
        uint8_t *qr = row ? outp(r.q) : nullptr, *qc = col ? outp(c.q) : nullptr;
        float *sr = row ? outp<float>(r.s) : nullptr, *sc = col ? outp<float>(c.s) : nullptr;
        const void* xp = in(*x);
        void* st = stream();
        jet_status e;
        Py_BEGIN_ALLOW_THREADS
        e = jet_quant_act(xp, xs, fp8 ? JET_SRC_FP8_ROW : JET_SRC_BF16, M, K, qr, sr, qc, sc, st);
        Py_END_ALLOW_THREADS
        return finish(e, "jet_quant_act", e == JET_OK ? same_or(out, row ? &r : nullptr, col ? &c : nullptr) : nullptr);
    });
}

// out: None or a dict that holds the row pair
bool row_pair(PyObject* out, int64_t M, int64_t K, const at::Tensor& like, Pair& r) {
    if (out == Py_None) {
        r = {make(M, K, at::kByte, like), make(M, std::max<int64_t>(K / kGroup, 1), at::kFloat, like)};
        return true;
    }
    return PyDict_CheckExact(out) && take_pair(out, "q_row", "s_row", M, K, like, r);
}

// rmsnorm_quant(x, gamma, eps, out | None)
PyObject* rmsnorm_quant(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!args(n, 4)) return nullptr;
    return guarded([&]() -> PyObject* {
        const at::Tensor *x = plain2d(a[0], at::kBFloat16), *g = plain(a[1], at::kBFloat16);
        if (!x || !g || !PyFloat_CheckExact(a[2]) || modes_active()) Py_RETURN_NONE;
        const int64_t M = x->size(0), K = x->size(1);
        if (g->dim() != 1 || g->size(0) != K || !g->is_contiguous() || g->device() != x->device()) Py_RETURN_NONE;
        Pair r;
        if (!row_pair(a[3], M, K, *x, r)) Py_RETURN_NONE;
        const float eps = (float)PyFloat_AS_DOUBLE(a[2]);
        const void *xp = in(*x), *gp = in(*g);
        uint8_t* q = outp(r.q);
        float* s = outp<float>(r.s);
        void* st = stream();
        jet_status e;
        Py_BEGIN_ALLOW_THREADS
        e = jet_rmsnorm_quant(xp, gp, eps, M, K, q, s, st);
        Py_END_ALLOW_THREADS
        return finish(e, "jet_rmsnorm_quant", e == JET_OK ? same_or(a[3], &r, nullptr) : nullptr);
    });
}

// gate and up: bf16 [M, K] on one GPU, of unit column stride and one row stride
bool gate_up(PyObject* const* a, const at::Tensor*& g, const at::Tensor*& u) {
    g = plain(a[0], at::kBFloat16);
    u = plain(a[1], at::kBFloat16);
    return g && u && g->dim() == 2 && u->dim() == 2 && g->stride(1) == 1 && u->stride(1) == 1 &&
           g->sizes() == u->sizes() && g->stride(0) == u->stride(0) && g->device() == u->device();
}

// silu_mul_quant(gate, up, out | None)
PyObject* silu_mul_quant(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!args(n, 3)) return nullptr;
    return guarded([&]() -> PyObject* {
        const at::Tensor *g, *u;
        if (!gate_up(a, g, u) || modes_active()) Py_RETURN_NONE;
        const int64_t M = g->size(0), K = g->size(1), ld = g->stride(0);
        Pair r;
        if (!row_pair(a[2], M, K, *g, r)) Py_RETURN_NONE;
        const void *gp = in(*g), *up = in(*u);
        uint8_t* q = outp(r.q);
        float* s = outp<float>(r.s);
        void* st = stream();
        jet_status e;
        Py_BEGIN_ALLOW_THREADS
        e = jet_silu_mul_quant(gp, up, ld, M, K, q, s, st);
        Py_END_ALLOW_THREADS
        return finish(e, "jet_silu_mul_quant", e == JET_OK ? same_or(a[2], &r, nullptr) : nullptr);
    });
}

// silu_mul_bwd(gate, up, dh, out | None)
PyObject* silu_mul_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!args(n, 4)) return nullptr;
    return guarded([&]() -> PyObject* {
        const at::Tensor *g, *u, *dh = plain2d(a[2], at::kBFloat16);
        if (!gate_up(a, g, u) || !dh || dh->sizes() != g->sizes() || dh->device() != g->device() || modes_active()) Py_RETURN_NONE;
        const int64_t M = g->size(0), K = g->size(1), ld = g->stride(0);
        at::Tensor o;
        if (a[3] == Py_None) {
            o = make(M, 2 * K, at::kBFloat16, *g);
        } else {
            const at::Tensor* t = plain2d(a[3], at::kBFloat16);
            if (!t || t->size(0) != M || t->size(1) != 2 * K || t->device() != g->device()) Py_RETURN_NONE;
            o = *t;
        }
        const void *gp = in(*g), *up = in(*u), *dp = in(*dh);
        uint8_t* op = outp(o);
        void* st = stream();
        jet_status e;
        Py_BEGIN_ALLOW_THREADS
        e = jet_silu_mul_bwd(gp, up, ld, dp, M, K, op, op + 2 * K, 2 * K, st);
        Py_END_ALLOW_THREADS
        if (e != JET_OK) return finish(e, "jet_silu_mul_bwd", nullptr);
        if (a[3] == Py_None) return THPVariable_Wrap(o);
        Py_INCREF(a[3]);
        return a[3];
    });
}

// quant_weight(w, transposed, out | None); out: a tuple of 2 or 4 tensors
PyObject* quant_weight(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!args(n, 3)) return nullptr;
    return guarded([&]() -> PyObject* {
        const int transposed = PyObject_IsTrue(a[1]);
        if (transposed < 0) return nullptr;
        const at::Tensor* w = plain2d(a[0], at::kBFloat16);
        if (!w || modes_active()) Py_RETURN_NONE;
        const int64_t N = w->size(0), K = w->size(1);
        at::Tensor t[4];
        PyObject* o[4] = {nullptr, nullptr, nullptr, nullptr};
        int have = transposed ? 4 : 2;
        if (a[2] == Py_None) {
            t[0] = make(N, K, at::kByte, *w);
            t[1] = make(std::max<int64_t>(N / kGroup, 1), std::max<int64_t>(K / kGroup, 1), at::kFloat, *w);
            if (transposed) {
                t[2] = make(K, N, at::kByte, *w);
                t[3] = make(std::max<int64_t>(K / kGroup, 1), std::max<int64_t>(N / kGroup, 1), at::kFloat, *w);
            }
        } else {
            // the tuple says what is written, `transposed` what is returned
            if (!PyTuple_CheckExact(a[2])) Py_RETURN_NONE;
            have = (int)PyTuple_GET_SIZE(a[2]);
            if (have != 4 && !(have == 2 && !transposed)) Py_RETURN_NONE;
            for (int i = 0; i < have; ++i) {
                o[i] = PyTuple_GET_ITEM(a[2], i);
                if (!THPVariable_CheckExact(o[i])) Py_RETURN_NONE;
                t[i] = THPVariable_Unpack(o[i]);
            }
            if (!holds(t[0], kCodes, N, K, *w) || !holds(t[1], kScales, N / kGroup, K / kGroup, *w) ||
                (have == 4 && !(holds(t[2], kCodes, K, N, *w) && holds(t[3], kScales, K / kGroup, N / kGroup, *w))))
                Py_RETURN_NONE;
        }
        const void* wp = in(*w);
        uint8_t *q = outp(t[0]), *qT = have == 4 ? outp(t[2]) : nullptr;
        float *s = outp<float>(t[1]), *sT = have == 4 ? outp<float>(t[3]) : nullptr;
        void* st = stream();
        jet_status e;
        Py_BEGIN_ALLOW_THREADS
        e = jet_quant_weight(wp, N, K, q, s, qT, sT, st);
        Py_END_ALLOW_THREADS
        if (e != JET_OK) return finish(e, "jet_quant_weight", nullptr);
        const int ret = transposed ? 4 : 2;
        PyObject* r = PyTuple_New(ret);
        for (int i = 0; r && i < ret; ++i) {
            PyObject* v = o[i];
            if (v) Py_INCREF(v);
            else v = THPVariable_Wrap(t[i]);
            if (!v) {
                Py_DECREF(r);
                return nullptr;
            }
            PyTuple_SET_ITEM(r, i, v);
        }
        return r;
    });
}

// codes [rows, R] with scales [rows / per, R / 128]
bool operand(PyObject* qo, PyObject* so, int64_t per, const at::Tensor*& q, const at::Tensor*& s) {
    q = plain2d(qo, at::kByte);
    s = plain2d(so, at::kFloat);
    if (!q || !s) return false;
    const int64_t rows = q->size(0), R = q->size(1);
    return R % kGroup == 0 && rows % per == 0 && s->size(0) == rows / per && s->size(1) == R / kGroup && s->device() == q->device();
}

// gemm(kind, a, sa, b, sb, out | None): kind 0 FProp, 1 DGrad, 2 WGrad; OUT[i,j] = sum_r A[i,r] B[j,r]
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!args(n, 6)) return nullptr;
    return guarded([&]() -> PyObject* {
        const long kind = PyLong_AsLong(a[0]);
        if (kind == -1 && PyErr_Occurred()) return nullptr;
        const at::Tensor *qa, *sa, *qb, *sb;
        if (!operand(a[1], a[2], 1, qa, sa) || !operand(a[3], a[4], kind == 2 ? 1 : kGroup, qb, sb) || modes_active()) Py_RETURN_NONE;
        const int64_t I = qa->size(0), J = qb->size(0), R = qa->size(1);
        if (qb->size(1) != R || qa->device() != qb->device()) Py_RETURN_NONE;
        at::Tensor o;
        if (a[5] == Py_None) {
            o = make(I, J, at::kBFloat16, *qa);
        } else {
            const at::Tensor* t = plain2d(a[5], at::kBFloat16);
            if (!t || t->size(0) != I || t->size(1) != J || t->device() != qa->device()) Py_RETURN_NONE;
            o = *t;
        }
        const uint8_t *pa = in(*qa), *pb = in(*qb);
        const float *psa = in<float>(*sa), *psb = in<float>(*sb);
        void *po = outp(o), *st = stream();
        jet_status e;
        Py_BEGIN_ALLOW_THREADS
        e = kind == 0   ? jet_fp8_linear_fwd(pa, psa, pb, psb, po, I, J, R, st)
            : kind == 1 ? jet_fp8_linear_dgrad(pa, psa, pb, psb, po, I, R, J, st)
                        : jet_fp8_linear_wgrad(pa, psa, pb, psb, po, R, I, J, st);
        Py_END_ALLOW_THREADS
        if (e != JET_OK)
            return finish(e, kind == 0 ? "jet_fp8_linear_fwd" : kind == 1 ? "jet_fp8_linear_dgrad" : "jet_fp8_linear_wgrad", nullptr);
        if (a[5] == Py_None) return THPVariable_Wrap(o);
        Py_INCREF(a[5]);
        return a[5];
    });
}

// init(JetError, torch.OutOfMemoryError)
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (!args(n, 2)) return nullptr;
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    Py_XDECREF(g_error);
    Py_XDECREF(g_oom);
    g_error = a[0];
    g_oom = a[1];
    Py_RETURN_NONE;
}

#define JET_FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr
PyMethodDef kMethods[] = {{"init", JET_FAST(init)},
                          {"quant_act", JET_FAST(quant_act)},
                          {"rmsnorm_quant", JET_FAST(rmsnorm_quant)},
                          {"silu_mul_quant", JET_FAST(silu_mul_quant)},
                          {"silu_mul_bwd", JET_FAST(silu_mul_bwd)},
                          {"quant_weight", JET_FAST(quant_weight)},
                          {"gemm", JET_FAST(gemm)},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_jet_host", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__jet_host() { return PyModule_Create(&kModule); }
