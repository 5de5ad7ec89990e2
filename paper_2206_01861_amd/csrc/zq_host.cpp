// The binding's calls on plain torch tensors: checks, output allocation and the call of the C entry point without the
// interpreter in between.  At the smallest sizes a call is host time: LayerNorm + quantizer and a 768x768 GeMM at 128
// tokens are 5.6 us on the GPU and 18.6 us issued call by call through ctypes.
//
// Each function returns None for anything but the plain case (another tensor class, type, shape or device, wrapped tensors);
// the caller then takes its ctypes path, which raises what is to be raised.  Errors of the library go to the callable that
// init() received.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/zq.h"

namespace {

struct {
    decltype(&zq_layernorm_quant_tokenwise) layernorm;
    decltype(&zq_gelu_quant_tokenwise) gelu;
    decltype(&zq_quantize_tokenwise) quantize;
    decltype(&zq_gemm_i8_dequant) gemm_i8;
    decltype(&zq_gemm_w4a8_dequant) gemm_w4;
    decltype(&zq_gemm_gelu_quant_tokenwise) gemm_gelu;
    decltype(&zq_gemm_w8a16_dequant) gemm_a16;
    decltype(&zq_quantize_weight_groupwise) weight;
} zq;
PyObject *check = nullptr;                     // raises for an error code

// A dense CUDA tensor whose memory is its own: no wrapper of a transform, no view that is resolved when it is read.
const at::Tensor *plain(PyObject *o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    static const c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::Functionalize,
                                              c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                              c10::DispatchKey::Batched, c10::DispatchKey::Conjugate,
                                              c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.layout() != at::kStrided || !t.has_storage() ||
        t.key_set().has_any(wrapped) || !t.is_contiguous())
        return nullptr;
    return &t;
}
// The same for an argument that may be None: false if it is neither.
bool plain_or_none(PyObject *o, at::ScalarType type, const at::Tensor **t) {
    *t = nullptr;
    if (o == Py_None) return true;
    return (*t = plain(o, type)) != nullptr;
}
bool matrix(const at::Tensor *t) { return t != nullptr && t->dim() == 2 && t->size(0) <= INT_MAX && t->size(1) <= INT_MAX; }
void *ptr(const at::Tensor *t) { return t != nullptr ? t->mutable_data_ptr() : nullptr; }
void *ptr(const at::Tensor &t) { return t.defined() ? t.mutable_data_ptr() : nullptr; }

at::Tensor empty(const at::Tensor &like, at::IntArrayRef size, at::ScalarType type) {
    return at::empty(size, like.options().dtype(type));
}
zq_stream stream() { return c10::hip::getCurrentHIPStream().stream(); }

// (tensor | None, ...), or what `check` raises
PyObject *result(zq_status st, std::initializer_list<at::Tensor *> outs) {
    if (st != ZQ_OK) {
        PyObject *r = PyObject_CallFunction(check, "i", (int)st);
        Py_XDECREF(r);
        if (r != nullptr) PyErr_SetString(PyExc_RuntimeError, "libzq error");
        return nullptr;
    }
    if (outs.size() == 1) return THPVariable_Wrap(std::move(**outs.begin()));
    PyObject *tuple = PyTuple_New((Py_ssize_t)outs.size());
    if (tuple == nullptr) return nullptr;
    Py_ssize_t i = 0;
    for (at::Tensor *t : outs) {
        PyObject *o = t->defined() ? THPVariable_Wrap(std::move(*t)) : Py_NewRef(Py_None);
        if (o == nullptr) {
            Py_DECREF(tuple);
            return nullptr;
        }
        PyTuple_SET_ITEM(tuple, i++, o);
    }
    return tuple;
}

// The tap of the row kernels: None, torch.float16 or torch.float32; false for anything else.
bool tap(PyObject *o, bool *want, int *code) {
    *want = o != Py_None;
    *code = 0;
    if (!*want) return true;
    if (!THPDtype_Check(o)) return false;
    const at::ScalarType type = reinterpret_cast<THPDtype *>(o)->scalar_type;
    *code = type == at::kFloat ? 1 : 0;
    return type == at::kFloat || type == at::kHalf;
}

#define ZQ_TAKEN(cond) \
    if (!(cond)) Py_RETURN_NONE

// layernorm(x, gamma, beta | None, eps, y_dtype) -> (xq, s_tok, y | None)
PyObject *layernorm(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    bool want;
    int code;
    const at::Tensor *beta;
    ZQ_TAKEN(n == 5 && PyFloat_Check(a[3]) && tap(a[4], &want, &code));
    const at::Tensor *x = plain(a[0], at::kHalf), *gamma = plain(a[1], at::kHalf);
    ZQ_TAKEN(matrix(x) && gamma != nullptr && plain_or_none(a[2], at::kHalf, &beta));
    const float eps = (float)PyFloat_AS_DOUBLE(a[3]);
    const int64_t M = x->size(0), K = x->size(1);
    at::Tensor xq, s, y;
    zq_status st;
    {
        pybind11::gil_scoped_release no_gil;
        xq = empty(*x, {M, K}, at::kChar);
        s = empty(*x, {M}, at::kFloat);
        if (want) y = empty(*x, {M, K}, code == 1 ? at::kFloat : at::kHalf);
        st = zq.layernorm(ptr(x), ptr(gamma), ptr(beta), eps, (int)M, (int)K, static_cast<int8_t *>(ptr(xq)),
                          static_cast<float *>(ptr(s)), ptr(y), code, stream());
    }
    return result(st, {&xq, &s, &y});
    END_HANDLE_TH_ERRORS
}

// gelu(h, bias | None, approx_tanh, y_dtype) -> (xq, s_tok, y | None)
PyObject *gelu(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    bool want;
    int code;
    const at::Tensor *bias;
    ZQ_TAKEN(n == 4 && PyBool_Check(a[2]) && tap(a[3], &want, &code));
    const at::Tensor *h = plain(a[0], at::kHalf);
    ZQ_TAKEN(matrix(h) && plain_or_none(a[1], at::kHalf, &bias));
    const int64_t M = h->size(0), N = h->size(1);
    at::Tensor xq, s, y;
    zq_status st;
    {
        pybind11::gil_scoped_release no_gil;
        xq = empty(*h, {M, N}, at::kChar);
        s = empty(*h, {M}, at::kFloat);
        if (want) y = empty(*h, {M, N}, code == 1 ? at::kFloat : at::kHalf);
        st = zq.gelu(ptr(h), ptr(bias), a[2] == Py_True, (int)M, (int)N, static_cast<int8_t *>(ptr(xq)),
                     static_cast<float *>(ptr(s)), ptr(y), code, stream());
    }
    return result(st, {&xq, &s, &y});
    END_HANDLE_TH_ERRORS
}

// quantize(x) -> (xq, s_tok)
PyObject *quantize(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    ZQ_TAKEN(n == 1);
    const at::Tensor *x = plain(a[0], at::kHalf);
    ZQ_TAKEN(matrix(x));
    const int64_t M = x->size(0), K = x->size(1);
    at::Tensor xq, s;
    zq_status st;
    {
        pybind11::gil_scoped_release no_gil;
        xq = empty(*x, {M, K}, at::kChar);
        s = empty(*x, {M}, at::kFloat);
        st = zq.quantize(ptr(x), (int)M, (int)K, static_cast<int8_t *>(ptr(xq)), static_cast<float *>(ptr(s)), stream());
    }
    return result(st, {&xq, &s});
    END_HANDLE_TH_ERRORS
}

// What every linear takes: weights [N, K] or packed [N, K/2], group scales, bias and workspace that fit the activations.
struct Linear {
    const at::Tensor *x, *wq, *s_w, *bias, *workspace;
    int64_t M, N, K;
    size_t ws_bytes() const { return workspace != nullptr ? (size_t)workspace->numel() : 0; }
    bool take(PyObject *x_, at::ScalarType xt, PyObject *wq_, int bits, PyObject *sw_, PyObject *bias_, PyObject *ws_) {
        x = plain(x_, xt);
        wq = plain(wq_, bits == 8 ? at::kChar : at::kByte);
        s_w = plain(sw_, at::kFloat);
        if (!matrix(x) || !matrix(wq) || s_w == nullptr || s_w->numel() > INT_MAX) return false;
        if (!plain_or_none(bias_, at::kHalf, &bias) || !plain_or_none(ws_, at::kByte, &workspace)) return false;
        M = x->size(0);
        K = x->size(1);
        N = wq->size(0);
        return wq->size(1) * (8 / bits) == K && (bias == nullptr || bias->numel() == N);
    }
};

// gemm(bits, xq, s_tok, wq, s_w, bias | None, requant, workspace | None) -> (out, None, out_q | None, out_s_tok | None)
PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    ZQ_TAKEN(n == 8 && PyLong_Check(a[0]) && PyBool_Check(a[6]));
    const int bits = PyLong_AsLong(a[0]) == 8 ? 8 : 4;
    const bool requant = a[6] == Py_True;
    Linear l;
    ZQ_TAKEN(l.take(a[1], at::kChar, a[3], bits, a[4], a[5], a[7]));
    const at::Tensor *s_tok = plain(a[2], at::kFloat);
    ZQ_TAKEN(s_tok != nullptr && s_tok->numel() == l.M);
    at::Tensor out, none, q, s;
    zq_status st;
    {
        pybind11::gil_scoped_release no_gil;
        out = empty(*l.x, {l.M, l.N}, at::kHalf);
        if (requant) {
            q = empty(*l.x, {l.M, l.N}, at::kChar);
            s = empty(*l.x, {l.M}, at::kFloat);
        }
        const auto *x = static_cast<const int8_t *>(ptr(l.x));
        const auto *stk = static_cast<const float *>(ptr(s_tok)), *sw = static_cast<const float *>(ptr(l.s_w));
        const int groups = (int)l.s_w->numel(), M = (int)l.M, N = (int)l.N, K = (int)l.K;
        auto *qp = static_cast<int8_t *>(ptr(q));
        auto *sp = static_cast<float *>(ptr(s));
        st = bits == 8 ? zq.gemm_i8(x, stk, static_cast<const int8_t *>(ptr(l.wq)), sw, groups, ptr(l.bias), M, N, K,
                                    ptr(out), nullptr, qp, sp, ptr(l.workspace), l.ws_bytes(), stream())
                       : zq.gemm_w4(x, stk, static_cast<const uint8_t *>(ptr(l.wq)), sw, groups, ptr(l.bias), M, N, K,
                                    ptr(out), nullptr, qp, sp, ptr(l.workspace), l.ws_bytes(), stream());
    }
    return result(st, {&out, &none, &q, &s});
    END_HANDLE_TH_ERRORS
}

// gemm_gelu(bits, xq, s_tok, wq, s_w, bias | None, approx_tanh, workspace | None, keep_g) -> (g | None, gq, s_tok)
PyObject *gemm_gelu(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    ZQ_TAKEN(n == 9 && PyLong_Check(a[0]) && PyBool_Check(a[6]) && PyBool_Check(a[8]));
    const int bits = PyLong_AsLong(a[0]) == 8 ? 8 : 4;
    const bool keep = a[8] == Py_True, tanh = a[6] == Py_True;
    Linear l;
    ZQ_TAKEN(l.take(a[1], at::kChar, a[3], bits, a[4], a[5], a[7]));
    const at::Tensor *s_tok = plain(a[2], at::kFloat);
    ZQ_TAKEN(s_tok != nullptr && s_tok->numel() == l.M);
    at::Tensor g, q, s;
    zq_status st;
    {
        pybind11::gil_scoped_release no_gil;
        if (keep) g = empty(*l.x, {l.M, l.N}, at::kHalf);
        q = empty(*l.x, {l.M, l.N}, at::kChar);
        s = empty(*l.x, {l.M}, at::kFloat);
        st = zq.gemm_gelu(static_cast<const int8_t *>(ptr(l.x)), static_cast<const float *>(ptr(s_tok)), ptr(l.wq), bits,
                          static_cast<const float *>(ptr(l.s_w)), (int)l.s_w->numel(), ptr(l.bias), tanh, (int)l.M, (int)l.N,
                          (int)l.K, ptr(g), static_cast<int8_t *>(ptr(q)), static_cast<float *>(ptr(s)), ptr(l.workspace),
                          l.ws_bytes(), stream());
    }
    return result(st, {&g, &q, &s});
    END_HANDLE_TH_ERRORS
}

// gemm_a16(x, wq, s_w, bias | None, workspace | None) -> out
PyObject *gemm_a16(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Linear l;
    ZQ_TAKEN(n == 5 && l.take(a[0], at::kHalf, a[1], 8, a[2], a[3], a[4]));
    at::Tensor out;
    zq_status st;
    {
        pybind11::gil_scoped_release no_gil;
        out = empty(*l.x, {l.M, l.N}, at::kHalf);
        st = zq.gemm_a16(ptr(l.x), static_cast<const int8_t *>(ptr(l.wq)), static_cast<const float *>(ptr(l.s_w)),
                         (int)l.s_w->numel(), ptr(l.bias), (int)l.M, (int)l.N, (int)l.K, ptr(out), ptr(l.workspace),
                         l.ws_bytes(), stream());
    }
    return result(st, {&out});
    END_HANDLE_TH_ERRORS
}

// weight(w, groups, bits) -> (wq, s_w)
PyObject *weight(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    ZQ_TAKEN(n == 3 && PyLong_CheckExact(a[1]) && PyLong_CheckExact(a[2]));
    const at::Tensor *w = plain(a[0], at::kHalf);
    int overflow = 0;
    const long groups = PyLong_AsLongAndOverflow(a[1], &overflow);
    ZQ_TAKEN(matrix(w) && overflow == 0 && groups > 0 && groups <= 65535);
    const long bits = PyLong_AsLongAndOverflow(a[2], &overflow);
    ZQ_TAKEN(overflow == 0 && (bits == 8 || bits == 4));
    const int64_t N = w->size(0), K = w->size(1);
    at::Tensor wq, s;
    zq_status st;
    {
        pybind11::gil_scoped_release no_gil;
        wq = empty(*w, {N, bits == 4 ? K / 2 : K}, bits == 4 ? at::kByte : at::kChar);
        s = empty(*w, {groups}, at::kFloat);
        st = zq.weight(ptr(w), (int)N, (int)K, (int)groups, (int)bits, ptr(wq), static_cast<float *>(ptr(s)), stream());
    }
    return result(st, {&wq, &s});
    END_HANDLE_TH_ERRORS
}

// init(check, addresses in the order of the members above)
PyObject *init(PyObject *, PyObject *args) {
    unsigned long long p[8];
    PyObject *c;
    if (!PyArg_ParseTuple(args, "OKKKKKKKK", &c, p, p + 1, p + 2, p + 3, p + 4, p + 5, p + 6, p + 7)) return nullptr;
    Py_INCREF(c);
    Py_XSETREF(check, c);
    zq.layernorm = reinterpret_cast<decltype(zq.layernorm)>(p[0]);
    zq.gelu = reinterpret_cast<decltype(zq.gelu)>(p[1]);
    zq.quantize = reinterpret_cast<decltype(zq.quantize)>(p[2]);
    zq.gemm_i8 = reinterpret_cast<decltype(zq.gemm_i8)>(p[3]);
    zq.gemm_w4 = reinterpret_cast<decltype(zq.gemm_w4)>(p[4]);
    zq.gemm_gelu = reinterpret_cast<decltype(zq.gemm_gelu)>(p[5]);
    zq.gemm_a16 = reinterpret_cast<decltype(zq.gemm_a16)>(p[6]);
    zq.weight = reinterpret_cast<decltype(zq.weight)>(p[7]);
    Py_RETURN_NONE;
}

#define ZQ_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"init", init, METH_VARARGS, nullptr}, ZQ_FAST(layernorm), ZQ_FAST(gelu), ZQ_FAST(quantize), ZQ_FAST(gemm),
    ZQ_FAST(gemm_gelu), ZQ_FAST(gemm_a16), ZQ_FAST(weight), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_zq_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__zq_host() { return PyModule_Create(&module); }
