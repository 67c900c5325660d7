// Argument marshalling of the calls a serving loop makes eagerly, once per draft position and once per round
// (binding.py has the same in Python, which is the reference for what is accepted).  In Python the some forty
// attribute look-ups and the ctypes call of a draft step take about 10 us of host time, twice what its kernels run
// at small batches; here about 1 us.
//
// Every function returns the call's svip_status, or DECLINED without having done anything where an argument is not plainly
// right: the Python path then takes the call, or says what is wrong with it.  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/svip.h"

namespace {

constexpr long DECLINED = -1;
decltype(&svip_draft_step) g_draft_step;
decltype(&svip_draft_step_greedy) g_draft_step_greedy;
decltype(&svip_verify) g_verify;
decltype(&svip_verify_greedy) g_verify_greedy;

// A plain dense device tensor, or nullptr: no subclass, nothing wrapped by a transform (those have no pointer to give).
const at::Tensor *device_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    const c10::TensorImpl *impl = t.unsafeGetTensorImpl();
    const c10::DispatchKeySet keys = impl->key_set();
    constexpr c10::DispatchKeySet wrapped = c10::DispatchKeySet(
        {c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
         c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
         c10::DispatchKey::ZeroTensor});
    if (!keys.has_all(c10::DispatchKeySet(c10::DispatchKey::CUDA)) || keys.has_any(wrapped) || !impl->has_storage() ||
        impl->has_symbolic_sizes_strides())
        return nullptr;
    return &t;
}

int dtype_of(const at::Tensor &t)
{
    switch (t.scalar_type()) {
        case at::kFloat: return SVIP_F32;
        case at::kBFloat16: return SVIP_BF16;
        case at::kHalf: return SVIP_F16;
        default: return -1;
    }
}

// Reads arguments one after the other; `ok` turns false at the first that is not plainly right.
struct Args {
    PyObject *const *v;
    bool ok = true;
    int i = 0;

    const at::Tensor *logits(int dims, int *dtype)
    {
        const at::Tensor *t = device_tensor(v[i++]);
        if (!t || t->dim() != dims || t->stride(dims - 1) != 1 || (*dtype = dtype_of(*t)) < 0) {
            ok = false;
            return nullptr;
        }
        return t;
    }
    // [B], [B, k]: contiguous, of the given type; None (if optional) gives nullptr
    template <typename T>
    T *array(at::ScalarType type, bool optional, long long B, long long k = -1)
    {
        PyObject *o = v[i++];
        if (!ok) return nullptr;
        if (o == Py_None && optional) return nullptr;
        const at::Tensor *t = device_tensor(o);
        if (!t || t->scalar_type() != type || t->dim() != (k < 0 ? 1 : 2) || t->size(0) != B || (k >= 0 && t->size(1) != k) ||
            !t->is_contiguous()) {
            ok = false;
            return nullptr;
        }
        return static_cast<T *>(t->data_ptr());
    }
    // [B], possibly a column of a larger array; all of a call's share one stride (-1: none seen yet)
    template <typename T>
    T *column(at::ScalarType type, bool optional, long long B, long long *stride)
    {
        PyObject *o = v[i++];
        if (!ok) return nullptr;
        if (o == Py_None && optional) return nullptr;
        const at::Tensor *t = device_tensor(o);
        if (!t || t->scalar_type() != type || t->dim() != 1 || t->size(0) != B || (B > 1 && (t->stride(0) == 0 || (*stride >= 0 && t->stride(0) != *stride)))) {
            ok = false;
            return nullptr;
        }
        if (*stride < 0) *stride = B > 1 ? t->stride(0) : 1;
        return static_cast<T *>(t->data_ptr());
    }
    const at::Tensor *workspace()
    {
        const at::Tensor *t = device_tensor(v[i++]);
        if (!t || t->scalar_type() != at::kByte) ok = false;
        return t;
    }
    float real()
    {
        PyObject *o = v[i++];
        if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
        return (float)whole();
    }
    int whole(bool again = true)
    {
        PyObject *o = v[again ? i - 1 : i++];
        int over = 0;
        const long n = PyLong_CheckExact(o) ? PyLong_AsLongAndOverflow(o, &over) : 0;
        if (!PyLong_CheckExact(o) || over || n < INT32_MIN || n > INT32_MAX) ok = false;
        return (int)n;
    }
    void *stream()          // None: the current one; otherwise its handle
    {
        PyObject *o = v[i++];
        if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
        if (!PyLong_CheckExact(o)) {
            ok = false;
            return nullptr;
        }
        void *p = PyLong_AsVoidPtr(o);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            ok = false;
        }
        return p;
    }
};

bool fits(long long n) { return n >= 0 && n <= INT32_MAX; }

template <typename F>
PyObject *answer(F f)
{
    long status = DECLINED;
    try {
        status = f();
    } catch (const std::exception &) {       // (a tensor without a pointer to give)
        status = DECLINED;
    }
    return PyLong_FromLong(status);
}

// draft_step(draft_logits, temperature, h, step_j, k_max, u_sample or None for greedy, token_out, entropy_out, q_tok_out, lse_out,
//            stop_in, stop_out, draft_len_out, workspace, stream)
PyObject *draft_step(PyObject *, PyObject *const *argv, Py_ssize_t n)
{
    return answer([&]() -> long {
        if (n != 15) return DECLINED;
        Args a{argv};
        int dtype = -1;
        const at::Tensor *z = a.logits(2, &dtype);
        if (!a.ok) return DECLINED;
        const long long B = z->size(0), V = z->size(1), s0 = z->stride(0), row_stride = B > 1 ? s0 : (V > s0 ? V : s0);
        const float temperature = a.real(), h = a.real();
        const int step_j = a.whole(false), k_max = a.whole(false);
        const bool greedy = argv[5] == Py_None;
        long long stride = -1;
        const float *u = a.column<float>(at::kFloat, true, B, &stride);
        int *token = a.column<int>(at::kInt, false, B, &stride);
        float *entropy = a.column<float>(at::kFloat, true, B, &stride), *q_tok = a.column<float>(at::kFloat, true, B, &stride);
        double *lse = a.column<double>(at::kDouble, false, B, &stride);
        const unsigned char *stop_in = a.array<unsigned char>(at::kByte, true, B);
        unsigned char *stop_out = a.array<unsigned char>(at::kByte, false, B);
        int *draft_len = a.array<int>(at::kInt, true, B);
        const at::Tensor *ws = a.workspace();
        void *stream = a.stream();
        if (!a.ok || !fits(B) || !fits(V)) return DECLINED;
        const void *logits = z->data_ptr();
        void *wp = ws->data_ptr();
        const size_t wn = (size_t)ws->numel();
        long status;
        Py_BEGIN_ALLOW_THREADS
        status = greedy ? g_draft_step_greedy(logits, dtype, (int)B, (int)V, row_stride, temperature, h, step_j, k_max, stop_in, token, entropy,
                                              q_tok, lse, stop_out, draft_len, stride, wp, wn, stream)
                        : g_draft_step(logits, dtype, (int)B, (int)V, row_stride, temperature, h, step_j, k_max, u, stop_in, token, entropy,
                                       q_tok, lse, stop_out, draft_len, stride, wp, wn, stream);
        Py_END_ALLOW_THREADS
        return status;
    });
}

// verify(target_logits, draft_logits, temperature, draft_tokens, draft_len, draft_lse, u_accept, u_resample, n_accepted_out,
//        next_token_out, accept_prob_out, workspace, stream)
PyObject *verify(PyObject *, PyObject *const *argv, Py_ssize_t n)
{
    return answer([&]() -> long {
        if (n != 13) return DECLINED;
        Args a{argv};
        int dtype = -1, dtype_q = -1;
        const at::Tensor *p = a.logits(3, &dtype), *q = a.logits(3, &dtype_q);
        if (!a.ok || dtype != dtype_q) return DECLINED;
        const long long B = p->size(0), k = p->size(1) - 1, V = p->size(2), row_stride = p->stride(1);
        if (q->size(0) != B || q->size(1) != k || q->size(2) != V || (k > 1 && q->stride(1) != row_stride)) return DECLINED;
        const long long seq_t = B > 1 ? p->stride(0) : (k + 1) * row_stride, seq_d = B > 1 ? q->stride(0) : k * row_stride;
        const float temperature = a.real();
        const int *tokens = a.array<int>(at::kInt, false, B, k), *len = a.array<int>(at::kInt, false, B);
        const double *lse = a.array<double>(at::kDouble, true, B, k);
        const float *ua = a.array<float>(at::kFloat, false, B, k), *ur = a.array<float>(at::kFloat, false, B);
        int *nacc = a.array<int>(at::kInt, false, B), *next = a.array<int>(at::kInt, false, B);
        float *prob = a.array<float>(at::kFloat, true, B, k);
        const at::Tensor *ws = a.workspace();
        void *stream = a.stream();
        if (!a.ok || !fits(B) || !fits(k) || !fits(V)) return DECLINED;
        const void *pp = p->data_ptr(), *qp = q->data_ptr();
        void *wp = ws->data_ptr();
        const size_t wn = (size_t)ws->numel();
        long status;
        Py_BEGIN_ALLOW_THREADS
        status = g_verify(pp, qp, dtype, (int)B, (int)k, (int)V, seq_t, seq_d, row_stride, temperature, tokens, len, lse, ua, ur, nacc, next,
                          prob, wp, wn, stream);
        Py_END_ALLOW_THREADS
        return status;
    });
}

// verify_greedy(target_logits, draft_tokens, draft_len, n_accepted_out, next_token_out, workspace, stream)
PyObject *verify_greedy(PyObject *, PyObject *const *argv, Py_ssize_t n)
{
    return answer([&]() -> long {
        if (n != 7) return DECLINED;
        Args a{argv};
        int dtype = -1;
        const at::Tensor *p = a.logits(3, &dtype);
        if (!a.ok) return DECLINED;
        const long long B = p->size(0), k = p->size(1) - 1, V = p->size(2), row_stride = p->stride(1);
        const long long seq_t = B > 1 ? p->stride(0) : (k + 1) * row_stride;
        if (!fits(k)) return DECLINED;
        const int *tokens = a.array<int>(at::kInt, false, B, k), *len = a.array<int>(at::kInt, false, B);
        int *nacc = a.array<int>(at::kInt, false, B), *next = a.array<int>(at::kInt, false, B);
        const at::Tensor *ws = a.workspace();
        void *stream = a.stream();
        if (!a.ok || !fits(B) || !fits(V)) return DECLINED;
        const void *pp = p->data_ptr();
        void *wp = ws->data_ptr();
        const size_t wn = (size_t)ws->numel();
        long status;
        Py_BEGIN_ALLOW_THREADS
        status = g_verify_greedy(pp, dtype, (int)B, (int)k, (int)V, seq_t, row_stride, tokens, len, nacc, next, wp, wn, stream);
        Py_END_ALLOW_THREADS
        return status;
    });
}

// bind(addresses of svip_draft_step, svip_draft_step_greedy, svip_verify, svip_verify_greedy)
PyObject *bind(PyObject *, PyObject *const *argv, Py_ssize_t n)
{
    void *f[4];
    if (n != 4) {
        PyErr_SetString(PyExc_TypeError, "bind takes four addresses");
        return nullptr;
    }
    for (int i = 0; i < 4; ++i) {
        f[i] = PyLong_AsVoidPtr(argv[i]);
        if (!f[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: a null address");
            return nullptr;
        }
    }
    g_draft_step = reinterpret_cast<decltype(g_draft_step)>(f[0]);
    g_draft_step_greedy = reinterpret_cast<decltype(g_draft_step_greedy)>(f[1]);
    g_verify = reinterpret_cast<decltype(g_verify)>(f[2]);
    g_verify_greedy = reinterpret_cast<decltype(g_verify_greedy)>(f[3]);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(bind)), METH_FASTCALL, nullptr},
    {"draft_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(draft_step)), METH_FASTCALL, nullptr},
    {"verify", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(verify)), METH_FASTCALL, nullptr},
    {"verify_greedy", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(verify_greedy)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "native argument marshalling of binding.py", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
