// Native side of the Python binding: the common call of every entry point, from tensors to launch.
//
// A call of a small rollout is bound by its host side: argument checks, two output
// allocations and a ctypes call of some sixteen arguments took 8 to 12 us in Python against 2 to
// 5 us on the GPU (GAE 8 x 128: 9.7 us a call; 4096 x 256: 10.3). These functions do the same
// checks, allocate the missing outputs and call the C interface on the current stream.
//
// They only take calls that are plain in every respect (tensors of exactly torch's own type on
// the current GPU, right shapes and types, no active dispatch mode, no function mode but torch's
// default device) and return NotImplemented for any other, having done nothing: the Python function then runs its own checks
// and reports what is wrong, or handles the call. So every error a caller sees about its arguments
// comes from one place. Errors of the C interface are raised here as they are there.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/PyInterpreter.h>
#include <torch/csrc/autograd/python_variable.h>

#include "rlcs.h"

namespace {

PyObject* g_error = nullptr;   // RlcsError(fn, code)
PyObject* g_device = nullptr;  // torch.utils._device.DeviceContext

// The library's functions, looked up in the handle the package loaded.
struct Library {
    decltype(&rlcs_gae) gae;
    decltype(&rlcs_vtrace) vtrace;
    decltype(&rlcs_retrace) retrace;
    decltype(&rlcs_retrace_full) retrace_full;
    decltype(&rlcs_td_lambda) td_lambda;
    decltype(&rlcs_discounted) discounted;
    decltype(&rlcs_elig_trace) elig_trace;
    decltype(&rlcs_episodic_prefix) episodic_prefix;
    decltype(&rlcs_affine_scan) affine_scan;
    decltype(&rlcs_gae_strided) gae_strided;
    decltype(&rlcs_vtrace_strided) vtrace_strided;
    decltype(&rlcs_retrace_strided) retrace_strided;
    decltype(&rlcs_td_lambda_strided) td_lambda_strided;
    decltype(&rlcs_discounted_strided) discounted_strided;
    decltype(&rlcs_elig_trace_strided) elig_trace_strided;
    decltype(&rlcs_episodic_prefix_strided) episodic_prefix_strided;
    decltype(&rlcs_elig_trace_vec) elig_trace_vec;
    decltype(&rlcs_gae_masked) gae_masked;
    decltype(&rlcs_gae_masked_noalloc) gae_masked_noalloc;
} g_lib;
bool g_bound = false;

struct NoGil {
    PyThreadState* state = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(state); }
};

// Keys of tensors whose memory is not simply theirs (function transforms, subclasses, lazy
// negation and the like).
const c10::DispatchKeySet kSpecial({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot,
                                    c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                    c10::DispatchKey::Functionalize, c10::DispatchKey::Conjugate,
                                    c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});

// Whether the function modes in force leave the call as it is: none, or torch's default device
// (torch.set_default_device, `with torch.device(...)`), which only gives a device to factory
// functions called without one. Every allocation here names its device.
bool modes_pass() {
    using TLS = at::impl::PythonTorchFunctionTLS;
    for (int64_t i = 0, n = TLS::stack_len(); i < n; ++i)
        if (reinterpret_cast<PyObject*>(Py_TYPE(TLS::get_stack_at(i)->ptr(getPyInterpreter()))) != g_device) return false;
    return true;
}

// One call: its shape, and whether every argument seen so far is a plain one.
struct Call {
    bool ok = true;
    const bool strided;
    int64_t N = 0, T = 0, sn = 0, st = 0;
    int64_t inner = 0;  // last dimension of a 3-D first input, or 0
    at::ScalarType dtype = at::kFloat;
    at::Device device = at::kCPU;

    explicit Call(bool s) : strided(s) {
        ok = g_bound && !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
             modes_pass();
    }

    bool bf16() const { return dtype == at::kBFloat16; }
    rlcs_dtype type() const { return bf16() ? RLCS_BF16 : RLCS_F32; }

    // A plain tensor, or null (None, or not plain: then ok is false).
    const at::Tensor* plain(PyObject* o) {
        if (!ok || o == Py_None) return nullptr;
        if (!THPVariable_CheckExact(o)) {
            ok = false;
            return nullptr;
        }
        const at::Tensor& t = THPVariable_Unpack(o);
        if (t.key_set().has_any(kSpecial) || t.layout() != at::kStrided || !t.has_storage()) {
            ok = false;
            return nullptr;
        }
        return &t;
    }

    // (stride_n, stride_t) of an [N, T] view; a dimension of one step takes the stride that nests
    // the two (it never multiplies an index other than 0).
    void strides(const at::Tensor& t, int64_t& a, int64_t& b) const {
        a = t.stride(0);
        b = t.stride(1);
        if (T == 1) b = std::max<int64_t>(1, N * std::max<int64_t>(a, 1));
        if (N == 1) a = std::max<int64_t>(1, T * std::max<int64_t>(b, 1));
    }

    // The first data input decides shape, type and device.
    void* first(PyObject* o, int dims = 2) {
        const at::Tensor* t = plain(o);
        if (!t) {
            ok = false;
            return nullptr;
        }
        dtype = t->scalar_type();
        device = t->device();
        if (t->dim() != dims || (dtype != at::kFloat && dtype != at::kBFloat16) || !device.is_cuda() ||
            device.index() != c10::hip::current_device()) {
            ok = false;
            return nullptr;
        }
        N = t->size(0);
        T = t->size(1);
        if (dims == 3) inner = t->size(2);
        if (strided) strides(*t, sn, st);
        return same_layout(*t) ? t->data_ptr() : nullptr;
    }

    // Whether a tensor of the call's shape lies as the call says it does.
    bool same_layout(const at::Tensor& t) {
        if (strided) {
            int64_t a, b;
            strides(t, a, b);
            ok = ok && a == sn && b == st;
        } else {
            ok = ok && t.is_contiguous();
        }
        return ok;
    }

    void* checked(PyObject* o, at::ScalarType type, at::IntArrayRef shape, bool of_call) {
        const at::Tensor* t = plain(o);
        if (!t) return nullptr;
        ok = ok && t->scalar_type() == type && t->sizes() == shape && t->device() == device;
        if (!ok) return nullptr;
        if (of_call) same_layout(*t);
        else ok = t->is_contiguous();
        return ok ? t->data_ptr() : nullptr;
    }
    void* data(PyObject* o) { return checked(o, dtype, {N, T}, true); }
    void* actions_axis(PyObject* o, int64_t A) { return checked(o, dtype, {N, T, A}, false); }
    int32_t* actions(PyObject* o) { return static_cast<int32_t*>(checked(o, at::kInt, {N, T}, false)); }
    void* per_row(PyObject* o) { return checked(o, dtype, {N}, false); }
    const uint8_t* flags(PyObject* o) {
        const at::Tensor* t = plain(o);
        if (!t) return nullptr;
        const at::ScalarType s = t->scalar_type();
        ok = ok && (s == at::kByte || s == at::kBool);
        return static_cast<const uint8_t*>(checked(o, s, {N, T}, true));
    }
    void* workspace(PyObject* o, size_t& bytes) {
        bytes = 0;
        const at::Tensor* t = plain(o);
        if (!t) return nullptr;
        ok = ok && t->device() == device && t->is_contiguous();
        if (!ok) return nullptr;
        bytes = t->nbytes();
        return t->data_ptr();
    }
    float number(PyObject* o) {
        if (PyFloat_CheckExact(o)) return float(PyFloat_AS_DOUBLE(o));
        if (PyLong_CheckExact(o)) {
            const double v = PyLong_AsDouble(o);
            if (v != -1.0 || !PyErr_Occurred()) return float(v);
            PyErr_Clear();
        }
        ok = false;
        return 0.f;
    }
    bool truth(PyObject* o) {
        if (o != Py_True && o != Py_False) ok = false;
        return o == Py_True;
    }
};

// An output: given by the caller, allocated by the call, or not wanted.
struct Out {
    PyObject* given = nullptr;
    bool make = false;
    at::Tensor made;
    float* ptr = nullptr;

    Out(Call& c, PyObject* o, bool want) {
        if (o == Py_None) {
            make = want;
            return;
        }
        given = o;
        if (c.inner) ptr = static_cast<float*>(c.checked(o, at::kFloat, {c.N, c.T, c.inner}, false));
        else ptr = static_cast<float*>(c.checked(o, at::kFloat, {c.N, c.T}, true));
    }
    void allocate(const Call& c) {
        if (!make) return;
        const auto options = at::TensorOptions().dtype(at::kFloat).device(c.device);
        if (c.inner) made = at::empty({c.N, c.T, c.inner}, options);
        else if (c.strided) made = at::empty_strided({c.N, c.T}, {c.sn, c.st}, options);
        else made = at::empty({c.N, c.T}, options);
        ptr = static_cast<float*>(made.data_ptr());
    }
    // A new reference: the tensor, or None.
    PyObject* object() {
        if (make) return THPVariable_Wrap(made);
        PyObject* o = given ? given : Py_None;
        Py_INCREF(o);
        return o;
    }
};

// Allocates, calls `fn(stream)` and returns the outputs: one tensor, or a pair with `second`.
template <class Fn>
PyObject* run(Call& c, const char* name, Out& a, Out* second, Fn&& fn) {
    if (!c.ok) Py_RETURN_NOTIMPLEMENTED;
    int code = 0;
    try {
        NoGil no_gil;
        a.allocate(c);
        if (second) second->allocate(c);
        code = fn(static_cast<rlcs_stream_t>(c10::hip::getCurrentHIPStream(c.device.index()).stream()));
    } catch (...) {  // an allocation that failed: the Python function meets it again and reports it
        Py_RETURN_NOTIMPLEMENTED;
    }
    if (code != RLCS_OK) {
        PyObject* e = PyObject_CallFunction(g_error, "si", name, code);
        if (e) {
            PyErr_SetObject(g_error, e);
            Py_DECREF(e);
        }
        return nullptr;
    }
    PyObject* x = a.object();
    if (!second || !x) return x;
    PyObject* y = second->object();
    if (!y) {
        Py_DECREF(x);
        return nullptr;
    }
    PyObject* pair = PyTuple_New(2);
    if (!pair) {
        Py_DECREF(x);
        Py_DECREF(y);
        return nullptr;
    }
    PyTuple_SET_ITEM(pair, 0, x);
    PyTuple_SET_ITEM(pair, 1, y);
    return pair;
}

typedef PyObject* const* Argv;

// A function of the module: F, or NotImplemented where an accessor of an exotic tensor throws.
template <PyObject* (*F)(Argv, Py_ssize_t)>
PyObject* entry(PyObject*, Argv x, Py_ssize_t nargs) {
    try {
        return F(x, nargs);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NOTIMPLEMENTED;
    }
}

#define RLCS_ARGS(n) \
    if (nargs != (n)) Py_RETURN_NOTIMPLEMENTED

// gae(r, v, term, trunc, bv, boot, adv, ret, gamma, lam, ws, want_ret)
template <bool S>
PyObject* gae(Argv x, Py_ssize_t nargs) {
    RLCS_ARGS(12);
    Call c(S);
    void *r = c.first(x[0]), *v = c.data(x[1]);
    const uint8_t *te = c.flags(x[2]), *tr = c.flags(x[3]);
    void *bv = c.data(x[4]), *b = c.per_row(x[5]);
    Out o0(c, x[6], true), o1(c, x[7], c.truth(x[11]));
    const float g = c.number(x[8]), l = c.number(x[9]);
    size_t wb;
    void* ws = c.workspace(x[10], wb);
    return run(c, S ? "rlcs_gae_strided" : "rlcs_gae", o0, &o1, [&](rlcs_stream_t s) {
        if constexpr (S) return g_lib.gae_strided(r, v, te, tr, bv, b, o0.ptr, o1.ptr, c.N, c.T, c.sn, c.st, g, l, c.type(), ws, wb, s);
        else return g_lib.gae(r, v, te, tr, bv, b, o0.ptr, o1.ptr, c.N, c.T, g, l, c.type(), ws, wb, s);
    });
}

// vtrace(r, v, log_rho, term, trunc, bv, boot, vs, pg, gamma, rho_bar, c_bar, ws, want_pg)
template <bool S>
PyObject* vtrace(Argv x, Py_ssize_t nargs) {
    RLCS_ARGS(14);
    Call c(S);
    void *r = c.first(x[0]), *v = c.data(x[1]), *lr = c.data(x[2]);
    const uint8_t *te = c.flags(x[3]), *tr = c.flags(x[4]);
    void *bv = c.data(x[5]), *b = c.per_row(x[6]);
    Out o0(c, x[7], true), o1(c, x[8], c.truth(x[13]));
    const float g = c.number(x[9]), rb = c.number(x[10]), cb = c.number(x[11]);
    size_t wb;
    void* ws = c.workspace(x[12], wb);
    return run(c, S ? "rlcs_vtrace_strided" : "rlcs_vtrace", o0, &o1, [&](rlcs_stream_t s) {
        if constexpr (S) return g_lib.vtrace_strided(r, v, lr, te, tr, bv, b, o0.ptr, o1.ptr, c.N, c.T, c.sn, c.st, g, rb, cb, c.type(), ws, wb, s);
        else return g_lib.vtrace(r, v, lr, te, tr, bv, b, o0.ptr, o1.ptr, c.N, c.T, g, rb, cb, c.type(), ws, wb, s);
    });
}

// retrace(r, q, eq, log_rho, term, trunc, bv, boot, delta, q_ret, gamma, lam, c_bar, ws, want_q_ret)
template <bool S>
PyObject* retrace(Argv x, Py_ssize_t nargs) {
    RLCS_ARGS(15);
    Call c(S);
    void *r = c.first(x[0]), *q = c.data(x[1]), *eq = c.data(x[2]), *lr = c.data(x[3]);
    const uint8_t *te = c.flags(x[4]), *tr = c.flags(x[5]);
    void *bv = c.data(x[6]), *b = c.per_row(x[7]);
    Out o0(c, x[8], true), o1(c, x[9], c.truth(x[14]));
    const float g = c.number(x[10]), l = c.number(x[11]), cb = c.number(x[12]);
    size_t wb;
    void* ws = c.workspace(x[13], wb);
    return run(c, S ? "rlcs_retrace_strided" : "rlcs_retrace", o0, &o1, [&](rlcs_stream_t s) {
        if constexpr (S) return g_lib.retrace_strided(r, q, eq, lr, te, tr, bv, b, o0.ptr, o1.ptr, c.N, c.T, c.sn, c.st, g, l, cb, c.type(), ws, wb, s);
        else return g_lib.retrace(r, q, eq, lr, te, tr, bv, b, o0.ptr, o1.ptr, c.N, c.T, g, l, cb, c.type(), ws, wb, s);
    });
}

// retrace_full(r, q, pi, actions, mu, term, trunc, bv, boot, delta, q_ret, gamma, lam, c_bar, ws,
// want_q_ret)
PyObject* retrace_full(Argv x, Py_ssize_t nargs) {
    RLCS_ARGS(16);
    Call c(false);
    void* r = c.first(x[0]);
    const at::Tensor* qt = c.plain(x[1]);
    if (!qt || qt->dim() != 3 || x[2] == Py_None || x[3] == Py_None) Py_RETURN_NOTIMPLEMENTED;
    const int64_t A = qt->size(2);
    void *q = c.actions_axis(x[1], A), *pi = c.actions_axis(x[2], A);
    int32_t* act = c.actions(x[3]);
    void* mu = c.data(x[4]);
    const uint8_t *te = c.flags(x[5]), *tr = c.flags(x[6]);
    void *bv = c.data(x[7]), *b = c.per_row(x[8]);
    Out o0(c, x[9], true), o1(c, x[10], c.truth(x[15]));
    const float g = c.number(x[11]), l = c.number(x[12]), cb = c.number(x[13]);
    size_t wb;
    void* ws = c.workspace(x[14], wb);
    return run(c, "rlcs_retrace_full", o0, &o1, [&](rlcs_stream_t s) {
        return g_lib.retrace_full(r, q, pi, act, mu, te, tr, bv, b, o0.ptr, o1.ptr, c.N, c.T, A, g, l, cb, c.type(), ws, wb, s);
    });
}

// td_lambda(r, v, term, trunc, bv, boot, ret, gamma, lam, ws)
template <bool S>
PyObject* td_lambda(Argv x, Py_ssize_t nargs) {
    RLCS_ARGS(10);
    Call c(S);
    void *r = c.first(x[0]), *v = c.data(x[1]);
    const uint8_t *te = c.flags(x[2]), *tr = c.flags(x[3]);
    void *bv = c.data(x[4]), *b = c.per_row(x[5]);
    Out o(c, x[6], true);
    const float g = c.number(x[7]), l = c.number(x[8]);
    size_t wb;
    void* ws = c.workspace(x[9], wb);
    return run(c, S ? "rlcs_td_lambda_strided" : "rlcs_td_lambda", o, nullptr, [&](rlcs_stream_t s) {
        if constexpr (S) return g_lib.td_lambda_strided(r, v, te, tr, bv, b, o.ptr, c.N, c.T, c.sn, c.st, g, l, c.type(), ws, wb, s);
        else return g_lib.td_lambda(r, v, te, tr, bv, b, o.ptr, c.N, c.T, g, l, c.type(), ws, wb, s);
    });
}

// discounted(r, term, trunc, bv, boot, ret, gamma, ws)
template <bool S>
PyObject* discounted(Argv x, Py_ssize_t nargs) {
    RLCS_ARGS(8);
    Call c(S);
    void* r = c.first(x[0]);
    const uint8_t *te = c.flags(x[1]), *tr = c.flags(x[2]);
    void *bv = c.data(x[3]), *b = c.per_row(x[4]);
    Out o(c, x[5], true);
    const float g = c.number(x[6]);
    size_t wb;
    void* ws = c.workspace(x[7], wb);
    return run(c, S ? "rlcs_discounted_strided" : "rlcs_discounted", o, nullptr, [&](rlcs_stream_t s) {
        if constexpr (S) return g_lib.discounted_strided(r, te, tr, bv, b, o.ptr, c.N, c.T, c.sn, c.st, g, c.type(), ws, wb, s);
        else return g_lib.discounted(r, te, tr, bv, b, o.ptr, c.N, c.T, g, c.type(), ws, wb, s);
    });
}

// elig_trace(x, term, trunc, z, gamma, lam, ws)
template <bool S>
PyObject* elig_trace(Argv x, Py_ssize_t nargs) {
    RLCS_ARGS(7);
    Call c(S);
    void* in = c.first(x[0]);
    const uint8_t *te = c.flags(x[1]), *tr = c.flags(x[2]);
    Out o(c, x[3], true);
    const float g = c.number(x[4]), l = c.number(x[5]);
    size_t wb;
    void* ws = c.workspace(x[6], wb);
    return run(c, S ? "rlcs_elig_trace_strided" : "rlcs_elig_trace", o, nullptr, [&](rlcs_stream_t s) {
        if constexpr (S) return g_lib.elig_trace_strided(in, te, tr, o.ptr, c.N, c.T, c.sn, c.st, g, l, c.type(), ws, wb, s);
        else return g_lib.elig_trace(in, te, tr, o.ptr, c.N, c.T, g, l, c.type(), ws, wb, s);
    });
}

// episodic_prefix(x, term, trunc, c, starts_at, ws)
template <bool S>
PyObject* episodic_prefix(Argv x, Py_ssize_t nargs) {
    RLCS_ARGS(6);
    Call c(S);
    void* in = c.first(x[0]);
    const uint8_t *te = c.flags(x[1]), *tr = c.flags(x[2]);
    Out o(c, x[3], true);
    const rlcs_boundary b = c.truth(x[4]) ? RLCS_STARTS_AT : RLCS_ENDS_AT;
    size_t wb;
    void* ws = c.workspace(x[5], wb);
    return run(c, S ? "rlcs_episodic_prefix_strided" : "rlcs_episodic_prefix", o, nullptr, [&](rlcs_stream_t s) {
        if constexpr (S) return g_lib.episodic_prefix_strided(in, te, tr, o.ptr, c.N, c.T, c.sn, c.st, b, c.type(), ws, wb, s);
        else return g_lib.episodic_prefix(in, te, tr, o.ptr, c.N, c.T, b, c.type(), ws, wb, s);
    });
}

// affine_scan(alpha, beta, carry, out, reverse, ws)
PyObject* affine_scan(Argv x, Py_ssize_t nargs) {
    RLCS_ARGS(6);
    Call c(false);
    void *al = c.first(x[0]), *be = c.data(x[1]), *carry = c.per_row(x[2]);
    Out o(c, x[3], true);
    const rlcs_direction d = c.truth(x[4]) ? RLCS_BACKWARD : RLCS_FORWARD;
    size_t wb;
    void* ws = c.workspace(x[5], wb);
    return run(c, "rlcs_affine_scan", o, nullptr, [&](rlcs_stream_t s) {
        return g_lib.affine_scan(al, be, carry, o.ptr, c.N, c.T, d, c.type(), ws, wb, s);
    });
}

// elig_trace_vec(x, term, trunc, z, gamma, lam, ws)
PyObject* elig_trace_vec(Argv x, Py_ssize_t nargs) {
    RLCS_ARGS(7);
    Call c(false);
    void* in = c.first(x[0], 3);
    const int64_t F = c.inner;
    if (!c.ok || F == 0) Py_RETURN_NOTIMPLEMENTED;
    const uint8_t *te = c.flags(x[1]), *tr = c.flags(x[2]);
    Out o(c, x[3], true);
    const float g = c.number(x[4]), l = c.number(x[5]);
    size_t wb;
    void* ws = c.workspace(x[6], wb);
    return run(c, "rlcs_elig_trace_vec", o, nullptr, [&](rlcs_stream_t s) {
        return g_lib.elig_trace_vec(in, te, tr, o.ptr, c.N, c.T, F, g, l, c.type(), ws, wb, s);
    });
}

// gae_masked(r, v, mask, term, trunc, bv, boot, adv, ret, gamma, lam, normalize, eps, want_ret[, ws])
PyObject* gae_masked(Argv x, Py_ssize_t nargs) {
    if (nargs != 14 && nargs != 15) Py_RETURN_NOTIMPLEMENTED;
    Call c(false);
    void *r = c.first(x[0]), *v = c.data(x[1]);
    const uint8_t *mk = c.flags(x[2]), *te = c.flags(x[3]), *tr = c.flags(x[4]);
    void *bv = c.data(x[5]), *b = c.per_row(x[6]);
    Out o0(c, x[7], true), o1(c, x[8], c.truth(x[13]));
    const float g = c.number(x[9]), l = c.number(x[10]), eps = c.number(x[12]);
    const int norm = c.truth(x[11]) ? 1 : 0;
    size_t wb = 0;
    void* ws = nargs == 15 ? c.workspace(x[14], wb) : nullptr;
    if (nargs == 14)
        return run(c, "rlcs_gae_masked_noalloc", o0, &o1, [&](rlcs_stream_t s) {
            return g_lib.gae_masked_noalloc(r, v, mk, te, tr, bv, b, o0.ptr, o1.ptr, c.N, c.T, g, l, norm, eps, c.type(), s);
        });
    if (norm && !ws) Py_RETURN_NOTIMPLEMENTED;  // the Python function makes one
    return run(c, "rlcs_gae_masked", o0, &o1, [&](rlcs_stream_t s) {
        return g_lib.gae_masked(r, v, mk, te, tr, bv, b, o0.ptr, o1.ptr, c.N, c.T, g, l, norm, eps, c.type(), ws, wb, s);
    });
}

// bind(handle, error, device): the dlopen handle of librlcs.so, the exception class of its status
// codes and the class of torch's default-device mode
PyObject* bind(PyObject*, PyObject* args) {
    unsigned long long handle = 0;
    PyObject *error = nullptr, *device = nullptr;
    if (!PyArg_ParseTuple(args, "KOO", &handle, &error, &device)) return nullptr;
    void* h = reinterpret_cast<void*>(handle);
    bool all = true;
    auto get = [&](auto& fn, const char* name) {
        fn = reinterpret_cast<std::decay_t<decltype(fn)>>(dlsym(h, name));
        all = all && fn;
    };
    get(g_lib.gae, "rlcs_gae");
    get(g_lib.vtrace, "rlcs_vtrace");
    get(g_lib.retrace, "rlcs_retrace");
    get(g_lib.retrace_full, "rlcs_retrace_full");
    get(g_lib.td_lambda, "rlcs_td_lambda");
    get(g_lib.discounted, "rlcs_discounted");
    get(g_lib.elig_trace, "rlcs_elig_trace");
    get(g_lib.episodic_prefix, "rlcs_episodic_prefix");
    get(g_lib.affine_scan, "rlcs_affine_scan");
    get(g_lib.gae_strided, "rlcs_gae_strided");
    get(g_lib.vtrace_strided, "rlcs_vtrace_strided");
    get(g_lib.retrace_strided, "rlcs_retrace_strided");
    get(g_lib.td_lambda_strided, "rlcs_td_lambda_strided");
    get(g_lib.discounted_strided, "rlcs_discounted_strided");
    get(g_lib.elig_trace_strided, "rlcs_elig_trace_strided");
    get(g_lib.episodic_prefix_strided, "rlcs_episodic_prefix_strided");
    get(g_lib.elig_trace_vec, "rlcs_elig_trace_vec");
    get(g_lib.gae_masked, "rlcs_gae_masked");
    get(g_lib.gae_masked_noalloc, "rlcs_gae_masked_noalloc");
    if (!all) {
        PyErr_SetString(PyExc_RuntimeError, "librlcs.so lacks a function of the binding");
        return nullptr;
    }
    Py_INCREF(error);
    Py_XSETREF(g_error, error);
    Py_INCREF(device);
    Py_XSETREF(g_device, device);
    g_bound = true;
    Py_RETURN_NONE;
}

template <PyObject* (*F)(Argv, Py_ssize_t)>
PyMethodDef fast(const char* name) {
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<F>)), METH_FASTCALL, nullptr};
}

PyMethodDef g_methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    fast<gae<false>>("gae"), fast<gae<true>>("gae_strided"),
    fast<vtrace<false>>("vtrace"), fast<vtrace<true>>("vtrace_strided"),
    fast<retrace<false>>("retrace"), fast<retrace<true>>("retrace_strided"),
    fast<retrace_full>("retrace_full"),
    fast<td_lambda<false>>("td_lambda"), fast<td_lambda<true>>("td_lambda_strided"),
    fast<discounted<false>>("discounted"), fast<discounted<true>>("discounted_strided"),
    fast<elig_trace<false>>("elig_trace"), fast<elig_trace<true>>("elig_trace_strided"),
    fast<episodic_prefix<false>>("episodic_prefix"), fast<episodic_prefix<true>>("episodic_prefix_strided"),
    fast<affine_scan>("affine_scan"), fast<elig_trace_vec>("elig_trace_vec"), fast<gae_masked>("gae_masked"),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&g_module); }
