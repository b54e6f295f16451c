// fastcall.cpp -- the binding's entry points for well-formed calls, in native code.
//
// A one-byte step takes the GPU a few microseconds, and marshalling its call in Python
// (argument checks, an output allocation and a ctypes call with 15 arguments) took about
// 10: decoding was bound by the host.  Each function here takes the arguments of the
// Python function of the same name, all positional.  If every tensor is a plain dense
// GPU tensor of the expected shape, type and layout on the current device, it allocates
// the outputs, calls the C ABI on the current stream and returns what the Python function
// returns.  Anything else returns None with nothing done, and the Python function goes on
// to its own checks, which raise the errors; a call that the library refuses returns its
// status (an int).  Per decoded byte (conv1d_step and scan_step, 3584 channels, batch 1):
// 21.3 us before, 10.0 now.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>

#include "mbscan.h"

namespace {

decltype(&mb_scan_fwd) scan_fwd_fn;
decltype(&mb_scan_fwd_states) scan_fwd_states_fn;
decltype(&mb_scan_fwd_ckpt) scan_fwd_ckpt_fn;
decltype(&mb_scan_step) scan_step_fn;
decltype(&mb_conv1d_fwd) conv1d_fwd_fn;
decltype(&mb_conv1d_step) conv1d_step_fn;
decltype(&mb_verify_rank) verify_rank_fn;
PyObject *current_device, *raw_stream, *parameter_type;   // torch's accessors and nn.Parameter

// A plain dense tensor on the GPU (no subclass, no transform's wrapper), or null.
const at::Tensor *plain(PyObject *o) {
    if (!THPVariable_CheckExact(o) && reinterpret_cast<PyObject *>(Py_TYPE(o)) != parameter_type) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    const auto ks = t.unsafeGetTensorImpl()->key_set();
    if (!t.defined() || !ks.has(c10::DispatchKey::CUDA) || ks.has(c10::DispatchKey::Python) || !t.has_storage())
        return nullptr;
    return &t;
}

// The checks of one call: ok stays true while every argument is as the library wants it.
struct Call {
    bool ok = true;
    c10::Device dev{c10::DeviceType::CPU};
    void *stream = nullptr;

    // The tensor that fixes the device: dims dimensions, on the current device.
    const at::Tensor *first(PyObject *o, int64_t dims) {
        const at::Tensor *t = plain(o);
        if (!t || t->dim() != dims || c10::impl::TorchDispatchModeTLS::any_modes_set()) { ok = false; return nullptr; }
        dev = t->device();
        PyObject *cur = PyObject_CallNoArgs(current_device);
        if (!cur) { PyErr_Clear(); ok = false; return nullptr; }
        const long index = PyLong_AsLong(cur);
        Py_DECREF(cur);
        if (index != dev.index()) { ok = false; return nullptr; }
        PyObject *at = PyLong_FromLong(index);
        PyObject *s = PyObject_CallOneArg(raw_stream, at);
        Py_DECREF(at);
        if (!s) { PyErr_Clear(); ok = false; return nullptr; }
        stream = PyLong_AsVoidPtr(s);
        Py_DECREF(s);
        return t;
    }
    // A required tensor of this shape and type; its data.
    void *need(PyObject *o, std::initializer_list<int64_t> shape, at::ScalarType type) {
        const at::Tensor *t = ok ? plain(o) : nullptr;
        if (!t || t->scalar_type() != type || t->device() != dev || t->sizes() != at::IntArrayRef(shape) ||
            !t->is_contiguous()) {
            ok = false;
            return nullptr;
        }
        return t->data_ptr();
    }
    // The same, or None: null.
    void *maybe(PyObject *o, std::initializer_list<int64_t> shape, at::ScalarType type) {
        return o == Py_None ? nullptr : need(o, shape, type);
    }
    static bool act(at::ScalarType t) { return t == at::kFloat || t == at::kBFloat16; }
    // An output given by the caller (any activation type), or its type when it is None.
    void *given(PyObject *o, std::initializer_list<int64_t> shape, at::ScalarType &type) {
        if (o == Py_None) return nullptr;
        const at::Tensor *t = ok ? plain(o) : nullptr;
        if (!t || !act(t->scalar_type())) { ok = false; return nullptr; }
        type = t->scalar_type();
        return need(o, shape, type);
    }
    void dtype(PyObject *o, at::ScalarType &type) {
        if (!THPDtype_Check(o) || !act(reinterpret_cast<THPDtype *>(o)->scalar_type)) ok = false;
        else type = reinterpret_cast<THPDtype *>(o)->scalar_type;
    }
    at::Tensor fresh(std::initializer_list<int64_t> shape, at::ScalarType type) const {
        return at::empty(at::IntArrayRef(shape), at::TensorOptions().dtype(type).device(dev));
    }
};

int32_t code(at::ScalarType t) { return t == at::kBFloat16 ? MB_BF16 : MB_F32; }
const float *f(void *p) { return static_cast<const float *>(p); }
PyObject *wrap(at::Tensor t) { return THPVariable_Wrap(std::move(t)); }
PyObject *same(PyObject *o) { Py_INCREF(o); return o; }

// Runs the library call without the interpreter lock.
template <class F> int unlocked(F call) {
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return st;
}

// No C++ exception leaves an entry: torch's errors become the Python errors they are for
// torch's own functions (OutOfMemoryError among them).
template <class F> PyObject *guarded(F body) {
    HANDLE_TH_ERRORS
    return body();
    END_HANDLE_TH_ERRORS
}

#define ARGS(n) if (nargs != (n)) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }
#define PLAIN_OR_NONE(c) if (!(c).ok) Py_RETURN_NONE

// h, u_t, delta_t, A, B_t, C_t, D, dt_bias, z_t, delta_softplus, out_dtype, out
PyObject *scan_step(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    ARGS(12)
    return guarded([&]() -> PyObject * {
        Call c;
        const at::Tensor *h = c.first(a[0], 3);
        const at::Tensor *u = c.ok ? plain(a[1]) : nullptr;
        if (!u || !Call::act(u->scalar_type())) Py_RETURN_NONE;
        const int64_t nb = h->size(0), dim = h->size(1), N = h->size(2);
        const auto act = u->scalar_type();
        void *hp = c.need(a[0], {nb, dim, N}, at::kFloat), *up = c.need(a[1], {nb, dim}, act);
        void *dp = c.need(a[2], {nb, dim}, act), *Ap = c.need(a[3], {dim, N}, at::kFloat);
        void *Bp = c.need(a[4], {nb, N}, act), *Cp = c.need(a[5], {nb, N}, act);
        void *Dp = c.maybe(a[6], {dim}, at::kFloat), *bp = c.maybe(a[7], {dim}, at::kFloat);
        void *zp = c.maybe(a[8], {nb, dim}, act);
        const int sp = PyObject_IsTrue(a[9]);
        at::ScalarType ot = at::kFloat;
        if (a[11] == Py_None) c.dtype(a[10], ot);
        void *op = c.given(a[11], {nb, dim}, ot);
        if (sp < 0) { PyErr_Clear(); c.ok = false; }
        PLAIN_OR_NONE(c);
        at::Tensor out;
        if (a[11] == Py_None) {
            out = c.fresh({nb, dim}, ot);
            op = out.data_ptr();
        }
        const int st = unlocked([&] {
            return scan_step_fn(nb, dim, N, code(act), code(ot), sp, up, dp, f(Ap), Bp, Cp, f(Dp), f(bp), zp,
                                static_cast<float *>(hp), op, c.stream);
        });
        if (st != MB_OK) return PyLong_FromLong(st);
        return a[11] == Py_None ? wrap(std::move(out)) : same(a[11]);
    });
}

// u, delta, A, B, C, D, dt_bias, z, h0, delta_softplus, out_dtype, return_last_state, out, h_last, positions, h_at,
// return_ckpt, ck
PyObject *scan_fwd(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    ARGS(18)
    return guarded([&]() -> PyObject * {
        Call c;
        const at::Tensor *u = c.first(a[0], 3);
        const at::Tensor *A = c.ok ? plain(a[2]) : nullptr;
        if (!A || A->dim() != 2 || !Call::act(u->scalar_type())) Py_RETURN_NONE;
        const int64_t nb = u->size(0), dim = u->size(1), L = u->size(2), N = A->size(1);
        const auto act = u->scalar_type();
        void *up = c.need(a[0], {nb, dim, L}, act), *dp = c.need(a[1], {nb, dim, L}, act);
        void *Ap = c.need(a[2], {dim, N}, at::kFloat);
        void *Bp = c.need(a[3], {nb, N, L}, act), *Cp = c.need(a[4], {nb, N, L}, act);
        void *Dp = c.maybe(a[5], {dim}, at::kFloat), *bp = c.maybe(a[6], {dim}, at::kFloat);
        void *zp = c.maybe(a[7], {nb, dim, L}, act), *h0 = c.maybe(a[8], {nb, dim, N}, at::kFloat);
        const int sp = PyObject_IsTrue(a[9]), want_last = PyObject_IsTrue(a[11]), want_ck = PyObject_IsTrue(a[16]);
        at::ScalarType ot = at::kFloat;
        if (a[12] == Py_None) c.dtype(a[10], ot);
        void *op = c.given(a[12], {nb, dim, L}, ot), *lp = c.maybe(a[13], {nb, dim, N}, at::kFloat);
        const bool has_pos = a[14] != Py_None, has_ck = want_ck > 0 || a[17] != Py_None;
        int64_t npos = 0;
        void *pp = nullptr, *hp = nullptr, *kp = nullptr;
        if (has_pos) {
            const at::Tensor *pos = c.ok ? plain(a[14]) : nullptr;
            if (!pos || pos->dim() != 2) Py_RETURN_NONE;
            npos = pos->size(0);
            pp = c.need(a[14], {npos, nb}, at::kInt);
            hp = c.maybe(a[15], {npos, nb, dim, N}, at::kFloat);
        } else if (a[15] != Py_None) {
            c.ok = false;
        }
        if (has_ck) kp = c.maybe(a[17], {L / 16, nb, dim, N}, at::kFloat);
        if (sp < 0 || want_last < 0 || want_ck < 0 || (has_ck && has_pos)) { PyErr_Clear(); c.ok = false; }
        PLAIN_OR_NONE(c);
        at::Tensor out, last, at_pos, ck;
        if (a[12] == Py_None) op = (out = c.fresh({nb, dim, L}, ot)).data_ptr();
        if (want_last && a[13] == Py_None) lp = (last = c.fresh({nb, dim, N}, at::kFloat)).data_ptr();
        if (has_pos && a[15] == Py_None) hp = (at_pos = c.fresh({npos, nb, dim, N}, at::kFloat)).data_ptr();
        if (has_ck && a[17] == Py_None) kp = (ck = c.fresh({L / 16, nb, dim, N}, at::kFloat)).data_ptr();
        const mb_scan_desc desc{nb, dim, L, N, code(act), code(ot), sp, 0};
        const int st = unlocked([&] {
            if (has_ck)
                return scan_fwd_ckpt_fn(&desc, up, dp, f(Ap), Bp, Cp, f(Dp), f(bp), zp, f(h0), op,
                                        static_cast<float *>(lp), static_cast<float *>(kp), c.stream);
            if (has_pos)
                return scan_fwd_states_fn(&desc, up, dp, f(Ap), Bp, Cp, f(Dp), f(bp), zp, f(h0), op,
                                          static_cast<float *>(lp), static_cast<const int32_t *>(pp), npos,
                                          static_cast<float *>(hp), c.stream);
            return scan_fwd_fn(&desc, up, dp, f(Ap), Bp, Cp, f(Dp), f(bp), zp, f(h0), op, static_cast<float *>(lp),
                               c.stream);
        });
        if (st != MB_OK) return PyLong_FromLong(st);
        PyObject *res[4];
        int n = 0;
        res[n++] = a[12] == Py_None ? wrap(std::move(out)) : same(a[12]);
        if (want_last || a[13] != Py_None) res[n++] = a[13] == Py_None ? wrap(std::move(last)) : same(a[13]);
        if (has_pos) res[n++] = a[15] == Py_None ? wrap(std::move(at_pos)) : same(a[15]);
        if (has_ck) res[n++] = a[17] == Py_None ? wrap(std::move(ck)) : same(a[17]);
        if (n == 1) return res[0];
        PyObject *t = PyTuple_New(n);
        for (int i = 0; i < n; ++i) PyTuple_SET_ITEM(t, i, res[i]);
        return t;
    });
}

// x, w, bias, state, apply_silu, out_dtype, return_state, out, state_out
PyObject *conv1d(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    ARGS(9)
    return guarded([&]() -> PyObject * {
        Call c;
        const at::Tensor *x = c.first(a[0], 3);
        const at::Tensor *w = c.ok ? plain(a[1]) : nullptr;
        if (!w || w->dim() != 2 || w->size(1) < 2 || !Call::act(x->scalar_type())) Py_RETURN_NONE;
        const int64_t nb = x->size(0), dim = x->size(1), L = x->size(2), K = w->size(1);
        const auto in = x->scalar_type();
        void *xp = c.need(a[0], {nb, dim, L}, in), *wp = c.need(a[1], {dim, K}, at::kFloat);
        void *bp = c.maybe(a[2], {dim}, at::kFloat), *sp = c.maybe(a[3], {nb, dim, K - 1}, at::kFloat);
        const int silu = PyObject_IsTrue(a[4]), want = PyObject_IsTrue(a[6]);
        at::ScalarType ot = in;
        if (a[7] == Py_None && a[5] != Py_None) c.dtype(a[5], ot);
        void *op = c.given(a[7], {nb, dim, L}, ot), *np = c.maybe(a[8], {nb, dim, K - 1}, at::kFloat);
        if (silu < 0 || want < 0 || K > INT32_MAX) { PyErr_Clear(); c.ok = false; }
        PLAIN_OR_NONE(c);
        at::Tensor out, next;
        if (a[7] == Py_None) op = (out = c.fresh({nb, dim, L}, ot)).data_ptr();
        if (want && a[8] == Py_None) np = (next = c.fresh({nb, dim, K - 1}, at::kFloat)).data_ptr();
        const mb_conv_desc desc{nb, dim, L, (int32_t)K, code(in), code(ot), silu, 0, 0};
        const int st = unlocked([&] {
            return conv1d_fwd_fn(&desc, xp, f(wp), f(bp), f(sp), op, static_cast<float *>(np), c.stream);
        });
        if (st != MB_OK) return PyLong_FromLong(st);
        PyObject *y = a[7] == Py_None ? wrap(std::move(out)) : same(a[7]);
        if (!want && a[8] == Py_None) return y;
        PyObject *t = PyTuple_New(2);
        PyTuple_SET_ITEM(t, 0, y);
        PyTuple_SET_ITEM(t, 1, a[8] == Py_None ? wrap(std::move(next)) : same(a[8]));
        return t;
    });
}

// state, x_t, w, bias, apply_silu, out_dtype, out
PyObject *conv1d_step(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    ARGS(7)
    return guarded([&]() -> PyObject * {
        Call c;
        const at::Tensor *x = c.first(a[1], 2);
        const at::Tensor *w = c.ok ? plain(a[2]) : nullptr;
        if (!w || w->dim() != 2 || w->size(1) < 2 || !Call::act(x->scalar_type())) Py_RETURN_NONE;
        const int64_t nb = x->size(0), dim = x->size(1), K = w->size(1);
        const auto in = x->scalar_type();
        void *xp = c.need(a[1], {nb, dim}, in), *wp = c.need(a[2], {dim, K}, at::kFloat);
        void *bp = c.maybe(a[3], {dim}, at::kFloat), *sp = c.need(a[0], {nb, dim, K - 1}, at::kFloat);
        const int silu = PyObject_IsTrue(a[4]);
        at::ScalarType ot = in;
        if (a[6] == Py_None && a[5] != Py_None) c.dtype(a[5], ot);
        void *op = c.given(a[6], {nb, dim}, ot);
        if (silu < 0 || K > INT32_MAX) { PyErr_Clear(); c.ok = false; }
        PLAIN_OR_NONE(c);
        at::Tensor out;
        if (a[6] == Py_None) op = (out = c.fresh({nb, dim}, ot)).data_ptr();
        const int st = unlocked([&] {
            return conv1d_step_fn(nb, dim, (int32_t)K, code(in), code(ot), silu, xp, f(wp), f(bp),
                                  static_cast<float *>(sp), op, c.stream);
        });
        if (st != MB_OK) return PyLong_FromLong(st);
        return a[6] == Py_None ? wrap(std::move(out)) : same(a[6]);
    });
}

// logits, draft, beta, return_ranks
PyObject *verify_rank(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    ARGS(4)
    return guarded([&]() -> PyObject * {
        if (!PyLong_CheckExact(a[2])) Py_RETURN_NONE;
        int over = 0;
        const long long beta = PyLong_AsLongLongAndOverflow(a[2], &over);
        if (over || beta < INT32_MIN || beta > INT32_MAX) Py_RETURN_NONE;
        Call c;
        const at::Tensor *lg = c.first(a[0], 3);
        if (!c.ok || !Call::act(lg->scalar_type())) Py_RETURN_NONE;
        const int64_t nb = lg->size(0), n = lg->size(1), V = lg->size(2);
        void *lp = c.need(a[0], {nb, n, V}, lg->scalar_type()), *dp = c.need(a[1], {nb, n}, at::kInt);
        const int want = PyObject_IsTrue(a[3]);
        if (want < 0) { PyErr_Clear(); c.ok = false; }
        PLAIN_OR_NONE(c);
        at::Tensor acc = c.fresh({nb}, at::kInt), pos = c.fresh({nb}, at::kInt), ranks;
        if (want) ranks = c.fresh({nb, n}, at::kInt);
        const int st = unlocked([&] {
            return verify_rank_fn(nb, n, V, code(lg->scalar_type()), (int32_t)beta, lp,
                                  static_cast<const int32_t *>(dp),
                                  want ? static_cast<int32_t *>(ranks.data_ptr()) : nullptr,
                                  static_cast<int32_t *>(acc.data_ptr()), static_cast<int32_t *>(pos.data_ptr()),
                                  c.stream);
        });
        if (st != MB_OK) return PyLong_FromLong(st);
        PyObject *t = PyTuple_New(want ? 3 : 2);
        PyTuple_SET_ITEM(t, 0, wrap(std::move(acc)));
        PyTuple_SET_ITEM(t, 1, wrap(std::move(pos)));
        if (want) PyTuple_SET_ITEM(t, 2, wrap(std::move(ranks)));
        return t;
    });
}

// setup(function addresses in the order below, current_device, raw_stream, Parameter)
PyObject *setup(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    ARGS(10)
    void *at[7];
    for (int i = 0; i < 7; ++i) {
        at[i] = PyLong_AsVoidPtr(a[i]);
        if (!at[i]) return PyErr_Occurred() ? nullptr : (PyErr_SetString(PyExc_ValueError, "null address"), nullptr);
    }
    scan_fwd_fn = reinterpret_cast<decltype(scan_fwd_fn)>(at[0]);
    scan_fwd_states_fn = reinterpret_cast<decltype(scan_fwd_states_fn)>(at[1]);
    scan_fwd_ckpt_fn = reinterpret_cast<decltype(scan_fwd_ckpt_fn)>(at[2]);
    scan_step_fn = reinterpret_cast<decltype(scan_step_fn)>(at[3]);
    conv1d_fwd_fn = reinterpret_cast<decltype(conv1d_fwd_fn)>(at[4]);
    conv1d_step_fn = reinterpret_cast<decltype(conv1d_step_fn)>(at[5]);
    verify_rank_fn = reinterpret_cast<decltype(verify_rank_fn)>(at[6]);
    current_device = same(a[7]);
    raw_stream = same(a[8]);
    parameter_type = same(a[9]);
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(setup),  METHOD(scan_step),   METHOD(scan_fwd),
                         METHOD(conv1d), METHOD(conv1d_step), METHOD(verify_rank),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() {
    PyObject *m = PyModule_Create(&module);
    // the torch whose object layouts this was compiled against: the binding uses no other
    if (m && PyModule_AddStringConstant(m, "torch_version", MB_TORCH_VERSION) != 0) Py_CLEAR(m);
    return m;
}
