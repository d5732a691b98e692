// binding.cpp -- the argument marshalling of the hot entry points in native
// code: from torch tensors to the C ABI of include/pi_attn.h.
//
// A call that launches one small kernel is bound by its host work: in Python
// the checks, the gate's broadcast view, the stream object and the ctypes
// conversion took 11 of a forward's 14.4 us, the launch itself 3.4; here the
// whole call takes 3.8 us.
//
// Each function takes the arguments of its namesake in __init__.py by
// position and serves the plain call: strided GPU tensors of one device,
// every argument of its documented type and valid.  For anything else --
// another type, another device, a tensor subclass or a wrapped tensor, an
// active torch function or dispatch mode, a given stream, an argument that
// the checks or the library refuse -- it returns None before anything is
// enqueued, and the Python code handles the call (and words the error).  A
// launch that the HIP runtime refuses (PI_ATTN_EHIP) raises PiAttnError here:
// of a call of several launches the first ones may be enqueued by then.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>

#include <array>
#include <cmath>
#include <string>

#include "pi_attn.h"

namespace {

using at::Tensor;

// A plain call's arguments, read in order; `ok` turns false at the first one
// that is not plain, and stays so.
struct Args {
    PyObject *const *a;
    Py_ssize_t i = 0;
    bool ok;
    c10::Device device = c10::Device(c10::kCPU);

    Args(PyObject *const *args, Py_ssize_t n, Py_ssize_t want) : a(args) {
        ok = n == want && !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled();
    }
    // A tensor on the device of the first one; an undefined tensor for None
    // where `optional`.
    Tensor tensor(bool optional = false) {
        PyObject *o = next();
        if (!o || (optional && o == Py_None)) return Tensor();
        if (!THPVariable_CheckExact(o)) return fail();
        const Tensor &t = THPVariable_Unpack(o);
        if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || !t.has_storage()) return fail();
        const auto keys = t.key_set();
        if (keys.has(c10::DispatchKey::Python) || keys.has_any(c10::functorch_transforms_ks)) return fail();
        if (device.is_cpu()) device = t.device();
        if (t.device() != device) return fail();
        return t;
    }
    int32_t integer() {
        PyObject *o = next();
        if (!o || !PyLong_CheckExact(o)) return fail(), 0;
        int overflow = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow || v < INT32_MIN || v > INT32_MAX) return fail(), 0;
        return (int32_t)v;
    }
    bool boolean() {
        PyObject *o = next();
        if (!o || !PyBool_Check(o)) return fail(), false;
        return o == Py_True;
    }
    // a float or an int; `none` for None (NaN: None is not taken)
    float real(float none) {
        PyObject *o = next();
        if (!o) return 0.0f;
        if (o == Py_None && !std::isnan(none)) return none;
        if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
        if (PyLong_CheckExact(o)) {
            int overflow = 0;
            const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
            if (!overflow) return (float)(double)v;
        }
        return fail(), 0.0f;
    }
    void none() {
        if (next() != Py_None) ok = false;
    }
    // the next argument; null once the call is not plain
    PyObject *next() { return ok ? a[i++] : nullptr; }
    Tensor fail() {
        ok = false;
        return Tensor();
    }
};

bool same_layout(const Tensor &x, const Tensor &y) { return x.sizes() == y.sizes() && x.strides() == y.strides(); }

int32_t dtype_of(const Tensor &t) {
    return t.scalar_type() == at::kFloat ? PI_ATTN_F32 : t.scalar_type() == at::kBFloat16 ? PI_ATTN_BF16 : -1;
}

// q, k, v [B, H, N, D]: one dtype, shape and strides, D contiguous, no empty
// extent.
struct Shape {
    int64_t B, H, N, D;
};

bool sequence_ok(const Tensor &q, const Tensor &k, const Tensor &v, Shape &s) {
    if (q.dim() != 4 || dtype_of(q) < 0 || k.scalar_type() != q.scalar_type() || v.scalar_type() != q.scalar_type())
        return false;
    if (!same_layout(q, k) || !same_layout(q, v) || q.stride(3) != 1) return false;
    s = Shape{q.size(0), q.size(1), q.size(2), q.size(3)};
    return q.numel() > 0 && s.B <= INT32_MAX && s.H <= INT32_MAX && s.N <= INT32_MAX && s.D <= INT32_MAX;
}

bool is_f32(const Tensor &t, at::IntArrayRef shape) {
    return t.scalar_type() == at::kFloat && t.sizes() == shape && t.is_contiguous();
}

// A float32 output buffer: the given one, checked, or a new one.
bool f32_out(Tensor &t, at::IntArrayRef shape, const c10::Device &device) {
    if (!t.defined()) {
        t = at::empty(shape, at::TensorOptions().dtype(at::kFloat).device(device));
        return true;
    }
    return is_f32(t, shape);
}

// The output in q's shape and dtype: the given one, checked, or a new one.
bool like_out(Tensor &out, const Tensor &q) {
    if (!out.defined()) {
        out = at::empty(q.sizes(), at::TensorOptions().dtype(q.scalar_type()).device(q.device()));
        return true;
    }
    return out.sizes() == q.sizes() && out.scalar_type() == q.scalar_type() && out.stride(3) == 1;
}

// Element strides of the gate logits: [H], or [B, H, N] (per_query).
bool gate_strides(const Tensor &g, const Shape &s, int64_t (&st)[3], bool &per_query) {
    if (g.scalar_type() != at::kFloat) return false;
    per_query = g.dim() == 3;
    if (g.dim() == 1 && g.size(0) == s.H) {
        st[0] = st[2] = 0;
        st[1] = g.stride(0);
        return true;
    }
    if (!per_query || g.size(0) != s.B || g.size(1) != s.H || g.size(2) != s.N) return false;
    for (int i = 0; i < 3; ++i) st[i] = g.stride(i);
    return true;
}

void *stream_of(const c10::Device &d) { return c10::hip::getCurrentHIPStream(d.index()).stream(); }

template <typename T>
T *ptr(const Tensor &t) {
    return t.defined() ? static_cast<T *>(t.data_ptr()) : nullptr;
}

PyObject *pack(std::initializer_list<Tensor> ts) {
    PyObject *r = PyTuple_New((Py_ssize_t)ts.size());
    Py_ssize_t i = 0;
    for (const Tensor &t : ts) PyTuple_SET_ITEM(r, i++, THPVariable_Wrap(t));
    return r;
}

// The result of a call whose status is not PI_ATTN_OK.
PyObject *refused(PyObject *self, int status, const char *where) {
    if (status != PI_ATTN_EHIP) Py_RETURN_NONE;
    const auto package = pybind11::handle(self).attr("__package__");
    const auto error = pybind11::module_::import(pybind11::str(package).cast<std::string>().c_str()).attr("PiAttnError");
    PyErr_SetObject(error.ptr(), error(status, where).ptr());
    return nullptr;
}

// q, k, v, gate, k_window, pi, scale, logit_clamp, out, return_lse, lse, stream, causal
PyObject *forward(PyObject *self, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Args a(args, n, 13);
    const Tensor q = a.tensor(), k = a.tensor(), v = a.tensor(), gate = a.tensor();
    const int32_t kw = a.integer(), pi = a.integer();
    Shape s{};
    if (!a.ok || !sequence_ok(q, k, v, s)) Py_RETURN_NONE;
    const float scale = a.real(pi_attn_default_scale((int32_t)s.D)), clamp = a.real(NAN);
    Tensor out = a.tensor(true);
    const bool want_lse = a.boolean();
    Tensor lse = a.tensor(true);
    a.none();
    const bool causal = a.boolean();
    int64_t gs[3];
    bool per_query;
    if (!a.ok || !gate_strides(gate, s, gs, per_query)) Py_RETURN_NONE;
    const bool with_lse = want_lse || lse.defined();
    int status = PI_ATTN_EINVAL;
    {
        pybind11::gil_scoped_release no_gil;
        if (like_out(out, q) && (!with_lse || f32_out(lse, {s.B, s.H, s.N}, a.device)))
            status = pi_attn_forward(dtype_of(q), s.B, s.H, s.N, s.D, kw, pi, causal, q.data_ptr(), k.data_ptr(),
                                     v.data_ptr(), q.stride(0), q.stride(1), q.stride(2), ptr<float>(gate), gs[0],
                                     gs[1], gs[2], scale, clamp, out.data_ptr(), out.stride(0), out.stride(1),
                                     out.stride(2), ptr<float>(lse), stream_of(a.device));
    }
    if (status != PI_ATTN_OK) return refused(self, status, "pi_attn_forward");
    return with_lse ? pack({out, lse}) : THPVariable_Wrap(out);
    END_HANDLE_TH_ERRORS
}

// q, k, v, u, w2, b2, k_window, pi, scale, logit_clamp, out, return_lse, lse, gate_out, stream, causal
PyObject *forward_gated(PyObject *self, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Args a(args, n, 16);
    const Tensor q = a.tensor(), k = a.tensor(), v = a.tensor(), u = a.tensor(), w2 = a.tensor();
    const Tensor b2 = a.tensor(true);
    const int32_t kw = a.integer(), pi = a.integer();
    Shape s{};
    if (!a.ok || !sequence_ok(q, k, v, s)) Py_RETURN_NONE;
    const float scale = a.real(pi_attn_default_scale((int32_t)s.D)), clamp = a.real(NAN);
    Tensor out = a.tensor(true);
    const bool want_lse = a.boolean();
    Tensor lse = a.tensor(true), gate = a.tensor(true);
    a.none();
    const bool causal = a.boolean();
    if (!a.ok || u.scalar_type() != q.scalar_type() || w2.scalar_type() != q.scalar_type()) Py_RETURN_NONE;
    if (u.dim() != 3 || u.size(0) != s.B || u.size(1) != s.N || u.stride(2) != 1) Py_RETURN_NONE;
    const int64_t dh = u.size(2);
    if (dh > INT32_MAX || w2.sizes() != at::IntArrayRef({s.H, dh}) || !w2.is_contiguous()) Py_RETURN_NONE;
    if (b2.defined() && !is_f32(b2, {s.H})) Py_RETURN_NONE;
    const bool with_lse = want_lse || lse.defined();
    int status = PI_ATTN_EINVAL;
    {
        pybind11::gil_scoped_release no_gil;
        if (like_out(out, q) && f32_out(gate, {s.B, s.H, s.N}, a.device) &&
            (!with_lse || f32_out(lse, {s.B, s.H, s.N}, a.device)))
            status = pi_attn_forward_gated(dtype_of(q), s.B, s.H, s.N, s.D, kw, pi, causal, q.data_ptr(), k.data_ptr(),
                                           v.data_ptr(), q.stride(0), q.stride(1), q.stride(2), u.data_ptr(),
                                           u.stride(0), u.stride(1), dh, w2.data_ptr(), ptr<float>(b2), scale, clamp,
                                           out.data_ptr(), out.stride(0), out.stride(1), out.stride(2), ptr<float>(lse),
                                           ptr<float>(gate), stream_of(a.device));
    }
    if (status != PI_ATTN_OK) return refused(self, status, "pi_attn_forward_gated");
    return with_lse ? pack({out, gate, lse}) : pack({out, gate});
    END_HANDLE_TH_ERRORS
}

// q, k, v, gate, k_window, pi, out, lse, dout, scale, logit_clamp, gate_grad_per_query, stream, causal, dq, dk, dv,
// dgate, rowterm
PyObject *backward(PyObject *self, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Args a(args, n, 19);
    const Tensor q = a.tensor(), k = a.tensor(), v = a.tensor(), gate = a.tensor();
    const int32_t kw = a.integer(), pi = a.integer();
    const Tensor out = a.tensor(), lse = a.tensor(), dout = a.tensor();
    Shape s{};
    if (!a.ok || !sequence_ok(q, k, v, s)) Py_RETURN_NONE;
    const float scale = a.real(pi_attn_default_scale((int32_t)s.D)), clamp = a.real(NAN);
    const bool keep_per_query = a.boolean();
    a.none();
    const bool causal = a.boolean();
    Tensor dq = a.tensor(true), dk = a.tensor(true), dv = a.tensor(true), dg = a.tensor(true), rt = a.tensor(true);
    int64_t gs[3];
    bool per_query;
    if (!a.ok || !gate_strides(gate, s, gs, per_query)) Py_RETURN_NONE;
    if (out.scalar_type() != q.scalar_type() || dout.scalar_type() != q.scalar_type() || !same_layout(out, dout) ||
        out.sizes() != q.sizes() || dout.stride(3) != 1 || !is_f32(lse, {s.B, s.H, s.N}))
        Py_RETURN_NONE;
    Tensor per_head;
    int status = PI_ATTN_EINVAL;
    const char *where = "pi_attn_backward";
    {
        pybind11::gil_scoped_release no_gil;
        const std::array<int64_t, 4> full{s.B, s.H, s.N, s.D};
        const std::array<int64_t, 3> rows{s.B, s.H, s.N};
        void *stream = stream_of(a.device);
        if (f32_out(dq, full, a.device) && f32_out(dk, full, a.device) && f32_out(dv, full, a.device) &&
            f32_out(dg, rows, a.device) && f32_out(rt, rows, a.device))
            status = pi_attn_backward(dtype_of(q), s.B, s.H, s.N, s.D, kw, pi, causal, q.data_ptr(), k.data_ptr(),
                                      v.data_ptr(), q.stride(0), q.stride(1), q.stride(2), ptr<float>(gate), gs[0],
                                      gs[1], gs[2], scale, clamp, ptr<float>(lse), out.data_ptr(), dout.data_ptr(),
                                      dout.stride(0), dout.stride(1), dout.stride(2), ptr<float>(dq), ptr<float>(dk),
                                      ptr<float>(dv), ptr<float>(dg), ptr<float>(rt), stream);
        if (status == PI_ATTN_OK && !per_query && !keep_per_query) {
            where = "pi_attn_gate_grad_per_head";   // of valid arguments: refused by the runtime or not at all
            f32_out(per_head, {s.H}, a.device);
            status = pi_attn_gate_grad_per_head(s.B, s.H, s.N, ptr<float>(dg), ptr<float>(per_head), stream);
        }
    }
    if (status != PI_ATTN_OK) return refused(self, status, where);
    return pack({dq, dk, dv, per_head.defined() ? per_head : dg});
    END_HANDLE_TH_ERRORS
}

// len_in, q_new, k_new, v_new, k_cache, v_cache, gate, k, pi, scale, logit_clamp, len_out, out, lse, stream
PyObject *decode_step(PyObject *self, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Args a(args, n, 15);
    const Tensor len_in = a.tensor(), q = a.tensor(), k = a.tensor(), v = a.tensor(), kc = a.tensor(),
                 vc = a.tensor(), gate = a.tensor();
    const int32_t kw = a.integer(), pi = a.integer();
    if (!a.ok || kc.dim() != 4 || dtype_of(kc) < 0 || kc.numel() == 0) Py_RETURN_NONE;
    const int64_t S = kc.size(0), H = kc.size(1), cap = kc.size(2), D = kc.size(3);
    if (S > INT32_MAX || H > INT32_MAX || cap > INT32_MAX || D > INT32_MAX) Py_RETURN_NONE;
    const float scale = a.real(pi_attn_default_scale((int32_t)D)), clamp = a.real(NAN);
    const Tensor len_out = a.tensor(true);
    Tensor out = a.tensor(true);
    const Tensor lse = a.tensor(true);
    a.none();
    if (!a.ok) Py_RETURN_NONE;
    const std::array<int64_t, 3> rows{S, H, D};
    const auto cached = [&](const Tensor &t, at::IntArrayRef shape) {
        return t.scalar_type() == kc.scalar_type() && t.sizes() == shape && t.is_contiguous();
    };
    const auto lengths = [&](const Tensor &t) {
        return t.scalar_type() == at::kInt && t.dim() == 1 && t.size(0) == S && t.is_contiguous();
    };
    if (!cached(q, rows) || !cached(k, rows) || !cached(v, rows) || !cached(vc, kc.sizes()) || !kc.is_contiguous())
        Py_RETURN_NONE;
    if (!lengths(len_in) || (len_out.defined() && !lengths(len_out)) || gate.scalar_type() != at::kFloat) Py_RETURN_NONE;
    int64_t gss, gsh;
    if (gate.dim() == 1 && gate.size(0) == H) {
        gss = 0;
        gsh = gate.stride(0);
    } else if (gate.dim() == 2 && gate.size(0) == S && gate.size(1) == H) {
        gss = gate.stride(0);
        gsh = gate.stride(1);
    } else {
        Py_RETURN_NONE;
    }
    if ((out.defined() && !cached(out, rows)) || (lse.defined() && !is_f32(lse, {S, H}))) Py_RETURN_NONE;
    int status;
    {
        pybind11::gil_scoped_release no_gil;
        if (!out.defined()) out = at::empty(rows, at::TensorOptions().dtype(kc.scalar_type()).device(a.device));
        status = pi_attn_decode_step(dtype_of(kc), S, H, D, cap, kw, pi, ptr<int32_t>(len_in), ptr<int32_t>(len_out),
                                     q.data_ptr(), k.data_ptr(), v.data_ptr(), kc.data_ptr(), vc.data_ptr(),
                                     ptr<float>(gate), gss, gsh, scale, clamp, out.data_ptr(), ptr<float>(lse),
                                     stream_of(a.device));
    }
    if (status != PI_ATTN_OK) return refused(self, status, "pi_attn_decode_step");
    return THPVariable_Wrap(out);
    END_HANDLE_TH_ERRORS
}

template <typename F>
PyCFunction fast(F f) {
    return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f));
}

PyMethodDef methods[] = {{"forward", fast(forward), METH_FASTCALL, nullptr},
                         {"forward_gated", fast(forward_gated), METH_FASTCALL, nullptr},
                         {"backward", fast(backward), METH_FASTCALL, nullptr},
                         {"decode_step", fast(decode_step), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
