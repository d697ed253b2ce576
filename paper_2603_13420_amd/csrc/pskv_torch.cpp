// Argument marshalling for torch tensors: the way from a Python call to the C ABI of include/pskv.h.
//
// One call of the library costs about 3 us on the host; reading some forty shapes, strides and pointers
// of its tensors through Python, checking them and filling in the parameters cost another 15 (19 us per
// forward call, 28 per backward call, and small problems take 6 on the GPU).  Here the same takes under
// one.  No check is lost: a function of this module either makes the call - when every argument is of
// the plain form it knows - or returns None having done nothing, and binding.py, whose own checks are the
// definition of what is allowed, goes on from there (and says what is wrong, if anything is).
//
// The library's entry points are handed over as addresses (bind), so that this module follows whichever
// build of it binding.py has loaded.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/DeviceGuard.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/pskv.h"

#include <cstring>

namespace {

decltype(&pskv_attn_fwd) lib_fwd;
decltype(&pskv_attn_fwd_multi) lib_fwd_multi;
decltype(&pskv_attn_bwd) lib_bwd;
decltype(&pskv_attn_bwd_multi) lib_bwd_multi;
decltype(&pskv_attn_bwd_noalloc) lib_bwd_noalloc;
decltype(&pskv_attn_bwd_workspace_bytes) lib_workspace_bytes;
PyObject *current_raw_stream; // torch._C._cuda_getCurrentRawStream

// A tensor argument: absent (None), or present; anything else is not of the plain form.
struct Arg {
    const at::Tensor *t = nullptr;
    bool read(PyObject *o)
    {
        if (o == Py_None)
            return true;
        if (!THPVariable_CheckExact(o)) // (a subclass may have its own empty_like)
            return false;
        t = &THPVariable_Unpack(o);
        return true;
    }
    // Throws for a tensor without storage (one that torch.vmap or torch.func.grad hands in is of the exact type Tensor).
    void *data() const { return t ? t->data_ptr() : nullptr; }
};

// The interpreter's lock given up for as long as the object lives, whatever ends that.
struct WithoutGil {
    PyThreadState *save = PyEval_SaveThread();
    WithoutGil() = default;
    WithoutGil(const WithoutGil &) = delete;
    ~WithoutGil() { PyEval_RestoreThread(save); }
};

bool same_layout(const at::Tensor &x, const at::Tensor &y)
{
    return x.scalar_type() == y.scalar_type() && x.device() == y.device() && x.sizes() == y.sizes() && x.strides() == y.strides();
}

// Element stride as the ABI wants it (see binding._stride); false: an expanded view.
bool stride_of(const at::Tensor &t, int dim, int64_t &dst)
{
    dst = t.size(dim) <= 1 ? 0 : t.stride(dim);
    return t.size(dim) <= 1 || dst != 0;
}
bool rows_contiguous(const at::Tensor &t) { return t.size(-1) <= 1 || t.stride(-1) == 1; }

bool is_index(const Arg &a, int64_t n, const at::Tensor &q)
{
    return !a.t || (a.t->scalar_type() == at::kInt && a.t->dim() == 1 && a.t->size(0) == n && a.t->is_contiguous() &&
                    a.t->device() == q.device());
}

bool impl_of(PyObject *o, int32_t &impl)
{
    const char *s = PyUnicode_Check(o) ? PyUnicode_AsUTF8(o) : nullptr;
    if (!s) {
        PyErr_Clear();
        return false;
    }
    if (!std::strcmp(s, "auto"))
        impl = PSKV_IMPL_AUTO;
    else if (!std::strcmp(s, "simple"))
        impl = PSKV_IMPL_SIMPLE;
    else if (!std::strcmp(s, "mfma"))
        impl = PSKV_IMPL_MFMA;
    else
        return false;
    return true;
}

// The parameters of a call, from tensors of the plain form (out: never absent here).
bool fill(pskv_multi_params &m, bool multi, const Arg &q, const Arg &ks, const Arg &vs, const Arg &kp, const Arg &vp, const Arg &pre_len,
          const Arg &suf_len, const at::Tensor &out, const Arg &lse, PyObject *impl, PyObject *scale)
{
    std::memset(&m, 0, sizeof m);
    pskv_attn_params &p = m.base;
    if (!q.t || !ks.t || !vs.t || !impl_of(impl, p.impl) || !PyFloat_Check(scale))
        return false;
    const at::Tensor &Q = *q.t, &K = *ks.t;
    if (!Q.is_cuda() || Q.dim() != 4 || K.dim() != 4 || out.dim() != 4)
        return false;
    if (Q.scalar_type() == at::kBFloat16)
        p.dtype = PSKV_DTYPE_BF16;
    else if (Q.scalar_type() == at::kFloat)
        p.dtype = PSKV_DTYPE_F32;
    else
        return false;
    const int64_t B = Q.size(0), S = Q.size(1), Hq = Q.size(2), D = Q.size(3), Hkv = K.size(2);
    if (K.scalar_type() != Q.scalar_type() || K.device() != Q.device() || K.size(0) != B || K.size(1) != S || K.size(3) != D ||
        !same_layout(K, *vs.t))
        return false;
    if (out.scalar_type() != Q.scalar_type() || out.device() != Q.device() || out.sizes() != Q.sizes())
        return false;
    if (!rows_contiguous(Q) || !rows_contiguous(K) || !rows_contiguous(out))
        return false;
    if (!is_index(suf_len, B, Q))
        return false;
    if (lse.t && !(lse.t->scalar_type() == at::kFloat && lse.t->dim() == 3 && lse.t->size(0) == B && lse.t->size(1) == Hq &&
                   lse.t->size(2) == S && lse.t->is_contiguous() && lse.t->device() == Q.device()))
        return false;
    int64_t P = 0;
    m.Np = 1;
    if (kp.t) {
        const at::Tensor &KP = *kp.t;
        const int d0 = multi ? 1 : 0; // the dimension of the prefix rows
        if (!vp.t || KP.dim() != 3 + d0 || KP.size(d0 + 1) != Hkv || KP.size(d0 + 2) != D || KP.scalar_type() != Q.scalar_type() ||
            KP.device() != Q.device() || !same_layout(KP, *vp.t) || !rows_contiguous(KP))
            return false;
        P = KP.size(d0);
        if (P > 0 && !(stride_of(KP, d0, p.kp_stride_p) && stride_of(KP, d0 + 1, p.kp_stride_h)))
            return false;
        if (multi) {
            m.Np = (int32_t)KP.size(0);
            if (!stride_of(KP, 0, m.kp_stride_n) || !is_index(pre_len, KP.size(0), Q))
                return false;
        }
    } else if (vp.t || multi) {
        return false;
    }
    for (int64_t n : {B, S, P, Hq, Hkv, D})
        if (n > 0x7fffffff)
            return false;
    p.B = (int32_t)B, p.S = (int32_t)S, p.P = (int32_t)P, p.Hq = (int32_t)Hq, p.Hkv = (int32_t)Hkv, p.D = (int32_t)D;
    p.scale = (float)PyFloat_AS_DOUBLE(scale);
    return stride_of(Q, 0, p.q_stride_b) && stride_of(Q, 1, p.q_stride_s) && stride_of(Q, 2, p.q_stride_h) &&
           stride_of(K, 0, p.ks_stride_b) && stride_of(K, 1, p.ks_stride_s) && stride_of(K, 2, p.ks_stride_h) &&
           stride_of(out, 0, p.o_stride_b) && stride_of(out, 1, p.o_stride_s) && stride_of(out, 2, p.o_stride_h);
}

// The stream to launch on: the caller's raw handle, or torch's current one.  False with a Python error set.
bool stream_of(PyObject *given, const at::Tensor &q, void *&stream)
{
    PyObject *index = nullptr, *raw = given;
    if (given == Py_None) {
        index = PyLong_FromLong(q.device().index());
        raw = index ? PyObject_CallOneArg(current_raw_stream, index) : nullptr;
        Py_XDECREF(index);
        if (!raw)
            return false;
    }
    stream = PyLong_AsVoidPtr(raw);
    if (given == Py_None)
        Py_DECREF(raw);
    return !PyErr_Occurred();
}

// fwd(q, k_suf, v_suf, k_pre, v_pre, suf_len, out, lse, impl, scale, stream)
// fwd_multi(q, k_suf, v_suf, k_pre, v_pre, pre_len, suf_len, out, lse, impl, scale, stream)
// -> out; a status number when the library refuses the call; None when an argument is not of the plain form
template <bool MULTI> PyObject *forward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    constexpr int kLen = MULTI ? 1 : 0; // arguments behind pre_len are one further on
    if (n != 11 + kLen || !lib_fwd)
        Py_RETURN_NONE;
    Arg q, ks, vs, kp, vp, pl, sl, out, lse;
    if (!(q.read(args[0]) && ks.read(args[1]) && vs.read(args[2]) && kp.read(args[3]) && vp.read(args[4]) &&
          (!MULTI || pl.read(args[5])) && sl.read(args[5 + kLen]) && out.read(args[6 + kLen]) && lse.read(args[7 + kLen])))
        Py_RETURN_NONE;
    at::Tensor made;
    if (!out.t) {
        if (!q.t || !q.t->is_cuda())
            Py_RETURN_NONE;
        made = at::empty_like(*q.t);
        out.t = &made;
    }
    pskv_multi_params m;
    if (!fill(m, MULTI, q, ks, vs, kp, vp, pl, sl, *out.t, lse, args[8 + kLen], args[9 + kLen]))
        Py_RETURN_NONE;
    void *stream;
    if (!stream_of(args[10 + kLen], *q.t, stream))
        return nullptr;
    const void *q_p = q.data(), *ks_p = ks.data(), *vs_p = vs.data(), *kp_p = kp.data(), *vp_p = vp.data();
    const auto *pre_len = static_cast<const int32_t *>(pl.data()), *suf_len = static_cast<const int32_t *>(sl.data());
    void *out_p = out.data();
    auto *lse_p = static_cast<float *>(lse.data());
    pskv_status rc;
    {
        const c10::DeviceGuard guard(q.t->device());
        const WithoutGil no_gil;
        if constexpr (MULTI)
            rc = lib_fwd_multi(&m, q_p, ks_p, vs_p, kp_p, vp_p, pre_len, suf_len, out_p, lse_p, nullptr, 0, stream);
        else
            rc = lib_fwd(&m.base, q_p, ks_p, vs_p, kp_p, vp_p, suf_len, out_p, lse_p, nullptr, 0, stream);
    }
    if (rc != PSKV_OK)
        return PyLong_FromLong(rc);
    if (made.defined())
        return THPVariable_Wrap(made);
    Py_INCREF(args[6 + kLen]);
    return args[6 + kLen];
    END_HANDLE_TH_ERRORS
}

// bwd(q, k_suf, v_suf, k_pre, v_pre, suf_len, out, lse, dout, dq, dk_suf, dv_suf, impl, scale, stream, workspace)
// bwd_multi: with pre_len before suf_len.  bwd_noalloc: bwd without the workspace, every tensor given.
// -> (dq, dk_suf, dv_suf), or as forward
enum class Bwd { kSingle, kMulti, kNoAlloc };
template <Bwd KIND> PyObject *backward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    constexpr bool kMulti = KIND == Bwd::kMulti, kNoAlloc = KIND == Bwd::kNoAlloc;
    constexpr int kLen = kMulti ? 1 : 0;
    if (n != (kNoAlloc ? 15 : 16 + kLen) || !lib_bwd)
        Py_RETURN_NONE;
    Arg q, ks, vs, kp, vp, pl, sl, out, lse, dout, dq, dk, dv, ws;
    if (!(q.read(args[0]) && ks.read(args[1]) && vs.read(args[2]) && kp.read(args[3]) && vp.read(args[4]) &&
          (!kMulti || pl.read(args[5])) && sl.read(args[5 + kLen]) && out.read(args[6 + kLen]) && lse.read(args[7 + kLen]) &&
          dout.read(args[8 + kLen]) && dq.read(args[9 + kLen]) && dk.read(args[10 + kLen]) && dv.read(args[11 + kLen])))
        Py_RETURN_NONE;
    if (!out.t || !lse.t || !dout.t)
        Py_RETURN_NONE;
    pskv_multi_params m;
    if (!fill(m, kMulti, q, ks, vs, kp, vp, pl, sl, *out.t, lse, args[12 + kLen], args[13 + kLen]) || !same_layout(*out.t, *dout.t))
        Py_RETURN_NONE;
    if (kNoAlloc && !(dq.t && dk.t && dv.t))
        Py_RETURN_NONE;
    at::Tensor made[3], made_ws;
    const struct {
        Arg *a;
        const at::Tensor &like;
    } grads[3] = {{&dq, *q.t}, {&dk, *ks.t}, {&dv, *vs.t}};
    for (int i = 0; i < 3; ++i) {
        if (!grads[i].a->t) {
            made[i] = at::empty_like(grads[i].like);
            grads[i].a->t = &made[i];
        }
        // (a gradient made like a tensor with gaps between its rows has not its strides)
        if (!same_layout(*grads[i].a->t, i == 0 ? *q.t : *ks.t))
            Py_RETURN_NONE;
    }
    void *stream;
    if (!stream_of(args[14 + kLen], *q.t, stream))
        return nullptr;
    size_t ws_bytes = 0;
    if constexpr (!kNoAlloc) {
        PyObject *w = args[15 + kLen]; // a tensor, None: one of our own unless the stream is the caller's (see binding.py), False: none
        if (w == Py_None) {
            if (args[14 + kLen] == Py_None) {
                const size_t need = lib_workspace_bytes(&m.base);
                if (need < ((size_t)1 << 62)) { // (invalid parameters: the call itself reports what is wrong)
                    made_ws = at::empty({(int64_t)need}, at::TensorOptions().dtype(at::kByte).device(q.t->device()));
                    ws.t = &made_ws;
                }
            }
        } else if (w != Py_False && !(ws.read(w) && ws.t)) {
            Py_RETURN_NONE;
        }
        ws_bytes = ws.t ? (size_t)ws.t->numel() * ws.t->element_size() : 0;
    }
    const void *q_p = q.data(), *ks_p = ks.data(), *vs_p = vs.data(), *kp_p = kp.data(), *vp_p = vp.data(), *out_p = out.data(),
               *dout_p = dout.data();
    const auto *pre_len = static_cast<const int32_t *>(pl.data()), *suf_len = static_cast<const int32_t *>(sl.data());
    const auto *lse_p = static_cast<const float *>(lse.data());
    void *dq_p = dq.data(), *dk_p = dk.data(), *dv_p = dv.data(), *ws_p = ws.data();
    pskv_status rc;
    {
        const c10::DeviceGuard guard(q.t->device());
        const WithoutGil no_gil;
        if constexpr (kMulti)
            rc = lib_bwd_multi(&m, q_p, ks_p, vs_p, kp_p, vp_p, pre_len, suf_len, out_p, lse_p, dout_p, dq_p, dk_p, dv_p, ws_p, ws_bytes, stream);
        else if constexpr (kNoAlloc)
            rc = lib_bwd_noalloc(&m.base, q_p, ks_p, vs_p, kp_p, vp_p, suf_len, out_p, lse_p, dout_p, dq_p, dk_p, dv_p, stream);
        else
            rc = lib_bwd(&m.base, q_p, ks_p, vs_p, kp_p, vp_p, suf_len, out_p, lse_p, dout_p, dq_p, dk_p, dv_p, ws_p, ws_bytes, stream);
    }
    if (rc != PSKV_OK)
        return PyLong_FromLong(rc);
    PyObject *res = PyTuple_New(3);
    for (int i = 0; res && i < 3; ++i) {
        PyObject *o;
        if (made[i].defined()) {
            o = THPVariable_Wrap(made[i]);
        } else {
            o = args[9 + kLen + i];
            Py_INCREF(o);
        }
        PyTuple_SET_ITEM(res, i, o);
    }
    return res;
    END_HANDLE_TH_ERRORS
}

// bind(fwd, fwd_multi, bwd, bwd_multi, bwd_noalloc, bwd_workspace_bytes, current_raw_stream): addresses of the
// library's entry points, and torch's function for the current stream of a device.
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long f[6];
    PyObject *raw;
    if (!PyArg_ParseTuple(args, "KKKKKKO", &f[0], &f[1], &f[2], &f[3], &f[4], &f[5], &raw))
        return nullptr;
    lib_fwd_multi = reinterpret_cast<decltype(lib_fwd_multi)>(f[1]);
    lib_bwd = reinterpret_cast<decltype(lib_bwd)>(f[2]);
    lib_bwd_multi = reinterpret_cast<decltype(lib_bwd_multi)>(f[3]);
    lib_bwd_noalloc = reinterpret_cast<decltype(lib_bwd_noalloc)>(f[4]);
    lib_workspace_bytes = reinterpret_cast<decltype(lib_workspace_bytes)>(f[5]);
    Py_INCREF(raw);
    Py_XSETREF(current_raw_stream, raw);
    lib_fwd = reinterpret_cast<decltype(lib_fwd)>(f[0]);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         {"fwd", (PyCFunction)(void (*)())forward<false>, METH_FASTCALL, nullptr},
                         {"fwd_multi", (PyCFunction)(void (*)())forward<true>, METH_FASTCALL, nullptr},
                         {"bwd", (PyCFunction)(void (*)())backward<Bwd::kSingle>, METH_FASTCALL, nullptr},
                         {"bwd_multi", (PyCFunction)(void (*)())backward<Bwd::kMulti>, METH_FASTCALL, nullptr},
                         {"bwd_noalloc", (PyCFunction)(void (*)())backward<Bwd::kNoAlloc>, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pskv_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__pskv_torch() { return PyModule_Create(&module); }
