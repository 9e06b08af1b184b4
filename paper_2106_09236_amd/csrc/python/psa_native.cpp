// The Python entry points of the hot calls, in native code: tensors in, checks, allocation of what the caller did not
// bring, the current stream, one call of the C ABI.  For short utterances the GPU is done in 10 us; marshalling the
// same call through ctypes took 8 us of the interpreter's time on top of the launches (B=1 H=4 L=128, output and
// scratch given: 13.0 us per call, here 8.7, of which two launches are 5).
//
// A function returns None where anything is out of the ordinary before the library is called (an argument that is no
// contiguous device tensor, an unknown type, no memory); nothing has been enqueued then, and the caller's ctypes path takes
// over, which reports the error.  A status other than PSA_OK is raised from here: a launch that failed may come after
// stages that have been enqueued, and those are not enqueued again.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../../include/probsparse.h"

namespace {

// A device tensor argument: a contiguous tensor on a GPU, or None where `optional`.
struct Arg {
    const at::Tensor* t = nullptr;
    void* ptr = nullptr;
};
bool take(PyObject* o, Arg& a, bool optional)
{
    if (o == Py_None) return optional;
    if (!THPVariable_Check(o)) return false;
    a.t = &THPVariable_Unpack(o);
    if (!a.t->is_cuda() || !a.t->is_contiguous()) return false;
    a.ptr = a.t->data_ptr();
    return true;
}
bool dtype_of(const at::Tensor& t, int32_t* dtype)
{
    const auto s = t.scalar_type();
    if (s == at::kFloat) { *dtype = PSA_F32; return true; }
    if (s == at::kBFloat16) { *dtype = PSA_BF16; return true; }
    return false;
}
// shape of Q [B, H, L, D]; U is the last dimension of sample_idx, or 1
bool shape_of(const at::Tensor& q, const Arg& idx, psa_shape_t* s)
{
    if (q.dim() != 4 || (idx.t && idx.t->dim() < 1)) return false;
    s->B = (int32_t)q.size(0); s->H = (int32_t)q.size(1); s->L_Q = s->L_K = (int32_t)q.size(2); s->D = (int32_t)q.size(3);
    s->U = idx.t ? (int32_t)idx.t->size(-1) : 1;
    return dtype_of(q, &s->dtype);
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }
at::Tensor scratch(const at::Tensor& like, size_t bytes)
{
    return at::empty({(int64_t)bytes}, like.options().dtype(at::kByte));
}
PyObject* none() { Py_RETURN_NONE; }
// what raises the binding's exception for a status (set by the binding)
PyObject* raise_status = nullptr;
PyObject* failed(int rc)
{
    PyObject* r = raise_status ? PyObject_CallFunction(raise_status, "i", rc) : nullptr;
    Py_XDECREF(r);
    if (!PyErr_Occurred()) PyErr_Format(PyExc_RuntimeError, "libprobsparse: status %d", rc);
    return nullptr;
}
PyObject* on_status(PyObject*, PyObject* callable)
{
    Py_INCREF(callable);
    Py_XSETREF(raise_status, callable);
    Py_RETURN_NONE;
}
// Other Python threads run while a call allocates and enqueues: either may wait (for memory, for room in a queue).
// No Python object is touched inside; the caller holds the arguments.
struct Unlocked {
    PyThreadState* const state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};
// the caller's output object, or the one made here
PyObject* result(PyObject* given, at::Tensor&& made)
{
    if (given == Py_None) return THPVariable_Wrap(std::move(made));
    Py_INCREF(given);
    return given;
}

// The forward's common part: Q, K, V, lengths, sample_idx, options, out, workspace (the last two may be None).
PyObject* forward(PyObject* const* a, const psa_options_t& opt, PyObject* out_o, PyObject* ws_o)
{
    Arg q, k, v, len, idx, out, ws;
    if (!take(a[0], q, false) || !take(a[1], k, false) || !take(a[2], v, false) || !take(a[3], len, true) ||
        !take(a[4], idx, false) || !take(out_o, out, true) || !take(ws_o, ws, true)) return none();
    psa_shape_t s;
    if (!shape_of(*q.t, idx, &s)) return none();
    at::Tensor made, room;
    const size_t bytes = ws.t ? (size_t)ws.t->numel() : probsparse_attn_workspace_bytes_opt(&s, &opt);
    if (bytes == 0) return none();
    int rc;
    {
        const Unlocked unlocked;
        if (!ws.t) { room = scratch(*q.t, bytes); ws.ptr = room.data_ptr(); }
        if (!out.t) { made = at::empty_like(*q.t); out.ptr = made.data_ptr(); }
        rc = probsparse_attn_fwd_opt(q.ptr, k.ptr, v.ptr, static_cast<const int32_t*>(len.ptr),
                                     static_cast<const int32_t*>(idx.ptr), &opt, out.ptr, &s, ws.ptr, bytes, stream(),
                                     nullptr, nullptr, nullptr);
    }
    return rc == PSA_OK ? result(out_o, std::move(made)) : failed(rc);
}

// attn_fwd(Q, K, V, lengths, sample_idx, c, out, workspace)
PyObject* attn_fwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 8) return none();
    const double c = PyFloat_AsDouble(a[5]);
    if (PyErr_Occurred()) { PyErr_Clear(); return none(); }
    return forward(a, psa_options_t{PSA_U_LOG, PSA_FILL_MEAN, c}, a[6], a[7]);
}

bool option_args(PyObject* rule, PyObject* factor, PyObject* fill, psa_options_t* o)
{
    o->u_rule = (int32_t)PyLong_AsLong(rule);
    o->factor = PyFloat_AsDouble(factor);
    o->fill = (int32_t)PyLong_AsLong(fill);
    if (PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}

// attn_fwd_opt(Q, K, V, lengths, sample_idx, u_rule, factor, fill, out, workspace), without taps
PyObject* attn_fwd_opt(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    psa_options_t opt;
    if (n != 10 || !option_args(a[5], a[6], a[7], &opt)) return none();
    return forward(a, opt, a[8], a[9]);
}

// attn_fwd_with_indices(Q, K, V, lengths, sel, u, fill, out, workspace)
PyObject* attn_fwd_with_indices(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Arg q, k, v, len, sel, u, out, ws;
    if (n != 9 || !take(a[0], q, false) || !take(a[1], k, false) || !take(a[2], v, false) || !take(a[3], len, true) ||
        !take(a[4], sel, false) || !take(a[5], u, false) || !take(a[7], out, true) || !take(a[8], ws, true)) return none();
    const int32_t fill = (int32_t)PyLong_AsLong(a[6]);
    if (PyErr_Occurred()) { PyErr_Clear(); return none(); }
    psa_shape_t s;
    if (!shape_of(*q.t, Arg{}, &s) || sel.t->dim() < 1) return none();
    const int32_t stride = (int32_t)sel.t->size(-1);
    at::Tensor made, room;
    const size_t bytes = ws.t ? (size_t)ws.t->numel() : probsparse_attn_with_indices_workspace_bytes(&s, stride);
    if (bytes == 0) return none();
    int rc;
    {
        const Unlocked unlocked;
        if (!ws.t) { room = scratch(*q.t, bytes); ws.ptr = room.data_ptr(); }
        if (!out.t) { made = at::empty_like(*q.t); out.ptr = made.data_ptr(); }
        rc = probsparse_attn_fwd_with_indices(q.ptr, k.ptr, v.ptr, static_cast<const int32_t*>(len.ptr),
                                              static_cast<const int32_t*>(sel.ptr), static_cast<const int32_t*>(u.ptr),
                                              stride, fill, out.ptr, &s, ws.ptr, bytes, stream());
    }
    return rc == PSA_OK ? result(a[7], std::move(made)) : failed(rc);
}

// attn_bwd(Q, K, V, lengths, sel, u, dOut, fill, workspace) -> (dQ, dK, dV)
PyObject* attn_bwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Arg q, k, v, len, sel, u, g, ws;
    if (n != 9 || !take(a[0], q, false) || !take(a[1], k, false) || !take(a[2], v, false) || !take(a[3], len, true) ||
        !take(a[4], sel, false) || !take(a[5], u, false) || !take(a[6], g, false) || !take(a[8], ws, true)) return none();
    const int32_t fill = (int32_t)PyLong_AsLong(a[7]);
    if (PyErr_Occurred()) { PyErr_Clear(); return none(); }
    psa_shape_t s;
    if (!shape_of(*q.t, Arg{}, &s) || sel.t->dim() < 1) return none();
    const int32_t stride = (int32_t)sel.t->size(-1);
    at::Tensor room, dq, dk, dv;
    const size_t bytes = ws.t ? (size_t)ws.t->numel() : probsparse_attn_bwd_workspace_bytes(&s, stride);
    if (bytes == 0) return none();
    int rc;
    {
        const Unlocked unlocked;
        if (!ws.t) { room = scratch(*q.t, bytes); ws.ptr = room.data_ptr(); }
        dq = at::empty_like(*q.t); dk = at::empty_like(*q.t); dv = at::empty_like(*q.t);
        rc = probsparse_attn_bwd(q.ptr, k.ptr, v.ptr, static_cast<const int32_t*>(len.ptr),
                                 static_cast<const int32_t*>(sel.ptr), static_cast<const int32_t*>(u.ptr), stride, fill,
                                 g.ptr, dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), &s, ws.ptr, bytes, stream());
    }
    if (rc != PSA_OK) return failed(rc);
    PyObject* t = PyTuple_New(3);
    if (!t) return nullptr;
    PyTuple_SET_ITEM(t, 0, THPVariable_Wrap(std::move(dq)));
    PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(std::move(dk)));
    PyTuple_SET_ITEM(t, 2, THPVariable_Wrap(std::move(dv)));
    return t;
}

// mhsa_fwd(X, weights, lengths, sample_idx, u_rule, factor, fill, Y, workspace); `weights`: anything whose buffer is a
// psa_mhsa_weights_t (the ctypes structure of the binding)
PyObject* mhsa_fwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Arg x, len, idx, y, ws;
    psa_options_t opt;
    if (n != 9 || !take(a[0], x, false) || !take(a[2], len, true) || !take(a[3], idx, false) ||
        !option_args(a[4], a[5], a[6], &opt) || !take(a[7], y, true) || !take(a[8], ws, true)) return none();
    if (x.t->dim() != 3 || idx.t->dim() < 1) return none();
    psa_shape_t s;
    s.B = (int32_t)x.t->size(0); s.H = (int32_t)(x.t->size(2) / 64); s.L_Q = s.L_K = (int32_t)x.t->size(1); s.D = 64;
    s.U = (int32_t)idx.t->size(-1);
    if (!dtype_of(*x.t, &s.dtype)) return none();
    Py_buffer view;
    if (PyObject_GetBuffer(a[1], &view, PyBUF_SIMPLE) != 0) { PyErr_Clear(); return none(); }
    psa_mhsa_weights_t w;
    const bool whole = view.len == (Py_ssize_t)sizeof(w);
    if (whole) w = *static_cast<const psa_mhsa_weights_t*>(view.buf);
    PyBuffer_Release(&view);
    if (!whole) return none();
    at::Tensor made, room;
    const size_t bytes = ws.t ? (size_t)ws.t->numel() : probsparse_mhsa_workspace_bytes(&s, &opt);
    if (bytes == 0) return none();
    int rc;
    {
        const Unlocked unlocked;
        if (!ws.t) { room = scratch(*x.t, bytes); ws.ptr = room.data_ptr(); }
        if (!y.t) { made = at::empty_like(*x.t); y.ptr = made.data_ptr(); }
        rc = probsparse_mhsa_fwd(x.ptr, &w, static_cast<const int32_t*>(len.ptr), static_cast<const int32_t*>(idx.ptr),
                                 &opt, y.ptr, &s, ws.ptr, bytes, stream());
    }
    return rc == PSA_OK ? result(a[7], std::move(made)) : failed(rc);
}

// exceptions of the tensor library (no memory, say) must not cross into the interpreter: the caller's path meets them
// again and reports them
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    try {
        return F(self, a, n);
    } catch (const std::exception&) {
        return none();
    }
}
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyCFunction entry() { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<F>)); }

PyMethodDef methods[] = {
    {"attn_fwd", entry<attn_fwd>(), METH_FASTCALL, nullptr},
    {"attn_fwd_opt", entry<attn_fwd_opt>(), METH_FASTCALL, nullptr},
    {"attn_fwd_with_indices", entry<attn_fwd_with_indices>(), METH_FASTCALL, nullptr},
    {"attn_bwd", entry<attn_bwd>(), METH_FASTCALL, nullptr},
    {"mhsa_fwd", entry<mhsa_fwd>(), METH_FASTCALL, nullptr},
    {"on_status", on_status, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
