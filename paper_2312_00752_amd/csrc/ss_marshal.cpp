// The binding's hot calls without ctypes: tensors in, parameter struct filled, library called.  A call marshals ten to
// twenty tensors, and in Python the checks, the struct's fields and the foreign call were most of the time of a short one.
// us per call among others, through ctypes / here: one token of a layer, D 4096, batch 1 13.8 / 8.9, of the scan, batch 64 9.6 / 7.6 (its kernel
// 7.1); forward + backward of 1 x 64 x 256 float32 through autograd 199 / 144.
//
// Only the plain case is served: exact torch.Tensors (or Parameters) with memory of their own, on the GPU, contiguous, of the expected
// type and shape.  Everything else returns None before anything has been allocated or enqueued, and binding.py takes it
// through its own marshalling, which raises what is to be raised.  Results: the call's tensors, or the library's error code as an int.
#include <Python.h>

#include <initializer_list>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "ss_layer.h"
#include "ss_scan.h"

namespace {

typedef std::initializer_list<int64_t> Shape;
constexpr int64_t CHANNEL_SKEW_BYTES = 66560;   // as binding.empty_channel_skewed

// Arguments of one call; `ok` falls when one of them is not the plain case.
struct Args {
    PyObject* const* a;
    bool ok = true;
    const at::Tensor* tensor(int i)
    {
        if (!THPVariable_CheckExact(a[i])) { ok = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(a[i]);
        if (!t.is_cuda() || !t.has_storage() || !t.is_contiguous()) { ok = false; return nullptr; }
        return &t;
    }
    // device pointer of argument i; None gives a null pointer where `optional`
    void* ptr(int i, at::ScalarType type, Shape shape, bool optional = false)
    {
        if (optional && a[i] == Py_None) return nullptr;
        const at::Tensor* t = ok ? tensor(i) : nullptr;
        if (!t) return nullptr;
        if (t->scalar_type() != type || !t->sizes().equals(at::IntArrayRef(shape))) { ok = false; return nullptr; }
        return t->data_ptr();
    }
    bool none(int i) const { return a[i] == Py_None; }
    long number(int i)
    {
        const long v = PyLong_AsLong(a[i]);
        if (v == -1 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return v;
    }
    void* stream(int i)
    {
        void* v = PyLong_AsVoidPtr(a[i]);
        if (!v && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return v;
    }
};

bool io_type(const at::Tensor& t, int32_t& code)
{
    if (t.scalar_type() == at::kFloat) code = SS_F32;
    else if (t.scalar_type() == at::kBFloat16) code = SS_BF16;
    else return false;
    return true;
}
inline bool fits(int64_t v) { return v >= 0 && v <= 0x7fffffff; }

template <typename P, typename F>
int call(F f, const P& p, void* stream)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f(&p, stream);
    Py_END_ALLOW_THREADS
    return rc;
}
PyObject* wrapped(const at::Tensor& t) { return THPVariable_Wrap(t); }
at::Tensor empty_f32(at::IntArrayRef shape, const at::Tensor& like) { return at::empty(shape, like.options().dtype(at::kFloat).requires_grad(false)); }

// step(h, u_t, delta_t, A, B_t, C_t, Dskip, z_t, delta_bias, out_t, flags, stream) -> out_t
PyObject* py_step(PyObject*, PyObject* const* argv, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 12) Py_RETURN_NONE;
    Args a{argv};
    const at::Tensor *h = a.tensor(0), *u = a.ok ? a.tensor(1) : nullptr;
    if (!a.ok || h->dim() != 3) Py_RETURN_NONE;
    const int64_t nb = h->size(0), nd = h->size(1), nn = h->size(2);
    ss_step_params p{};
    if (!io_type(*u, p.io_dtype) || !fits(nb) || !fits(nd) || !fits(nn)) Py_RETURN_NONE;
    const at::ScalarType io = u->scalar_type(), f32 = at::kFloat;
    p.batch = (int32_t)nb; p.dim = (int32_t)nd; p.dstate = (int32_t)nn;
    p.flags = (uint32_t)a.number(10);
    const bool bfix = p.flags & SS_B_FIXED, cfix = p.flags & SS_C_FIXED;
    p.h = static_cast<float*>(a.ptr(0, f32, {nb, nd, nn}));
    p.u_t = a.ptr(1, io, {nb, nd});
    p.delta_t = a.ptr(2, io, {nb, nd});
    p.A = static_cast<const float*>(a.ptr(3, f32, {nd, nn}));
    p.B_t = bfix ? a.ptr(4, f32, {nd, nn}) : a.ptr(4, io, {nb, nn});
    p.C_t = cfix ? a.ptr(5, f32, {nd, nn}) : a.ptr(5, io, {nb, nn});
    p.Dskip = static_cast<const float*>(a.ptr(6, f32, {nd}, true));
    p.z_t = a.ptr(7, io, {nb, nd}, true);
    p.delta_bias = static_cast<const float*>(a.ptr(8, f32, {nd}, true));
    void* out = a.ptr(9, io, {nb, nd}, true);
    void* stream = a.stream(11);
    if (!a.ok) Py_RETURN_NONE;
    if (!a.none(6)) p.flags |= SS_HAS_D;
    if (!a.none(7)) p.flags |= SS_HAS_Z;
    if (!a.none(8)) p.flags |= SS_HAS_DELTA_BIAS;
    at::Tensor fresh;
    if (a.none(9)) {
        fresh = at::empty_like(*u);
        out = fresh.data_ptr();
    }
    p.out_t = out;
    const int rc = call(ss_step, p, stream);
    if (rc != SS_OK) return PyLong_FromLong(rc);
    if (a.none(9)) return wrapped(fresh);
    Py_INCREF(argv[9]);
    return argv[9];
    END_HANDLE_TH_ERRORS
}

// layer_step(h, conv_state, x_t, z_t, conv_w, conv_b, W_x, W_dt, dt_bias, A, Dskip, scratch, out_t, stream) -> out_t
PyObject* py_layer_step(PyObject*, PyObject* const* argv, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 14) Py_RETURN_NONE;
    Args a{argv};
    const at::Tensor* h = a.tensor(0);
    const at::Tensor* x = a.ok ? a.tensor(2) : nullptr;
    const at::Tensor* cw = a.ok ? a.tensor(4) : nullptr;
    const at::Tensor* wdt = a.ok ? a.tensor(7) : nullptr;
    const at::Tensor* scratch = a.ok ? a.tensor(11) : nullptr;
    if (!a.ok || h->dim() != 3 || cw->dim() != 2 || wdt->dim() != 2 || scratch->scalar_type() != at::kByte) Py_RETURN_NONE;
    const int64_t nb = h->size(0), nd = h->size(1), nn = h->size(2), width = cw->size(1), rank = wdt->size(1);
    ss_layer_step_params p{};
    if (!io_type(*x, p.io_dtype) || !fits(nb) || !fits(nd) || !fits(nn) || !fits(rank) || width < 1 || !fits(width)) Py_RETURN_NONE;
    const at::ScalarType io = x->scalar_type(), f32 = at::kFloat;
    p.batch = (int32_t)nb; p.dim = (int32_t)nd; p.dstate = (int32_t)nn; p.dt_rank = (int32_t)rank; p.conv_width = (int32_t)width;
    p.h = static_cast<float*>(a.ptr(0, f32, {nb, nd, nn}));
    p.conv_state = a.ptr(1, io, {nb, nd, width - 1});
    p.x_t = a.ptr(2, io, {nb, nd});
    p.z_t = a.ptr(3, io, {nb, nd});
    p.conv_w = static_cast<const float*>(a.ptr(4, f32, {nd, width}));
    p.conv_b = static_cast<const float*>(a.ptr(5, f32, {nd}));
    p.W_x = a.ptr(6, io, {rank + 2 * nn, nd});
    p.W_dt = a.ptr(7, io, {nd, rank});
    p.dt_bias = static_cast<const float*>(a.ptr(8, f32, {nd}));
    p.A = static_cast<const float*>(a.ptr(9, f32, {nd, nn}));
    p.Dskip = static_cast<const float*>(a.ptr(10, f32, {nd}));
    void* out = a.ptr(12, io, {nb, nd}, true);
    void* stream = a.stream(13);
    if (!a.ok) Py_RETURN_NONE;
    p.scratch = scratch->data_ptr();
    p.scratch_bytes = (size_t)scratch->numel();
    at::Tensor fresh;
    if (a.none(12)) {
        fresh = at::empty_like(*x);
        out = fresh.data_ptr();
    }
    p.out_t = out;
    const int rc = call(ss_layer_step, p, stream);
    if (rc != SS_OK) return PyLong_FromLong(rc);
    if (a.none(12)) return wrapped(fresh);
    Py_INCREF(argv[12]);
    return argv[12];
    END_HANDLE_TH_ERRORS
}

// The scan's inputs: u, delta, A, B, C, Dskip, z, delta_bias, h0 from argument `at` on; real state.
bool scan_inputs(Args& a, int at, uint32_t flags, ss_fwd_params& p)
{
    const at::Tensor *u = a.tensor(at), *A = a.ok ? a.tensor(at + 2) : nullptr;
    const at::Tensor *B = a.ok ? a.tensor(at + 3) : nullptr, *C = a.ok ? a.tensor(at + 4) : nullptr;
    if (!a.ok || u->dim() != 3 || A->dim() != 2 || !io_type(*u, p.io_dtype)) return false;
    const int64_t nb = u->size(0), nd = u->size(1), nl = u->size(2), nn = A->size(1);
    if (!fits(nb) || !fits(nd) || !fits(nl) || !fits(nn)) return false;
    const at::ScalarType io = u->scalar_type(), f32 = at::kFloat;
    p.batch = (int32_t)nb; p.dim = (int32_t)nd; p.seqlen = (int32_t)nl; p.dstate = (int32_t)nn;
    p.flags = flags;
    p.u = a.ptr(at, io, {nb, nd, nl});
    p.delta = a.ptr(at + 1, io, {nb, nd, nl});
    p.A = static_cast<const float*>(a.ptr(at + 2, f32, {nd, nn}));
    if (B->dim() == 2) p.flags |= SS_B_FIXED;   // (D,N): the time-invariant form
    if (C->dim() == 2) p.flags |= SS_C_FIXED;
    p.Bmat = B->dim() == 2 ? a.ptr(at + 3, f32, {nd, nn}) : a.ptr(at + 3, io, {nb, nn, nl});
    p.Cmat = C->dim() == 2 ? a.ptr(at + 4, f32, {nd, nn}) : a.ptr(at + 4, io, {nb, nn, nl});
    p.Dskip = static_cast<const float*>(a.ptr(at + 5, f32, {nd}, true));
    p.z = a.ptr(at + 6, io, {nb, nd, nl}, true);
    p.delta_bias = static_cast<const float*>(a.ptr(at + 7, f32, {nd}, true));
    p.h0 = static_cast<const float*>(a.ptr(at + 8, f32, {nb, nd, nn}, true));
    if (!a.none(at + 5)) p.flags |= SS_HAS_D;
    if (!a.none(at + 6)) p.flags |= SS_HAS_Z;
    if (!a.none(at + 7)) p.flags |= SS_HAS_DELTA_BIAS;
    if (!a.none(at + 8)) p.flags |= SS_HAS_H0;
    return a.ok;
}
bool workspace_of(Args& a, int i, ss_fwd_params& p)
{
    const at::Tensor* ws = a.tensor(i);
    if (!ws || ws->scalar_type() != at::kByte) return false;
    p.workspace = ws->data_ptr();
    p.workspace_bytes = (size_t)ws->numel();
    return true;
}

// scan_fwd(u, delta, A, B, C, Dskip, z, delta_bias, h0, workspace, flags, want_last, stream) -> (out, h_last or None)
PyObject* py_scan_fwd(PyObject*, PyObject* const* argv, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 13) Py_RETURN_NONE;
    Args a{argv};
    ss_fwd_params p{};
    const uint32_t flags = (uint32_t)a.number(10);
    const bool last = argv[11] == Py_True;
    void* stream = a.stream(12);
    if (!a.ok || !scan_inputs(a, 0, flags, p)) Py_RETURN_NONE;
    if (a.none(9)) p.flags &= ~(uint32_t)SS_SAVE_FOR_BWD;
    else if (!workspace_of(a, 9, p)) Py_RETURN_NONE;
    const at::Tensor& u = *a.tensor(0);
    at::Tensor out = at::empty_like(u), h_last;
    p.out = out.data_ptr();
    if (last) {
        h_last = empty_f32({p.batch, p.dim, p.dstate}, u);
        p.h_last = static_cast<float*>(h_last.data_ptr());
        p.flags |= SS_WRITE_H_LAST;
    }
    const int rc = call(ss_scan_fwd, p, stream);
    if (rc != SS_OK) return PyLong_FromLong(rc);
    PyObject* res = PyTuple_New(2);
    if (!res) return nullptr;
    PyTuple_SET_ITEM(res, 0, wrapped(out));
    if (last) PyTuple_SET_ITEM(res, 1, wrapped(h_last));
    else { Py_INCREF(Py_None); PyTuple_SET_ITEM(res, 1, Py_None); }
    return res;
    END_HANDLE_TH_ERRORS
}

// scan_bwd(u, delta, A, B, C, Dskip, z, delta_bias, h0, workspace, dout, dh_last, flags, want_dh0, stream) -> dict of gradients
PyObject* py_scan_bwd(PyObject*, PyObject* const* argv, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 15) Py_RETURN_NONE;
    Args a{argv};
    ss_bwd_params q{};
    const uint32_t flags = (uint32_t)a.number(12);
    const bool want_dh0 = argv[13] == Py_True;
    void* stream = a.stream(14);
    if (!a.ok || !scan_inputs(a, 0, flags, q.fwd) || !workspace_of(a, 9, q.fwd)) Py_RETURN_NONE;
    const at::Tensor &u = *a.tensor(0), &A = *a.tensor(2), &B = *a.tensor(3), &C = *a.tensor(4);
    const int64_t nb = u.size(0), nd = u.size(1), nl = u.size(2), nn = A.size(1);
    q.dout = a.ptr(10, u.scalar_type(), {nb, nd, nl});
    q.dh_last = static_cast<const float*>(a.ptr(11, at::kFloat, {nb, nd, nn}, true));
    if (!a.ok) Py_RETURN_NONE;
    // du, ddelta and dz in one allocation, 65 KiB further apart than their size (binding.empty_channel_skewed)
    const bool has_z = !a.none(6);
    const int64_t esz = (int64_t)u.element_size(), pitch = ((u.numel() * esz + 255) / 256 * 256 + CHANNEL_SKEW_BYTES) / esz;
    const at::Tensor pool = at::empty({(has_z ? 3 : 2) * pitch}, u.options().requires_grad(false));
    const int64_t row = nl > 1 ? nl : 1, entry = row * (nd > 1 ? nd : 1);
    auto carve = [&](int64_t i) { return at::as_strided(pool, u.sizes(), {entry, row, 1}, i * pitch); };
    at::Tensor du = carve(0), ddelta = carve(1), dz, dD, dbias, dh0;
    at::Tensor dB = empty_f32(B.sizes(), u), dC = empty_f32(C.sizes(), u), dA = empty_f32(A.sizes(), u);
    if (has_z) dz = carve(2);
    if (!a.none(5)) dD = empty_f32({nd}, u);
    if (!a.none(7)) dbias = empty_f32({nd}, u);
    if (want_dh0) dh0 = empty_f32({nb, nd, nn}, u);
    auto f = [](const at::Tensor& t) { return t.defined() ? static_cast<float*>(t.data_ptr()) : nullptr; };
    q.du = du.data_ptr(); q.ddelta = ddelta.data_ptr(); q.dz = has_z ? dz.data_ptr() : nullptr;
    q.dB = f(dB); q.dC = f(dC); q.dA = f(dA); q.dD = f(dD); q.ddelta_bias = f(dbias); q.dh0 = f(dh0);
    const int rc = call(ss_scan_bwd, q, stream);
    if (rc != SS_OK) return PyLong_FromLong(rc);
    PyObject* res = PyDict_New();
    if (!res) return nullptr;
    auto put = [&](const char* name, const at::Tensor& t) {
        PyObject* o = t.defined() ? wrapped(t) : (Py_INCREF(Py_None), Py_None);
        const bool good = o && PyDict_SetItemString(res, name, o) == 0;
        Py_XDECREF(o);
        return good;
    };
    if (!(put("du", du) && put("ddelta", ddelta) && put("dz", dz) && put("dB", dB) && put("dC", dC) && put("dA", dA) && put("dD", dD) &&
          put("ddelta_bias", dbias) && put("dh0", dh0))) {
        Py_DECREF(res);
        return nullptr;
    }
    return res;
    END_HANDLE_TH_ERRORS
}

// The layer's inputs from argument `at` on: x, z, conv_w, conv_b, W_x, W_dt, dt_bias, A, Dskip, scratch, saved (or None).
bool layer_inputs(Args& a, int at, ss_layer_params& p)
{
    const at::Tensor* x = a.tensor(at);
    const at::Tensor* cw = a.ok ? a.tensor(at + 2) : nullptr;
    const at::Tensor* wdt = a.ok ? a.tensor(at + 5) : nullptr;
    const at::Tensor* A = a.ok ? a.tensor(at + 7) : nullptr;
    const at::Tensor* scratch = a.ok ? a.tensor(at + 9) : nullptr;
    if (!a.ok || x->dim() != 3 || cw->dim() != 2 || wdt->dim() != 2 || A->dim() != 2 || scratch->scalar_type() != at::kByte) return false;
    const int64_t nb = x->size(0), nd = x->size(1), nl = x->size(2), nn = A->size(1), width = cw->size(1), rank = wdt->size(1);
    if (!io_type(*x, p.io_dtype) || !fits(nb) || !fits(nd) || !fits(nl) || !fits(nn) || !fits(rank) || width < 1 || !fits(width)) return false;
    const at::ScalarType io = x->scalar_type(), f32 = at::kFloat;
    p.batch = (int32_t)nb; p.dim = (int32_t)nd; p.seqlen = (int32_t)nl; p.dstate = (int32_t)nn; p.dt_rank = (int32_t)rank; p.conv_width = (int32_t)width;
    p.x = a.ptr(at, io, {nb, nd, nl});
    p.z = a.ptr(at + 1, io, {nb, nd, nl});
    p.conv_w = static_cast<const float*>(a.ptr(at + 2, f32, {nd, width}));
    p.conv_b = static_cast<const float*>(a.ptr(at + 3, f32, {nd}));
    p.W_x = a.ptr(at + 4, io, {rank + 2 * nn, nd});
    p.W_dt = a.ptr(at + 5, io, {nd, rank});
    p.dt_bias = static_cast<const float*>(a.ptr(at + 6, f32, {nd}));
    p.A = static_cast<const float*>(a.ptr(at + 7, f32, {nd, nn}));
    p.Dskip = static_cast<const float*>(a.ptr(at + 8, f32, {nd}));
    p.scratch = scratch->data_ptr();
    p.scratch_bytes = (size_t)scratch->numel();
    if (a.ok && !a.none(at + 10)) {
        const at::Tensor* saved = a.tensor(at + 10);
        if (!saved || saved->scalar_type() != at::kByte) return false;
        p.saved = saved->data_ptr();
        p.saved_bytes = (size_t)saved->numel();
    }
    return a.ok;
}

// layer_fwd(x .. saved, return_states, stream) -> out, or (out, h_last, conv_state)
PyObject* py_layer_fwd(PyObject*, PyObject* const* argv, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 13) Py_RETURN_NONE;
    Args a{argv};
    ss_layer_params p{};
    const bool states = argv[11] == Py_True;
    void* stream = a.stream(12);
    if (!a.ok || !layer_inputs(a, 0, p)) Py_RETURN_NONE;
    const at::Tensor& x = *a.tensor(0);
    at::Tensor out = at::empty_like(x), h_last, conv_state;
    p.out = out.data_ptr();
    if (states) {
        h_last = empty_f32({p.batch, p.dim, p.dstate}, x);
        conv_state = at::empty({p.batch, p.dim, p.conv_width - 1}, x.options().requires_grad(false));
        p.h_last = static_cast<float*>(h_last.data_ptr());
        p.conv_state = conv_state.data_ptr();
    }
    const int rc = call(ss_layer_fwd, p, stream);
    if (rc != SS_OK) return PyLong_FromLong(rc);
    if (!states) return wrapped(out);
    PyObject* res = PyTuple_New(3);
    if (!res) return nullptr;
    PyTuple_SET_ITEM(res, 0, wrapped(out));
    PyTuple_SET_ITEM(res, 1, wrapped(h_last));
    PyTuple_SET_ITEM(res, 2, wrapped(conv_state));
    return res;
    END_HANDLE_TH_ERRORS
}

// layer_bwd(x .. saved, dout, stream) -> dict of gradients
PyObject* py_layer_bwd(PyObject*, PyObject* const* argv, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 13) Py_RETURN_NONE;
    Args a{argv};
    ss_layer_bwd_params q{};
    void* stream = a.stream(12);
    if (!a.ok || !layer_inputs(a, 0, q.fwd)) Py_RETURN_NONE;
    const at::Tensor &x = *a.tensor(0), &cw = *a.tensor(2), &cb = *a.tensor(3), &wx = *a.tensor(4), &wdt = *a.tensor(5), &bias = *a.tensor(6),
                     &A = *a.tensor(7), &D = *a.tensor(8);
    q.dout = a.ptr(11, x.scalar_type(), {q.fwd.batch, q.fwd.dim, q.fwd.seqlen});
    if (!a.ok) Py_RETURN_NONE;
    const char* const names[] = {"dx", "dz", "dconv_w", "dconv_b", "dW_x", "dW_dt", "ddt_bias", "dA", "dD"};
    const at::Tensor g[] = {at::empty_like(x), at::empty_like(x), at::empty_like(cw), at::empty_like(cb), empty_f32(wx.sizes(), x),
                            empty_f32(wdt.sizes(), x), at::empty_like(bias), at::empty_like(A), at::empty_like(D)};
    auto f = [&](int i) { return static_cast<float*>(g[i].data_ptr()); };
    q.dx = g[0].data_ptr(); q.dz = g[1].data_ptr();
    q.dconv_w = f(2); q.dconv_b = f(3); q.dW_x = f(4); q.dW_dt = f(5); q.ddt_bias = f(6); q.dA = f(7); q.dD = f(8);
    const int rc = call(ss_layer_bwd, q, stream);
    if (rc != SS_OK) return PyLong_FromLong(rc);
    PyObject* res = PyDict_New();
    if (!res) return nullptr;
    for (int i = 0; i < 9; ++i) {
        PyObject* o = wrapped(g[i]);
        const bool good = o && PyDict_SetItemString(res, names[i], o) == 0;
        Py_XDECREF(o);
        if (!good) {
            Py_DECREF(res);
            return nullptr;
        }
    }
    return res;
    END_HANDLE_TH_ERRORS
}

#define SS_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(py_##name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SS_METHOD(step), SS_METHOD(layer_step), SS_METHOD(scan_fwd), SS_METHOD(scan_bwd),
                         SS_METHOD(layer_fwd), SS_METHOD(layer_bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
