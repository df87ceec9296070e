// The attention calls' way from Python to the C entry points: layout checks, outputs and argument blocks of memo_attn_fwd,
// memo_attn_bwd and memo_attn_bwd_static in one native call each.  The kernels of a short forward and backward take 13 to 16 us, and
// with the same work in Python (ctypes, some 60 property reads) the host took 17.6 us to queue a forward and a static backward, 26.2 with the outputs
// allocated; now 10.6 and 16.5, launches included.
//
// Only plain device tensors that pass every check are taken.  For anything else (another layout or type, subclasses, wrapped
// or lazy tensors, modes that intercept calls) the functions return None, and the Python code beside the call does what
// it does for every tensor, errors included.  A call that the library refuses returns the status.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

#include <algorithm>
#include <initializer_list>

#include "../../include/memo.h"

namespace {

using FwdFn = decltype(&memo_attn_fwd);
using BwdFn = decltype(&memo_attn_bwd);
using StaticFn = decltype(&memo_attn_bwd_static);
using BytesFn = decltype(&memo_attn_bwd_workspace_bytes);

bool intercepted()
{
    return c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled();
}

// The tensor of obj if it is a plain strided one on a device, else null.
const at::Tensor *plain(PyObject *obj)
{
    if (!THPVariable_CheckExact(obj)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(obj);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda()) return nullptr;
    const c10::DispatchKeySet usual({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::ADInplaceOrView,
                                     c10::DispatchKey::AutocastCUDA});
    if (t.key_set().raw_repr() & ~usual.raw_repr()) return nullptr;
    return &t;
}

bool same_layout(const at::Tensor &ref, std::initializer_list<const at::Tensor *> others)
{
    for (const at::Tensor *t : others)
        if (!t || t->sizes() != ref.sizes() || t->strides() != ref.strides() || t->scalar_type() != ref.scalar_type() ||
            t->device() != ref.device())
            return false;
    return true;
}

bool describe(const at::Tensor &q, PyObject *scale, memo_attn_desc *d)
{
    if (q.dim() != 4 || q.stride(3) != 1 || !PyFloat_CheckExact(scale)) return false;
    if (q.scalar_type() != at::kFloat && q.scalar_type() != at::kBFloat16) return false;
    if (q.size(0) > INT32_MAX || q.size(2) > INT32_MAX || q.size(3) > INT32_MAX) return false;
    *d = {};
    d->B = (int32_t)q.size(0);
    d->S = q.size(1);
    d->H = (int32_t)q.size(2);
    d->d = (int32_t)q.size(3);
    d->dtype = q.scalar_type() == at::kFloat ? MEMO_F32 : MEMO_BF16;
    d->scale = (float)PyFloat_AS_DOUBLE(scale);
    d->stride_b = q.stride(0);
    d->stride_s = q.stride(1);
    d->stride_h = q.stride(2);
    d->causal = 1;
    return true;
}

// The logsumexp of the problem `d` on q's device.
bool holds_lse(const at::Tensor &lse, const at::Tensor &q, const memo_attn_desc &d)
{
    return lse.scalar_type() == at::kFloat && lse.is_contiguous() && lse.device() == q.device() && lse.numel() == (int64_t)d.B * d.H * d.S;
}

// A workspace on q's device with as many bytes behind its first element as it has elements, which is the size it is passed on with.
bool holds_bytes(const at::Tensor &t, const at::Tensor &q)
{
    return t.device() == q.device() && t.scalar_type() == at::kByte && t.is_contiguous() &&
           (int64_t)t.storage().nbytes() - t.storage_offset() >= t.numel();
}

template <typename Fn>
Fn address(PyObject *obj)
{
    return reinterpret_cast<Fn>(PyLong_AsVoidPtr(obj));
}

// Outputs and workspaces are allocated without the interpreter's lock, as torch's own functions do: the allocator may have to wait for the
// device.
struct OthersMayRun {
    PyThreadState *const state = PyEval_SaveThread();
    ~OthersMayRun() { PyEval_RestoreThread(state); }
};

at::Tensor new_like(at::Tensor like)     // a copy: nothing that another thread does to the Python object takes it away
{
    const OthersMayRun here;
    return at::empty_like(like);
}

at::Tensor new_tensor(at::IntArrayRef sizes, const at::TensorOptions &options)
{
    const OthersMayRun here;
    return at::empty(sizes, options);
}

// The stream's handle, as the binding finds it (find(stream)): after the checks, so that their errors come first.
// kOther: no integer that fits a pointer; the Python code takes what ctypes takes (None, a c_void_p ..).
enum Handle { kFound, kOther, kFailed };
Handle stream_handle(PyObject *find, PyObject *stream, void **out)
{
    PyObject *handle = PyObject_CallOneArg(find, stream);
    if (!handle) return kFailed;
    Handle found = kOther;
    if (PyLong_Check(handle)) {
        *out = PyLong_AsVoidPtr(handle);
        if (PyErr_Occurred()) PyErr_Clear();
        else found = kFound;
    }
    Py_DECREF(handle);
    return found;
}

PyObject *wrap(PyObject *given, const at::Tensor &t)
{
    if (given == Py_None) return THPVariable_Wrap(t);
    Py_INCREF(given);
    return given;
}

// (address, find stream, q, k, v, scale, o or None, lse or None, stream) -> (o, lse), a status or None
PyObject *attn_fwd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 9 || intercepted()) Py_RETURN_NONE;
    const at::Tensor *q = plain(a[2]), *k = plain(a[3]), *v = plain(a[4]);
    memo_attn_desc desc;
    if (!q || !same_layout(*q, {k, v}) || !describe(*q, a[5], &desc)) Py_RETURN_NONE;
    const at::Tensor *given_o = a[6] == Py_None ? nullptr : plain(a[6]), *given_lse = a[7] == Py_None ? nullptr : plain(a[7]);
    if ((a[6] != Py_None && !given_o) || (a[7] != Py_None && !given_lse)) Py_RETURN_NONE;
    const at::Tensor o = given_o ? *given_o : new_like(*q);
    const at::Tensor lse = given_lse ? *given_lse : new_tensor({desc.B, desc.H, desc.S}, q->options().dtype(at::kFloat));
    if (!same_layout(*q, {&o}) || !holds_lse(lse, *q, desc) || lse.dim() != 3 || lse.size(0) != desc.B || lse.size(1) != desc.H)
        Py_RETURN_NONE;
    void *stream = nullptr;
    const Handle found = stream_handle(a[1], a[8], &stream);
    if (found == kFailed) return nullptr;
    if (found == kOther) Py_RETURN_NONE;
    const FwdFn fn = address<FwdFn>(a[0]);
    const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr();
    void *op = o.data_ptr();
    float *lp = static_cast<float *>(lse.data_ptr());
    memo_status st;
    Py_BEGIN_ALLOW_THREADS
    st = fn(&desc, qp, kp, vp, op, lp, stream);
    Py_END_ALLOW_THREADS
    if (st != MEMO_OK) return PyLong_FromLong(st);
    return Py_BuildValue("(NN)", wrap(a[6], o), wrap(a[7], lse));
    END_HANDLE_TH_ERRORS
}

// (address, address of the workspace query, find stream, q, k, v, o, lse, d_o, scale, dq, dk, dv, workspace, stream) -> (dq, dk, dv), a
// status or None; dq, dk, dv and the workspace may be None.  Without a workspace query the call is the static one, whose outputs
// are all given.
PyObject *attn_bwd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 15 || intercepted()) Py_RETURN_NONE;
    const at::Tensor *q = plain(a[3]), *k = plain(a[4]), *v = plain(a[5]), *o = plain(a[6]), *lse = plain(a[7]), *g = plain(a[8]);
    memo_attn_desc desc;
    if (!q || !lse || !same_layout(*q, {k, v, o, g}) || !describe(*q, a[9], &desc) || !holds_lse(*lse, *q, desc)) Py_RETURN_NONE;
    const bool is_static = a[1] == Py_None;
    at::Tensor out[3], workspace;
    for (int i = 0; i < 3; ++i) {
        const at::Tensor *t = a[10 + i] == Py_None ? nullptr : plain(a[10 + i]);
        if (!t && (a[10 + i] != Py_None || is_static)) Py_RETURN_NONE;
        out[i] = t ? *t : new_like(*q);
    }
    if (!same_layout(*q, {&out[0], &out[1], &out[2]})) Py_RETURN_NONE;
    if (!is_static) {
        const at::Tensor *t = a[13] == Py_None ? nullptr : plain(a[13]);
        if (a[13] != Py_None && (!t || !holds_bytes(*t, *q))) Py_RETURN_NONE;
        workspace = t ? *t : new_tensor({(int64_t)std::max<size_t>(address<BytesFn>(a[1])(&desc), 256)}, q->options().dtype(at::kByte));
    }
    void *stream = nullptr;
    const Handle found = stream_handle(a[2], a[14], &stream);
    if (found == kFailed) return nullptr;
    if (found == kOther) Py_RETURN_NONE;
    const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr(), *op = o->data_ptr(), *gp = g->data_ptr();
    const float *lp = static_cast<const float *>(lse->data_ptr());
    void *dq = out[0].data_ptr(), *dk = out[1].data_ptr(), *dv = out[2].data_ptr(), *ws = is_static ? nullptr : workspace.data_ptr();
    const size_t ws_bytes = is_static ? 0 : (size_t)workspace.numel();
    void *fn = PyLong_AsVoidPtr(a[0]);
    memo_status st;
    Py_BEGIN_ALLOW_THREADS
    if (is_static) st = reinterpret_cast<StaticFn>(fn)(&desc, qp, kp, vp, op, lp, gp, dq, dk, dv, stream);
    else st = reinterpret_cast<BwdFn>(fn)(&desc, qp, kp, vp, op, lp, gp, dq, dk, dv, ws, ws_bytes, stream);
    Py_END_ALLOW_THREADS
    if (st != MEMO_OK) return PyLong_FromLong(st);
    return Py_BuildValue("(NNN)", wrap(a[10], out[0]), wrap(a[11], out[1]), wrap(a[12], out[2]));
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"attn_fwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(attn_fwd)), METH_FASTCALL, nullptr},
    {"attn_bwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(attn_bwd)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
