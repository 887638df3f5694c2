// The Python calls of a layer's step - forward, input gradient, weight gradient, both gradients - without the interpreter:
// the checks of binding.py, the output allocation and the C call in one native function.  A call through binding.py is some
// thirty Python-level calls, about half of what a small call took from the host (B1 C256 L4096 K64 fp32 forward 7.0 us a call,
// 4.5-5.1 here, its kernel 4.7; B4 C64 L1024 K16, three calls 22.0 us, 12.7-14.8 here, its kernels 3.2 each).
//
// A function here does the call or returns None: anything but plain strided device tensors of a supported type, laid out as the
// library takes them, on the current device (subclasses, wrappers of transforms, active torch function or dispatch modes, traces,
// arguments that are not exact ints, mismatched shapes) is left to binding.py, whose checks and messages are the only ones.
// A status other than 0 is raised by binding.py's own exception.
//
// Built for one PyTorch and one Python (DWCONV_BUILT_FOR names them): it reads their objects by its headers' layouts.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include <climits>

namespace {

typedef int (*CorrFn)(const void *, const void *, void *, int, int, int, int, int, int, void *);
typedef int (*WeightFn)(const void *, const void *, void *, void *, size_t, int, int, int, int, int, int, void *);
typedef int (*BothFn)(const void *, const void *, const void *, void *, void *, void *, size_t, int, int, int, int, int, int, void *);

CorrFn fn_fwd, fn_bwd_input;
WeightFn fn_bwd_weight;
BothFn fn_bwd;
PyObject *current_device, *raw_stream, *check;       // binding.py's queries and its check of a status

// A tensor the library can take as it is, or nullptr.
const at::Tensor *plain(PyObject *o, int64_t dim, long device)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || t.get_device() != device) return nullptr;
    // (nothing but a device tensor under autograd and autocast: no wrapper of a transform, no lazy conjugate or negative)
    if ((t.key_set() - c10::autograd_dispatch_keyset_with_ADInplaceOrView - c10::autocast_dispatch_keyset).highestPriorityTypeId() !=
        c10::DispatchKey::CUDA)
        return nullptr;
    if ((dim >= 0 && t.dim() != dim) || !t.is_contiguous()) return nullptr;
    return &t;
}

int dtype_code(const at::Tensor &t)
{
    return t.scalar_type() == at::kFloat ? 0 : t.scalar_type() == at::kBFloat16 ? 1 : -1;
}

bool exact_int(PyObject *o, int &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long l = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || l < INT_MIN || l > INT_MAX) return false;
    v = (int)l;
    return true;
}

struct Call {
    long device = -1;
    void *stream = nullptr;
    // False (no error set): binding.py's turn; with an error set: the error.
    bool begin(PyObject *first)
    {
        // (the queries are there to be asked once a device tensor is)
        if (!THPVariable_CheckExact(first) || !THPVariable_Unpack(first).is_cuda()) return false;
        if (at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set() || torch::jit::tracer::isTracing())
            return false;
        PyObject *d = PyObject_CallNoArgs(current_device);
        if (!d) return false;
        device = PyLong_AsLong(d);
        PyObject *s = PyErr_Occurred() ? nullptr : PyObject_CallOneArg(raw_stream, d);
        Py_DECREF(d);
        if (!s) return false;
        stream = PyLong_AsVoidPtr(s);
        Py_DECREF(s);
        return !PyErr_Occurred();
    }
    bool bad() const { return PyErr_Occurred() != nullptr; }
};

// Without the interpreter's lock while it lives: around allocation and launch, either of which may wait (for memory, for a place in the
// queue, for code to be loaded) while other threads, or a host function the queue waits for, want the lock.
struct Unlocked {
    PyThreadState *state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked &) = delete;
    Unlocked &operator=(const Unlocked &) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

PyObject *decline() { Py_RETURN_NONE; }
bool raised(int status)
{
    if (status == 0) return false;
    PyObject *s = PyLong_FromLong(status), *r = s ? PyObject_CallOneArg(check, s) : nullptr;
    Py_XDECREF(s);
    Py_XDECREF(r);
    return true;
}

struct Dims {
    int B, C, L, K;
};
bool dims_of(const at::Tensor &x, int64_t K, Dims &d)
{
    if (x.size(0) > INT_MAX || x.size(1) > INT_MAX || x.size(2) > INT_MAX || K > INT_MAX) return false;
    d = Dims{(int)x.size(0), (int)x.size(1), (int)x.size(2), (int)K};
    return true;
}

// (in, filter, pad_left, out or None) -> out
PyObject *corr(CorrFn fn, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Call call;
    int pad;
    Dims d;
    if (n != 4 || !exact_int(a[2], pad)) return decline();
    if (!call.begin(a[0])) return call.bad() ? nullptr : decline();
    const at::Tensor *x = plain(a[0], 3, call.device), *w = plain(a[1], 2, call.device);
    if (!x || !w || w->scalar_type() != x->scalar_type() || w->size(0) != x->size(1) || !dims_of(*x, w->size(1), d)) return decline();
    const int code = dtype_code(*x);
    if (code < 0) return decline();
    const at::Tensor *out = nullptr;
    if (a[3] != Py_None) {
        out = plain(a[3], 3, call.device);
        if (!out || out->sizes() != x->sizes() || out->scalar_type() != x->scalar_type()) return decline();
    }
    const void *px = x->const_data_ptr(), *pw = w->const_data_ptr();
    void *py = out ? out->mutable_data_ptr() : nullptr;
    at::Tensor made;
    int status;
    {
        Unlocked unlocked;
        if (!out) {
            made = at::empty_like(*x);
            py = made.mutable_data_ptr();
        }
        status = fn(px, pw, py, d.B, d.C, d.L, d.K, pad, code, call.stream);
    }
    if (raised(status)) return nullptr;
    if (a[3] == Py_None) return THPVariable_Wrap(std::move(made));
    Py_INCREF(a[3]);
    return a[3];
    END_HANDLE_TH_ERRORS
}
PyObject *fwd(PyObject *, PyObject *const *a, Py_ssize_t n) { return corr(fn_fwd, a, n); }
PyObject *bwd_input(PyObject *, PyObject *const *a, Py_ssize_t n) { return corr(fn_bwd_input, a, n); }

// A [C, K] output of the caller's.
const at::Tensor *weight_out(PyObject *o, const at::Tensor &x, const Dims &d, long device)
{
    const at::Tensor *dw = plain(o, 2, device);
    return dw && dw->size(0) == d.C && dw->size(1) == d.K && dw->scalar_type() == x.scalar_type() ? dw : nullptr;
}

// (x, dy, K, pad_left, workspace, out or None) -> out
PyObject *bwd_weight(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Call call;
    int K, pad;
    Dims d;
    if (n != 6 || a[4] == Py_None || !exact_int(a[2], K) || K < 1 || !exact_int(a[3], pad)) return decline();
    if (!call.begin(a[0])) return call.bad() ? nullptr : decline();
    const at::Tensor *x = plain(a[0], 3, call.device), *dy = plain(a[1], 3, call.device), *ws = plain(a[4], -1, call.device);
    if (!x || !dy || !ws || dy->sizes() != x->sizes() || dy->scalar_type() != x->scalar_type() || !dims_of(*x, K, d)) return decline();
    const int code = dtype_code(*x);
    if (code < 0) return decline();
    const at::Tensor *out = nullptr;
    if (a[5] != Py_None && !(out = weight_out(a[5], *x, d, call.device))) return decline();
    const void *px = x->const_data_ptr(), *pdy = dy->const_data_ptr();
    void *pdw = out ? out->mutable_data_ptr() : nullptr, *pws = ws->mutable_data_ptr();
    const size_t bytes = ws->nbytes();
    at::Tensor made;
    int status;
    {
        Unlocked unlocked;
        if (!out) {
            made = at::empty({d.C, d.K}, x->options());
            pdw = made.mutable_data_ptr();
        }
        status = fn_bwd_weight(px, pdy, pdw, pws, bytes, d.B, d.C, d.L, d.K, pad, code, call.stream);
    }
    if (raised(status)) return nullptr;
    if (a[5] == Py_None) return THPVariable_Wrap(std::move(made));
    Py_INCREF(a[5]);
    return a[5];
    END_HANDLE_TH_ERRORS
}

// (dy, x, w, pad_left, workspace, out_dx or None, out_dw or None) -> (dx, dw)
PyObject *bwd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Call call;
    int pad;
    Dims d;
    if (n != 7 || a[4] == Py_None || !exact_int(a[3], pad)) return decline();
    if (!call.begin(a[0])) return call.bad() ? nullptr : decline();
    const at::Tensor *dy = plain(a[0], 3, call.device), *x = plain(a[1], 3, call.device), *w = plain(a[2], 2, call.device),
                     *ws = plain(a[4], -1, call.device);
    if (!dy || !x || !w || !ws || dy->sizes() != x->sizes() || dy->scalar_type() != x->scalar_type() || w->scalar_type() != x->scalar_type() ||
        w->size(0) != x->size(1) || !dims_of(*x, w->size(1), d))
        return decline();
    const int code = dtype_code(*x);
    if (code < 0) return decline();
    const at::Tensor *dx = nullptr, *dw = nullptr;
    if (a[5] != Py_None) {
        dx = plain(a[5], 3, call.device);
        if (!dx || dx->sizes() != dy->sizes() || dx->scalar_type() != dy->scalar_type()) return decline();
    }
    if (a[6] != Py_None && !(dw = weight_out(a[6], *x, d, call.device))) return decline();
    const void *pdy = dy->const_data_ptr(), *px = x->const_data_ptr(), *pw = w->const_data_ptr();
    void *pdx = dx ? dx->mutable_data_ptr() : nullptr, *pdw = dw ? dw->mutable_data_ptr() : nullptr, *pws = ws->mutable_data_ptr();
    const size_t bytes = ws->nbytes();
    at::Tensor made_dx, made_dw;
    int status;
    {
        Unlocked unlocked;
        if (!dx) {
            made_dx = at::empty_like(*dy);
            pdx = made_dx.mutable_data_ptr();
        }
        if (!dw) {
            made_dw = at::empty({d.C, d.K}, x->options());
            pdw = made_dw.mutable_data_ptr();
        }
        status = fn_bwd(pdy, px, pw, pdx, pdw, pws, bytes, d.B, d.C, d.L, d.K, pad, code, call.stream);
    }
    if (raised(status)) return nullptr;
    PyObject *out_dx = a[5], *out_dw = a[6];
    if (out_dx == Py_None) out_dx = THPVariable_Wrap(std::move(made_dx));
    else Py_INCREF(out_dx);
    if (out_dw == Py_None) out_dw = THPVariable_Wrap(std::move(made_dw));
    else Py_INCREF(out_dw);
    PyObject *pair = out_dx && out_dw ? PyTuple_Pack(2, out_dx, out_dw) : nullptr;
    Py_XDECREF(out_dx);
    Py_XDECREF(out_dw);
    return pair;
    END_HANDLE_TH_ERRORS
}

// setup(address of dwconv_fwd, dwconv_bwd_input, dwconv_bwd_weight, dwconv_bwd, current_device, raw_stream, check)
PyObject *setup(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 7) {
        PyErr_SetString(PyExc_TypeError, "setup takes seven arguments");
        return nullptr;
    }
    void *p[4];
    for (int i = 0; i < 4; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) return PyErr_Occurred() ? nullptr : decline();
    }
    fn_fwd = (CorrFn)p[0];
    fn_bwd_input = (CorrFn)p[1];
    fn_bwd_weight = (WeightFn)p[2];
    fn_bwd = (BothFn)p[3];
    PyObject **to[3] = {&current_device, &raw_stream, &check};
    for (int i = 0; i < 3; ++i) {
        Py_INCREF(a[4 + i]);
        Py_XSETREF(*to[i], a[4 + i]);
    }
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"setup", (PyCFunction)(void (*)())setup, METH_FASTCALL, nullptr},
    {"fwd", (PyCFunction)(void (*)())fwd, METH_FASTCALL, nullptr},
    {"bwd_input", (PyCFunction)(void (*)())bwd_input, METH_FASTCALL, nullptr},
    {"bwd_weight", (PyCFunction)(void (*)())bwd_weight, METH_FASTCALL, nullptr},
    {"bwd", (PyCFunction)(void (*)())bwd, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// (binding.py compares `built_for` with the PyTorch and the Python that are there before it calls anything)
PyMODINIT_FUNC PyInit__fastcall()
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", DWCONV_BUILT_FOR) < 0) Py_CLEAR(m);
    return m;
}
