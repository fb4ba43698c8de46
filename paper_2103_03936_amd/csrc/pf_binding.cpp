// The layers' calls from Python: argument checks, output tensors, workspace and the call into libpufferfish.so, natively.
// A small layer's kernels take 10 to 20 us; marshalling its arguments in Python (ctypes, torch.empty, current_stream)
// took 10 us forward and 15 us backward on top and bounded every small call.  Here a call costs its outputs' allocations and
// the launches.  Nothing is computed here.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "../../include/pufferfish.h"

namespace {

PyObject *g_error = nullptr, *g_no_memory = nullptr; // the package's PfError, torch.OutOfMemoryError

struct Fail { // a Python exception to raise
    PyObject *type;
    std::string what;
};
[[noreturn]] void fail(const std::string &what) { throw Fail{g_error, what}; }

using at::Tensor;
constexpr auto F32 = at::kFloat;
constexpr auto ANY = at::ScalarType::Undefined;

const Tensor &tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) throw Fail{PyExc_TypeError, "expected a tensor"};
    return THPVariable_Unpack(o);
}
void *address(const Tensor &t, at::ScalarType want)
{
    if (!t.is_cuda()) fail("tensors must live on the GPU; there is no CPU path");
    if (!t.is_contiguous()) fail("tensors must be contiguous");
    if (want != ANY && t.scalar_type() != want)
        fail(std::string("expected ") + c10::toString(want) + ", got " + c10::toString(t.scalar_type()));
    return t.data_ptr();
}
void *ptr(PyObject *o, at::ScalarType want = ANY) { return o == Py_None ? nullptr : address(tensor(o), want); }

int dtype_code(const Tensor &t)
{
    if (t.scalar_type() == at::kFloat) return PF_F32;
    if (t.scalar_type() == at::kBFloat16) return PF_BF16;
    fail(std::string("unsupported dtype ") + c10::toString(t.scalar_type()));
}
void dims(const Tensor &t, int n, const char *name)
{
    if (t.dim() != n) throw Fail{PyExc_ValueError, std::string(name) + " must have " + std::to_string(n) + " dimensions"};
}

// An output tensor (owned by Python once given out)
struct Out {
    Tensor t;
    void *p = nullptr;
    Out() {}
    Out(at::IntArrayRef size, at::ScalarType type, const at::Device &dev)
    {
        if (!dev.is_cuda()) fail("tensors must live on the GPU; there is no CPU path");
        t = Tensor(at::detail::empty_cuda(size, type, dev, std::nullopt));
        p = t.data_ptr();
    }
    PyObject *give()
    {
        if (!t.defined()) Py_RETURN_NONE;
        return THPVariable_Wrap(std::move(t));
    }
};
PyObject *tuple(std::initializer_list<PyObject *> items)
{
    PyObject *t = PyTuple_New((Py_ssize_t)items.size());
    Py_ssize_t i = 0;
    for (PyObject *o : items) PyTuple_SET_ITEM(t, i++, o);
    return t;
}
PyObject *borrowed(PyObject *o)
{
    Py_INCREF(o);
    return o;
}
PyObject *give_or(Out &o, PyObject *given) { return given ? borrowed(given) : o.give(); }

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

void check(int status, const char *what)
{
    if (status != PF_OK)
        fail(std::string(what) + ": status " + std::to_string(status) + " (" + pf_status_string(status) + "), hip error " +
             std::to_string(pf_last_hip_error()));
}

// A reusable byte buffer per (device, stream): calls enqueued on one stream are ordered, so they may share scratch
// memory; calls on different streams get different buffers.  It grows and never shrinks; one that is outgrown is kept
// alive rather than freed, so that graphs captured through these calls stay valid when a later call needs more.  Every call
// of the package takes it from here, those that Python marshals through lend(), and holds it until its launches are
// enqueued: of two threads' calls on one stream the second's launches follow the first's.
struct Space {
    void *p;
    size_t n;
};
struct Scratch {
    std::recursive_mutex busy; // (recursive: a finalizer may run a call while its thread has the buffer lent)
    Tensor t;
    std::vector<Tensor> retired;
    Space get(size_t bytes, const at::Device &dev)
    {
        if (!t.defined() || (size_t)t.numel() < bytes) {
            if (t.defined()) retired.push_back(t);
            t = Tensor(at::detail::empty_cuda({(int64_t)(bytes < 256 ? 256 : bytes)}, at::kByte, dev, std::nullopt));
        }
        return Space{t.data_ptr(), (size_t)t.numel()};
    }
};
Scratch &scratch(const at::Device &dev)
{
    static std::mutex lock;
    static auto &all = *new std::map<std::pair<int, void *>, Scratch>; // (never destroyed: the allocator may be gone)
    std::lock_guard<std::mutex> hold(lock);
    return all[{dev.index(), (void *)c10::hip::getCurrentHIPStream(dev.index()).stream()}];
}

// The interpreter runs other threads meanwhile
struct NoGil {
    PyThreadState *state = PyEval_SaveThread();
    NoGil() {}
    NoGil(const NoGil &) = delete;
    ~NoGil() { PyEval_RestoreThread(state); }
};
// f(scratch memory): the call into the library, which touches no Python object
template <class F>
void call(const char *what, size_t bytes, const at::Device &dev, F f)
{
    if (!dev.is_cuda()) fail("tensors must live on the GPU; there is no CPU path");
    int status;
    {
        NoGil released;
        Scratch &s = scratch(dev);
        std::lock_guard<std::recursive_mutex> hold(s.busy);
        status = f(s.get(bytes, dev));
    }
    check(status, what);
}
bool truth(PyObject *o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Fail{nullptr, ""};
    return v != 0;
}
long integer(PyObject *o)
{
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw Fail{nullptr, ""};
    return v;
}

template <PyObject *(*F)(PyObject *const *), int N>
PyObject *entry(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    try {
        return F(a);
    } catch (const Fail &f) {
        if (f.type) PyErr_SetString(f.type, f.what.c_str());
    } catch (const c10::OutOfMemoryError &e) {
        PyErr_SetString(g_no_memory, e.what());
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

// An owned reference
struct Ref {
    PyObject *o;
    explicit Ref(PyObject *owned = nullptr) : o(owned) {}
    Ref(const Ref &) = delete;
    Ref(Ref &&r) : o(r.o) { r.o = nullptr; }
    ~Ref() { Py_XDECREF(o); }
};

// parameter gradients: new tensors, or those of a given sequence of n (accumulated into; None: not wanted)
struct Grads {
    Ref items; // a list or tuple, which keeps them
    PyObject *g[3] = {nullptr, nullptr, nullptr};
    Out o[3];
    void *p[3] = {nullptr, nullptr, nullptr};
    bool given;
    Grads(PyObject *grads, int n) : given(grads != Py_None)
    {
        if (!given) return;
        items.o = PySequence_Fast(grads, "grads must be a sequence");
        if (!items.o) throw Fail{nullptr, ""};
        const Py_ssize_t have = PySequence_Fast_GET_SIZE(items.o);
        if (have != n)
            throw Fail{PyExc_ValueError, "grads must hold " + std::to_string(n) + " entries, not " + std::to_string(have)};
        for (int i = 0; i < n; ++i) {
            g[i] = PySequence_Fast_GET_ITEM(items.o, i);
            p[i] = ptr(g[i], F32);
        }
    }
    void make(int i, at::IntArrayRef size, const at::Device &dev)
    {
        o[i] = Out(size, F32, dev);
        p[i] = o[i].p;
    }
    PyObject *give(int i) { return give_or(o[i], g[i]); }
};

// ------------------------------------------------------------------ linear
pf_linear_desc linear_desc(const Tensor &X, const Tensor &U, bool bias)
{
    dims(X, 2, "X");
    dims(U, 2, "U");
    pf_linear_desc d = {};
    d.M = X.size(0);
    d.in = X.size(1);
    d.out = U.size(0);
    d.r = U.size(1);
    d.dtype = dtype_code(X);
    d.wgrad_dtype = PF_F32;
    d.has_bias = bias;
    return d;
}

// X, V, U, bias, residual, act, save_T, with epilogue
PyObject *linear_fwd(PyObject *const *a)
{
    const Tensor &X = tensor(a[0]), &U = tensor(a[2]);
    const pf_linear_desc d = linear_desc(X, U, a[3] != Py_None);
    const auto dt = X.scalar_type();
    const auto dev = X.device();
    Out Y({d.M, d.out}, dt, dev), T;
    if (truth(a[6])) T = Out({d.M, d.r}, dt, dev);
    void *const p[5] = {ptr(a[0], dt), ptr(a[1], dt), ptr(a[2], dt), ptr(a[3], dt), ptr(a[4], dt)}, *const st = stream();
    const size_t need = pf_lowrank_linear_fwd_workspace_bytes(&d);
    const int act = (int)integer(a[5]);
    if (truth(a[7]))
        call("pf_lowrank_linear_fwd_ep", need, dev, [&](Space ws) {
            return pf_lowrank_linear_fwd_ep(&d, p[0], p[1], p[2], p[3], p[4], act, Y.p, T.p, ws.p, ws.n, st);
        });
    else
        call("pf_lowrank_linear_fwd", need, dev,
             [&](Space ws) { return pf_lowrank_linear_fwd(&d, p[0], p[1], p[2], p[3], Y.p, T.p, ws.p, ws.n, st); });
    return tuple({Y.give(), T.give()});
}

// X, V, U, dY, T_saved, dX_add, x_is_relu, need_dX, has_bias, grads, with epilogue
PyObject *linear_bwd(PyObject *const *a)
{
    const Tensor &X = tensor(a[0]), &U = tensor(a[2]);
    const pf_linear_desc d = linear_desc(X, U, truth(a[8]));
    const auto dt = X.scalar_type();
    const auto dev = X.device();
    Out dX;
    if (truth(a[7])) dX = Out(X.sizes(), dt, dev);
    Grads g(a[9], 3);
    if (!g.given) {
        g.make(0, {d.out, d.r}, dev);
        g.make(1, {d.in, d.r}, dev);
        if (d.has_bias) g.make(2, {d.out}, dev);
    }
    void *const p[6] = {ptr(a[0], dt), ptr(a[1], dt), ptr(a[2], dt), ptr(a[3], dt), ptr(a[4], dt), ptr(a[5], dt)}, *const st = stream();
    const size_t need = pf_lowrank_linear_bwd_workspace_bytes(&d);
    const bool relu = truth(a[6]);
    if (truth(a[10]))
        call("pf_lowrank_linear_bwd_ep", need, dev, [&](Space ws) {
            return pf_lowrank_linear_bwd_ep(&d, p[0], p[1], p[2], p[3], p[4], p[5], relu, dX.p, g.p[0], g.p[1], g.p[2], g.given, ws.p, ws.n, st);
        });
    else
        call("pf_lowrank_linear_bwd", need, dev, [&](Space ws) {
            return pf_lowrank_linear_bwd(&d, p[0], p[1], p[2], p[3], p[4], dX.p, g.p[0], g.p[1], g.p[2], g.given, ws.p, ws.n, st);
        });
    return tuple({dX.give(), g.give(0), g.give(1), g.give(2)});
}

pf_linear_shared_desc shared_desc(const Tensor &X, const Tensor &U, bool bias)
{
    dims(X, 2, "X");
    dims(U, 3, "U");
    pf_linear_shared_desc d = {};
    d.M = X.size(0);
    d.n_in = X.size(1);
    d.groups = (int)U.size(0);
    d.n_out = U.size(1);
    d.r = U.size(2);
    d.dtype = dtype_code(X);
    d.has_bias = bias;
    return d;
}

// X, V, U, bias, save_T
PyObject *shared_fwd(PyObject *const *a)
{
    const Tensor &X = tensor(a[0]), &U = tensor(a[2]);
    const pf_linear_shared_desc d = shared_desc(X, U, a[3] != Py_None);
    const auto dt = X.scalar_type();
    const auto dev = X.device();
    Out Y({d.groups, d.M, d.n_out}, dt, dev), T;
    if (truth(a[4])) T = Out({d.groups, d.M, d.r}, dt, dev);
    void *const p[4] = {ptr(a[0]), ptr(a[1], dt), ptr(a[2], dt), ptr(a[3], dt)}, *const st = stream();
    call("pf_lowrank_linear_shared_fwd", pf_lowrank_linear_shared_fwd_workspace_bytes(&d), dev,
         [&](Space ws) { return pf_lowrank_linear_shared_fwd(&d, p[0], p[1], p[2], p[3], Y.p, T.p, ws.p, ws.n, st); });
    return tuple({Y.give(), T.give()});
}

// X, V, U, dY, T_saved, need_dX, has_bias, grads
PyObject *shared_bwd(PyObject *const *a)
{
    const Tensor &X = tensor(a[0]), &V = tensor(a[1]), &U = tensor(a[2]);
    const pf_linear_shared_desc d = shared_desc(X, U, truth(a[6]));
    const auto dt = X.scalar_type();
    const auto dev = X.device();
    Out dX;
    if (truth(a[5])) dX = Out(X.sizes(), dt, dev);
    Grads g(a[7], 3);
    if (!g.given) {
        g.make(0, U.sizes(), dev);
        g.make(1, V.sizes(), dev);
        if (d.has_bias) g.make(2, {d.groups, d.n_out}, dev);
    }
    void *const p[5] = {ptr(a[0]), ptr(a[1], dt), ptr(a[2], dt), ptr(a[3], dt), ptr(a[4], dt)}, *const st = stream();
    call("pf_lowrank_linear_shared_bwd", pf_lowrank_linear_shared_bwd_workspace_bytes(&d), dev, [&](Space ws) {
        return pf_lowrank_linear_shared_bwd(&d, p[0], p[1], p[2], p[3], p[4], dX.p, g.p[0], g.p[1], g.p[2], g.given, ws.p, ws.n, st);
    });
    return tuple({dX.give(), g.give(0), g.give(1), g.give(2)});
}

// ------------------------------------------------------------------ convolution
pf_conv_desc conv_desc(const Tensor &X, const Tensor &Uk, const Tensor &Vp, long stride, long pad)
{
    dims(X, 4, "X");
    dims(Uk, 4, "Uk");
    pf_conv_desc d = {};
    d.N = X.size(0);
    d.Cin = X.size(1);
    d.H = X.size(2);
    d.W = X.size(3);
    d.Cout = Vp.size(0);
    d.r = Uk.size(0);
    d.k = (int)Uk.size(2);
    d.stride = (int)stride;
    d.pad = (int)pad;
    d.layout = PF_NCHW;
    d.dtype = dtype_code(X);
    d.wgrad_dtype = PF_F32;
    return d;
}

// X, Uk, Vp, scale, shift, residual, act, stride, pad, save_T, save_W, with epilogue
PyObject *conv_fwd(PyObject *const *a)
{
    const Tensor &X = tensor(a[0]), &Uk = tensor(a[1]), &Vp = tensor(a[2]);
    const long stride_ = integer(a[7]), pad = integer(a[8]);
    if (stride_ <= 0) fail("stride must be positive");
    const pf_conv_desc d = conv_desc(X, Uk, Vp, stride_, pad);
    const int64_t Ho = (d.H + 2 * pad - d.k) / d.stride + 1, Wo = (d.W + 2 * pad - d.k) / d.stride + 1;
    const auto dt = X.scalar_type();
    const auto dev = X.device();
    const bool save_W = truth(a[10]);
    Out Y({d.N, d.Cout, Ho, Wo}, dt, dev), T, W;
    if (truth(a[9])) T = Out({d.N, d.r, Ho, Wo}, dt, dev);
    const size_t nW = save_W ? pf_lowrank_conv_saved_weights_bytes(&d) : 0;
    if (nW) W = Out({(int64_t)nW}, at::kByte, dev);
    void *const p[6] = {ptr(a[0], dt), ptr(a[1], dt), ptr(a[2], dt), ptr(a[3], F32), ptr(a[4], F32), ptr(a[5], dt)}, *const st = stream();
    const size_t need = pf_lowrank_conv_fwd_workspace_bytes(&d);
    const int act = (int)integer(a[6]);
    if (truth(a[11]))
        call("pf_lowrank_conv_fwd_ep", need, dev, [&](Space ws) {
            return pf_lowrank_conv_fwd_ep(&d, p[0], p[1], p[2], p[3], p[4], p[5], act, Y.p, T.p, W.p, ws.p, ws.n, st);
        });
    else
        call("pf_lowrank_conv_fwd", need, dev,
             [&](Space ws) { return pf_lowrank_conv_fwd(&d, p[0], p[1], p[2], Y.p, T.p, W.p, ws.p, ws.n, st); });
    return save_W ? tuple({Y.give(), T.give(), W.give()}) : tuple({Y.give(), T.give()});
}

// X, Uk, Vp, scale, dZ, T_saved, stride, pad, dX_add, x_is_relu, need_dX, need_dshift, grads, W_saved, with epilogue
PyObject *conv_bwd(PyObject *const *a)
{
    const Tensor &X = tensor(a[0]), &Uk = tensor(a[1]), &Vp = tensor(a[2]);
    const pf_conv_desc d = conv_desc(X, Uk, Vp, integer(a[6]), integer(a[7]));
    const auto dt = X.scalar_type();
    const auto dev = X.device();
    const bool ep = truth(a[14]);
    Out dX;
    if (truth(a[10])) dX = Out(X.sizes(), dt, dev);
    Grads g(a[12], ep ? 3 : 2);
    if (!g.given) {
        g.make(0, Uk.sizes(), dev);
        g.make(1, Vp.sizes(), dev);
        if (ep && truth(a[11])) g.make(2, {d.Cout}, dev);
    }
    void *const p[6] = {ptr(a[0], dt), ptr(a[1], dt), ptr(a[2], dt), ptr(a[4], dt), ptr(a[5], dt), ptr(a[13])}, *const st = stream();
    if (ep) {
        void *const scale = ptr(a[3], F32), *const add = ptr(a[8], dt);
        const bool relu = truth(a[9]);
        call("pf_lowrank_conv_bwd_ep", pf_lowrank_conv_bwd_ep_workspace_bytes(&d), dev, [&](Space ws) {
            return pf_lowrank_conv_bwd_ep(&d, p[0], p[1], p[2], scale, p[3], p[4], p[5], add, relu, dX.p, g.p[0], g.p[1], g.p[2], g.given,
                                          ws.p, ws.n, st);
        });
        return tuple({dX.give(), g.give(0), g.give(1), g.give(2)});
    }
    call("pf_lowrank_conv_bwd", pf_lowrank_conv_bwd_workspace_bytes(&d), dev, [&](Space ws) {
        return pf_lowrank_conv_bwd(&d, p[0], p[1], p[2], p[3], p[4], p[5], dX.p, g.p[0], g.p[1], g.given, ws.p, ws.n, st);
    });
    return tuple({dX.give(), g.give(0), g.give(1)});
}

// ------------------------------------------------------------------ LSTM
const char *const GRAD_NAMES[5] = {"dVx", "dUx", "dVh", "dUh", "dbias"};

// The five parameter gradients of a layer: a given dict's tensors, or new ones in a new dict
struct LstmGrads {
    Ref dict, items[5];
    void *p[5];
    LstmGrads(PyObject *given, const Tensor &Vx, const Tensor &Ux, const Tensor &Vh, const Tensor &Uh, int64_t h)
    {
        if (given != Py_None) {
            dict.o = borrowed(given);
            for (int i = 0; i < 5; ++i) {
                items[i].o = PyMapping_GetItemString(given, GRAD_NAMES[i]);
                if (!items[i].o) throw Fail{nullptr, ""};
                p[i] = ptr(items[i].o, F32);
            }
            return;
        }
        dict.o = PyDict_New();
        const at::IntArrayRef sizes[4] = {Vx.sizes(), Ux.sizes(), Vh.sizes(), Uh.sizes()};
        for (int i = 0; i < 5; ++i) {
            const int64_t nb[1] = {4 * h};
            Out o(i < 4 ? sizes[i] : at::IntArrayRef(nb), F32, Vx.device());
            p[i] = o.p;
            PyObject *t = o.give();
            PyDict_SetItemString(dict.o, GRAD_NAMES[i], t);
            Py_DECREF(t);
        }
    }
    LstmGrads(LstmGrads &&) = default;
    PyObject *give() { return std::exchange(dict.o, nullptr); }
};

pf_lstm_desc cell_desc(const Tensor &x, const Tensor &h, const Tensor &Ux, long groups, bool bias)
{
    dims(x, 2, "x");
    pf_lstm_desc d = {};
    d.B = x.size(0);
    d.d_in = x.size(1);
    d.h = h.size(1);
    d.r = Ux.size(1);
    d.groups = (int)groups;
    d.dtype = dtype_code(x);
    d.has_bias = bias;
    return d;
}

// x, h_prev, c_prev, Vx, Ux, Vh, Uh, bias, groups
PyObject *cell_fwd(PyObject *const *a)
{
    const Tensor &x = tensor(a[0]);
    const pf_lstm_desc d = cell_desc(x, tensor(a[1]), tensor(a[4]), integer(a[8]), a[7] != Py_None);
    const auto dev = x.device();
    const int64_t gr = d.groups * d.r;
    Out h({d.B, d.h}, F32, dev), c({d.B, d.h}, F32, dev), g({d.B, 4 * d.h}, F32, dev), Tx({d.B, gr}, F32, dev),
        Th({d.B, gr}, F32, dev);
    void *p[8], *const st = stream();
    for (int i = 0; i < 8; ++i) p[i] = ptr(a[i], F32);
    call("pf_lowrank_lstm_cell_fwd", pf_lowrank_lstm_cell_fwd_workspace_bytes(&d), dev, [&](Space ws) {
        return pf_lowrank_lstm_cell_fwd(&d, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], h.p, c.p, g.p, Tx.p, Th.p, ws.p, ws.n, st);
    });
    return tuple({h.give(), c.give(), g.give(), Tx.give(), Th.give()});
}

// x, h_prev, c_prev, c_out, gates, Tx, Th, Vx, Ux, Vh, Uh, dh, dc_next, groups, need_dx, grads
PyObject *cell_bwd(PyObject *const *a)
{
    const Tensor &x = tensor(a[0]), &hp = tensor(a[1]);
    const pf_lstm_desc d = cell_desc(x, hp, tensor(a[8]), integer(a[13]), true);
    const auto dev = x.device();
    Out dx, dh(hp.sizes(), F32, dev), dc(tensor(a[2]).sizes(), F32, dev);
    if (truth(a[14])) dx = Out(x.sizes(), F32, dev);
    LstmGrads g(a[15], tensor(a[7]), tensor(a[8]), tensor(a[9]), tensor(a[10]), d.h);
    void *p[13], *const st = stream();
    for (int i = 0; i < 13; ++i) p[i] = ptr(a[i], F32);
    const bool given = a[15] != Py_None;
    call("pf_lowrank_lstm_cell_bwd", pf_lowrank_lstm_cell_bwd_workspace_bytes(&d), dev, [&](Space ws) {
        return pf_lowrank_lstm_cell_bwd(&d, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], p[8], p[9], p[10], p[11], p[12], dx.p, dh.p,
                                        dc.p, g.p[0], g.p[1], g.p[2], g.p[3], g.p[4], given, ws.p, ws.n, st);
    });
    return tuple({dx.give(), dh.give(), dc.give(), g.give()});
}

// A list with one tensor (or None) per layer and the host array of its pointers
struct Layers {
    PyObject *seq = nullptr;
    std::vector<Tensor> keep; // (another thread may change the list during the call)
    std::vector<void *> p;
    bool present;
    explicit Layers(PyObject *o, at::ScalarType want = F32) : present(o != Py_None)
    {
        if (!present) return;
        seq = PySequence_Fast(o, "expected a list with one tensor per layer");
        if (!seq) throw Fail{nullptr, ""};
        for (Py_ssize_t i = 0; i < size(); ++i) {
            PyObject *t = PySequence_Fast_GET_ITEM(seq, i);
            p.push_back(ptr(t, want));
            if (t != Py_None) keep.push_back(tensor(t));
        }
    }
    Layers(const Layers &) = delete;
    ~Layers() { Py_XDECREF(seq); }
    Py_ssize_t size() const { return PySequence_Fast_GET_SIZE(seq); }
    const Tensor &at(Py_ssize_t i) const { return tensor(PySequence_Fast_GET_ITEM(seq, i)); }
    template <class T>
    T *arr()
    {
        return present ? (T *)p.data() : nullptr;
    }
};
// One new tensor per layer
struct Outs {
    std::vector<Out> o;
    std::vector<void *> p;
    void add(at::IntArrayRef size, const at::Device &dev)
    {
        o.emplace_back(size, F32, dev);
        p.push_back(o.back().p);
    }
    PyObject *give()
    {
        PyObject *l = PyList_New((Py_ssize_t)o.size());
        for (size_t i = 0; i < o.size(); ++i) PyList_SET_ITEM(l, (Py_ssize_t)i, o[i].give());
        return l;
    }
};

pf_lstm_stack_desc stack_desc(const Tensor &x, const Layers &h0, const Layers &Ux, long groups, bool bias)
{
    dims(x, 3, "x");
    pf_lstm_stack_desc d = {};
    if (Ux.size() == 0 || h0.size() < Ux.size()) throw Fail{PyExc_ValueError, "one tensor per layer is wanted"};
    d.T = x.size(0);
    d.B = x.size(1);
    d.d_in = x.size(2);
    d.h = h0.at(0).size(1);
    d.r = Ux.at(0).size(1);
    d.groups = (int)groups;
    d.layers = (int)Ux.size();
    d.dtype = dtype_code(x);
    d.has_bias = bias;
    return d;
}
void per_layer(const pf_lstm_stack_desc &d, std::initializer_list<const Layers *> ls)
{
    for (const Layers *l : ls)
        if (l->present && l->size() < d.layers) throw Fail{PyExc_ValueError, "one tensor per layer is wanted"};
}

// x, h0, c0, Vx, Ux, Vh, Uh, bias, groups
PyObject *stack_fwd(PyObject *const *a)
{
    const Tensor &x = tensor(a[0]);
    Layers h0(a[1]), c0(a[2]), Vx(a[3]), Ux(a[4]), Vh(a[5]), Uh(a[6]), bias(a[7]);
    const pf_lstm_stack_desc d = stack_desc(x, h0, Ux, integer(a[8]), bias.present);
    per_layer(d, {&h0, &c0, &Vx, &Ux, &Vh, &Uh, &bias});
    const auto dev = x.device();
    const int64_t n[5] = {d.h, d.h, 4 * d.h, d.groups * d.r, d.groups * d.r};
    Outs o[5];
    for (int i = 0; i < 5; ++i)
        for (int l = 0; l < d.layers; ++l) o[i].add({d.T, d.B, n[i]}, dev);
    void *const px = ptr(a[0], F32), *const st = stream();
    call("pf_lowrank_lstm_stack_fwd", pf_lowrank_lstm_stack_fwd_workspace_bytes(&d), dev, [&](Space ws) {
        return pf_lowrank_lstm_stack_fwd(&d, px, h0.arr<const void *>(), c0.arr<const void *>(), Vx.arr<const void *>(),
                                         Ux.arr<const void *>(), Vh.arr<const void *>(), Uh.arr<const void *>(),
                                         bias.arr<const void *>(), o[0].p.data(), o[1].p.data(), o[2].p.data(), o[3].p.data(),
                                         o[4].p.data(), ws.p, ws.n, st);
    });
    return tuple({o[0].give(), o[1].give(), o[2].give(), o[3].give(), o[4].give()});
}

// x, h0, c0, h_all, c_all, gates_all, Tx_all, Th_all, Vx, Ux, Vh, Uh, dh_top, dhT, dcT, groups, need_dx, grads
PyObject *stack_bwd(PyObject *const *a)
{
    const Tensor &x = tensor(a[0]);
    Layers h0(a[1]), c0(a[2]), h(a[3]), c(a[4]), g(a[5]), Tx(a[6]), Th(a[7]), Vx(a[8]), Ux(a[9]), Vh(a[10]), Uh(a[11]),
        dhT(a[13]), dcT(a[14]);
    const pf_lstm_stack_desc d = stack_desc(x, h0, Ux, integer(a[15]), true);
    per_layer(d, {&h0, &c0, &h, &c, &g, &Tx, &Th, &Vx, &Ux, &Vh, &Uh, &dhT, &dcT});
    const auto dev = x.device();
    Out dx;
    if (truth(a[16])) dx = Out(x.sizes(), F32, dev);
    Outs dh0, dc0;
    for (int l = 0; l < d.layers; ++l) dh0.add(h0.at(l).sizes(), dev);
    for (int l = 0; l < d.layers; ++l) dc0.add(c0.at(l).sizes(), dev);
    std::vector<LstmGrads> gr;
    gr.reserve(d.layers);
    for (int l = 0; l < d.layers; ++l) {
        Ref given(a[17] != Py_None ? PySequence_GetItem(a[17], l) : borrowed(Py_None));
        if (!given.o) throw Fail{nullptr, ""};
        gr.emplace_back(given.o, Vx.at(l), Ux.at(l), Vh.at(l), Uh.at(l), d.h);
    }
    std::vector<void *> gp[5];
    for (int i = 0; i < 5; ++i)
        for (int l = 0; l < d.layers; ++l) gp[i].push_back(gr[l].p[i]);
    void *const px = ptr(a[0], F32), *const pdh = ptr(a[12], F32), *const st = stream();
    const bool given = a[17] != Py_None;
    call("pf_lowrank_lstm_stack_bwd", pf_lowrank_lstm_stack_bwd_workspace_bytes(&d), dev, [&](Space ws) {
        return pf_lowrank_lstm_stack_bwd(&d, px, h0.arr<const void *>(), c0.arr<const void *>(), h.arr<const void *>(),
                                         c.arr<const void *>(), g.arr<const void *>(), Tx.arr<const void *>(), Th.arr<const void *>(),
                                         Vx.arr<const void *>(), Ux.arr<const void *>(), Vh.arr<const void *>(), Uh.arr<const void *>(),
                                         pdh, dhT.arr<const void *>(), dcT.arr<const void *>(), dx.p, dh0.p.data(), dc0.p.data(),
                                         gp[0].data(), gp[1].data(), gp[2].data(), gp[3].data(), gp[4].data(), given, ws.p, ws.n, st);
    });
    PyObject *grads = a[17];
    if (grads == Py_None) {
        grads = PyList_New(d.layers);
        for (int l = 0; l < d.layers; ++l) PyList_SET_ITEM(grads, l, gr[l].give());
    } else {
        Py_INCREF(grads);
    }
    return tuple({dx.give(), dh0.give(), dc0.give(), grads});
}

// bytes, a tensor on the device: the scratch buffer of the current stream, held by this thread until it gives it back
PyObject *lend(PyObject *const *a)
{
    const size_t bytes = (size_t)integer(a[0]);
    const auto dev = tensor(a[1]).device();
    if (!dev.is_cuda()) fail("tensors must live on the GPU; there is no CPU path");
    Scratch *s;
    {
        NoGil released;
        s = &scratch(dev);
        s->busy.lock();
    }
    try {
        s->get(bytes, dev);
    } catch (...) {
        s->busy.unlock();
        throw;
    }
    return tuple({PyLong_FromVoidPtr(s), THPVariable_Wrap(s->t)});
}
PyObject *give_back(PyObject *const *a)
{
    ((Scratch *)PyLong_AsVoidPtr(a[0]))->busy.unlock();
    Py_RETURN_NONE;
}

// The exceptions to raise: PfError, torch.OutOfMemoryError
PyObject *set_errors(PyObject *, PyObject *args)
{
    PyObject *e, *m;
    if (!PyArg_ParseTuple(args, "OO", &e, &m)) return nullptr;
    g_error = borrowed(e);
    g_no_memory = borrowed(m);
    Py_RETURN_NONE;
}

#define CALL(name, n) {#name, (PyCFunction)(void (*)(void))entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {CALL(linear_fwd, 8),
                         CALL(linear_bwd, 11),
                         CALL(shared_fwd, 5),
                         CALL(shared_bwd, 8),
                         CALL(conv_fwd, 12),
                         CALL(conv_bwd, 15),
                         CALL(cell_fwd, 9),
                         CALL(cell_bwd, 16),
                         CALL(stack_fwd, 9),
                         CALL(stack_bwd, 18),
                         CALL(lend, 2),
                         CALL(give_back, 1),
                         {"set_errors", set_errors, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
