// The binding's calls on torch tensors, in native code: argument checks,
// buffers and the library call of noble_linear_fwd / _fwd_static / _bwd and
// of the module's forward and backward.
//
// In Python they took longer than the GPU works on a layer of few tokens.  Host
// time of one pass, before and after (us): noble_linear_fwd_static 23.9 -> 8.3,
// the module's inference 35.5 -> 16.0, its forward and backward 301 -> 167 (the
// rest is torch's autograd).  These functions serve the well-formed call
// on ordinary tensors and return None for every other one (a tensor subclass,
// a wrapped or traced tensor, an active dispatch mode, a wrong shape, dtype or
// device): the Python code then runs and raises its own errors.
//
// The library's entry points come in as addresses (init), so this file does
// not link libnoble.so.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ops/empty.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <initializer_list>

#include "noble_binding.h"

namespace {

decltype(&noble_linear_fwd) p_fwd;
decltype(&noble_linear_fwd_static) p_fwd_static;
decltype(&noble_linear_bwd) p_bwd;
decltype(&noble_linear_bwd_storage) p_bwd_storage;
decltype(&noble_linear_workspace_size) p_sizes;
decltype(&noble_linear_fwd_scratch_size) p_fwd_size;

// Releases the GIL for its lifetime.
struct NoGil {
    PyThreadState* s = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(s); }
};

// An ordinary strided CUDA tensor, or nullptr (anything else).
const at::Tensor* plain(PyObject* o) {
    static const c10::DispatchKeySet special({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                              c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                              c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                              c10::DispatchKey::ZeroTensor});
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != c10::kStrided || !t.device().is_cuda() || !t.has_storage() ||
        t.key_set().has_any(special) || !t.is_contiguous())
        return nullptr;
    return &t;
}

// The tensors of one call as they are checked; ok turns false at the first
// argument that the native path does not take.
struct Call {
    bool ok = true;
    at::Device dev{c10::kCUDA};
    at::ScalarType sd = at::kBFloat16;
    int64_t T = 0, din = 0, dout = 0, R = 0, r = 0, G = 1, dog = 0;
    int act = 0, layers = 1;
    noble_linear_desc d{};

    const at::Tensor* tensor(PyObject* o) {
        const at::Tensor* t = plain(o);
        if (!t) ok = false;
        return t;
    }
    // Data pointer of an argument of the given dtype and shape (None: NULL).
    void* ptr(PyObject* o, at::ScalarType dt, std::initializer_list<int64_t> shape) {
        if (o == Py_None || !ok) return nullptr;
        const at::Tensor* t = tensor(o);
        if (!t || t->scalar_type() != dt || t->device() != dev || !t->sizes().equals(shape)) {
            ok = false;
            return nullptr;
        }
        return t->data_ptr();
    }
    void* bytes(PyObject* o, size_t* n = nullptr) {   // a work buffer: any dtype and shape
        if (n) *n = 0;
        if (o == Py_None || !ok) return nullptr;
        const at::Tensor* t = tensor(o);
        if (!t || t->device() != dev) {
            ok = false;
            return nullptr;
        }
        if (n) *n = (size_t)t->numel() * t->element_size();
        return t->data_ptr();
    }
    float* vec(PyObject* o) { return static_cast<float*>(ptr(o, at::kFloat, {R})); }
    float* vec2(PyObject* o) {
        return static_cast<float*>(layers == 3 ? ptr(o, at::kFloat, {2, R}) : ptr(o, at::kFloat, {R}));
    }
    void* mix(PyObject* o, at::ScalarType dt) {
        if (layers == 3) return G == 1 ? ptr(o, dt, {2, r, r}) : ptr(o, dt, {2, G, r, r});
        return G == 1 ? ptr(o, dt, {r, r}) : ptr(o, dt, {G, r, r});
    }
    // Sizes from act, layers, groups, x, W and W_down.
    Call(PyObject* a, PyObject* l, PyObject* g, PyObject* x, PyObject* W, PyObject* Wd) {
        if (!PyLong_CheckExact(a) || !PyLong_CheckExact(l) || !PyLong_CheckExact(g) ||
            c10::impl::TorchDispatchModeTLS::any_modes_set()) {
            ok = false;
            return;
        }
        act = (int)PyLong_AsLong(a);
        layers = (int)PyLong_AsLong(l);
        int wide = 0;   // past a long: G is -1, which is refused below
        G = PyLong_AsLongAndOverflow(g, &wide);
        const at::Tensor *tx = tensor(x), *tw = tensor(W), *td = Wd == Py_None ? nullptr : tensor(Wd);
        if (!ok || tx->dim() != 2 || tw->dim() != 2 || (td && td->dim() != 2) || G < 1 || G > INT32_MAX) {
            ok = false;
            return;
        }
        dev = tx->device();
        sd = tx->scalar_type();
        T = tx->size(0);
        din = tx->size(1);
        dout = tw->size(1);
        R = td ? td->size(1) : 0;
        ok = (sd == at::kBFloat16 || sd == at::kFloat) && R % G == 0 && dout % G == 0;
        r = R / G;
        dog = dout / G;
        d.T = T;
        d.d_in = din;
        d.d_out = dout;
        d.r = r;
        d.dtype = sd == at::kBFloat16 ? NOBLE_BF16 : NOBLE_F32;
        d.activation = act;
        d.groups = (int32_t)G;
    }
    void* stream() const { return at::hip::getCurrentHIPStreamMasqueradingAsCUDA(dev.index()).stream(); }
    at::Tensor empty(c10::IntArrayRef shape, at::ScalarType dt) const {
        return at::empty(shape, at::TensorOptions().dtype(dt).device(dev));
    }
    at::Tensor work(size_t n) const { return empty({(int64_t)std::max<size_t>(n, 16)}, at::kByte); }
};

// The parameters W_down .. W_up in the order of every call.
struct Branch {
    void *Wd, *M, *Wu;
    float *o1, *p1, *o2, *p2;
    Branch(Call& c, PyObject* const* a)
        : Wd(c.ptr(a[0], c.sd, {c.din, c.R})), M(c.mix(a[3], c.sd)), Wu(c.ptr(a[6], c.sd, {c.R, c.dog})),
          o1(c.vec(a[1])), p1(c.vec(a[2])), o2(c.vec2(a[4])), p2(c.vec2(a[5])) {}
};

// forward(static, act, layers, groups, x, W, b, W_down, omega1, phi1, M, omega2, phi2, W_up, y, reserve, scratch)
// -> status or None.
PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 17) Py_RETURN_NONE;
    const bool fixed = a[0] == Py_True;
    Call c(a[1], a[2], a[3], a[4], a[5], a[7]);
    if (!c.ok) Py_RETURN_NONE;
    const void* x = c.ptr(a[4], c.sd, {c.T, c.din});
    const void* W = c.ptr(a[5], c.sd, {c.din, c.dout});
    const float* b = static_cast<float*>(c.ptr(a[6], at::kFloat, {c.dout}));
    const Branch p(c, a + 7);
    void* y = c.ptr(a[14], c.sd, {c.T, c.dout});
    void* reserve = c.bytes(a[15]);
    size_t sbytes = 0;
    void* scratch = c.bytes(a[16], &sbytes);
    if (!c.ok || a[14] == Py_None) Py_RETURN_NONE;
    noble_status st;
    {
        NoGil nogil;
        const c10::DeviceGuard guard(c.dev);
        st = fixed ? p_fwd_static(&c.d, x, W, b, p.Wd, p.o1, p.p1, p.M, p.o2, p.p2, p.Wu, y, reserve, c.stream())
                   : p_fwd(&c.d, x, W, b, p.Wd, p.o1, p.p1, p.M, p.o2, p.p2, p.Wu, y, reserve, scratch, sbytes,
                           c.stream());
    }
    return PyLong_FromLong(st);
    END_HANDLE_TH_ERRORS
}

// backward(act, layers, groups, dy, x, W, W_down, omega1, phi1, M, omega2, phi2, W_up, reserve, dx, dW, db, dW_down,
// dM, dW_up, domega1, dphi1, domega2, dphi2, scratch) -> status or None.
PyObject* backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 25) Py_RETURN_NONE;
    Call c(a[0], a[1], a[2], a[4], a[5], a[6]);
    if (!c.ok) Py_RETURN_NONE;
    const auto f32 = at::kFloat;
    const void* dy = c.ptr(a[3], c.sd, {c.T, c.dout});
    const void* x = c.ptr(a[4], c.sd, {c.T, c.din});
    const void* W = c.ptr(a[5], c.sd, {c.din, c.dout});
    const Branch p(c, a + 6);
    const void* reserve = c.bytes(a[13]);
    void* dx = c.ptr(a[14], c.sd, {c.T, c.din});
    auto f = [](void* q) { return static_cast<float*>(q); };
    float* dW = f(c.ptr(a[15], f32, {c.din, c.dout}));
    float* db = f(c.ptr(a[16], f32, {c.dout}));
    float* dWd = f(c.ptr(a[17], f32, {c.din, c.R}));
    float* dM = f(c.mix(a[18], f32));
    float* dWu = f(c.ptr(a[19], f32, {c.R, c.dog}));
    float *do1 = c.vec(a[20]), *dp1 = c.vec(a[21]), *do2 = c.vec2(a[22]), *dp2 = c.vec2(a[23]);
    size_t sbytes = 0;
    void* scratch = c.bytes(a[24], &sbytes);
    if (!c.ok) Py_RETURN_NONE;
    noble_status st;
    {
        NoGil nogil;
        const c10::DeviceGuard guard(c.dev);
        st = p_bwd(&c.d, dy, x, W, p.Wd, p.o1, p.p1, p.M, p.o2, p.p2, p.Wu, reserve, dx, dW, db, dWd, dM, dWu, do1, dp1,
                   do2, dp2, scratch, sbytes, c.stream());
    }
    return PyLong_FromLong(st);
    END_HANDLE_TH_ERRORS
}

// module_forward(keep, act, layers, groups, x, W, b, W_down, ..., W_up) -> (y, reserve) (reserve None unless `keep`),
// a status, or None.
PyObject* module_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 14) Py_RETURN_NONE;
    const bool keep = a[0] == Py_True;
    Call c(a[1], a[2], a[3], a[4], a[5], a[7]);
    // A recorded plain layer has a W_down of no columns (the backward needs it); None is an error.
    if (!c.ok || (keep && a[7] == Py_None)) Py_RETURN_NONE;
    const void* x = c.ptr(a[4], c.sd, {c.T, c.din});
    const void* W = c.ptr(a[5], c.sd, {c.din, c.dout});
    const float* b = static_cast<float*>(c.ptr(a[6], at::kFloat, {c.dout}));
    const Branch p(c, a + 7);
    size_t res = 0, scr = 0;
    if (!c.ok || p_sizes(&c.d, &res, nullptr) != NOBLE_OK || p_fwd_size(&c.d, &scr) != NOBLE_OK) Py_RETURN_NONE;
    noble_status st;
    at::Tensor y, reserve;
    {
        NoGil nogil;
        const c10::DeviceGuard guard(c.dev);
        const at::Tensor scratch = c.work(scr);
        if (keep) reserve = c.work(res);
        y = c.empty({c.T, c.dout}, c.sd);
        st = p_fwd(&c.d, x, W, b, p.Wd, p.o1, p.p1, p.M, p.o2, p.p2, p.Wu, y.data_ptr(),
                   keep ? reserve.data_ptr() : nullptr, scratch.data_ptr(), (size_t)scratch.numel(), c.stream());
    }
    if (st != NOBLE_OK) return PyLong_FromLong(st);
    PyObject* out = PyTuple_New(2);
    if (!out) return nullptr;
    PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(y));
    if (!keep) Py_INCREF(Py_None);
    PyTuple_SET_ITEM(out, 1, keep ? THPVariable_Wrap(reserve) : Py_None);
    return out;
    END_HANDLE_TH_ERRORS
}

// module_backward(has_bias, act, layers, groups, dy, x, W, W_down, omega1, phi1, M, omega2, phi2, W_up, reserve) ->
// (dx, dW, db, dW_down, domega1, dphi1, dM, domega2, dphi2, dW_up), dW, dW_down, dM and dW_up in the storage dtype and
// the vectors in float32 (None for those the form does not have), a status, or None.
PyObject* module_backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 15) Py_RETURN_NONE;
    const bool bias = a[0] == Py_True;
    Call c(a[1], a[2], a[3], a[5], a[6], a[7]);
    if (!c.ok || a[7] == Py_None || c.T == 0) Py_RETURN_NONE;
    const void* dy = c.ptr(a[4], c.sd, {c.T, c.dout});
    const void* x = c.ptr(a[5], c.sd, {c.T, c.din});
    const void* W = c.ptr(a[6], c.sd, {c.din, c.dout});
    const Branch p(c, a + 7);
    const void* reserve = c.bytes(a[14]);
    size_t scr = 0;
    if (!c.ok || p_sizes(&c.d, nullptr, &scr) != NOBLE_OK) Py_RETURN_NONE;
    noble_status st;
    at::Tensor g[10];   // in the order returned
    {
        NoGil nogil;
        const c10::DeviceGuard guard(c.dev);
        const auto f32 = at::kFloat;
        const at::Tensor scratch = c.work(scr);
        g[0] = c.empty({c.T, c.din}, c.sd);
        g[1] = c.empty({c.din, c.dout}, c.sd);
        if (bias) g[2] = c.empty({c.dout}, f32);
        g[3] = c.empty({c.din, c.R}, c.sd);
        g[4] = c.empty({c.R}, f32);
        g[5] = c.empty({c.R}, f32);
        if (c.layers >= 2) {
            const bool three = c.layers == 3;
            c10::SmallVector<int64_t, 4> ms;
            if (three) ms.push_back(2);
            if (c.G > 1) ms.push_back(c.G);
            ms.push_back(c.r);
            ms.push_back(c.r);
            g[6] = c.empty(ms, c.sd);
            for (int i : {7, 8}) g[i] = three ? c.empty({2, c.R}, f32) : c.empty({c.R}, f32);
        }
        g[9] = c.empty({c.R, c.dog}, c.sd);
        auto v = [&](int i) { return g[i].defined() ? g[i].data_ptr() : nullptr; };
        auto f = [&](int i) { return static_cast<float*>(v(i)); };
        st = p_bwd_storage(&c.d, dy, x, W, p.Wd, p.o1, p.p1, p.M, p.o2, p.p2, p.Wu, reserve, v(0), v(1), f(2), v(3),
                           v(6), v(9), f(4), f(5), f(7), f(8), scratch.data_ptr(), (size_t)scratch.numel(), c.stream());
    }
    if (st != NOBLE_OK) return PyLong_FromLong(st);
    PyObject* out = PyTuple_New(10);
    if (!out) return nullptr;
    for (int i = 0; i < 10; ++i) {
        if (!g[i].defined()) Py_INCREF(Py_None);
        PyTuple_SET_ITEM(out, i, g[i].defined() ? THPVariable_Wrap(g[i]) : Py_None);
    }
    return out;
    END_HANDLE_TH_ERRORS
}

// init(fwd, fwd_static, bwd, bwd_storage, workspace_size, fwd_scratch_size): the library's entry points, as addresses.
PyObject* init(PyObject*, PyObject* args) {
    unsigned long long p[6];
    if (!PyArg_ParseTuple(args, "KKKKKK", &p[0], &p[1], &p[2], &p[3], &p[4], &p[5])) return nullptr;
    p_fwd = reinterpret_cast<decltype(p_fwd)>(p[0]);
    p_fwd_static = reinterpret_cast<decltype(p_fwd_static)>(p[1]);
    p_bwd = reinterpret_cast<decltype(p_bwd)>(p[2]);
    p_bwd_storage = reinterpret_cast<decltype(p_bwd_storage)>(p[3]);
    p_sizes = reinterpret_cast<decltype(p_sizes)>(p[4]);
    p_fwd_size = reinterpret_cast<decltype(p_fwd_size)>(p[5]);
    Py_RETURN_NONE;
}

#define NOBLE_FAST(fn) {#fn, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"init", init, METH_VARARGS, nullptr},
                         NOBLE_FAST(forward),
                         NOBLE_FAST(backward),
                         NOBLE_FAST(module_forward),
                         NOBLE_FAST(module_backward),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_noble_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__noble_torch(void) { return PyModule_Create(&module_def); }
