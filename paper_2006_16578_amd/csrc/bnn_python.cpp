// The calls of binding.py whose kernels are short, for the arguments that programs pass nearly always.
//
// What a small call costs is host work: 8 x 4096 x 4096 runs 3.1 us on the GPU, its launch takes 2.6 us of host time, and checking, allocating and marshalling
// from Python took 3.6 more (torch.empty 1.4, three tensors' checks 0.65, pointers 0.45, devices and stream 0.5, ctypes 0.4).  Here they take about 1.
// Each function takes exactly what its namesake in binding.py would after its defaults, and returns None for everything out of the ordinary --
// anything but plain contiguous device tensors of the expected types and shapes on the current device, numbers that are no int --: the
// Python function then does as it always did, errors included.  Nothing is kept from one call to the next.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/DeviceGuardImplInterface.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "../../include/bnn.h"

namespace {

#define BNN_ENTRIES(X)                                                                                                                   \
    X(bnn_bmm_ex) X(bnn_bmm_thr_ex) X(bnn_bconv_ex) X(bnn_bconv_thr_ex) X(bnn_threshold_pack) X(bnn_maxpool_or)                            \
    X(bnn_bmm_general_workspace_bytes) X(bnn_bmm_general_f32) X(bnn_bwn_workspace_bytes) X(bnn_bwn_conv_thr)                               \
    X(bnn_conv_f32_split_workspace_bytes) X(bnn_conv_f32_split_thr_ex) X(bnn_net_workspace_bytes) X(bnn_net_forward)
#define DECLARE(name) decltype(&::name) p_##name = nullptr;
BNN_ENTRIES(DECLARE)

PyObject* raw_stream = nullptr;      // torch's current raw stream of a device index
PyObject* check = nullptr;           // binding._check: raises a status

using at::Tensor;

// One call's arguments: each getter gives up (ok = false) at the first thing that is not plain.
struct Call {
    bool ok = true;
    int device = -1;

    const Tensor* tensor(PyObject* o, at::ScalarType type, int dims) {
        static const Tensor none;
        if (!ok || !THPVariable_CheckExact(o)) { ok = false; return &none; }
        const Tensor& t = THPVariable_Unpack(o);
        const at::TensorImpl* impl = t.unsafeGetTensorImpl();
        ok = t.defined() && t.is_cuda() && t.scalar_type() == type && (dims < 0 || t.dim() == dims) && t.layout() == at::kStrided && impl->has_storage() &&
             !impl->is_python_dispatch() && t.is_contiguous() && (device < 0 || t.get_device() == device);
        if (!ok) return &none;
        device = t.get_device();
        for (const int64_t n : t.sizes()) ok = ok && n <= INT_MAX;
        return &t;
    }
    int number(PyObject* o) {
        if (!ok || !PyLong_CheckExact(o)) { ok = false; return 0; }
        int overflow = 0;
        const long v = PyLong_AsLongAndOverflow(o, &overflow);
        ok = !overflow && v >= INT_MIN && v <= INT_MAX;
        return (int)v;
    }
    // The tensors' device is the current one, and nobody listens for torch functions (torch.empty would be one)
    bool ready() {
        if (!ok || at::impl::PythonTorchFunctionTLS::stack_len() != 0) return false;
        return c10::impl::getDeviceGuardImpl(at::kCUDA)->getDevice().index() == device;
    }
    bool stream(void** s) const {
        PyObject* index = PyLong_FromLong(device);
        PyObject* v = index ? PyObject_CallOneArg(raw_stream, index) : nullptr;
        Py_XDECREF(index);
        if (!v) return false;
        *s = PyLong_AsVoidPtr(v);
        Py_DECREF(v);
        return !PyErr_Occurred();
    }
};

Tensor empty(const Tensor& like, at::IntArrayRef sizes, at::ScalarType type) {
    return at::empty(sizes, at::TensorOptions().dtype(type).device(like.device()));
}

inline int words(int bits) { return (int)(((long long)bits + 31) / 32); }
template <class T> T* ptr(const Tensor& t) { return static_cast<T*>(t.data_ptr()); }

// The library's call, without the GIL; false: a Python error is set.  The arguments come by value: whatever reading them may throw (a tensor whose storage was freed
// has no pointer) it throws in the caller, with the GIL held.
template <class F, class... Args>
bool run(const Call& c, const char* what, F f, Args... args) {
    void* s = nullptr;
    int status = 0;
    if (!c.stream(&s)) return false;
    Py_BEGIN_ALLOW_THREADS
    status = f(args..., s);
    Py_END_ALLOW_THREADS
    if (status == 0) return true;
    PyObject* r = PyObject_CallFunction(check, "is", status, what);
    Py_XDECREF(r);
    if (r) PyErr_SetString(PyExc_RuntimeError, what);
    return false;
}

// C++ exceptions (an allocation that fails, a tensor without memory) become Python's.
template <class F>
PyObject* guarded(F f) {
    HANDLE_TH_ERRORS
    return f();
    END_HANDLE_TH_ERRORS
}

#define ARGS(n)                                              \
    if (nargs != n) {                                        \
        PyErr_SetString(PyExc_TypeError, "argument count");  \
        return nullptr;                                      \
    }
#define PLAIN(c) \
    if (!(c).ready()) Py_RETURN_NONE

constexpr at::ScalarType BITS = at::kInt;

PyObject* bmm(PyObject*, PyObject* const* a, Py_ssize_t nargs) {          // A, B, K, path
    ARGS(4)
    return guarded([&]() -> PyObject* {
        Call c;
        const Tensor &A = *c.tensor(a[0], BITS, 2), &B = *c.tensor(a[1], BITS, 2);
        const int K = c.number(a[2]), path = c.number(a[3]);
        PLAIN(c);
        const int M = (int)A.size(0), N = (int)B.size(0);
        const Tensor out = empty(A, {M, N}, at::kInt);
        const bool done = run(c, "bnn_bmm", p_bnn_bmm_ex, ptr<uint32_t>(A), ptr<uint32_t>(B), ptr<int32_t>(out), M, N, K, (int)A.size(1), (int)B.size(1), N, path);
        return done ? THPVariable_Wrap(out) : nullptr;
    });
}

PyObject* bmm_thr(PyObject*, PyObject* const* a, Py_ssize_t nargs) {      // A, B, thr, K, path
    ARGS(5)
    return guarded([&]() -> PyObject* {
        Call c;
        const Tensor &A = *c.tensor(a[0], BITS, 2), &B = *c.tensor(a[1], BITS, 2), &thr = *c.tensor(a[2], at::kInt, 1);
        const int K = c.number(a[3]), path = c.number(a[4]);
        PLAIN(c);
        const int M = (int)A.size(0), N = (int)B.size(0);
        if (thr.size(0) != N) Py_RETURN_NONE;
        const int ld = (words(N) + 3) / 4 * 4;
        const Tensor out = empty(A, {M, ld}, BITS);
        const bool done = run(c, "bnn_bmm_thr", p_bnn_bmm_thr_ex, ptr<uint32_t>(A), ptr<uint32_t>(B), ptr<int32_t>(thr), ptr<uint32_t>(out), M, N, K, (int)A.size(1),
                              (int)B.size(1), ld, path);
        return done ? THPVariable_Wrap(out) : nullptr;
    });
}

struct Conv {
    int N, H, W, O, k, P, Q;
    // x [N][H][W][.], filters [O][k][k][.], whose last sizes are compared by the caller; false: not an ordinary convolution
    bool set(const Tensor& x, const Tensor& f, int stride, int pad) {
        N = (int)x.size(0); H = (int)x.size(1); W = (int)x.size(2); O = (int)f.size(0); k = (int)f.size(1);
        if (f.size(2) != k || stride < 1 || pad < 0 || pad > 1 << 20 || k < 1 || H + 2LL * pad < k || W + 2LL * pad < k) return false;
        const long long p = (H + 2LL * pad - k) / stride + 1, q = (W + 2LL * pad - k) / stride + 1;
        if (p > INT_MAX || q > INT_MAX) return false;
        P = (int)p; Q = (int)q;
        return true;
    }
};

PyObject* bconv(PyObject*, PyObject* const* a, Py_ssize_t nargs) {        // x, filt, C, stride, pad, pad_mode, path
    ARGS(7)
    return guarded([&]() -> PyObject* {
        Call c;
        const Tensor &x = *c.tensor(a[0], BITS, 4), &f = *c.tensor(a[1], BITS, 4);
        const int C = c.number(a[2]), stride = c.number(a[3]), pad = c.number(a[4]), mode = c.number(a[5]), path = c.number(a[6]);
        PLAIN(c);
        Conv v;
        if (C < 1 || x.size(3) != words(C) || f.size(3) != x.size(3) || !v.set(x, f, stride, pad)) Py_RETURN_NONE;
        const Tensor y = empty(x, {v.N, v.P, v.Q, v.O}, at::kInt);
        const bool done = run(c, "bnn_bconv", p_bnn_bconv_ex, ptr<uint32_t>(x), ptr<uint32_t>(f), ptr<int32_t>(y), v.N, v.H, v.W, C, v.O, v.k, stride, pad, mode, path);
        return done ? THPVariable_Wrap(y) : nullptr;
    });
}

PyObject* bconv_thr(PyObject*, PyObject* const* a, Py_ssize_t nargs) {    // x, filt, thr, C, stride, pad, pad_mode, residual, want_sum, path
    ARGS(10)
    return guarded([&]() -> PyObject* {
        Call c;
        const Tensor &x = *c.tensor(a[0], BITS, 4), &f = *c.tensor(a[1], BITS, 4), &thr = *c.tensor(a[2], at::kInt, 1);
        const int C = c.number(a[3]), stride = c.number(a[4]), pad = c.number(a[5]), mode = c.number(a[6]), path = c.number(a[9]);
        const bool add = a[7] != Py_None, sum = a[8] == Py_True;
        const Tensor& r = add ? *c.tensor(a[7], at::kInt, 4) : x;
        if (!sum && a[8] != Py_False) Py_RETURN_NONE;
        PLAIN(c);
        Conv v;
        if (C < 1 || x.size(3) != words(C) || f.size(3) != x.size(3) || !v.set(x, f, stride, pad)) Py_RETURN_NONE;
        if (add && (r.size(0) != v.N || r.size(1) != v.P || r.size(2) != v.Q || r.size(3) != v.O)) Py_RETURN_NONE;
        Tensor y;
        if (sum) y = empty(x, {v.N, v.P, v.Q, v.O}, at::kInt);
        const Tensor bits = empty(x, {v.N, v.P, v.Q, words(v.O)}, BITS);
        if (!run(c, "bnn_bconv_thr", p_bnn_bconv_thr_ex, ptr<uint32_t>(x), ptr<uint32_t>(f), add ? ptr<int32_t>(r) : nullptr, sum ? ptr<int32_t>(y) : nullptr,
                 ptr<int32_t>(thr), ptr<uint32_t>(bits), v.N, v.H, v.W, C, v.O, v.k, stride, pad, mode, path))
            return nullptr;
        if (!sum) return THPVariable_Wrap(bits);
        PyObject* result = PyTuple_New(2);
        if (!result) return nullptr;
        PyTuple_SET_ITEM(result, 0, THPVariable_Wrap(bits));
        PyTuple_SET_ITEM(result, 1, THPVariable_Wrap(y));
        return result;
    });
}

PyObject* threshold_pack(PyObject*, PyObject* const* a, Py_ssize_t nargs) {   // X, thr
    ARGS(2)
    return guarded([&]() -> PyObject* {
        Call c;
        const Tensor &X = *c.tensor(a[0], at::kInt, -1), &thr = *c.tensor(a[1], at::kInt, 1);
        PLAIN(c);
        if (X.dim() < 1 || X.size(-1) < 1) Py_RETURN_NONE;
        const int cols = (int)X.size(-1), ld = words(cols);
        const int64_t rows = X.numel() / cols;
        std::vector<int64_t> sizes = X.sizes().vec();
        sizes.back() = ld;
        const Tensor bits = empty(X, sizes, BITS);
        const bool done = run(c, "bnn_threshold_pack", p_bnn_threshold_pack, ptr<int32_t>(X), ptr<int32_t>(thr), ptr<uint32_t>(bits), rows, cols, cols, ld);
        return done ? THPVariable_Wrap(bits) : nullptr;
    });
}

PyObject* maxpool_or(PyObject*, PyObject* const* a, Py_ssize_t nargs) {   // bits, C, win, stride
    ARGS(4)
    return guarded([&]() -> PyObject* {
        Call c;
        const Tensor& x = *c.tensor(a[0], BITS, 4);
        const int C = c.number(a[1]), win = c.number(a[2]), stride = c.number(a[3]);
        PLAIN(c);
        const int N = (int)x.size(0), H = (int)x.size(1), W = (int)x.size(2);
        if (stride < 1 || win < 1 || win > H || win > W) Py_RETURN_NONE;
        const Tensor out = empty(x, {N, (H - win) / stride + 1, (W - win) / stride + 1, x.size(3)}, BITS);
        const bool done = run(c, "bnn_maxpool_or", p_bnn_maxpool_or, ptr<uint32_t>(x), ptr<uint32_t>(out), N, H, W, C, win, stride);
        return done ? THPVariable_Wrap(out) : nullptr;
    });
}

PyObject* bmm_general_f32(PyObject*, PyObject* const* a, Py_ssize_t nargs) {  // A, B
    ARGS(2)
    return guarded([&]() -> PyObject* {
        Call c;
        const Tensor &A = *c.tensor(a[0], at::kFloat, 2), &B = *c.tensor(a[1], at::kFloat, 2);
        PLAIN(c);
        const int M = (int)A.size(0), N = (int)B.size(0), K = (int)A.size(1);
        if (B.size(1) != K) Py_RETURN_NONE;
        const Tensor out = empty(A, {M, N}, at::kFloat);
        const Tensor work = empty(A, {std::max<int64_t>((int64_t)p_bnn_bmm_general_workspace_bytes(M, N, K), 256)}, at::kByte);
        const bool done = run(c, "bnn_bmm_general_f32", p_bnn_bmm_general_f32, ptr<float>(A), ptr<float>(B), ptr<float>(out), M, N, K, K, K, N, ptr<void>(work),
                              (size_t)work.numel());
        return done ? THPVariable_Wrap(out) : nullptr;
    });
}

PyObject* bwn_conv_thr(PyObject*, PyObject* const* a, Py_ssize_t nargs) {     // x, wbits, thr, C, stride, pad
    ARGS(6)
    return guarded([&]() -> PyObject* {
        Call c;
        const Tensor &x = *c.tensor(a[0], at::kFloat, 4), &w = *c.tensor(a[1], BITS, 4), &thr = *c.tensor(a[2], at::kFloat, 1);
        const int C = c.number(a[3]), stride = c.number(a[4]), pad = c.number(a[5]);
        PLAIN(c);
        Conv v;
        if (C < 1 || x.size(3) != C || w.size(3) != words(C) || !v.set(x, w, stride, pad)) Py_RETURN_NONE;
        const Tensor bits = empty(x, {v.N, v.P, v.Q, words(v.O)}, BITS);
        const Tensor work = empty(x, {std::max<int64_t>((int64_t)p_bnn_bwn_workspace_bytes(C, v.O, v.k), 16)}, at::kByte);
        const bool done = run(c, "bnn_bwn_conv_thr", p_bnn_bwn_conv_thr, ptr<float>(x), ptr<uint32_t>(w), ptr<float>(thr), nullptr, ptr<uint32_t>(bits), v.N, v.H, v.W, C,
                              v.O, v.k, stride, pad, ptr<void>(work), (size_t)work.numel());
        return done ? THPVariable_Wrap(bits) : nullptr;
    });
}

PyObject* conv_f32_split_thr(PyObject*, PyObject* const* a, Py_ssize_t nargs) {   // x, w, thr, stride, pad, products
    ARGS(6)
    return guarded([&]() -> PyObject* {
        Call c;
        const Tensor &x = *c.tensor(a[0], at::kFloat, 4), &w = *c.tensor(a[1], at::kFloat, 4), &thr = *c.tensor(a[2], at::kFloat, 1);
        const int stride = c.number(a[3]), pad = c.number(a[4]), products = c.number(a[5]);
        PLAIN(c);
        Conv v;
        const int C = (int)x.size(3);
        if (w.size(3) != C || !v.set(x, w, stride, pad)) Py_RETURN_NONE;
        const Tensor bits = empty(x, {v.N, v.P, v.Q, words(v.O)}, BITS);
        const Tensor work = empty(x, {std::max<int64_t>((int64_t)p_bnn_conv_f32_split_workspace_bytes(C, v.O, v.k), 16)}, at::kByte);
        const bool done = run(c, "bnn_conv_f32_split_thr_ex", p_bnn_conv_f32_split_thr_ex, ptr<float>(x), ptr<float>(w), ptr<float>(thr), nullptr, ptr<uint32_t>(bits),
                              v.N, v.H, v.W, C, v.O, v.k, stride, pad, products, ptr<void>(work), (size_t)work.numel());
        return done ? THPVariable_Wrap(bits) : nullptr;
    });
}

// handle, x, its type (uint8, int32 or float32 as 0, 1, 2), the workspace, columns and type of the output (int32 or float32 as 1, 2), path.  A workspace too
// small, or of another device, is the Python function's to replace.
PyObject* net_forward(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    ARGS(7)
    return guarded([&]() -> PyObject* {
        constexpr at::ScalarType TYPES[] = {at::kByte, at::kInt, at::kFloat};
        Call c;
        const int in = c.number(a[2]), cols = c.number(a[4]), kind = c.number(a[5]), path = c.number(a[6]);
        if (!c.ok || in < 0 || in > 2 || kind < 1 || kind > 2) Py_RETURN_NONE;
        bnn_net* net = static_cast<bnn_net*>(PyLong_AsVoidPtr(a[0]));
        if (PyErr_Occurred()) return nullptr;
        const Tensor &x = *c.tensor(a[1], TYPES[in], -1), &work = *c.tensor(a[3], at::kByte, 1);
        PLAIN(c);
        if (net == nullptr || x.dim() < 1) Py_RETURN_NONE;
        const int batch = (int)x.size(0);
        size_t need = 0;
        if (p_bnn_net_workspace_bytes(net, batch, &need) != 0 || (size_t)work.numel() < need) Py_RETURN_NONE;
        const Tensor out = empty(x, {batch, cols}, TYPES[kind]);
        const bool done = run(c, "bnn_net_forward", p_bnn_net_forward, net, x.data_ptr(), out.data_ptr(), batch, work.data_ptr(), (size_t)work.numel(), path);
        return done ? THPVariable_Wrap(out) : nullptr;
    });
}

PyObject* init(PyObject*, PyObject* args) {        // {name: address}, the raw stream function, _check
    PyObject *addresses, *stream_fn, *check_fn;
    if (!PyArg_ParseTuple(args, "O!OO", &PyDict_Type, &addresses, &stream_fn, &check_fn)) return nullptr;
    auto address = [&](const char* name) -> void* {
        PyObject* v = PyDict_GetItemString(addresses, name);
        if (!v) { PyErr_SetString(PyExc_KeyError, name); return nullptr; }
        return PyLong_AsVoidPtr(v);
    };
#define FETCH(name) \
    if (!(p_##name = reinterpret_cast<decltype(&::name)>(address(#name)))) return nullptr;
    BNN_ENTRIES(FETCH)
    Py_INCREF(stream_fn); Py_INCREF(check_fn);
    Py_XDECREF(raw_stream); Py_XDECREF(check);
    raw_stream = stream_fn; check = check_fn;
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bmm), METHOD(bmm_thr), METHOD(bconv), METHOD(bconv_thr), METHOD(threshold_pack), METHOD(maxpool_or), METHOD(bmm_general_f32),
                         METHOD(bwn_conv_thr), METHOD(conv_f32_split_thr), METHOD(net_forward), {"init", init, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", BNN_BUILT_FOR) < 0) Py_CLEAR(m);       // binding.py compares it
    return m;
}
