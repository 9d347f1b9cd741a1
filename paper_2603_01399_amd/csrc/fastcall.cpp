// The linears' and fused linears' argument marshalling in native code: what binding.py does for an ordinary call - plain CUDA tensors, an output
// given - without its Python and ctypes steps.  Scratch that a call uses comes from torch's allocator, on the stream of the call.
//
// Every function returns the status of the C entry point it calls, or -1 for "not an ordinary call": binding.py then goes its
// own way, which raises what is to be raised.  Nothing is kept from one call for the next.
//
// What it measured, one 1024 x 1024 linear of 8 tokens through the binding, us of host time: 6.1 -> 4.0, of which the launch
// itself takes 2.9 (the kernel 3.4 on the GPU); a decoder block whose six calls are host-bound 40.9 -> 33.8.  A call with scratch and two
// launches (1024 x 8256 with a residual, 9 tokens; 7.3 in a graph): 13.0 through Python, 7.9 so.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/core/Allocator.h>
#include <c10/util/Exception.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "../../include/quasar.h"
#include "unlocked.hpp"

namespace {

using quasar::call;
using quasar::status_of;

// entry points of the library that binding.py has loaded, and torch's own two functions for the current stream
decltype(&quasar_w8_linear) p_w8_linear;
decltype(&quasar_bf16_linear) p_bf16_linear;
decltype(&quasar_w8a8_linear_split) p_w8a8_linear;
decltype(&quasar_w4_linear_split) p_w4_linear;
decltype(&quasar_w4_packed_bytes) p_w4_packed_bytes;
decltype(&quasar_w8a8_workspace_bytes) p_w8a8_workspace_bytes;
decltype(&quasar_w4_workspace_bytes) p_w4_workspace_bytes;
decltype(&quasar_w8_linear_fused_split) p_w8_linear_fused;
decltype(&quasar_w8_gateup_swiglu_split) p_w8_gateup_swiglu;
decltype(&quasar_w8_fused_workspace_bytes) p_w8_fused_workspace_bytes;
decltype(&quasar_w8_gateup_workspace_bytes) p_w8_gateup_workspace_bytes;
PyObject *g_device, *g_stream;

struct NotOrdinary {};

// a tensor of exactly torch's class (or a parameter) on the GPU; a subclass may stand for something else
const at::Tensor &cuda_tensor(PyObject *o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) throw NotOrdinary{};
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type) throw NotOrdinary{};
    return t;
}
const at::Tensor &any_tensor(PyObject *o) {
    if (!THPVariable_CheckExact(o)) throw NotOrdinary{};
    return THPVariable_Unpack(o);
}
int64_t integer(PyObject *o) {
    if (!PyLong_CheckExact(o)) throw NotOrdinary{};
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow) throw NotOrdinary{};
    return v;
}

struct Activations {
    const uint16_t *x;
    int64_t M, K, ldx;
    explicit Activations(PyObject *o) {
        const at::Tensor &t = cuda_tensor(o, at::kBFloat16);
        if (t.dim() != 2) throw NotOrdinary{};
        x = static_cast<const uint16_t *>(t.data_ptr());
        M = t.size(0);
        K = t.size(1);
        ldx = t.stride(0);
    }
};
struct Output {
    uint16_t *y;
    int64_t ldy;
    explicit Output(PyObject *o) {
        const at::Tensor &t = any_tensor(o);
        if (t.dim() < 1) throw NotOrdinary{};
        y = static_cast<uint16_t *>(t.data_ptr());
        ldy = t.stride(0);
    }
};
struct Workspace {
    void *p = nullptr;
    size_t bytes = 0;
    explicit Workspace(PyObject *o) {
        if (o == Py_None) return;
        const at::Tensor &t = any_tensor(o);
        p = t.data_ptr();
        bytes = t.nbytes();
    }
};

void *current_stream() {
    PyObject *dev = PyObject_CallNoArgs(g_device);
    PyObject *raw = dev ? PyObject_CallOneArg(g_stream, dev) : nullptr;
    Py_XDECREF(dev);
    if (!raw) throw NotOrdinary{};
    void *s = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    if (PyErr_Occurred()) throw NotOrdinary{};
    return s;
}

// A call with `need` bytes of scratch: entry(.., scratch, bytes, stream).  The scratch is given back behind the launch, for work that
// follows on the same stream.  Scratch makes a call faster and no call needs it: where memory is short it runs without.
template <typename Entry, typename... Args>
int call_with_scratch(Entry entry, size_t need, void *stream, Args... args) {
    quasar::Unlocked unlocked;
    c10::DataPtr scratch;
    if (need) {
        try {
            scratch = c10::GetAllocator(c10::DeviceType::CUDA)->allocate(need);
        } catch (const c10::OutOfMemoryError &) {
        }
    }
    return entry(args..., scratch.get(), scratch ? need : 0, stream);
}

// (x, wq_packed, scales, N, y, workspace)
PyObject *w8_linear(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return status_of(n, 6, [&] {
        const Activations x(a[0]);
        const void *w = cuda_tensor(a[1], at::kChar).data_ptr(), *sc = cuda_tensor(a[2], at::kBFloat16).data_ptr();
        const Output y(a[4]);
        const Workspace ws(a[5]);
        return call(p_w8_linear, x.x, x.M, x.K, x.ldx, static_cast<const int8_t *>(w), static_cast<const uint16_t *>(sc), integer(a[3]), y.y,
                           y.ldy, ws.p, ws.bytes, current_stream());
    });
}

// (x, w_packed, N, y, workspace)
PyObject *bf16_linear(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return status_of(n, 5, [&] {
        const Activations x(a[0]);
        const void *w = cuda_tensor(a[1], at::kBFloat16).data_ptr();
        const Output y(a[3]);
        const Workspace ws(a[4]);
        return call(p_bf16_linear, x.x, x.M, x.K, x.ldx, static_cast<const uint16_t *>(w), integer(a[2]), y.y, y.ldy, ws.p, ws.bytes,
                             current_stream());
    });
}

// (x, wq_packed, scales, N, smooth, y)
PyObject *w8a8_linear(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return status_of(n, 6, [&] {
        const Activations x(a[0]);
        const int64_t N = integer(a[3]);
        const void *w = cuda_tensor(a[1], at::kChar).data_ptr(), *sc = cuda_tensor(a[2], at::kBFloat16).data_ptr();
        const float *smooth = nullptr;
        if (a[4] != Py_None) {
            const at::Tensor &s = cuda_tensor(a[4], at::kFloat);
            if (s.numel() != x.K || !s.is_contiguous()) throw NotOrdinary{};
            smooth = static_cast<const float *>(s.data_ptr());
        }
        const Output y(a[5]);
        return call_with_scratch(p_w8a8_linear, p_w8a8_workspace_bytes(x.M, N, x.K), current_stream(), x.x, x.M, x.K, x.ldx, smooth,
                                 static_cast<const int8_t *>(w), static_cast<const uint16_t *>(sc), N, y.y, y.ldy);
    });
}

// (x, w4_packed, N, y)
PyObject *w4_linear(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return status_of(n, 4, [&] {
        const Activations x(a[0]);
        const at::Tensor &w = cuda_tensor(a[1], at::kByte);
        const int64_t N = integer(a[2]);
        if (w.numel() < (int64_t)p_w4_packed_bytes(N, x.K)) throw NotOrdinary{};
        const Output y(a[3]);
        return call_with_scratch(p_w4_linear, p_w4_workspace_bytes(x.M, N, x.K), current_stream(), x.x, x.M, x.K, x.ldx,
                                 static_cast<const void *>(w.data_ptr()), N, y.y, y.ldy);
    });
}

struct Gamma {
    const uint16_t *p = nullptr;
    Gamma(PyObject *o, int64_t K) {
        if (o == Py_None) return;
        const at::Tensor &t = cuda_tensor(o, at::kBFloat16);
        if (t.numel() != K || !t.is_contiguous()) throw NotOrdinary{};
        p = static_cast<const uint16_t *>(t.data_ptr());
    }
};
float real(PyObject *o) {
    if (!PyFloat_CheckExact(o)) throw NotOrdinary{};
    return static_cast<float>(PyFloat_AS_DOUBLE(o));
}

// (x, wq_packed, scales, N, gamma, eps, residual, y)
PyObject *w8_linear_fused(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return status_of(n, 8, [&] {
        const Activations x(a[0]);
        const void *w = cuda_tensor(a[1], at::kChar).data_ptr(), *sc = cuda_tensor(a[2], at::kBFloat16).data_ptr();
        const int64_t N = integer(a[3]);
        const Gamma gamma(a[4], x.K);
        const uint16_t *residual = nullptr;
        int64_t ldr = 0;
        if (a[6] != Py_None) {
            const at::Tensor &r = cuda_tensor(a[6], at::kBFloat16);
            if (r.dim() != 2 || r.size(0) != x.M || r.size(1) != N || r.stride(1) != 1) throw NotOrdinary{};
            residual = static_cast<const uint16_t *>(r.data_ptr());
            ldr = r.stride(0);
        }
        const float eps = real(a[5]);
        const Output y(a[7]);
        return call_with_scratch(p_w8_linear_fused, p_w8_fused_workspace_bytes(x.M, N, x.K, gamma.p != nullptr, residual != nullptr),
                                 current_stream(), x.x, x.M, x.K, x.ldx, gamma.p, eps, static_cast<const int8_t *>(w),
                                 static_cast<const uint16_t *>(sc), N, residual, ldr, y.y, y.ldy);
    });
}

// (x, wq_packed, scales, I, gamma, eps, y)
PyObject *w8_gateup_swiglu(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return status_of(n, 7, [&] {
        const Activations x(a[0]);
        const void *w = cuda_tensor(a[1], at::kChar).data_ptr(), *sc = cuda_tensor(a[2], at::kBFloat16).data_ptr();
        const int64_t I = integer(a[3]);
        const Gamma gamma(a[4], x.K);
        const float eps = real(a[5]);
        const Output y(a[6]);
        return call_with_scratch(p_w8_gateup_swiglu, p_w8_gateup_workspace_bytes(x.M, I, x.K, gamma.p != nullptr), current_stream(),
                                 x.x, x.M, x.K, x.ldx, gamma.p, eps, static_cast<const int8_t *>(w), static_cast<const uint16_t *>(sc), I,
                                 y.y, y.ldy);
    });
}

// (addresses of the eleven entry points, current device, current raw stream)
PyObject *bind(PyObject *, PyObject *args) {
    unsigned long long f[11];
    PyObject *device, *stream;
    if (!PyArg_ParseTuple(args, "(KKKKKKKKKKK)OO", &f[0], &f[1], &f[2], &f[3], &f[4], &f[5], &f[6], &f[7], &f[8], &f[9], &f[10], &device, &stream)) return nullptr;
    p_w8_linear = reinterpret_cast<decltype(p_w8_linear)>(f[0]);
    p_bf16_linear = reinterpret_cast<decltype(p_bf16_linear)>(f[1]);
    p_w8a8_linear = reinterpret_cast<decltype(p_w8a8_linear)>(f[2]);
    p_w4_linear = reinterpret_cast<decltype(p_w4_linear)>(f[3]);
    p_w4_packed_bytes = reinterpret_cast<decltype(p_w4_packed_bytes)>(f[4]);
    p_w8a8_workspace_bytes = reinterpret_cast<decltype(p_w8a8_workspace_bytes)>(f[5]);
    p_w4_workspace_bytes = reinterpret_cast<decltype(p_w4_workspace_bytes)>(f[6]);
    p_w8_linear_fused = reinterpret_cast<decltype(p_w8_linear_fused)>(f[7]);
    p_w8_gateup_swiglu = reinterpret_cast<decltype(p_w8_gateup_swiglu)>(f[8]);
    p_w8_fused_workspace_bytes = reinterpret_cast<decltype(p_w8_fused_workspace_bytes)>(f[9]);
    p_w8_gateup_workspace_bytes = reinterpret_cast<decltype(p_w8_gateup_workspace_bytes)>(f[10]);
    Py_INCREF(device);
    Py_INCREF(stream);
    Py_XSETREF(g_device, device);
    Py_XSETREF(g_stream, stream);
    Py_RETURN_NONE;
}

// the addresses that bind() was given
PyObject *bound(PyObject *, PyObject *) {
    auto at = [](auto *entry) { return static_cast<unsigned long long>(reinterpret_cast<uintptr_t>(entry)); };
    return Py_BuildValue("(KKKKKKKKKKK)", at(p_w8_linear), at(p_bf16_linear), at(p_w8a8_linear), at(p_w4_linear), at(p_w4_packed_bytes),
                         at(p_w8a8_workspace_bytes), at(p_w4_workspace_bytes), at(p_w8_linear_fused), at(p_w8_gateup_swiglu),
                         at(p_w8_fused_workspace_bytes), at(p_w8_gateup_workspace_bytes));
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(w8_linear), FAST(bf16_linear), FAST(w8a8_linear), FAST(w4_linear),
                         FAST(w8_linear_fused), FAST(w8_gateup_swiglu),
                         {"bind", bind, METH_VARARGS, nullptr}, {"bound", bound, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&module); }
