"""The linears' native marshalling: only calls of plain CUDA tensors are taken, every other one is left to the Python path, which
raises as it did (CPU), and the ordinary calls give the same bits and the same errors (GPU)."""
import ctypes
import importlib.util
import os
import shutil
import subprocess
import sysconfig

import pytest
import torch


@pytest.fixture(scope="module")
def qb():
    from paper_2603_01399_amd import binding
    return binding


class _Sub(torch.Tensor):
    pass


def test_not_on_a_gpu_or_not_enough_arguments(qb):
    f = qb._fast
    x, w, s, y = torch.zeros(2, 128).bfloat16(), torch.zeros(4096, dtype=torch.int8), torch.zeros(16).bfloat16(), torch.zeros(2, 16).bfloat16()
    for call in (lambda: f.w8_linear(x, w, s, 16, y, None), lambda: f.bf16_linear(x, s, 16, y, None), lambda: f.w8a8_linear(x, w, s, 16, None, y),
                 lambda: f.w4_linear(x, w, 16, y), lambda: f.w8_linear_fused(x, w, s, 16, None, 1e-6, None, y),
                 lambda: f.w8_gateup_swiglu(x, w, s, 16, None, 1e-6, y), lambda: f.w8_linear(None, w, s, 16, y, None)):
        assert call() == -1
    assert f.w8_linear(x, w, s, 16, y) == -1 and f.w4_linear() == -1
    with pytest.raises(TypeError):
        qb.w8_linear(x, w, s, 16, y=y)                                           # what the Python path says of it
    with pytest.raises(TypeError):
        qb.w4_linear(x, w, 16, y=y)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["int8", "bf16", "w8a8", "int4", "fused", "gated"])
def test_what_is_not_an_ordinary_call(qb, kind):
    """One thing wrong or unusual in a call that is ordinary otherwise: the native side leaves it, and the public function does what the
    Python path does - raises (on the host, before any launch) or gives the ordinary call's bits."""
    M, N, K = 3, 48, 256
    gen = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn(M, K, generator=gen, device="cuda").bfloat16()
    w = torch.randn(N, K, generator=gen, device="cuda") * 0.02
    wq, sc = qb.quantize_weights(torch.cat([w, w]) if kind == "gated" else w)
    wp, w4 = qb.pack_bf16_weights(w), qb.quantize_weights_w4(w)
    smooth = torch.rand(K, generator=gen, device="cuda") + 0.5
    gamma = (torch.rand(K, generator=gen, device="cuda") + 0.5).bfloat16()
    res = torch.randn(M, N, generator=gen, device="cuda").bfloat16()
    y = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    good = {"int8": dict(x=x, wq_packed=wq, scales=sc, N=N, y=y, workspace=None), "bf16": dict(x=x, w_packed=wp, N=N, y=y, workspace=None),
            "w8a8": dict(x=x, wq_packed=wq, scales=sc, N=N, smooth=smooth, y=y), "int4": dict(x=x, w4_packed=w4, N=N, y=y),
            "fused": dict(x=x, wq_packed=wq, scales=sc, N=N, gamma=gamma, eps=0.0, residual=res, y=y),
            "gated": dict(x=x, wq_packed=wq, scales=sc, I=N, gamma=gamma, eps=0.0, y=y)}[kind]
    name = {"int8": "w8_linear", "bf16": "bf16_linear", "w8a8": "w8a8_linear", "int4": "w4_linear", "fused": "w8_linear_fused",
            "gated": "w8_gateup_swiglu"}[kind]
    native, public = getattr(qb._fast, name), getattr(qb, name)
    assert native(*good.values()) == 0
    want = y.clone()

    rows = "I" if kind == "gated" else "N"
    same = [("x", x.as_subclass(_Sub))]
    wrong = [(rows, 2 ** 80), (rows, float(N)), (rows, True), (rows, None), ("x", x[0]), ("x", x.half()), ("x", None)]
    weights = {"bf16": "w_packed", "int4": "w4_packed"}.get(kind, "wq_packed")
    wrong += [(weights, good[weights].float()), (weights, good[weights].cpu())]
    if "scales" in good:
        wrong += [("scales", sc.float()), ("scales", None)]
    if kind == "int4":
        wrong += [("w4_packed", w4.flatten()[:-1])]
    if kind == "w8a8":
        wrong += [("smooth", smooth[:-1]), ("smooth", smooth.bfloat16()), ("smooth", torch.cat([smooth, smooth])[::2])]
    if "gamma" in good:
        wrong += [("gamma", gamma[:-1]), ("gamma", gamma.float()), ("gamma", torch.cat([gamma, gamma])[::2])]
        same += [("eps", 0)]
    if kind == "fused":
        wrong += [("residual", torch.cat([res, res])[:M + 1]), ("residual", res[:, :-1]), ("residual", res.t().contiguous().t()), ("residual", res.float()),
                  ("residual", res[0])]
    for key, value in same + wrong:
        print("not ordinary", kind, key, flush=True)
        call = dict(good, **{key: value})
        y.fill_(7.0)
        assert native(*call.values()) == -1
        if any(value is v for _, v in same):
            assert torch.equal(public(**call).view(torch.int16), want.view(torch.int16))
        else:
            with pytest.raises((TypeError, ValueError, ctypes.ArgumentError, qb.QuasarError)):
                public(**call)
            assert bool((y == 7.0).all())


_THROWING = """
#include "unlocked.hpp"
#include <new>
static int throws(int) { throw std::bad_alloc(); }
static PyObject *run(PyObject *, PyObject *) {
    PyObject *status = quasar::status_of(1, 1, [] { return quasar::call(throws, 0); });
    const int held = PyGILState_Check();
    if (!held) PyGILState_Ensure();
    return Py_BuildValue("(iN)", held, status);
}
static PyMethodDef methods[] = {{"run", run, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "throwing", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_throwing(void) { return PyModule_Create(&module); }
"""


def test_lock_after_an_exception(tmp_path):
    """An entry point that throws leaves the interpreter's lock held by the caller, and the call is not an ordinary one."""
    src, so = tmp_path / "throwing.cpp", tmp_path / "throwing.so"
    src.write_text(_THROWING)
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_01399_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-fPIC", "-shared", "-I" + csrc, "-I" + sysconfig.get_paths()["include"], "-o", str(so), str(src)], check=True)
    spec = importlib.util.spec_from_file_location("throwing", so)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    assert module.run() == (1, -1)


def test_another_build_of_the_library(qb, tmp_path):
    """use_library: the native side calls the library that the ctypes calls go to; a file that cannot be loaded changes nothing."""
    path, lib = qb.LIB_PATH, qb.lib()
    assert qb._fast.bound() == qb._native_addresses(lib)
    other = tmp_path / "other.so"
    shutil.copy(path, other)
    try:
        qb.use_library(str(other))
        assert qb.lib() is not lib and qb.LIB_PATH == str(other)
        assert qb._fast.bound() == qb._native_addresses(qb.lib()) and not set(qb._fast.bound()) & set(qb._native_addresses(lib))
        with pytest.raises(ImportError):
            qb.use_library(str(tmp_path / "none.so"))
        assert qb.LIB_PATH == str(other) and qb._fast.bound() == qb._native_addresses(qb.lib())
    finally:
        qb.use_library(path)
    assert qb._fast.bound() == qb._native_addresses(lib)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["int8", "bf16", "w8a8", "smoothed", "int4", "fused", "residual", "gated"])
def test_ordinary_calls(qb, kind):
    M, N, K = 5, 48, 256
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(M, K + 8, generator=gen, device="cuda").bfloat16()[:, :K]
    w = torch.randn(N, K, generator=gen, device="cuda") * 0.02
    smooth = torch.rand(K, generator=gen, device="cuda") + 0.5
    gamma = (torch.rand(K, generator=gen, device="cuda") + 0.5).bfloat16()
    res = torch.randn(M, N + 8, generator=gen, device="cuda").bfloat16()
    wq, sc = qb.quantize_weights(w)
    wq2, sc2 = qb.quantize_weights(torch.cat([w, w]))
    packed = {"bf16": qb.pack_bf16_weights(w), "int4": qb.quantize_weights_w4(w)}.get(kind, wq)
    calls = {"int8": lambda x, N, y: qb.w8_linear(x, wq, sc, N, y=y), "bf16": lambda x, N, y: qb.bf16_linear(x, packed, N, y=y),
             "w8a8": lambda x, N, y: qb.w8a8_linear(x, wq, sc, N, y=y), "smoothed": lambda x, N, y: qb.w8a8_linear(x, wq, sc, N, smooth=smooth, y=y),
             "int4": lambda x, N, y: qb.w4_linear(x, packed, N, y=y),
             "fused": lambda x, N, y: qb.w8_linear_fused(x, wq, sc, N, gamma=gamma, eps=1e-5, residual=res[:, :N], y=y),
             "residual": lambda x, N, y: qb.w8_linear_fused(x, wq, sc, N, residual=res[:, :N], y=y),
             "gated": lambda x, N, y: qb.w8_gateup_swiglu(x, wq2, sc2, N, gamma=gamma, y=y)}
    call = calls[kind]
    want = call(x, N, None)                                                      # without an output: the Python path
    y = torch.full((M, N + 16), 7.0, dtype=torch.bfloat16, device="cuda")
    out = y[:, :N]
    assert call(x, N, out) is out and torch.equal(out.view(torch.int16), want.view(torch.int16)) and bool((y[:, N:] == 7.0).all())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                                                # torch's current stream is the one that is used
        y2 = torch.zeros(M, N, dtype=torch.bfloat16, device="cuda")
        call(x, N, y2)
        got = y2.clone()
    side.synchronize()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    for bad in (lambda: call(x, N + 8, out), lambda: call(x[:, 8:K // 2 + 8 - 4], N, out), lambda: call(x[:, 1:129], N, out),
                lambda: call(x[0], N, out), lambda: call(x.float(), N, out), lambda: call(x.cpu(), N, out)):
        with pytest.raises((qb.QuasarError, TypeError, ValueError)):
            bad()
    param = torch.nn.Parameter(x.contiguous(), requires_grad=False)
    assert torch.equal(call(param, N, out.contiguous()).view(torch.int16), want.view(torch.int16))
    meta = torch.empty(M, K, dtype=torch.bfloat16, device="meta")
    with pytest.raises(TypeError):
        call(meta, N, out)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["w8a8", "int4", "norm", "residual", "gated"])
def test_calls_with_scratch(qb, kind):
    """Calls that use scratch are ordinary ones: taken by the native side, and the bits are those of the Python path (to which a
    subclass of Tensor goes)."""
    M, N, K = 20, 16 * 40, 8192
    gen = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn(M, K, generator=gen, device="cuda").bfloat16()
    w = torch.randn(N, K, generator=gen, device="cuda") * 0.02
    wq, sc = qb.quantize_weights(w)
    w4 = qb.quantize_weights_w4(w)
    gamma = (torch.rand(K, generator=gen, device="cuda") + 0.5).bfloat16()
    res = torch.randn(M, N, generator=gen, device="cuda").bfloat16()
    y = torch.empty((M, N // 2 if kind == "gated" else N), dtype=torch.bfloat16, device="cuda")
    native = {"w8a8": lambda: qb._fast.w8a8_linear(x, wq, sc, N, None, y), "int4": lambda: qb._fast.w4_linear(x, w4, N, y),
              "norm": lambda: qb._fast.w8_linear_fused(x, wq, sc, N, gamma, 1e-6, None, y),
              "residual": lambda: qb._fast.w8_linear_fused(x, wq, sc, N, None, 1e-6, res, y),
              "gated": lambda: qb._fast.w8_gateup_swiglu(x, wq, sc, N // 2, gamma, 1e-6, y)}[kind]
    call = {"w8a8": lambda x, y: qb.w8a8_linear(x, wq, sc, N, y=y), "int4": lambda x, y: qb.w4_linear(x, w4, N, y=y),
            "norm": lambda x, y: qb.w8_linear_fused(x, wq, sc, N, gamma=gamma, y=y),
            "residual": lambda x, y: qb.w8_linear_fused(x, wq, sc, N, residual=res, y=y),
            "gated": lambda x, y: qb.w8_gateup_swiglu(x, wq, sc, N // 2, gamma=gamma, y=y)}[kind]
    lib = qb.lib()
    assert {"w8a8": lib.quasar_w8a8_workspace_bytes(M, N, K), "int4": lib.quasar_w4_workspace_bytes(M, N, K),
            "gated": lib.quasar_w8_gateup_workspace_bytes(M, N // 2, K, 1)}.get(
                kind, lib.quasar_w8_fused_workspace_bytes(M, N, K, kind != "residual", kind == "residual")) > 0
    y.fill_(7.0)
    assert native() == 0
    want = call(x.as_subclass(_Sub), torch.empty_like(y))
    for got in (y, call(x, torch.empty_like(y)), call(x, None)):
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
