"""The native form of the binding's calls against their Python form: same outputs, same refusals."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2512_06443_amd import binding as B


def test_native_form_is_built_and_declines_what_it_does_not_know():
    B.lib()
    if torch.version.hip is None:
        pytest.skip("built with a torch for ROCm only")
    n = B._native
    assert n is not None
    x = torch.zeros(2, 8)                                     # not on the GPU: the Python form decides (and raises)
    p = torch.zeros(64, dtype=torch.uint8)
    assert n.quantize_act(x, None, None) is None
    assert n.quantize_act("x", None, None) is None
    assert n.mpgemm_f32(p, 1.0, x, 4, None, False, False, None) is None
    assert n.mpgemm(p, 1.0, x, x, 4, None, None, False, None) is None
    assert n.mpgemm(p) is None
    assert n.pack_weights(torch.zeros(4, 8, dtype=torch.int8)) is None
    with pytest.raises(AssertionError):
        B.quantize_act(x)
    with pytest.raises(TypeError):
        n.bind(1)


def test_native_form_of_another_torch_is_not_used(monkeypatch):
    """A file whose symbols all resolve can hold the layouts of another torch's headers."""
    L = B.lib()
    if torch.version.hip is None:
        pytest.skip("built with a torch for ROCm only")
    monkeypatch.setattr(B, "_native", None)
    B._load_native(L)
    assert B._native is not None and B._native.built_for == B.built_for()
    for name, value in (("__version__", "2.99.0"), ("version.git_version", "0" * 40)):
        with monkeypatch.context() as m:
            m.setattr("torch." + name, value)
            m.setattr(B, "_native", None)
            B._load_native(L)
            assert B._native is None


# The native form as it is, on CPU tensors: in place of the GPU tests of its arguments, of torch's allocator and of the stream are ones that
# count, and functions of the library that count.  Counted is whether the thread holds the interpreter's lock.
ON_CPU = r"""
#include <Python.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <stdexcept>
#include "vlut.h"
#define SHOWN extern "C" __attribute__((visibility("default")))
static int allocations_, calls_, held_, fail_at_;
static int called() { ++calls_; held_ += PyGILState_Check(); return 0; }
namespace at {
static Tensor counted_empty(c10::IntArrayRef size, TensorOptions o) {
    held_ += PyGILState_Check();
    if (++allocations_ == fail_at_) throw std::runtime_error("no memory");
    return at::empty(size, o);
}
}
namespace c10 { namespace hip { struct NoStream { void* stream() { return nullptr; } }; static NoStream no_stream() { return {}; } } }
static int quantize(const float*, int64_t, int64_t, int64_t, int8_t*, float*, void*) { return called(); }
static int mpgemm(const uint8_t*, float, const int8_t*, const float*, const int16_t*, int64_t, int64_t, int64_t, float*, int64_t, int32_t*, void*,
                  size_t, void*) { return called(); }
static int mpgemm5(const uint8_t*, float, const int8_t*, const float*, int64_t, int64_t, int64_t, float*, int64_t, int32_t*, void*, size_t,
                   void*) { return called(); }
static int mpgemm_f32(const uint8_t*, float, const float*, const float*, int64_t, int64_t, int64_t, int64_t, float*, int64_t, int32_t*, float*,
                      void*, size_t, void*) { return called(); }
static int pack(const int8_t*, int64_t, int64_t, uint8_t*, size_t, void*) { return called(); }
static size_t bytes3(int64_t, int64_t, int64_t) { return 64; }
static size_t bytes2(int64_t, int64_t) { return 64; }
SHOWN void* address(int i) {
    void* const a[] = {(void*)quantize, (void*)mpgemm, (void*)bytes3, (void*)mpgemm_f32, (void*)bytes3, (void*)mpgemm5, (void*)bytes3,
                       (void*)mpgemm5, (void*)bytes3, (void*)pack, (void*)bytes2, (void*)pack, (void*)bytes2, (void*)pack, (void*)bytes2};
    return a[i];
}
SHOWN void start(int fail_at) { allocations_ = calls_ = held_ = 0; fail_at_ = fail_at; }
SHOWN int allocations() { return allocations_; }
SHOWN int calls() { return calls_; }
SHOWN int held() { return held_; }
#define is_cuda is_cpu
#define empty counted_empty
#define getCurrentHIPStream no_stream
#include "torch_calls.cpp"
"""


@pytest.fixture(scope="module")
def on_cpu(tmp_path_factory):
    """(the module, its counting library, the library's path)"""
    import ctypes
    import importlib.util
    import os

    from paper_2512_06443_amd import build
    if torch.version.hip is None:
        pytest.skip("built with a torch for ROCm only")
    tmp_path = tmp_path_factory.mktemp("on_cpu")
    (tmp_path / "on_cpu.cpp").write_text(ON_CPU)
    path = str(tmp_path / "_vlut_torch.so")
    own = {build.TORCH_SRC: str(tmp_path / "on_cpu.cpp"), build.TORCH_LIB: path, "-O2": "-O0"}
    build._run([own.get(a, a) for a in build.torch_command()] + ["-I" + os.path.dirname(build.TORCH_SRC)])
    lib = ctypes.CDLL(path)
    lib.address.restype = ctypes.c_void_p
    spec = importlib.util.spec_from_file_location("_vlut_torch", path)
    n = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(n)
    n.bind(*[lib.address(i) for i in range(len(B._NATIVE_ORDER))])
    return n, lib, path


def test_native_form_allocates_and_calls_with_the_interpreter_released(on_cpu):
    """An allocation may wait for the device, as the call may: other threads run Python meanwhile, as they do in the Python form.  An
    allocation that fails leaves the call to that form, with the lock taken back."""
    import ctypes
    n, lib, path = on_cpu
    M, K, N = 8, 16, 3
    w, x, p = torch.zeros(M, K, dtype=torch.int8), torch.zeros(N, K), torch.zeros(64, dtype=torch.uint8)
    q, s = torch.zeros(1, K, 8, dtype=torch.int8), torch.zeros(N)
    product = (p, 0.5, q, s, M, None, None, True, None)
    for f, args, allocations in ((n.quantize_act, (x, None, None), 2), (n.mpgemm, product, 3), (n.mpgemm_g5, product, 3), (n.mpgemm_mixed, product, 3),
                                 (n.mpgemm_f32, (p, 0.5, x, M, None, True, True, None), 4), (n.pack_weights, (w,), 1), (n.pack_weights_g5, (w,), 1),
                                 (n.pack_weights_mixed, (w,), 1)):
        lib.start(0)
        out = f(*args)
        assert isinstance(out, tuple) and all(isinstance(t, torch.Tensor) for t in out), f
        assert (lib.allocations(), lib.calls(), lib.held()) == (allocations, 1, 0), f
        lib.start(allocations)
        assert f(*args) is None and lib.calls() == 0, f
    assert ctypes.PyDLL(path).calls() == 0 and ctypes.pythonapi.PyGILState_Check() == 1


def test_native_form_leaves_a_workspace_without_memory_to_the_python_form(on_cpu):
    """The Python form hands it over and the call refuses it; the lean call would run without one."""
    n, lib, _ = on_cpu
    M, K, N = 8, 16, 3
    p, q, s = torch.zeros(64, dtype=torch.uint8), torch.zeros(1, K, 8, dtype=torch.int8), torch.zeros(N)
    for f in (n.mpgemm, n.mpgemm_g5, n.mpgemm_mixed):
        lib.start(0)
        assert f(p, 0.5, q, s, M, None, None, False, torch.empty(0, dtype=torch.uint8)) is None
        assert (lib.allocations(), lib.calls()) == (0, 0)
        assert f(p, 0.5, q, s, M, None, None, False, torch.empty(64, dtype=torch.uint8)) is not None and lib.calls() == 1


def _both(monkeypatch, f):
    assert B._native is not None
    native = f()
    with monkeypatch.context() as m:
        m.setattr(B, "_native", None)
        return native, f()


def _same(a, b):
    assert type(a) is type(b) and len(a) == len(b)
    for u, v in zip(a, b):
        assert (u is None) == (v is None)
        if u is not None:
            assert u.dtype == v.dtype and u.shape == v.shape and u.device == v.device and torch.equal(u, v)


@pytest.mark.gpu
@pytest.mark.parametrize("N", [1, 9, 70])
@pytest.mark.parametrize("want", [False, True])
def test_native_form_gives_what_the_python_form_gives(monkeypatch, N, want):
    B.lib()
    torch.manual_seed(N)
    M, K = 203, 320
    W = torch.randint(-1, 2, (M, K), dtype=torch.int8, device="cuda")
    x = torch.randn(N, K + 4, device="cuda")[:, :K]            # row stride above K
    packed, mixed = B.pack_weights(W), B.pack_weights_mixed(W)
    for pack in (B.pack_weights, B.pack_weights_g5, B.pack_weights_mixed):
        assert torch.equal(*_both(monkeypatch, lambda: pack(W)))
    rows = torch.rand(M, device="cuda") + 0.5
    q = _both(monkeypatch, lambda: B.quantize_act(x))
    _same(*q)
    a_q, a_s = q[0]
    y = torch.empty(N, M + 5, device="cuda")
    for f in (lambda: B.mpgemm(packed, 0.25, a_q, a_s, M, want_acc=want), lambda: B.mpgemm(packed, np.float32(0.25), a_q, a_s, M),
              lambda: B.mpgemm(packed, 2, a_q, a_s, M, y=y[:, :M]), lambda: B.mpgemm_g5(B.pack_weights_g5(W), 0.5, a_q, a_s, M, want_acc=want),
              lambda: B.mpgemm_mixed(mixed, 0.5, a_q, a_s, M, want_acc=want),
              lambda: B.mpgemm_f32(packed, 0.25, x, M, want_acc=want, want_scales=want), lambda: B.mpgemm_f32(packed, rows, x, M)):
        n, p = _both(monkeypatch, lambda: [t.clone() if t is not None else None for t in f()])
        _same(n, p)


@pytest.mark.gpu
def test_native_form_refuses_what_the_python_form_refuses(monkeypatch):
    B.lib()
    M, K, N = 64, 128, 40
    packed = B.pack_weights(torch.zeros(M, K, dtype=torch.int8, device="cuda"))
    x = torch.randn(N, K, device="cuda")
    a_q, a_s = B.quantize_act(x)
    wrong = torch.full((M, K), 2, dtype=torch.int8, device="cuda")
    small = torch.empty(4, dtype=torch.uint8, device="cuda")
    for f in (lambda: B.mpgemm_f32(packed, 1.0, x, M, workspace=small), lambda: B.mpgemm_f32(packed, 1.0, x[:, :126], M),
              lambda: B.mpgemm_f32(packed, 1.0, x.half(), M), lambda: B.mpgemm_f32(packed, 1.0, x.t(), M), lambda: B.mpgemm_f32(packed, 1.0, x.cpu(), M),
              lambda: B.mpgemm_f32(packed, torch.ones(M - 1, device="cuda"), x, M), lambda: B.mpgemm_f32(packed, 1.0, x[:0], M),
              lambda: B.mpgemm(packed[1:], 1.0, a_q, a_s, M), lambda: B.mpgemm(packed, 1.0, a_q, a_s, 0),
              lambda: B.mpgemm(packed, 1.0, a_q, a_s, M, y=torch.empty(N, M - 1, device="cuda")), lambda: B.mpgemm(packed, None, a_q, a_s, M), lambda: B.pack_weights(wrong),
              lambda: B.pack_weights(wrong[:, :126]), lambda: B.pack_weights_g5(wrong), lambda: B.pack_weights_mixed(wrong)):
        def outcome():
            try:
                f()
            except Exception as e:
                return type(e), getattr(e, "status", None)
            return None
        n, p = _both(monkeypatch, outcome)
        assert n is not None and n == p


@pytest.mark.gpu
def test_native_form_leaves_modes_and_subclasses_to_the_python_form():
    from torch.overrides import TorchFunctionMode
    B.lib()
    n = B._native
    M, K, N = 64, 128, 5
    W = torch.randint(-1, 2, (M, K), dtype=torch.int8, device="cuda")
    x = torch.randn(N, K, device="cuda")
    packed = B.pack_weights(W)
    a_q, a_s = B.quantize_act(x)
    args = {"quantize_act": (x, None, None), "pack_weights": (W,), "mpgemm": (packed, 0.5, a_q, a_s, M, None, None, False, None),
            "mpgemm_f32": (packed, 0.5, x, M, None, False, False, None)}
    want = B.mpgemm_f32(packed, 0.5, x, M)[0]

    class Seen(TorchFunctionMode):
        functions = []

        def __torch_function__(self, func, types, args=(), kwargs=None):
            self.functions.append(func)
            return func(*args, **(kwargs or {}))

    class Sub(torch.Tensor):
        pass

    for name, a in args.items():
        assert getattr(n, name)(*a) is not None
        with Seen():
            assert getattr(n, name)(*a) is None, name
        for i, t in enumerate(a):
            if isinstance(t, torch.Tensor):
                assert getattr(n, name)(*a[:i], t.as_subclass(Sub), *a[i + 1:]) is None, (name, i)
    with Seen() as mode:
        y = B.mpgemm_f32(packed, 0.5, x, M)[0]
    assert torch.empty in mode.functions and torch.equal(y, want)
    assert torch.equal(B.mpgemm_f32(packed, 0.5, x.as_subclass(Sub), M)[0], want)
    assert torch.equal(B.mpgemm_f32(torch.nn.Parameter(packed, requires_grad=False), 0.5, x, M)[0], want)


@pytest.mark.gpu
def test_native_form_from_two_threads_and_streams():
    import threading
    B.lib()
    M, K = 640, 2560
    packed = B.pack_weights(torch.randint(-1, 2, (M, K), dtype=torch.int8, device="cuda"))
    xs = [torch.randn(N, K, device="cuda") for N in (5, 40)]
    want = [B.mpgemm_f32(packed, 0.5, x, M, want_acc=True, want_scales=True) for x in xs]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(100):
                    got = B.mpgemm_f32(packed, 0.5, xs[i], M, want_acc=True, want_scales=True)
                    a_q, a_s = B.quantize_act(xs[i])
                    y, acc = B.mpgemm(packed, 0.5, a_q, a_s, M, want_acc=True)
                    stream.synchronize()
                    if not (all(torch.equal(u, v) for u, v in zip(got, want[i])) and torch.equal(y, got[0]) and torch.equal(acc, got[1])):
                        bad.append(i)
        except Exception as e:
            bad.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
