"""The binding's native marshalling (csrc/sqcall.cpp): arguments that are not
plain go to the ctypes path, which refuses them as before (CPU); plain ones give
what the ctypes path gives, errors included (GPU)."""
import ctypes
import os
import subprocess
import sys
import timeit

import pytest
import torch

from paper_2609_39056_amd import _build
from paper_2609_39056_amd import binding as B


@pytest.fixture(scope="module", autouse=True)
def _built():
    if not (os.path.exists(B.LIB_PATH) and os.path.exists(B.CALL_PATH)):
        _build.build()
    B.lib()
    assert not isinstance(B._call, B._NoCall)


def layer(dev, M=40, K=256, N=128, bits=8):
    g = torch.Generator(device=dev)
    g.manual_seed(3)
    x = torch.randn((M, K), generator=g, device=dev).to(torch.bfloat16)
    act = B.ActParams(tok2stream=torch.arange(M, device=dev, dtype=torch.int32) % 3,
                      gamma=torch.rand((4, 3), generator=g, device=dev) + 0.5, step=2, act_bits=bits,
                      clip=torch.full((4,), 2.0, device=dev), dinv=torch.rand((K,), generator=g, device=dev) + 0.5)
    w = B.Weight(qw=torch.randint(0, 256, (N, K // 2), generator=g, device=dev, dtype=torch.uint8),
                 w_scale=(torch.rand((K // 128, N), generator=g, device=dev) * 0.01).half(), w_group=128,
                 bias=torch.randn((N,), generator=g, device=dev).to(torch.bfloat16))
    return x, act, w, torch.empty((M, N), device=dev), torch.empty(1 << 20, dtype=torch.uint8, device=dev)


def test_not_plain_goes_to_ctypes():
    x, act, w, y, ws = layer("cpu")
    addr = B.lib().sq_address["sq_linear_w4a8"]
    assert B._call.linear(addr, x, act, w, y, 0, ws, None) is NotImplemented  # host tensors
    assert B._call.linear(addr, None, act, w, y, 0, ws, None) is NotImplemented
    assert B._call.linear(addr, x, act) is NotImplemented
    with pytest.raises(ValueError, match="device tensors"):
        B.sq_linear_w4a8(x, act, w, y, B.SQ_OUT_F32, ws)
    with pytest.raises(ValueError, match="device tensors"):
        B.sq_quantize_act(x, act, ws, y)


def test_a_refusal_is_cheap():
    """Arguments that are not plain cost little before the ctypes path takes
    them: about a Python call, not a C++ exception (50 times that).  The least of
    many runs, so that a busy machine does not matter."""

    class Act(B.ActParams):
        pass

    x, act, w, y, ws = layer("cpu")
    sub = Act(**act.__dict__)
    addr = B.lib().sq_address["sq_linear_w4a8"]

    def least(f):
        return min(timeit.repeat(f, number=1000, repeat=30))

    plain = least(lambda: max(1, 2, 3, 4))
    for args in ((x, act, w, y, 0, ws, None), (x, sub, w, y, 0, ws, None), (x, act, w, y, 0, None, None)):
        assert B._call.linear(addr, *args) is NotImplemented
        assert least(lambda: B._call.linear(addr, *args)) < 15 * plain


@pytest.mark.parametrize("why", ["missing", "not a module", "another torch"])
def test_without_the_module(why, tmp_path, monkeypatch):
    """The binding loads without a usable module, with a warning, and the
    ctypes code takes every call."""
    path = tmp_path / "sqcall.so"
    if why == "not a module":
        path.write_bytes(b"no ELF")
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_call", None)
    if why == "another torch":
        monkeypatch.setattr(torch, "__version__", "0.0.0")
    else:
        monkeypatch.setattr(B, "CALL_PATH", str(path))
    with pytest.warns(RuntimeWarning, match="marshalled with ctypes"):
        B.lib()
    assert B.sq_workspace_bytes(B.SQ_VARIANT_FUSED, 40, 256, 128, 8) > 0
    x, act, w, y, ws = layer("cpu")
    for fn in (B.sq_linear_w4a8, B.sq_linear_w4a4):
        with pytest.raises(ValueError, match="device tensors"):
            fn(x, act, w, y, B.SQ_OUT_F32, ws)


@pytest.mark.parametrize("why", ["no compiler", "no torch headers"])
def test_build_without_the_module(why, tmp_path, monkeypatch):
    """Where the module cannot be built the build warns, and no module of an
    earlier build stays."""
    old = tmp_path / "sqcall.so"
    old.write_bytes(b"")
    monkeypatch.setattr(_build, "CALL", str(old))
    if why == "no compiler":
        monkeypatch.setenv("PATH", str(tmp_path))
    else:
        monkeypatch.setitem(sys.modules, "torch.utils.cpp_extension", None)
        monkeypatch.delattr(torch.utils, "cpp_extension", raising=False)
    with pytest.warns(RuntimeWarning, match="sqcall.cpp was not built"):
        _build._build_call()
    assert not old.exists()


# A module around sqcall.cpp's own call wrapper: nap() is a call that takes 0.6 s.
# The process is kept alive past the interpreter's end, so that the call returns
# to a finalized interpreter.
NAP = """
#include "sqcall.cpp"
#include <unistd.h>
#include <cstdlib>
PyObject* nap(PyObject*, PyObject* const*, Py_ssize_t n) {
  return guarded(n, 0, [] { return true; }, [] { usleep(600000); return SQ_OK; });
}
PyMethodDef nap_methods[] = {
    {"setup", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(setup)), METH_FASTCALL, nullptr},
    {"nap", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(nap)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef nap_def = {PyModuleDef_HEAD_INIT, "nap", nullptr, -1, nap_methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_nap() {
  atexit([] { usleep(1500000); });
  return PyModule_Create(&nap_def);
}
"""


def test_daemon_thread_in_a_call_at_exit(tmp_path):
    """The interpreter ends while a daemon thread is inside a call: the process
    exits normally, as with a call through ctypes."""
    src = tmp_path / "nap.cpp"
    src.write_text(NAP)
    subprocess.run(_build.call_command(str(src), str(tmp_path / "nap.so")), check=True)
    main = ("import sys, threading, time, torch\n"
            f"sys.path.insert(0, {str(tmp_path)!r})\n"
            "import nap\n"
            "nap.setup(int, str)\n"
            "assert nap.nap(1) is NotImplemented and nap.nap() == 0\n"
            "threading.Thread(target=nap.nap, daemon=True).start()\n"
            "time.sleep(0.2)\n")
    r = subprocess.run([sys.executable, "-c", main], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M", [40, 300])
def test_native_equals_ctypes(M, bits, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    K, N = 256, 128
    x, act, w, y, _ = layer("cuda", M, K, N, bits)
    down = layer("cuda", M, N, K, bits)
    nxt = down[1]
    nxt.range_mode = B.SQ_RANGE_STATIC
    ws = B.alloc_workspace(B.SQ_VARIANT_FUSED, M, K, N, bits)
    side = torch.cuda.Stream()

    def calls(stream):
        qx, sc = B.act_buffers(M, K, bits)
        B.sq_quantize_act(x, act, qx, sc, stream)
        out = [qx, sc]
        for d, dt in ((B.SQ_OUT_F32, torch.float32), (B.SQ_OUT_BF16, torch.bfloat16)):
            y1, y2 = torch.empty((M, N), dtype=dt, device="cuda"), torch.empty((M, N), dtype=dt, device="cuda")
            (B.sq_linear_w4a8 if bits == 8 else B.sq_linear_w4a4)(x, act, w, y1, d, ws, stream)
            if bits == 8:
                B.sq_gemm_w4a8(qx, sc, w, y2, d, None, stream)
            else:
                B.sq_gemm_w4a4(qx, sc, act, w, y2, d, None, stream)
            out += [y1, y2]
        q2, s2 = B.act_buffers(M, N, bits)
        y3 = torch.empty((M, K), device="cuda")
        if bits == 8:
            B.sq_linear_w4a8_gelu_quant(x, act, w, nxt, q2, s2, ws, stream)
        elif M <= 128:
            B.sq_linear_w4a4_gelu_quant(x, act, w, nxt, q2, s2, None, ws, stream)
        else:
            q2 = torch.empty((M, N), dtype=torch.uint8, device="cuda")
            s2, kc = torch.empty((M, N // 64), device="cuda"), torch.empty((M, N // 64), device="cuda")
            B.sq_linear_w4a4_gelu_quant(x, act, w, nxt, q2, s2, kc, ws, stream)
            B.sq_gemm_w4a4_fp8(q2, s2, kc, nxt, down[2], y3, B.SQ_OUT_F32, None, stream)
            out += [kc, y3]
        torch.cuda.synchronize()
        return out + [q2, s2]

    class Recorder:
        """The module, noting every call's name; none of them may fall back."""

        def __getattr__(self, name):
            def call(*args):
                made.add(name)
                st = getattr(real, name)(*args)
                assert st is not NotImplemented, name
                return st

            return call

    Ctypes, real, made = B._NoCall, B._call, set()
    monkeypatch.setattr(B, "_call", Recorder())
    native = [calls(s) for s in (None, side, side.cuda_stream)]
    with torch.cuda.stream(side):
        native.append(calls(None))
    assert made == {"quantize", "linear"} | ({"gemm8", "gelu8"} if bits == 8 else {"gemm4", "gelu4"}) | (
        {"gemm4_fp8"} if bits == 4 and M > 128 else set())
    # the stream of None is the current one: the calls come after the work before them there
    x0, big = x.clone(), torch.randn((4096, 4096), device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        x.zero_()
        for _ in range(20):
            big = big @ big * 1e-3
        x.copy_(x0)
        native.append(calls(None))
    monkeypatch.setattr(B, "_call", Ctypes())
    want = calls(None)
    for got in native:
        assert len(got) == len(want)
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    # errors: the same from both
    for call in (real, Ctypes()):
        monkeypatch.setattr(B, "_call", call)
        fn = B.sq_linear_w4a8 if bits == 8 else B.sq_linear_w4a4
        with pytest.raises(B.SqError) as e:
            fn(x, act, w, y, 7, ws)
        assert e.value.status == -4
        bad = B.ActParams(tok2stream=act.tok2stream, gamma=act.gamma, step=9, act_bits=bits)
        with pytest.raises(B.SqError) as e:
            fn(x, bad, w, y, B.SQ_OUT_F32, ws)
        assert e.value.status == -2
        with pytest.raises(ValueError, match="contiguous"):
            fn(x.t(), act, w, y, B.SQ_OUT_F32, ws)
        with pytest.raises(B.SqError) as e:
            fn(x, act, w, y, B.SQ_OUT_F32, ws[:128])
        assert e.value.status == -5
    assert ctypes.sizeof(B.sq_weight) == 40  # the struct both paths fill
