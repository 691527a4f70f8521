"""The binding's native marshalling (csrc/py_marshal.cpp): declines what it does not take, so that binding.py's own code raises what it always has, and
gives the library the same arguments as that code for what it takes."""
import os
import subprocess
import sys
import sysconfig

import numpy as np
import pytest

from paper_2604_01489_amd import binding


def _plain(args, name="gemm_epilogue_f32"):
    binding.load()
    return binding._native.plain(binding._entry[name], binding._raw, *args)


def test_declines_on_the_host():
    import torch
    t = torch.zeros(64, 64)
    good = [64, 64, 64, t, 64, t, 64, None, 1.0, "relu", t, 64, 1, None]
    assert _plain(good) is None                                   # tensors on the CPU
    for i, bad in [(0, np.int64(64)), (0, 2 ** 31), (0, True), (3, np.zeros(4)), (3, None), (8, "1"), (9, "tanh"), (9, 1)]:
        args = list(good)
        args[i] = bad
        assert _plain(args) is None, (i, bad)
    with pytest.raises(TypeError):
        _plain(good[:-1])
    with pytest.raises(ValueError):
        binding.gemm_epilogue_f32(*good[:-1])


def _fresh(monkeypatch):
    for name, value in (("_lib", None), ("_native", None), ("_entry", {}), ("_raw", None)):
        monkeypatch.setattr(binding, name, value)


def test_the_library_loads_without_it(monkeypatch, tmp_path):
    """No module, something else in its place, or one for another torch: a warning, and binding.py's own code takes every call."""
    import torch
    broken = tmp_path / "broken.so"
    broken.write_bytes(b"no module")
    t = torch.zeros(64, 64)
    for what, value in ((binding, str(tmp_path / "missing.so")), (binding, str(broken)), (torch, "0.0")):
        with monkeypatch.context() as m:
            _fresh(m)
            m.setattr(what, "MARSHAL_PATH" if what is binding else "__version__", value)
            with pytest.warns(RuntimeWarning, match="no native marshalling"):
                assert binding.status_string(0) == "ok"
            assert binding._native is None
            with pytest.raises(ValueError):
                binding.gemm_epilogue_f32(64, 64, 64, t, 64, t, 64, None, 1.0, "none", t, 64)
    with monkeypatch.context() as m:
        _fresh(m)
        binding.load()
        assert binding._native is not None


def test_a_call_that_outlives_the_interpreter(tmp_path):
    """A daemon thread that comes back from the library while the interpreter shuts down is ended by it there, as it is in a call through ctypes: the
    process ends with its own status and does not abort.  (The last object of the module to go keeps the interpreter in its shutdown until the thread is back.)"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    probe = str(tmp_path / "py_call_probe.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I" + sysconfig.get_paths()["include"], "-o", probe,
                    os.path.join(root, "tests", "py_call_probe.cpp")], check=True)
    code = """
import threading, time, sys
sys.path.insert(0, %r)
import py_call_probe
assert py_call_probe.call(0) == 7 and py_call_probe.call(-1) is None
class Last:
    def __del__(self, sleep=time.sleep): sleep(1.5)
last = Last()
threading.Thread(target=py_call_probe.call, args=(700000,), daemon=True).start()
time.sleep(0.2)
print("done", flush=True)
""" % str(tmp_path)
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=60)
    assert res.stdout == "done\n" and res.returncode == 0, (res.returncode, res.stdout, res.stderr)


def _calls():
    import torch
    g = torch.Generator(device="cuda").manual_seed(5)
    bf = lambda *s: torch.randn(*s, device="cuda", generator=g).bfloat16()
    f = lambda *s: torch.rand(*s, device="cuda", generator=g)
    A, B, F, bias, R = bf(72, 136), bf(136, 88), f(136, 136), f(136), bf(72, 88)
    ws = torch.empty(1 << 20, device="cuda")
    X, W = bf(2, 9, 9, 32), bf(40, 3, 3, 32)
    S = bf(512, 512)
    C = lambda *s, dtype=torch.float32: torch.full(s, -1.0, device="cuda", dtype=dtype)
    fused = binding.gemm_epilogue_bf16_fused

    def run(call, *outs):
        call(*outs)
        return outs
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())

    def on_side(c):
        binding.gemm_epilogue_f32(136, 136, 136, F, 136, F, 136, bias, 1, "none", c, 136, stream=side)
        side.synchronize()
    return [
        lambda: run(lambda c: binding.gemm_epilogue_bf16(72, 88, 136, A, 136, B, 88, bias, 0.5, "gelu_tanh", c, 88), C(72, 88)),
        lambda: run(lambda c: binding.gemm_epilogue_f32(136, 136, 136, F, 136, F, 136, None, 2, "relu", c, 136, 1), C(136, 136)),
        lambda: run(on_side, C(136, 136)),
        lambda: run(lambda c: fused(72, 88, 136, A, 136, B, 88, c, 88, row_scale=bias, bias=bias, residual=R, ldr=88, beta=-0.5, alpha=0.75, clamp=(-0.25, 1)),
                    C(72, 88, dtype=torch.bfloat16)),
        lambda: run(lambda c: fused(88, 72, 136, B, 88, A, 136, c, 72, transA=1, transB=True, act="relu", plan="splitk", split_k=2, workspace=ws), C(88, 72)),
        lambda: run(lambda c: fused(512, 3, 512, S, 512, A, 3, c, 3, a_structure="sym_upper"), C(512, 3)),
        lambda: run(lambda y: binding.conv2d_epilogue_bf16(X, W, y, stride=(2, 1), pad=(1, 0), dil=(1, 2), alpha=0.5, bias=bias, act="relu", clamp=(0.0, 2.5)),
                    C(2, 5, 5, 40, dtype=torch.bfloat16)),
        lambda: run(lambda p, y: (binding.gemm_rowsum_params_bf16(72, 136, A, 136, True, bias, p, workspace=ws), binding.gemm_rowsum_bf16(72, 136, A, 136, p, 0.5, y)),
                    C(137), C(72)),
    ]


@pytest.mark.gpu
def test_same_calls_as_the_python_code(monkeypatch):
    import torch
    binding.load()
    taken = []
    native = binding._native

    class Counting:
        def __getattr__(self, name):
            def call(*args):
                status = getattr(native, name)(*args)
                taken.append(status)
                return status
            return call
    for call in _calls():
        taken.clear()
        with monkeypatch.context() as m:
            m.setattr(binding, "_native", Counting())
            fast = call()
        assert taken and all(s == 0 for s in taken)
        with monkeypatch.context() as m:
            m.setattr(binding, "_native", None)
            slow = call()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(fast, slow))


@pytest.mark.gpu
def test_what_was_refused_still_is():
    import torch
    A, C = torch.zeros(64, 64, device="cuda", dtype=torch.bfloat16), torch.zeros(64, 64, device="cuda")
    with pytest.raises(ValueError):
        binding.gemm_epilogue_bf16(64, 64, 65, A, 65, A, 64, None, 1.0, "none", C, 64)
    with pytest.raises(ValueError):
        binding.gemm_epilogue_bf16_fused(64, 64, 64, A, 64, A, 64, C, 64, row_scale=torch.zeros(63, device="cuda"))
    with pytest.raises(ValueError):
        binding.gemm_rowsum_params_bf16(64, 64, A, 64, True, None, torch.zeros(64, device="cuda"))
    with pytest.raises(ValueError):
        binding.gemm_epilogue_bf16(64, 64, 64, A.cpu(), 64, A, 64, None, 1.0, "none", C, 64)
    with pytest.raises(KeyError):
        binding.gemm_epilogue_bf16(64, 64, 64, A, 64, A, 64, None, 1.0, "tanh", C, 64)
    with pytest.raises(ValueError):
        binding.conv2d_epilogue_bf16(A, A, C)
    with pytest.raises(binding.GemmEpilogueError) as err:
        binding.gemm_epilogue_bf16(64, 64, 64, A, 63, A, 64, None, 1.0, "none", C, 64)
    assert err.value.status == 3
    # and other ints than exact ones are taken as before
    binding.gemm_epilogue_bf16(np.int32(64), 64, 64, A, 64, A, 64, None, 1.0, "none", C, 64)
    torch.cuda.synchronize()
