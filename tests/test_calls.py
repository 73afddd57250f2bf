"""The binding's native calls (csrc/calls.cpp) against its Python code: the same bits, and None for whatever is out of the ordinary."""
import builtins
import os
import shutil
import time

import numpy as np
import pytest
import torch

from paper_2305_16513_amd import binding as B


@pytest.fixture(scope="module")
def native():
    B.lib()
    if B._calls is None and shutil.which("g++") is None:
        pytest.skip("not built")
    assert B._calls is not None, "not built, or for another torch"
    return B._calls


ODD = {"slide1d": (0, None, 3, 1.0), "slide1d_16": (0, None, 3, 1.0), "slide1d_padded": (0, None, 3, 1, 1, 0, 1.0), "pool2d": (0, None, 3, 3, 1, 1, 1, 1, 1.0),
       "pool2d_16": (0, None, 3, 3, 1, 1, 1, 1, 1.0), "maxpool2d_grad": (None, None, 3, 3, 1, 1, 1, 1), "avgpool2d_grad": (None, 4, 4, 3, 3, 1, 1, 1, 1, 0, 1.0),
       "conv1d": (None, None, 1, 0, 1, 2), "conv1d_16": (None, None, 1, 0, 1, 2), "conv1d_grad_input": (None, None, 9, 1, 0, 1, 2),
       "conv1d_grad_weight": (None, None, 3, 1, 0, 1, 2)}


@pytest.mark.parametrize("name", ODD)
def test_calls_out_of_the_ordinary_are_left_to_python(native, name):
    f, args = getattr(native, name), ODD[name]
    for x in (None, 3, "x", torch.zeros(2, 2, 9), torch.zeros(2, 2, 4, 4), np.zeros((2, 9), np.float32)):
        assert f(*[x if a is None else a for a in args]) is None
    assert f() is None and f(*args, 1) is None


@pytest.mark.parametrize("name", ODD)
def test_refusing_takes_next_to_nothing(native, name):
    """The Python code's time is all that a call costs that is left to it.  (By a C++ exception a refusal took 35 times as long as a call of len().)"""
    def least(f):
        def once():
            t = time.perf_counter()
            for _ in range(50):
                f()
            return time.perf_counter() - t
        return min(once() for _ in range(200))

    f, args = getattr(native, name), ODD[name]
    x = [torch.zeros(2, 2, 9) if a is None else a for a in args]
    assert least(lambda: f(*x)) < 15 * least(lambda: len(()))


def _loaded(monkeypatch):
    """What a first use of the library takes the native calls to be."""
    real = B.lib()
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_calls", None)
    monkeypatch.setattr(B.ctypes, "CDLL", lambda path: real)
    assert B.lib() is real
    return B._calls


def test_native_calls_are_not_taken_for_another_torch(native, monkeypatch):
    assert _loaded(monkeypatch) is native
    monkeypatch.setattr(torch, "__version__", torch.__version__ + ".other")
    assert _loaded(monkeypatch) is None


def test_native_calls_are_not_taken_for_another_library(native, monkeypatch, tmp_path):
    """They call the library that they are linked to; options would go to the other one."""
    (tmp_path / "libother.so").write_bytes(b"")
    with monkeypatch.context() as m:                  # another file, in the folder that the native calls are looked for beside
        m.setattr(B, "_HERE", str(tmp_path))
        m.setattr(B, "LIB_PATH", str(tmp_path / "libother.so"))
        assert _loaded(m) is None
    with monkeypatch.context() as m:                  # a path without a folder
        m.chdir(tmp_path)
        m.setattr(B, "LIB_PATH", "libother.so")
        assert _loaded(m) is None


@pytest.mark.parametrize("missing", ["torch", "g++", "headers"])
def test_the_library_is_built_without_what_only_the_native_calls_need(monkeypatch, tmp_path, capsys, missing):
    """... and old native calls don't stay beside a new library."""
    from paper_2305_16513_amd import build
    lib, calls = tmp_path / "libsws.so", tmp_path / "_calls.so"
    calls.write_bytes(b"old")
    real_run, real_import = build.subprocess.run, builtins.__import__

    def run(cmd, **k):
        if cmd[0] == "hipcc":                         # (compiling and linking the library: as if)
            if "-shared" in cmd:
                lib.write_bytes(b"new")
            return build.subprocess.CompletedProcess(cmd, 0, "", "")
        if missing == "g++":
            raise FileNotFoundError("g++")
        return real_run(["false"], **k)

    def imports(name, *a):
        if missing == "torch" and name == "torch":
            raise ImportError("no torch")
        return real_import(name, *a)

    monkeypatch.setattr(build, "LIB", str(lib))
    monkeypatch.setattr(build, "CALLS", str(calls), raising=False)
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "OBJ", str(tmp_path / "obj"))
    monkeypatch.setattr(build.subprocess, "run", run)
    monkeypatch.setattr(builtins, "__import__", imports)
    assert build.build() == str(lib)
    assert lib.read_bytes() == b"new" and not os.path.exists(calls) and "without native calls" in capsys.readouterr().err


def _all():
    """name of the native function, keyword of the output, the call"""
    g = torch.Generator(device="cuda").manual_seed(5)
    r = lambda *s: torch.randn(s, generator=g, device="cuda")
    x, p, w, gy = r(3, 4, 1001), r(2, 5, 9, 11), r(4, 1, 7), r(3, 4, 1001)
    h, ph, ones = x.bfloat16(), p.half(), torch.ones(2, 5, 5, 6, device="cuda")
    yield "slide1d", "y", lambda **k: B.sws_slide1d(B.OP_ADD, x, 5, 0.2, **k)
    yield "slide1d", "y", lambda **k: B.sws_slide1d(B.OP_MAX, x, 5, 2, **k)
    yield "slide1d_16", "y", lambda **k: B.sws_slide1d_16(B.OP_ADD, h, 64, 1 / 64, **k)
    yield "slide1d_padded", "y", lambda **k: B.sws_slide1d_padded(B.OP_MIN, x, 6, 2, 3, B.SWS_PAD_MIRROR, **k)
    yield "pool2d", "y", lambda **k: B.sws_pool2d(B.OP_ADD, p, 3, 2, 2, 1, 1, 0, 1 / 6, **k)
    yield "pool2d_16", "y", lambda **k: B.sws_pool2d_16(B.OP_MAX, ph, 3, 3, 2, 2, 1, 1, **k)
    yield "conv1d", "y", lambda **k: B.sws_conv1d(x, w, 1, 3, 1, 4, **k)
    yield "conv1d_16", "y", lambda **k: B.sws_conv1d_16(h, w, 1, 3, 1, 4, **k)
    yield "conv1d", "y", lambda **k: B.sws_conv1d(x, w, 2, 3, 2, 4, **k)
    yield "maxpool2d_grad", "gx", lambda **k: B.sws_maxpool2d_grad(p, ones, 3, 3, 2, 2, 1, 1, **k)
    yield "avgpool2d_grad", "gx", lambda **k: B.sws_avgpool2d_grad(p, 9, 11, 3, 3, 1, 1, 1, 1, B.SWS_DIV_REAL_CELLS, 1.0, **k)
    yield "conv1d_grad_input", "gx", lambda **k: B.sws_conv1d_grad_input(gy, w, 1001, 1, 3, 1, 4, **k)
    yield "conv1d_grad_weight", "gw", lambda **k: B.sws_conv1d_grad_weight(x, gy, 7, 1, 3, 1, 4, **k)


class _Noting:
    """The native calls, and which of them were asked and which of those answered."""

    def __init__(self, native):
        self.native, self.asked, self.answered = native, [], []

    def __getattr__(self, name):
        def f(*a):
            self.asked.append(name)
            y = getattr(self.native, name)(*a)
            if y is not None:
                self.answered.append(name)
            return y
        return f


@pytest.mark.gpu
def test_native_calls_give_the_bits_of_the_python_code(native, monkeypatch):
    side, seen = torch.cuda.Stream(), set()
    for name, key, f in _all():
        noting = _Noting(native)
        monkeypatch.setattr(B, "_calls", None)
        want = f()
        monkeypatch.setattr(B, "_calls", noting)
        got = f()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            other = f()
        side.synchronize()
        assert noting.answered == [name, name], name
        seen.add(name)
        out = torch.empty_like(want)                  # an output of the caller's, a stream handed over: the Python code, without asking
        assert f(**{key: out}) is out
        torch.cuda.synchronize()
        handed = f(stream=side)
        side.synchronize()
        assert noting.asked == [name, name], name
        for y in (got, other, out, handed):
            assert type(y) is torch.Tensor and y.shape == want.shape and y.dtype == want.dtype and y.is_contiguous() and not y.requires_grad
            if name == "conv1d_grad_weight":          # (atomic adds: no fixed order)
                assert torch.allclose(y, want, rtol=1e-5, atol=1e-4)
            else:
                assert torch.equal(y, want), name
    assert seen == set(ODD)


@pytest.mark.gpu
def test_native_calls_leave_watched_and_wrapped_tensors_to_python(native, monkeypatch):
    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode

    class Functions(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    class Dispatch(TorchDispatchMode):
        seen = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            Dispatch.seen += 1
            return func(*args, **(kwargs or {}))

    class Sub(torch.Tensor):
        pass

    x = torch.randn(3, 200, device="cuda")
    want = native.slide1d(B.OP_ADD, x, 5, 0.2)
    assert torch.equal(native.slide1d(B.OP_ADD, torch.nn.Parameter(x), 5, 0.2), want)        # (a plain tensor)
    noting = _Noting(native)
    monkeypatch.setattr(B, "_calls", noting)
    with Functions():
        y = B.sws_slide1d(B.OP_ADD, x, 5, 0.2)
    with Dispatch():
        z = B.sws_slide1d(B.OP_ADD, x, 5, 0.2)
    assert torch.equal(y, want) and torch.equal(z, want) and Dispatch.seen > 0               # (the output's allocation is seen)
    assert torch.equal(B.sws_slide1d(B.OP_ADD, x.as_subclass(Sub), 5, 0.2).as_subclass(torch.Tensor), want)
    assert noting.asked == ["slide1d"] * 3 and not noting.answered
    inside = []
    torch.func.vmap(lambda t: inside.append(native.slide1d(B.OP_ADD, t, 5, 0.2)) or t)(x)
    torch.func.functionalize(lambda t: inside.append(native.slide1d(B.OP_ADD, t, 5, 0.2)) or t)(x)
    torch.func.jvp(lambda t: inside.append(native.slide1d(B.OP_ADD, t, 5, 0.2)) or t, (x,), (x,))
    inside.append(native.slide1d(B.OP_ADD, torch.empty(3, 200, device="meta"), 5, 0.2))
    inside.append(native.slide1d(B.OP_ADD, x.to_sparse(), 5, 0.2))
    inside.append(native.slide1d(B.OP_ADD, x.t(), 5, 0.2))
    if torch.cuda.device_count() > 1:
        inside.append(native.slide1d(B.OP_ADD, x.to("cuda:1"), 5, 0.2))
    assert inside == [None] * len(inside) and len(inside) >= 6


@pytest.mark.gpu
def test_native_calls_refuse_what_python_refuses(native):
    x = torch.randn(2, 4, 64, device="cuda")
    w = torch.randn(4, 1, 7, device="cuda")
    for bad, err in ((lambda: B.sws_slide1d(0, x, 65), B.SwsError), (lambda: B.sws_slide1d(0, x, 0), B.SwsError), (lambda: B.sws_slide1d(7, x, 3), B.SwsError),
                     (lambda: B.sws_slide1d(0, x.double(), 3), TypeError), (lambda: B.sws_slide1d(0, x[:, :, ::2], 3), TypeError),
                     (lambda: B.sws_slide1d(0, x.cpu(), 3), TypeError), (lambda: B.sws_conv1d(x, w, 1, 0, 1, 2), B.SwsError),
                     (lambda: B.sws_conv1d(x, w, 0, 0, 1, 4), B.SwsError), (lambda: B.sws_conv1d(x, w, 1, 0, 11, 4), B.SwsError),
                     (lambda: B.sws_slide1d_padded(0, x, 3, -1, 1, 0), B.SwsError), (lambda: B.sws_slide1d_padded(0, x, 3, 70, 70, 1), B.SwsError)):
        with pytest.raises(err):
            bad()
    y = B.sws_slide1d(0, x, np.int64(5), np.float32(0.5))                    # numbers of other types: as before
    assert torch.equal(y, B.sws_slide1d(0, x, 5, 0.5))
    with torch.inference_mode():
        assert B.sws_slide1d(0, x, 5).is_inference()
    graph = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=s):
        y = B.sws_slide1d(0, x, 9, 1.0)
    for _ in range(3):
        x.normal_()
        want = B.sws_slide1d(0, x, 9, 1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)


@pytest.mark.gpu
def test_native_calls_take_the_numbers_that_the_python_code_takes(native):
    """Scales of types derived from float, negative whole ones and truth values; what is refused has not allocated an output."""
    x = torch.randn(2, 64, device="cuda")
    for scale in (np.float64(0.25), -2, True):
        y = native.slide1d(B.OP_ADD, x, 5, scale)
        assert y is not None and torch.equal(y, B.sws_slide1d(B.OP_ADD, x, 5, float(scale)))
    assert torch.equal(native.slide1d(True, x, True, 1.0), B.sws_slide1d(B.OP_MAX, x, 1))
    torch.cuda.synchronize()
    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    assert native.slide1d(B.OP_ADD, x, 5, np.float32(0.25)) is None and native.slide1d(B.OP_ADD, x, 5, 1 << 70) is None
    assert native.slide1d(B.OP_ADD, x, 5, "1") is None and native.slide1d(B.OP_ADD, x, 1 << 31, 1.0) is None
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == before


@pytest.mark.gpu
def test_other_threads_run_while_an_output_is_allocated(native):
    """16 GB from the device take half a millisecond, in which the allocator may also wait for it.  The longest time that another thread's loop stands still is 4 - 17 % of
    the call; with the interpreter locked it was 87 %."""
    import sys
    import threading
    x = torch.zeros(8, 1 << 29, device="cuda")
    native.slide1d(B.OP_ADD, x[:, :64].contiguous(), 5, 1.0)
    interval, shares = sys.getswitchinterval(), []
    sys.setswitchinterval(1e-5)
    try:
        for _ in range(6):
            torch.cuda.synchronize()
            torch.cuda.empty_cache()
            ticks, done = [], threading.Event()

            def watch():
                while not done.is_set() and len(ticks) < 1000000:
                    ticks.append(time.perf_counter())

            other = threading.Thread(target=watch)
            other.start()
            time.sleep(0.005)
            begin = time.perf_counter()
            y = native.slide1d(B.OP_ADD, x, 5, 1.0)
            end = time.perf_counter()
            time.sleep(0.002)
            done.set()
            other.join()
            assert y is not None
            del y
            shares.append(max(b - a for a, b in zip(ticks, ticks[1:]) if b > begin and a < end) / (end - begin))
    finally:
        sys.setswitchinterval(interval)
    assert min(shares) < 0.5, shares
