"""Host-side checks of the C ABI that need no GPU: the library loads, exports every
symbol the header declares, and rejects bad arguments before anything is launched."""
import ctypes
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADERS = [os.path.join(ROOT, "include", n) for n in ("sws.h", "sws_dev.h")]


@pytest.fixture(scope="module")
def L():
    from paper_2305_16513_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2305_16513_amd import build
        build.build()
    return binding.lib()


def _declared():
    names = set()
    for h in HEADERS:
        text = re.sub(r"/\*.*?\*/", "", open(h).read(), flags=re.S)
        names |= set(re.findall(r"\b(sws_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_header_symbols_are_exported(L):
    from paper_2305_16513_amd import binding
    names = _declared()
    assert set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(L, n) is not None


def test_the_binding_and_the_library_agree_on_output_lengths(L):
    """The binding works the length out by itself: every sign and both sides of every limit."""
    from paper_2305_16513_amd import binding
    for n in (-1, 0, 1, 2, 5, 6, 7, 112, 2 ** 31 + 5, 2 ** 40):
        for w in (-1, 0, 1, 2, 3, 7, 50, 2 ** 31 - 1):
            for s in (-1, 0, 1, 2, 3, 64):
                for p in (-1, 0, 1, 3, 1000):
                    for d in (0, 1, 2, 8):
                        assert binding._out_len(n, w, s, p, d) == L.sws_out_len(n, w, s, p, d), (n, w, s, p, d)
                    want = L.sws_out_len(n, w, s, p, 1)
                    assert binding._out_hw(n, 50, w, 3, s, 2, p, 1) == (want, 25) and binding._out_hw(50, n, 3, w, 2, s, 1, p) == (25, want)


def test_output_lengths_of_numbers_that_are_not_plain_ints(L):
    """numpy's fixed-width numbers and numbers beyond 32 bits: an output is as long as the library will write, whatever the
    call's numbers become on their way in (a shorter one would be written behind its end)."""
    from paper_2305_16513_amd import binding
    for a in [(100, 3, 1, np.uint8(200), 1), (np.int8(100), 3, 1, 20, 1), (np.int16(30000), 3, 1, 1000, 1), (100, np.uint8(1), 1, 0, 1),
              (2 ** 31, np.int32(5000), 1, 0, np.int32(2 ** 20)), (100, 3, np.int64(2), np.int8(100), 1), (100, 3, 2 ** 32 + 2, 0, 1),
              (100, 2 ** 32 + 3, 1, 0, 1), (100, 3, 1, 2 ** 32 + 1, 1), (100, 3, 1, 0, 2 ** 32 + 1), (100, 1 - 2 ** 32, 1, 0, 1),
              (100, 3, 1, -2 ** 32, 1), (2 ** 64 + 100, 3, 1, 0, 1), (100, 3, True, False, True)]:
        assert binding._out_len(*a) == L.sws_out_len(*a), a
        if a[4] == 1:
            n, w, st, p, _ = a
            want = L.sws_out_len(n, w, st, p, 1)
            assert binding._out_hw(n, 50, w, 3, st, 2, p, 1) == (want, 25) and binding._out_hw(50, n, 3, w, 2, st, 1, p) == (25, want), a


def test_out_len(L):
    assert L.sws_out_len(1048576, 5, 1, 0, 1) == 1048572
    assert L.sws_out_len(4096, 3, 1, 0, 1) == 4094
    assert L.sws_out_len(112, 3, 2, 1, 1) == 56
    assert L.sws_out_len(112, 3, 1, 1, 1) == 112
    assert L.sws_out_len(16384, 255, 1, 0, 1) == 16130
    assert L.sws_out_len(10, 3, 1, 0, 4) == 2
    assert L.sws_out_len(4, 5, 1, 0, 1) == -1
    assert L.sws_out_len(4, 0, 1, 0, 1) == -1
    assert L.sws_out_len(4, 2, 0, 0, 1) == -1
    assert L.sws_out_len(-1, 2, 1, 0, 1) == -1


def test_status_strings(L):
    seen = {L.sws_status_string(i) for i in range(4)}
    assert len(seen) == 4 and all(s for s in seen)
    assert L.sws_status_string(99)


def test_slide1d_argument_checks(L):
    one = ctypes.c_void_p(16)      # never dereferenced: every call below fails or is empty
    nul = ctypes.c_void_p(0)
    assert L.sws_slide1d(0, one, one, 0, 100, 3, 1.0, nul) == 0            # no rows: nothing to do
    assert L.sws_slide1d(7, one, one, 1, 100, 3, 1.0, nul) == 1            # unknown op
    assert L.sws_slide1d(0, one, one, 1, 100, 0, 1.0, nul) == 1            # w < 1
    assert L.sws_slide1d(0, one, one, 1, 100, 101, 1.0, nul) == 1          # w > len
    assert L.sws_slide1d(0, one, one, -1, 100, 3, 1.0, nul) == 1
    assert L.sws_slide1d(0, one, one, 1, -5, 3, 1.0, nul) == 1
    assert L.sws_slide1d(0, nul, one, 1, 100, 3, 1.0, nul) == 1            # NULL with output
    assert L.sws_slide1d(0, one, nul, 1, 100, 3, 1.0, nul) == 1
    assert L.sws_slide1d(0, one, one, 1, 2 ** 31, 3, 1.0, nul) == 1        # row too long for int32
    assert L.sws_slide1d(0, one, one, 2 ** 40, 2 ** 30, 3, 1.0, nul) == 1  # size overflow


def test_slide1d_padded_argument_checks(L):
    one = ctypes.c_void_p(16)
    nul = ctypes.c_void_p(0)
    f = L.sws_slide1d_padded
    assert f(0, one, one, 0, 100, 3, 1, 1, 0, 1.0, nul) == 0               # no rows: nothing to do
    assert f(0, one, one, 1, 100, 3, -1, 1, 0, 1.0, nul) == 1              # negative pad
    assert f(0, one, one, 1, 100, 3, 1, 1, 5, 1.0, nul) == 1               # unknown mode
    assert f(0, one, one, 1, 100, 3, 3, 1, 4, 1.0, nul) == 1               # shrinking window: pad not below w
    assert f(0, one, one, 1, 100, 103, 1, 1, 0, 1.0, nul) == 1             # w longer than the extended row
    assert f(0, one, one, 1, 100, 3, 100, 0, 1, 1.0, nul) == 1             # mirror pad reaches past the row
    assert f(0, one, one, 1, 100, 3, 0, 101, 2, 1.0, nul) == 1             # periodic pad longer than the row
    assert f(0, one, one, 1, 0, 1, 1, 1, 0, 1.0, nul) == 1                 # empty rows cannot be extended
    assert f(5, one, one, 1, 100, 3, 1, 1, 0, 1.0, nul) == 1               # unknown op
    assert f(0, nul, one, 1, 100, 3, 1, 1, 0, 1.0, nul) == 1               # NULL with output
    assert f(0, one, one, 1, 2 ** 31 - 10, 3, 100000, 0, 3, 1.0, nul) == 1  # extended row too long for int32


def test_slide1d_pair_argument_checks(L):
    one = ctypes.c_void_p(16)
    nul = ctypes.c_void_p(0)
    assert L.sws_slide1d_pair(one, one, one, one, 0, 100, 3, nul) == 0        # no rows: nothing to do
    assert L.sws_slide1d_pair(one, one, one, one, 1, 100, 0, nul) == 1        # w < 1
    assert L.sws_slide1d_pair(one, one, one, one, 1, 100, 101, nul) == 1      # w > len
    assert L.sws_slide1d_pair(one, one, one, one, -1, 100, 3, nul) == 1
    assert L.sws_slide1d_pair(one, one, one, one, 1, 2 ** 31, 3, nul) == 1    # row too long for int32
    for k in range(4):                                                       # any NULL plane with output
        args = [one, one, one, one]
        args[k] = nul
        assert L.sws_slide1d_pair(*args, 1, 100, 3, nul) == 1


def test_pool2d_argument_checks(L):
    one, nul = ctypes.c_void_p(16), ctypes.c_void_p(0)
    ok = (0, one, one, 0, 3, 8, 8, 3, 3, 1, 1, 1, 1, 1.0, nul)
    assert L.sws_pool2d(*ok) == 0                                          # N = 0
    bad = lambda **kw: L.sws_pool2d(*[kw.get(n, v) for n, v in zip(
        ("op", "x", "y", "N", "C", "H", "W", "kh", "kw", "sh", "sw", "ph", "pw", "scale", "s"),
        (0, one, one, 1, 3, 8, 8, 3, 3, 1, 1, 1, 1, 1.0, nul))])
    assert bad(op=5) == 1
    assert bad(kh=0) == 1
    assert bad(sw=0) == 1
    assert bad(ph=3) == 1                                                  # window wholly in padding
    assert bad(pw=-1) == 1
    assert bad(kh=11) == 1                                                 # window larger than padded input
    assert bad(x=nul) == 1
    assert bad(N=-1) == 1


def test_conv_argument_checks(L):
    one, nul = ctypes.c_void_p(16), ctypes.c_void_p(0)
    c1 = lambda **kw: L.sws_conv1d(*[kw.get(n, v) for n, v in zip(
        ("x", "w", "y", "B", "Cin", "L", "Cout", "k", "stride", "pad", "dil", "groups", "s"),
        (one, one, one, 1, 4, 32, 6, 3, 1, 0, 1, 1, nul))])
    assert c1(B=0) == 0
    assert c1(groups=3) == 1                                               # Cin % groups
    assert c1(groups=4) == 1                                               # Cout % groups
    assert c1(k=0) == 1 and c1(stride=0) == 1 and c1(dil=0) == 1 and c1(pad=-1) == 1
    assert c1(k=33) == 1                                                   # taps span more than the row
    assert c1(k=9, dil=4) == 1
    assert c1(w=nul) == 1 and c1(x=nul) == 1 and c1(y=nul) == 1
    c2 = lambda **kw: L.sws_conv2d(*[kw.get(n, v) for n, v in zip(
        ("x", "w", "y", "N", "Cin", "H", "W", "Cout", "kh", "kw", "sh", "sw", "ph", "pw", "s"),
        (one, one, one, 1, 4, 8, 8, 6, 3, 3, 1, 1, 1, 1, nul))])
    assert c2(N=0) == 0
    assert c2(kh=0) == 1 and c2(sw=0) == 1 and c2(ph=-1) == 1 and c2(Cin=0) == 1
    assert c2(kw=11) == 1
    assert c2(w=nul) == 1


def test_options_and_copy_checks(L):
    assert L.sws_set_option(b"slide_variant", 0) == 0
    assert L.sws_set_option(b"no_such_knob", 1) == 1
    assert L.sws_set_option(None, 1) == 1
    one, nul = ctypes.c_void_p(16), ctypes.c_void_p(0)
    assert L.sws_copy(one, one, 0, nul) == 0
    assert L.sws_copy(one, one, -1, nul) == 1
    assert L.sws_copy(nul, one, 8, nul) == 1


def test_binding_refuses_cpu_tensors():
    """The product path never computes on the CPU: host tensors are an error."""
    import torch
    from paper_2305_16513_amd import binding
    with pytest.raises(TypeError):
        binding.sws_slide1d(0, torch.zeros(8), 3)


def test_new_entry_points_argument_checks(L):
    """sws_slide1d_16, sws_pool2d_ex and the conv1d adjoints reject bad arguments before any launch."""
    one, nul = ctypes.c_void_p(16), ctypes.c_void_p(0)
    i64, i32, f32 = ctypes.c_int64, ctypes.c_int32, ctypes.c_float
    L.sws_slide1d_16.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, i64, i64, i32, f32, ctypes.c_void_p]
    assert L.sws_slide1d_16(0, 1, one, one, 0, 100, 3, 1.0, nul) == 0      # no rows
    assert L.sws_slide1d_16(0, 0, one, one, 1, 100, 3, 1.0, nul) == 1      # fp32 is not a 16-bit type
    assert L.sws_slide1d_16(0, 2, one, one, 1, 100, 101, 1.0, nul) == 1    # window longer than the row
    assert L.sws_slide1d_16(0, 2, nul, one, 1, 100, 3, 1.0, nul) == 1
    L.sws_pool2d_ex.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, i64, i64, i64, i64, i32, i32, i32, i32,
                                i32, i32, i32, i32, ctypes.c_int, f32, ctypes.c_void_p]
    pe = lambda **kw: L.sws_pool2d_ex(*[kw.get(n, v) for n, v in zip(
        ("op", "x", "y", "N", "C", "H", "W", "kh", "kw", "sh", "sw", "pt", "pl", "pb", "pr", "div", "scale", "s"),
        (0, one, one, 1, 3, 8, 8, 3, 3, 1, 1, 1, 0, 2, 1, 0, 1.0, nul))])
    assert pe(N=0) == 0
    assert pe(pt=3) == 1 and pe(pb=3) == 1 and pe(pl=3) == 1 and pe(pr=-1) == 1
    assert pe(div=2) == 1 and pe(op=4) == 1 and pe(y=nul) == 1 and pe(H=0) == 1
    for f in (L.sws_conv1d_grad_input, L.sws_conv1d_grad_weight):
        f.argtypes = [ctypes.c_void_p] * 3 + [i64, i64, i64, i64, i32, i32, i32, i32, i32, ctypes.c_void_p]
        g = lambda **kw: f(*[kw.get(n, v) for n, v in zip(
            ("a", "b", "c", "B", "Cin", "L", "Cout", "k", "stride", "pad", "dil", "groups", "s"),
            (one, one, one, 1, 4, 32, 6, 3, 1, 0, 1, 1, nul))])
        assert g(groups=3) == 1 and g(k=0) == 1 and g(k=40) == 1 and g(stride=0) == 1 and g(c=nul) == 1
    assert L.sws_conv1d_grad_input(one, one, one, 0, 4, 32, 6, 3, 1, 0, 1, 1, nul) == 0
    for f in (L.sws_conv2d_grad_input, L.sws_conv2d_grad_weight):
        f.argtypes = [ctypes.c_void_p] * 3 + [i64] * 5 + [i32] * 6 + [ctypes.c_void_p]
        g2 = lambda **kw: f(*[kw.get(n, v) for n, v in zip(
            ("a", "b", "c", "N", "Cin", "H", "W", "Cout", "kh", "kw", "sh", "sw", "ph", "pw", "s"),
            (one, one, one, 1, 4, 8, 8, 6, 3, 3, 1, 1, 1, 1, nul))])
        assert g2(kh=0) == 1 and g2(sw=0) == 1 and g2(kh=11) == 1 and g2(c=nul) == 1 and g2(Cin=0) == 1
    L.sws_maxpool2d_grad.argtypes = [ctypes.c_void_p] * 3 + [i64] * 4 + [i32] * 6 + [ctypes.c_void_p]
    mp = lambda **kw: L.sws_maxpool2d_grad(*[kw.get(n, v) for n, v in zip(
        ("x", "gy", "gx", "N", "C", "H", "W", "kh", "kw", "sh", "sw", "ph", "pw", "s"),
        (one, one, one, 1, 3, 8, 8, 3, 3, 1, 1, 1, 1, nul))])
    assert mp(N=0) == 0 and mp(ph=3) == 1 and mp(kw=0) == 1 and mp(gx=nul) == 1 and mp(kh=12) == 1
    L.sws_avgpool2d_grad.argtypes = [ctypes.c_void_p] * 2 + [i64] * 4 + [i32] * 6 + [ctypes.c_int, f32, ctypes.c_void_p]
    ap = lambda **kw: L.sws_avgpool2d_grad(*[kw.get(n, v) for n, v in zip(
        ("gy", "gx", "N", "C", "H", "W", "kh", "kw", "sh", "sw", "ph", "pw", "div", "scale", "s"),
        (one, one, 1, 3, 8, 8, 3, 3, 2, 2, 1, 1, 0, 1.0, nul))])
    assert ap(N=0) == 0 and ap(ph=3) == 1 and ap(sh=0) == 1 and ap(gx=nul) == 1 and ap(kh=12) == 1 and ap(div=2) == 1
    L.sws_pool2d_16.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, i64, i64, i64, i64,
                                i32, i32, i32, i32, i32, i32, f32, ctypes.c_void_p]
    assert L.sws_pool2d_16(0, 1, one, one, 0, 3, 8, 8, 3, 3, 1, 1, 1, 1, 1.0, nul) == 0
    assert L.sws_pool2d_16(0, 3, one, one, 1, 3, 8, 8, 3, 3, 1, 1, 1, 1, 1.0, nul) == 1
    assert L.sws_pool2d_16(0, 1, one, nul, 1, 3, 8, 8, 3, 3, 1, 1, 1, 1, 1.0, nul) == 1


def test_conv1d_16_argument_checks(L):
    one, nul = ctypes.c_void_p(16), ctypes.c_void_p(0)
    i64, i32 = ctypes.c_int64, ctypes.c_int32
    L.sws_conv1d_16.argtypes = [ctypes.c_int] + [ctypes.c_void_p] * 3 + [i64] * 4 + [i32] * 5 + [ctypes.c_void_p]
    c = lambda **kw: L.sws_conv1d_16(*[kw.get(n, v) for n, v in zip(
        ("dtype", "x", "w", "y", "B", "Cin", "L", "Cout", "k", "stride", "pad", "dil", "groups", "s"),
        (1, one, one, one, 1, 4, 32, 4, 3, 1, 0, 1, 4, nul))])
    assert c(B=0) == 0
    assert c(dtype=0) == 1 and c(dtype=3) == 1                             # fp32 / unknown storage type
    assert c(groups=3) == 1 and c(k=0) == 1 and c(k=33) == 1 and c(stride=0) == 1 and c(dil=0) == 1 and c(pad=-1) == 1
    assert c(x=nul) == 1 and c(w=nul) == 1 and c(y=nul) == 1
    assert c(L=2 ** 31) == 1


def test_headers_compile_as_plain_c(tmp_path):
    """The boundary is a C ABI: both headers must be valid C99 with no HIP include."""
    import shutil
    import subprocess
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no C compiler")
    src = tmp_path / "use.c"
    src.write_text('#include "sws.h"\n#include "sws_dev.h"\n'
                   'int f(sws_stream_t s) { return (int)sws_slide1d(SWS_OP_ADD, 0, 0, 0, 8, 3, 1.0f, s); }\n')
    subprocess.run([cc, "-std=c99", "-Wall", "-Werror", "-pedantic", "-fsyntax-only",
                    "-I", os.path.join(ROOT, "include"), str(src)], check=True)


def test_pool2d_padded_argument_checks(L):
    one, nul = ctypes.c_void_p(16), ctypes.c_void_p(0)
    i64, i32, f32 = ctypes.c_int64, ctypes.c_int32, ctypes.c_float
    L.sws_pool2d_padded.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, i64, i64, i64, i64, i32, i32, i32, i32,
                                    i32, i32, i32, i32, ctypes.c_int, f32, ctypes.c_void_p]
    pp = lambda **kw: L.sws_pool2d_padded(*[kw.get(n, v) for n, v in zip(
        ("op", "x", "y", "N", "C", "H", "W", "kh", "kw", "sh", "sw", "pt", "pl", "pb", "pr", "mode", "scale", "s"),
        (0, one, one, 1, 3, 8, 6, 3, 3, 1, 1, 1, 0, 2, 1, 1, 1.0, nul))])
    assert pp(N=0) == 0 and pp(C=0, mode=2) == 0
    assert pp(mode=5) == 1 and pp(mode=-1) == 1 and pp(op=3) == 1 and pp(H=0) == 1 and pp(pr=-1) == 1
    assert pp(pt=8) == 1 and pp(pb=8) == 1 and pp(pl=6) == 1 and pp(pr=6) == 1            # mirror: at most extent - 1
    assert pp(mode=2, pt=9) == 1 and pp(mode=2, pr=7) == 1                                # periodic: at most the extent
    assert pp(mode=4, pt=3) == 1 and pp(mode=4, pr=3) == 1                                # shrinking: below the window
    assert pp(kh=12) == 1 and pp(kw=8) == 1 and pp(sh=0) == 1 and pp(x=nul) == 1 and pp(y=nul) == 1


def test_conv1d_padded_argument_checks(L):
    one, nul = ctypes.c_void_p(16), ctypes.c_void_p(0)
    i64, i32 = ctypes.c_int64, ctypes.c_int32
    L.sws_conv1d_padded.argtypes = [ctypes.c_void_p] * 3 + [i64] * 4 + [i32] * 6 + [ctypes.c_int, ctypes.c_void_p]
    c = lambda **kw: L.sws_conv1d_padded(*[kw.get(n, v) for n, v in zip(
        ("x", "w", "y", "B", "Cin", "L", "Cout", "k", "stride", "pl", "pr", "dil", "groups", "mode", "s"),
        (one, one, one, 1, 4, 32, 4, 3, 1, 1, 1, 1, 4, 1, nul))])
    assert c(B=0) == 0
    assert c(mode=4) == 1 and c(mode=-1) == 1 and c(L=0) == 1 and c(pl=-1) == 1 and c(pr=-1) == 1
    assert c(pl=32) == 1 and c(pr=32) == 1 and c(mode=2, pl=33) == 1 and c(mode=2, pr=33) == 1
    assert c(groups=3) == 1 and c(k=0) == 1 and c(k=40) == 1 and c(stride=0) == 1 and c(dil=0) == 1 and c(y=nul) == 1


def test_conv2d_padded_argument_checks(L):
    one, nul = ctypes.c_void_p(16), ctypes.c_void_p(0)
    i64, i32 = ctypes.c_int64, ctypes.c_int32
    L.sws_conv2d_padded.argtypes = [ctypes.c_void_p] * 3 + [i64] * 5 + [i32] * 8 + [ctypes.c_int, ctypes.c_void_p]
    c = lambda **kw: L.sws_conv2d_padded(*[kw.get(n, v) for n, v in zip(
        ("x", "w", "y", "N", "Cin", "H", "W", "Cout", "kh", "kw", "sh", "sw", "pt", "pl", "pb", "pr", "mode", "s"),
        (one, one, one, 1, 4, 8, 6, 6, 3, 3, 1, 1, 1, 1, 1, 1, 1, nul))])
    assert c(N=0) == 0
    assert c(mode=4) == 1 and c(mode=-1) == 1 and c(H=0) == 1 and c(pt=-1) == 1 and c(Cin=0) == 1
    assert c(pt=8) == 1 and c(pr=6) == 1 and c(mode=2, pb=9) == 1 and c(mode=2, pl=7) == 1
    assert c(kh=11) == 1 and c(kw=9) == 1 and c(sh=0) == 1 and c(y=nul) == 1 and c(w=nul) == 1


def test_conv_workspace_and_argument_checks_of_the_ws_entries(L):
    one, nul = ctypes.c_void_p(16), ctypes.c_void_p(0)
    assert L.sws_conv_workspace(64, 64, 9, 1000) >= 6 * 64 * 64 * 9         # three bf16 pieces per weight
    assert L.sws_conv_workspace(64, 64, 65, 1000) == 0 and L.sws_conv_workspace(0, 64, 9, 1000) == 0
    assert L.sws_conv_workspace(2 ** 31, 2 ** 31, 9, 1000) == 0 and L.sws_conv_workspace(64, 64, 9, 0) == 0
    assert L.sws_conv_workspace(32, 64, 1, 1000) == 0                       # a contraction too short for it
    assert L.sws_conv2d_ws(one, one, one, 0, 3, 10, 10, 4, 3, 3, 1, 1, 1, 1, one, 64, nul) == 0     # no images: nothing to do
    assert L.sws_conv2d_ws(nul, one, one, 1, 3, 10, 10, 4, 3, 3, 1, 1, 1, 1, one, 64, nul) == 1
    assert L.sws_conv2d_grad_input_ws(one, one, one, 1, 3, 2, 2, 4, 5, 5, 1, 1, 1, 1, one, 64, nul) == 1
    assert L.sws_conv1d_ws(one, one, one, 1, 3, 10, 4, 11, 1, 0, 1, 1, one, 64, nul) == 1
    assert L.sws_conv1d_grad_input_ws(one, one, nul, 1, 3, 10, 4, 3, 1, 0, 1, 1, one, 64, nul) == 1


def test_grad_weight_workspace_goes_with_the_work(L):
    """Partial sums of as many runs as the layer has tiles for, and none where no kernel uses them."""
    conv2, conv1 = L.sws_conv2d_grad_weight_workspace, L.sws_conv1d_grad_weight_workspace
    gw = 4 * 64 * 64 * 9
    assert conv2(32, 64, 56, 56, 64, 3, 3, 1, 1, 1, 1) >= 64 * gw            # one block of gw, runs for the whole chip
    assert 0 < conv2(2, 64, 8, 8, 64, 3, 3, 1, 1, 1, 1) <= 8 * gw            # a few tiles (75 MB for any layer of these channels before)
    assert 0 < conv2(2, 8, 8, 8, 8, 3, 3, 1, 1, 1, 1) <= 8 * 4 * 32 * 32 * 9
    assert 0 < conv1(16, 64, 4096, 64, 3, 1, 0, 1, 1) <= 512 * 4 * 64 * 64 * 3
    assert conv2(32, 64, 56, 56, 64, 3, 3, 3, 3, 1, 1) == 0 and conv1(16, 64, 4096, 64, 3, 3, 0, 1, 1) == 0       # strides beyond 2
    assert conv2(32, 128, 56, 56, 128, 3, 3, 2, 2, 1, 1) == 0                # the kernel that reads its operands from memory
    assert conv1(16, 64, 4096, 64, 3, 1, 0, 1, 2) == 0 and conv1(16, 1, 4096, 64, 3, 1, 0, 1, 1) == 0
    assert conv2(1, 64, 30, 30, 64, 9, 9, 1, 1, 0, 0) == 0 and conv1(1, 64, 30, 64, 31, 1, 0, 1, 1) == 0          # 81 taps; invalid
    assert conv2(0, 64, 30, 30, 64, 3, 3, 1, 1, 0, 0) == 0


def test_grad_weight_plans_that_the_gpu_tests_count_on(L):
    """The layers of test_grad_weight_runs_and_images have as many blocks of partial sums as its comments say: as many runs, and tiles as large."""
    from tests.test_parity_conv_split import GW_RUNS
    for (n, cin, cout, h, w, kh, kw, s, p), blocks in GW_RUNS.items():
        ph, sh = (p, s) if h > 1 else (0, 1)
        taps = 5 if (kh, kw) == (5, 5) else kh * kw                          # (of a workgroup)
        assert L.sws_conv2d_grad_weight_workspace(n, cin, h, w, cout, kh, kw, sh, s, ph, p) == 4096 * taps * blocks, (n, cin, cout, h, w, kh, kw, s, p)


def test_grad_weight_runs_fill_whole_rounds_and_one_row_layers_go_to_the_faster_kernel(L):
    """A workgroup of the tiled kernel fills a compute unit: a few more workgroups than there are units would be a second round.  (Counted from
    the partial sums: 64 x 64 channels x 9 taps each.)"""
    for cin, cout in ((320, 192), (192, 320), (576, 192), (448, 448), (704, 192), (192, 192)):
        groups = L.sws_conv2d_grad_weight_workspace(32, cin, 56, 56, cout, 3, 3, 1, 1, 1, 1) / (4.0 * 64 * 64 * 9)
        assert 0 < groups <= 256 or 420 <= groups <= 512, (cin, cout, groups)
    conv1 = L.sws_conv1d_grad_weight_workspace
    assert conv1(32, 256, 3136, 256, 3, 1, 1, 1, 1) == 0 and conv1(16, 544, 6024, 128, 1, 1, 0, 1, 1) == 0
    assert conv1(16, 64, 4096, 64, 3, 1, 0, 1, 1) > 0 and conv1(64, 544, 1029, 32, 5, 1, 2, 1, 1) > 0
    assert conv1(32, 256, 3136, 250, 3, 1, 1, 1, 1) > 0                      # (channels that kernel does not take)


def test_no_memory_for_a_workspace_is_no_error(monkeypatch):
    import torch
    from paper_2305_16513_amd import binding as B

    class Full:
        def new_empty(self, n):
            raise torch.cuda.OutOfMemoryError("no %d floats" % n)

        def get_device(self):
            return 0

    monkeypatch.setattr(B, "_device", lambda: 0)
    assert B._scratch(1 << 20, Full(), None) == (None, None, 0)
    assert B._scratch(0, Full(), None) == (None, None, 0)


def test_a_tensor_of_another_device_gets_no_workspace(monkeypatch):
    """Memory of device 1 would be given back on device 1's stream while the call still runs on device 0's."""
    from paper_2305_16513_amd import binding as B

    class Elsewhere:
        def new_empty(self, n):
            raise AssertionError("allocated")

        def get_device(self):
            return 1

    monkeypatch.setattr(B, "_device", lambda: 0)
    assert B._scratch(1 << 20, Elsewhere(), None) == (None, None, 0)


def test_grad_weight_workspace_and_argument_checks(L):
    one, nul = ctypes.c_void_p(16), ctypes.c_void_p(0)
    assert L.sws_conv_grad_weight_workspace(64, 64, 3, 3) >= 4 * 64 * 64 * 9
    assert L.sws_conv_grad_weight_workspace(64, 64, 9, 9) == 0 and L.sws_conv_grad_weight_workspace(64, 0, 3, 3) == 0
    assert L.sws_conv2d_grad_weight_ws(one, one, nul, 1, 3, 10, 10, 4, 3, 3, 1, 1, 1, 1, one, 64, nul) == 1
    assert L.sws_conv1d_grad_weight_ws(nul, one, one, 1, 3, 10, 4, 3, 1, 0, 1, 1, one, 64, nul) == 1


def test_planning_of_a_launch_takes_microseconds(L):
    """Host time of an entry whose launcher looks for the best tiling, beside one that does not: without a GPU the launch itself
    is refused, so what is timed is the checks and the plan."""
    import time
    import torch
    if torch.cuda.is_available():
        pytest.skip("made-up pointers")
    one, nul = ctypes.c_void_p(4096), ctypes.c_void_p(0)

    def us(hw, k):
        best = 1e9
        for _ in range(9):
            t = time.perf_counter()
            for _ in range(60):
                assert L.sws_maxpool2d_grad(one, one, one, 1, 1, hw, hw, k, k, 1, 1, k // 2, k // 2, nul) != 0
            best = min(best, (time.perf_counter() - t) / 60 * 1e6)
        return best

    plain = us(112, 3)
    for hw, k in ((112, 7), (224, 13)):
        assert us(hw, k) < plain + 15, (hw, k, plain)       # 1 - 2 us; every pair of 64 x 64 cuts: 45 us
