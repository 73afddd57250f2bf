"""The split-operand convolution kernel for any dense layer (conv_split.hip): every tile configuration at the edges of
its tiles, against the C oracle.

Tolerance: an output is a sum of n products (Cin*kh*kw, adjoint Cout*kh*kw, at most 1170 here), each evaluated as six exact piece
products (what is dropped is below 2^-22 of it), accumulated with two roundings of the running sum per 16 products and a few at the
end.  Each is at most 2^-24 of sum|terms| and their signs differ, so twice the root of their number counts:
|err| <= (2^-22 + 2 sqrt(n/8 + 8) 2^-24) * sum|terms|, 0.6e-6 of it for n = 9 and 1.8e-6 for 1170; 2e-6 is used throughout.
"""
import numpy as np
import pytest

import oracle
from paper_2305_16513_amd import workloads
from tests.parity_util import assert_bit_exact, assert_within_tol, to_gpu, to_host

pytestmark = pytest.mark.gpu
SPLIT_TOL = 2e-6
FORWARD, PHASES = range(10), range(10, 14)


@pytest.fixture(scope="module")
def B():
    from paper_2305_16513_amd import binding
    return binding


@pytest.fixture(autouse=True)
def automatic(B):
    yield
    B.sws_set_option("conv2d_variant", 0)


@pytest.fixture
def lent(B, monkeypatch):
    """Every workspace that a test lends, filled with a value that no kernel leaves throughout: taken(t) tells whether one was used."""
    given, scratch = [], B._scratch

    def fill(n, like, stream):
        t, at, size = scratch(n, like, stream)
        if t is not None:
            t.fill_(12345.0)
            given.append(t)
        return t, at, size

    monkeypatch.setattr(B, "_scratch", fill)
    return given


def _taken(t):
    return bool((t != 12345.0).any())


def _guarded(shape):
    """A contiguous tensor between two bands of a value that no output takes."""
    import torch
    n = int(np.prod(shape))
    flat = torch.full((n + 128,), 12345.0, device="cuda")
    return flat, flat[64:64 + n].view(shape)


def _check(B, case, seed, integer, forward=True, adjoint=True):
    n, cin, cout, h, w, kh, kw, s, p = case
    ph, pw = (p if h > 1 else 0), p
    if integer:                                       # sums below 2^24: exact in any order
        x = workloads.integer_valued((n, cin, h, w), -3, 3, seed)
        wgt = workloads.integer_valued((cout, cin, kh, kw), -3, 3, seed + 1)
    else:
        rng = np.random.default_rng(seed)
        x = rng.standard_normal((n, cin, h, w)).astype(np.float32)
        wgt = rng.standard_normal((cout, cin, kh, kw)).astype(np.float32)
    sh = s if h > 1 else 1
    ref, mag = oracle.conv2d(x, wgt, sh, s, ph, pw)
    if forward:
        flat, y = _guarded(ref.shape)
        B.sws_conv2d(to_gpu(x), to_gpu(wgt), sh, s, ph, pw, y=y)
        if integer:
            assert_bit_exact(to_host(y), ref, "y %s" % (case,))
        else:
            assert_within_tol(to_host(y), ref, mag, "y %s" % (case,), tol=SPLIT_TOL)
        assert (flat[:64] == 12345.0).all() and (flat[-64:] == 12345.0).all()
    if adjoint:
        gy = workloads.integer_valued(ref.shape, -3, 3, seed + 2) if integer else \
            np.random.default_rng(seed + 2).standard_normal(ref.shape).astype(np.float32)
        gref, gmag = oracle.conv2d_grad_input(gy, wgt, h, w, sh, s, ph, pw)
        flat, gx = _guarded(gref.shape)
        B.sws_conv2d_grad_input(to_gpu(gy), to_gpu(wgt), h, w, sh, s, ph, pw, gx=gx)
        if integer:
            assert_bit_exact(to_host(gx), gref, "gx %s" % (case,))
        else:
            assert_within_tol(to_host(gx), gref, gmag, "gx %s" % (case,), tol=SPLIT_TOL)
        assert (flat[:64] == 12345.0).all() and (flat[-64:] == 12345.0).all()


# n, cin, cout, h, w, kh, kw, stride, pad: channels below, at and beyond blocks of 8, 16, 32 and 64; planes smaller than a
# tile, tiles across images, rows longer than a tile, strips; every residue of the strides
CASES = [
    (1, 1, 1, 1, 1, 1, 1, 1, 0),
    (2, 7, 33, 5, 6, 3, 3, 1, 1),
    (3, 24, 65, 7, 7, 3, 3, 1, 1),
    (5, 19, 31, 4, 3, 3, 3, 1, 0),
    (2, 40, 129, 14, 13, 3, 3, 1, 1),
    (1, 16, 32, 3, 300, 3, 3, 1, 1),
    (2, 33, 20, 1, 257, 1, 3, 1, 1),
    (1, 50, 64, 1, 1030, 1, 5, 1, 0),
    (2, 130, 40, 9, 11, 1, 1, 1, 0),
    (3, 17, 34, 8, 9, 5, 5, 1, 2),
    (2, 20, 48, 15, 18, 3, 3, 2, 1),
    (4, 9, 32, 7, 8, 3, 3, 2, 1),
    (3, 40, 24, 6, 5, 1, 1, 2, 0),
    (2, 12, 36, 11, 12, 2, 2, 2, 0),
    (2, 5, 40, 12, 9, 5, 5, 2, 2),
    (1, 6, 10, 9, 9, 7, 7, 2, 3),
    (2, 30, 18, 1, 77, 1, 3, 2, 1),
]


@pytest.mark.parametrize("case", CASES)
def test_chosen_configuration(B, case):
    for integer in (True, False):
        _check(B, case, 11, integer)


@pytest.mark.parametrize("cfg", FORWARD)
def test_every_forward_configuration(B, cfg, lent):
    """(A configuration whose tile does not fit a shape leaves it to the kernels without a workspace.)"""
    B.sws_set_option("conv2d_variant", 100 + cfg)
    for i, case in enumerate(CASES):
        _check(B, case, 20 + i, i % 2 == 0, adjoint=case[7] == 1)
    taken = [_taken(t) for t in lent]
    assert sum(taken) >= 19, taken                    # of 27 calls (the smallest tiles do not hold the widest lines)


@pytest.mark.parametrize("cfg", PHASES)
def test_every_phase_configuration(B, cfg, lent):
    B.sws_set_option("conv2d_variant", 100 + cfg)
    for i, case in enumerate(CASES):
        if case[7] == 2:
            _check(B, case, 50 + i, i % 2 == 0, forward=False)
    taken = [_taken(t) for t in lent]
    assert sum(taken) >= 6, taken                     # of 7 calls


def test_many_chunks_and_large_tiles(B, lent):
    """Several chunks of input channels through both staging buffers, tiles of every configuration filled."""
    for cfg in FORWARD:
        B.sws_set_option("conv2d_variant", 100 + cfg)
        _check(B, (2, 150, 130, 17, 19, 3, 3, 1, 1), 70, True)
    taken = [_taken(t) for t in lent]
    assert len(taken) == 2 * len(FORWARD) and all(taken[:16]), taken  # (likewise 8 and 9)
    B.sws_set_option("conv2d_variant", 0)
    _check(B, (2, 100, 70, 21, 18, 3, 3, 2, 1), 71, True)


def test_information_in_the_third_piece(B):
    """Values 1 + i 2^-23: their low bits live in the third bf16 piece; differences of neighbouring channels show them."""
    rng = np.random.default_rng(3)
    x = (1.0 + rng.integers(0, 1 << 23, (1, 32, 6, 40)) * 2.0 ** -23).astype(np.float32)
    wgt = np.zeros((32, 32, 3, 3), np.float32)
    for co in range(32):
        wgt[co, co, 1, 1], wgt[co, (co + 1) % 32, 1, 1] = 1.0, -1.0
    ref, _ = oracle.conv2d(x, wgt, 1, 1, 1, 1)
    y = to_host(B.sws_conv2d(to_gpu(x), to_gpu(wgt), 1, 1, 1, 1)).astype(np.float64)
    assert np.abs(y - ref).max() <= 2.0 ** -23


def test_weights_at_the_end_of_the_range(B):
    """Weights up to the largest finite number (their leading piece must not round to infinity) against small inputs."""
    # (both the kernel for any layer and, with 64 channels and enough positions, the one that keeps its weights in registers)
    big = np.array([3.4028235e38, -3.4028235e38, 3.3961775e38, 3.39e38, -1.0, 2.0 ** 127, float.fromhex("0x1.ff0001p127"), float.fromhex("-0x1.feffffp127")], np.float32)
    rng = np.random.default_rng(4)
    for c, (n, h, w) in ((32, (2, 9, 11)), (64, (2, 56, 56))):
        wgt = np.zeros((c, c, 3, 3), np.float32)
        for co in range(c):
            wgt[co, co, co % 3, 1] = big[co % 8]
        x = (rng.standard_normal((n, c, h, w)) * 2.0 ** -110).astype(np.float32)
        for var in (0, 18 if c == 64 else 0):         # (18: the streaming kernel on a small problem)
            B.sws_set_option("conv2d_variant", var)
            for ref, got in ((oracle.conv2d(x, wgt, 1, 1, 1, 1)[0], B.sws_conv2d(to_gpu(x), to_gpu(wgt), 1, 1, 1, 1)),
                             (oracle.conv2d_grad_input(x, wgt, h, w, 1, 1, 1, 1)[0], B.sws_conv2d_grad_input(to_gpu(x), to_gpu(wgt), h, w, 1, 1, 1, 1))):
                assert np.abs(to_host(got).astype(np.float64) - ref).max() <= 2.0 ** -21 * np.abs(ref).max(), (c, var)


def test_what_the_dropped_products_may_reach(B):
    """One product per output: three of the nine piece products are dropped, below 2^-21 of it where both operands are cut and 2^-22
    where the weights are rounded to nearest, and the rest takes a rounding or two.  Mantissas whose second and third pieces are
    as large as they can be, and random ones."""
    rng = np.random.default_rng(6)
    v = np.concatenate([[1 + 2.0 ** -7 - 2.0 ** -23, 1 + 2.0 ** -8 - 2.0 ** -23, 2 - 2.0 ** -23, 1 + 2.0 ** -7 - 2.0 ** -15 - 2.0 ** -23],
                        1.0 + rng.integers(0, 1 << 23, 4092) * 2.0 ** -23]).astype(np.float32)
    exact = v.astype(np.float64)
    # gw[co][0] = gy[co] * x for one position (kernel 100: the tiled one also for so few)
    B.sws_set_option("conv2d_variant", 100)
    for first in v[:4]:
        x = np.full((1, 2, 1, 1), first, np.float32)
        gw = to_host(B.sws_conv2d_grad_weight(to_gpu(x), to_gpu(v[:2048].reshape(1, 2048, 1, 1)), 1, 1)).astype(np.float64)[:, 0, 0, 0]
        off = np.abs(gw / (exact[:2048] * np.float64(first)) - 1)
        assert off.max() <= 2.0 ** -21 + 2.0 ** -23, off.max() * 2.0 ** 23
    B.sws_set_option("conv2d_variant", 0)
    # y[co] = wgt[co][c] * x[c], one non-zero input channel of 64, 3 x 3 so that the split-operand kernel takes it
    for first in v[:4]:
        x = np.zeros((1, 64, 1, 40), np.float32)
        x[0, 5] = first
        wgt = np.zeros((2048, 64, 1, 3), np.float32)
        wgt[:, 5, 0, 1] = v[:2048]
        y = to_host(B.sws_conv2d(to_gpu(x), to_gpu(wgt), 1, 1, 0, 1)).astype(np.float64)[0, :, 0, 7]
        off = np.abs(y / (exact[:2048] * np.float64(first)) - 1)
        assert off.max() <= 2.0 ** -22 + 2.0 ** -23, off.max() * 2.0 ** 23


def test_without_workspace_and_with_one_too_small(B):
    """The C entries take a NULL or a small workspace: the same result by the kernels that need none."""
    import ctypes
    import torch
    x = workloads.integer_valued((2, 24, 9, 10), -3, 3, 5)
    wgt = workloads.integer_valued((40, 24, 3, 3), -3, 3, 6)
    ref, _ = oracle.conv2d(x, wgt, 1, 1, 1, 1)
    xd, wd = to_gpu(x), to_gpu(wgt)
    small = torch.empty(4096, dtype=torch.uint8, device="cuda")
    for ws, size in ((None, 0), (small.data_ptr(), small.numel())):
        y = torch.full(ref.shape, 7.0, device="cuda")
        rc = B.lib().sws_conv2d_ws(xd.data_ptr(), wd.data_ptr(), y.data_ptr(), 2, 24, 9, 10, 40, 3, 3, 1, 1, 1, 1, ws, size,
                                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0
        assert_bit_exact(to_host(y), ref, "workspace of %d bytes" % size)


@pytest.mark.parametrize("cin,cout,k,stride", [(60, 32, 3, 1), (60, 32, 3, 2), (20, 24, 9, 1), (64, 64, 3, 1), (32, 64, 5, 1), (9, 70, 31, 1), (18, 33, 7, 3)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_a_workspace_too_small_gives_the_bits_of_none(B, cin, cout, k, stride, adjoint):
    """1-D layers, where another kernel is preferred when there is no workspace: lending too little or at a crooked address takes that one too."""
    import ctypes
    import torch
    gen = torch.Generator(device="cuda").manual_seed(cin + k)
    b, length = 3, 700
    lo = (length - k) // stride + 1
    x = torch.randn(b, cout if adjoint else cin, lo if adjoint else length, generator=gen, device="cuda")
    wgt = torch.randn(cout, cin, k, generator=gen, device="cuda")
    lent = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    entry = B.lib().sws_conv1d_grad_input_ws if adjoint else B.lib().sws_conv1d_ws
    got = []
    for at, size in ((None, 0), (lent.data_ptr(), 64), (lent.data_ptr() + 4, lent.numel() - 4)):
        y = torch.full((b, cin if adjoint else cout, length if adjoint else lo), 7.0, device="cuda")
        rc = entry(x.data_ptr(), wgt.data_ptr(), y.data_ptr(), b, cin, length, cout, k, stride, 0, 1, 1, at, size,
                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0
        got.append(to_host(y))
    assert_bit_exact(got[1], got[0], "64 bytes")
    assert_bit_exact(got[2], got[0], "not on a 16-byte boundary")


def test_any_object_with_a_stream_handle(B):
    """`stream` may be a torch Stream or anything with its handle, the default stream's too; the workspace is the stream's."""
    import types
    import torch
    x = to_gpu(workloads.integer_valued((4, 40, 13, 11), -3, 3, 8))
    wgt = to_gpu(workloads.integer_valued((48, 40, 3, 3), -3, 3, 9))
    g = to_gpu(workloads.integer_valued((4, 48, 13, 11), -3, 3, 10))

    def all_three(**kw):
        return (B.sws_conv2d(x, wgt, 1, 1, 1, 1, **kw), B.sws_conv2d_grad_input(g, wgt, 13, 11, 1, 1, 1, 1, **kw),
                B.sws_conv2d_grad_weight(x, g, 3, 3, 1, 1, 1, 1, **kw))

    want = all_three()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for stream in (side, types.SimpleNamespace(cuda_stream=side.cuda_stream), types.SimpleNamespace(cuda_stream=0), torch.cuda.default_stream()):
        got = all_three(stream=stream)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b)


def test_graph_replay(B):
    """Captured in a HIP graph (the workspace comes from the graph's pool) and replayed with eager work between."""
    import torch
    x = to_gpu(workloads.integer_valued((3, 40, 13, 11), -3, 3, 8))
    wgt = to_gpu(workloads.integer_valued((48, 40, 3, 3), -3, 3, 9))
    g = to_gpu(workloads.integer_valued((3, 48, 7, 6), -3, 3, 10))
    y, gx = torch.empty(3, 48, 7, 6, device="cuda"), torch.empty_like(x)

    def both():
        B.sws_conv2d(x, wgt, 2, 2, 1, 1, y=y)
        B.sws_conv2d_grad_input(g, wgt, 13, 11, 2, 2, 1, 1, gx=gx)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        both()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        both()
    for rep in range(4):
        wgt.copy_(to_gpu(workloads.integer_valued((48, 40, 3, 3), -3, 3, 30 + rep)))
        y.fill_(7.0)
        gx.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = y.clone(), gx.clone()
        both()
        torch.cuda.synchronize()
        assert torch.equal(got[0], y) and torch.equal(got[1], gx), "replay %d" % rep
        ref, _ = oracle.conv2d(to_host(x), to_host(wgt), 2, 2, 1, 1)
        assert_bit_exact(to_host(y), ref, "replay %d" % rep)


# (pad below the kernel; strides beyond 2 and more than 64 taps are other kernels' cases)
GW_CASES = CASES + [
    (2, 70, 33, 10, 9, 3, 3, 1, 1),                   # blocks of 64 and 32 channels, both ends ragged
    (1, 20, 70, 1, 700, 1, 11, 1, 5),                 # two runs of taps of one row
    (20, 33, 9, 7, 7, 3, 3, 1, 1),                    # tiles across images
    (2, 3, 5, 130, 140, 3, 3, 1, 1),                  # strips, fewer than eight channels
    (1, 40, 40, 2, 600, 2, 3, 2, 0),
    (2, 12, 34, 1, 300, 1, 2, 1, 0),                  # every number of taps that a workgroup takes at once: 2, 4, 6, 7, 8 ...
    (1, 20, 40, 9, 70, 2, 2, 1, 0),
    (2, 33, 10, 8, 40, 2, 3, 1, 1),
    (1, 10, 66, 1, 500, 1, 7, 1, 3),
    (2, 20, 40, 9, 37, 4, 4, 1, 1),
    (1, 18, 40, 20, 21, 8, 8, 1, 3),                  # ... and the most taps
]


@pytest.mark.parametrize("integer", [True, False])
@pytest.mark.parametrize("case", GW_CASES)
def test_grad_weight_through_transposing_reads(B, case, integer, lent):
    n, cin, cout, h, w, kh, kw, s, p = case
    ph, sh = (p, s) if h > 1 else (0, 1)
    rng = np.random.default_rng(41)
    x = workloads.integer_valued((n, cin, h, w), -3, 3, 42) if integer else rng.standard_normal((n, cin, h, w)).astype(np.float32)
    ho, wo = (h + 2 * ph - kh) // sh + 1, (w + 2 * p - kw) // s + 1
    gy = workloads.integer_valued((n, cout, ho, wo), -3, 3, 43) if integer else \
        rng.standard_normal((n, cout, ho, wo)).astype(np.float32)
    ref, mag = oracle.conv2d_grad_weight(x, gy, kh, kw, sh, s, ph, p)
    flat, gw = _guarded(ref.shape)
    B.sws_set_option("conv2d_variant", 100)           # (also where another kernel is preferred)
    B.sws_conv2d_grad_weight(to_gpu(x), to_gpu(gy), kh, kw, sh, s, ph, p, gw=gw)
    if integer:
        assert_bit_exact(to_host(gw), ref, "gw %s" % (case,))
    else:
        # sums of up to n*ho*wo = 36400 products, by a few hundred positions per run: the bound above, 2^-21 dropped
        assert_within_tol(to_host(gw), ref, mag, "gw %s" % (case,), tol=SPLIT_TOL)
    assert len(lent) == 1 and _taken(lent[0])
    assert (flat[:64] == 12345.0).all() and (flat[-64:] == 12345.0).all()


# n, cin, cout, h, w, kh, kw, stride, pad: blocks of partial sums (32 x 32 channels x the taps of a workgroup x runs; test_abi_cpu.py holds the planner
# to them).  Tiles that never meet two images (rows per tile divide a plane's), that just do and that always do; 3 x 3 at stride 2
# with tiles of five units a thread (the four behind the comment: 185 tiles of 5 x 25 positions hold 11 x 52 inputs, more than the 512 of four units;
# 188 of 11 x 11, 11 and 10 of 24 x 4), both widths of a block and both ways to multiply; few runs added in one pass (at most 8, 1 to 9 taps), 9 and many
GW_RUNS = {(4, 32, 64, 56, 54, 3, 3, 2, 1): 138, (3, 33, 32, 16, 16, 3, 3, 2, 1): 24, (2, 40, 32, 112, 42, 3, 3, 2, 1): 224, (2, 60, 30, 56, 56, 3, 3, 2, 1): 168,
           (5, 32, 32, 12, 28, 3, 3, 1, 1): 28, (7, 40, 30, 6, 60, 3, 3, 1, 1): 84, (3, 33, 64, 4, 30, 3, 3, 1, 1): 24, (1, 16, 24, 9, 9, 3, 3, 1, 1): 1,
           (40, 64, 32, 28, 28, 3, 3, 1, 1): 500, (12, 256, 256, 14, 14, 3, 3, 1, 1): 13 * 64, (9, 40, 72, 20, 20, 5, 5, 1, 2): 15 * 30,
           (24, 32, 40, 1, 1000, 1, 3, 1, 1): 216 * 2,
           # five units a thread
           (37, 10, 8, 50, 50, 3, 3, 2, 1): 185, (47, 10, 37, 43, 43, 3, 3, 2, 1): 188 * 2, (62, 224, 96, 7, 7, 3, 3, 2, 1): 11 * 21,
           (55, 320, 96, 7, 7, 3, 3, 2, 1): 10 * 40,
           # few runs, and one more than that
           (2, 20, 24, 10, 13, 3, 3, 1, 1): 5, (4, 20, 24, 9, 20, 3, 3, 1, 0): 8, (3, 20, 24, 9, 20, 3, 3, 1, 1): 9, (4, 256, 250, 14, 14, 3, 3, 1, 1): 7 * 64,
           (12, 300, 290, 9, 9, 3, 3, 1, 1): 8 * 100,
           (5, 20, 24, 10, 13, 1, 1, 1, 0): 8, (3, 20, 24, 12, 30, 1, 1, 1, 0): 9, (5, 9, 32, 9, 20, 1, 2, 1, 0): 8, (2, 20, 24, 30, 14, 1, 3, 1, 0): 8,
           (2, 20, 24, 17, 23, 2, 2, 1, 0): 8, (5, 9, 32, 9, 20, 1, 5, 1, 0): 8, (2, 20, 24, 17, 23, 2, 3, 1, 0): 8, (2, 20, 24, 12, 30, 1, 7, 1, 0): 8,
           (2, 9, 32, 17, 23, 2, 4, 1, 0): 8}


@pytest.mark.parametrize("integer", [True, False])
@pytest.mark.parametrize("case", GW_RUNS)
def test_grad_weight_runs_and_images(B, case, integer, lent):
    """By the library's own choice of kernel: a workspace is lent and used."""
    n, cin, cout, h, w, kh, kw, s, p = case
    ph, sh = (p, s) if h > 1 else (0, 1)
    rng = np.random.default_rng(51)
    x = workloads.integer_valued((n, cin, h, w), -3, 3, 52) if integer else rng.standard_normal((n, cin, h, w)).astype(np.float32)
    ho, wo = (h + 2 * ph - kh) // sh + 1, (w + 2 * p - kw) // s + 1
    gy = workloads.integer_valued((n, cout, ho, wo), -3, 3, 53) if integer else rng.standard_normal((n, cout, ho, wo)).astype(np.float32)
    ref, mag = oracle.conv2d_grad_weight(x, gy, kh, kw, sh, s, ph, p)
    flat, gw = _guarded(ref.shape)
    B.sws_conv2d_grad_weight(to_gpu(x), to_gpu(gy), kh, kw, sh, s, ph, p, gw=gw)
    if integer:
        assert_bit_exact(to_host(gw), ref, "gw %s" % (case,))
    else:
        assert_within_tol(to_host(gw), ref, mag, "gw %s" % (case,), tol=SPLIT_TOL)      # (at most 31360 products: the bound of the test above)
    assert len(lent) == 1 and _taken(lent[0])
    assert (flat[:64] == 12345.0).all() and (flat[-64:] == 12345.0).all()


def test_grad_weight_is_reproducible(B):
    """Partial sums are added in a fixed order: two calls give the same bits."""
    rng = np.random.default_rng(7)
    x, gy = (to_gpu(rng.standard_normal(s).astype(np.float32)) for s in ((8, 40, 30, 30), (8, 48, 30, 30)))
    a = to_host(B.sws_conv2d_grad_weight(x, gy, 3, 3, 1, 1, 1, 1))
    for _ in range(3):
        assert_bit_exact(to_host(B.sws_conv2d_grad_weight(x, gy, 3, 3, 1, 1, 1, 1)), a)


def _gw_exact(x, gy, kh, kw, s, ph, pw):
    """The gradient in 64 bits: per tap one product of matrices."""
    import torch
    import torch.nn.functional as F
    x, gy = x.double(), gy.double()
    cin, (cout, ho, wo) = x.shape[1], gy.shape[1:]
    xe = F.pad(x, (pw, pw, ph, ph)).transpose(0, 1).contiguous()
    g2 = gy.transpose(0, 1).reshape(cout, -1).contiguous()
    gw = torch.empty(cout, cin, kh, kw, dtype=torch.float64, device=x.device)
    for a in range(kh):
        for b in range(kw):
            xt = xe[:, :, a:a + s * (ho - 1) + 1:s, b:b + s * (wo - 1) + 1:s].reshape(cin, -1)
            gw[:, :, a, b] = g2 @ xt.t().contiguous()
    return gw


# n, cin, cout, h, w, kh, kw, stride, pad; channels that no multiple of 32 rounds, or taps other than 3 x 3: without a workspace these
# run on fp32 instructions; the last two by so many blocks of gw that runs are cut for the length of their sums alone
EXACT = [(8, 96, 72, 40, 40, 5, 5, 1, 2), (8, 61, 50, 28, 28, 3, 3, 1, 1), (4, 40, 90, 33, 33, 3, 3, 2, 1), (4, 60, 60, 30, 30, 7, 7, 1, 3),
         (8, 48, 100, 40, 40, 4, 4, 1, 1), (16, 24, 40, 1, 5574, 1, 1, 1, 0), (8, 40, 70, 1, 2156, 1, 3, 1, 0), (2, 60, 100, 1, 3136, 1, 11, 1, 5),
         (8, 260, 260, 28, 28, 3, 3, 1, 1), (4, 200, 260, 28, 28, 5, 5, 1, 2)]


@pytest.mark.parametrize("case", EXACT)
def test_grad_weight_is_as_exact_as_the_fp32_kernels(B, monkeypatch, case):
    """Error against 64 bits (2-norm) with the workspace and without: at most a tenth more, the spread between two inputs."""
    import torch
    n, cin, cout, h, w, kh, kw, s, p = case
    ph = p if h > 1 else 0
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(n, cin, h, w, generator=gen, device="cuda")
    sh = s if h > 1 else 1
    gy = torch.randn(n, cout, (h + 2 * ph - kh) // sh + 1, (w + 2 * p - kw) // s + 1, generator=gen, device="cuda")
    ref = _gw_exact(x, gy, kh, kw, s, ph, p)

    def error():
        return ((B.sws_conv2d_grad_weight(x, gy, kh, kw, sh, s, ph, p).double() - ref).norm() / ref.norm()).item()

    tiled = error()
    monkeypatch.setattr(B, "_scratch", lambda *a: (None, None, 0))
    plain = error()
    assert tiled <= 1.1 * plain, (tiled, plain)


# 3 x 3, stride 2, padded by one: a chunk's phases as straight-line code; one and several chunks, odd planes (a last row or column of one
# phase only), ragged channels
@pytest.mark.parametrize("integer", [True, False])
@pytest.mark.parametrize("cfg", (0,) + tuple(PHASES))
def test_phases_of_the_usual_strided_layer(B, cfg, integer, lent):
    B.sws_set_option("conv2d_variant", 100 + cfg if cfg else 0)
    for i, (n, cin, cout, h, w) in enumerate([(2, 40, 70, 15, 22), (3, 16, 16, 8, 8), (1, 33, 130, 31, 17), (5, 64, 48, 2, 3), (1, 20, 9, 2, 40)]):
        _check(B, (n, cin, cout, h, w, 3, 3, 2, 1), 80 + i, integer, forward=False)
    taken = [_taken(t) for t in lent]
    assert len(taken) == 5 and sum(taken) >= 4, taken
