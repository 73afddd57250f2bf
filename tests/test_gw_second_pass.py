"""The second pass of the tiled weight gradient (csrc/conv_gw_tile.hip, gw_reduce_kernel) at the edges of its batches of runs, with sixteen runs in
flight a wavefront and with four."""
import numpy as np
import pytest

import oracle
from paper_2305_16513_amd import workloads
from tests.parity_util import assert_bit_exact, assert_within_tol, to_gpu, to_host
from tests.test_parity_conv_split import SPLIT_TOL, B, _guarded, _taken, automatic, lent  # noqa: F401

# n, cin, cout, h, w, k, stride, pad: workgroups, runs.  A wavefront adds every fourth run.
DEEP = {(32, 32, 17, 9, 9, 1, 2, 0): (16, 9), (1, 16, 32, 35, 35, 1, 1, 0): (16, 10), (1, 24, 16, 1, 1255, 1, 1, 0): (16, 11), (8, 16, 24, 1, 402, 1, 1, 0): (16, 28),
        (32, 16, 32, 30, 30, 1, 2, 0): (16, 60), (1, 19, 32, 1, 7356, 3, 1, 1): (48, 61), (32, 16, 24, 11, 11, 3, 2, 1): (144, 64), (16, 16, 22, 1, 885, 1, 1, 0): (16, 128),
        (64, 32, 16, 44, 44, 1, 2, 0): (16, 256)}
FLAT = {(32, 44, 128, 9, 9, 5, 2, 2): (3200, 9), (8, 272, 40, 9, 9, 3, 2, 1): (2592, 10), (1, 48, 72, 25, 25, 5, 1, 2): (2400, 13), (1, 30, 416, 19, 45, 3, 2, 1): (1872, 15),
        (8, 196, 43, 11, 13, 3, 2, 1): (2016, 16), (32, 40, 64, 12, 8, 3, 2, 1): (576, 48), (32, 56, 43, 17, 17, 3, 2, 1): (576, 58)}


def _layer(case):
    n, cin, cout, h, w, k, s, p = case
    return (n, cin, h, w, cout, k, k, s, s, p, p) if h > 1 else (n, cin, h, w, cout, 1, k, 1, s, 0, p)


def test_the_plans_have_these_runs(B):  # noqa: F811
    """(256 bytes of partial sums a workgroup and run; the line between the two is at 512 workgroups or 24576 of those.)"""
    B.sws_set_option("conv2d_variant", 100)           # (also where another kernel is preferred)
    for cases, deep in ((DEEP, True), (FLAT, False)):
        for case, (wgs, runs) in cases.items():
            assert B.lib().sws_conv2d_grad_weight_workspace(*_layer(case)) == 256 * wgs * runs, case
            assert (wgs <= 512 or wgs * runs <= 24576) == deep, case


@pytest.mark.gpu
@pytest.mark.parametrize("case", [*DEEP, *FLAT])
def test_second_pass(B, case, lent):  # noqa: F811
    n, cin, h, w, cout, kh, kw, sh, sw, ph, pw = _layer(case)
    shape, gshape = (n, cin, h, w), (n, cout, (h + 2 * ph - kh) // sh + 1, (w + 2 * pw - kw) // sw + 1)
    B.sws_set_option("conv2d_variant", 100)           # (also where another kernel is preferred)
    for integer in (True, False):
        rng = np.random.default_rng(71)
        x = workloads.integer_valued(shape, -3, 3, 72) if integer else rng.standard_normal(shape).astype(np.float32)
        gy = workloads.integer_valued(gshape, -3, 3, 73) if integer else rng.standard_normal(gshape).astype(np.float32)
        ref, mag = oracle.conv2d_grad_weight(x, gy, kh, kw, sh, sw, ph, pw)
        flat, gw = _guarded(ref.shape)
        B.sws_conv2d_grad_weight(to_gpu(x), to_gpu(gy), kh, kw, sh, sw, ph, pw, gw=gw)
        if integer:
            assert_bit_exact(to_host(gw), ref, "gw %s" % (case,))
        else:
            # sums of up to 30976 products: the bound of test_parity_conv_split.py
            assert_within_tol(to_host(gw), ref, mag, "gw %s" % (case,), tol=SPLIT_TOL)
        assert len(lent) and _taken(lent[-1])
        assert (flat[:64] == 12345.0).all() and (flat[-64:] == 12345.0).all()
