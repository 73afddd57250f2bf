"""The weight gradient of 3 x 3 layers whose workgroups hold wavefronts that only stage (csrc/conv_gw_tile.hip), at the edges of its runs, groups
and tiles."""
import numpy as np
import pytest

import oracle
from paper_2305_16513_amd import workloads
from tests.parity_util import assert_bit_exact, assert_within_tol, kernels, to_gpu, to_host
from tests.test_parity_conv_split import SPLIT_TOL, B, _guarded, _taken, automatic, lent  # noqa: F401

# n, cin, cout, h, w, pad: runs of rows as the planner cuts them (of 32 x 32 channels: the blocks of partial sums beside them)
RUNS = {(3, 320, 128, 18, 60, 1): 12 * 40,            # two strips, runs of half an image
        (1, 192, 384, 31, 148, 0): 7 * 72,            # five strips, the last one of 26 columns; runs that begin inside a strip; no padding
        (16, 96, 384, 10, 42, 0): 13 * 36,            # four strips, tiles that hold parts of three images, groups of five images and a last one of one
        (4, 512, 64, 52, 64, 1): 16 * 32,             # a run is a strip of an image
        (7, 192, 128, 67, 34, 1): 21 * 24,            # a last strip of 10 columns
        (24, 256, 64, 55, 16, 0): 32 * 16,            # one strip, tiles that meet two images
        (16, 128, 256, 68, 6, 0): 16 * 32,            # rows of four positions, 24 of them per tile
        (16, 96, 160, 37, 38, 1): 17 * 15,            # one block of output channels, four wavefronts add up; four strips of groups of four images
        (24, 256, 32, 44, 30, 1): 32 * 8}             # the last strip six columns wide, groups of three images


# output channels in blocks of 32: four wavefronts add up
ONE_BLOCK = {(16, 96, 160, 37, 38, 1)}


def test_the_plans_are_those_that_the_runs_are_meant_for():
    from paper_2305_16513_amd import binding
    for (n, cin, cout, h, w, p), blocks in RUNS.items():
        assert binding.lib().sws_conv2d_grad_weight_workspace(n, cin, h, w, cout, 3, 3, 1, 1, p, p) == 4096 * 9 * blocks, (n, cin, cout, h, w, p)


def _one_float_on(a):
    """On the GPU, 4 bytes behind an address that allocations start at."""
    import torch
    flat = torch.empty(a.size + 1, device="cuda")
    t = flat[1:].view(a.shape)
    t.copy_(torch.from_numpy(a))
    assert t.data_ptr() % 16 == 4
    return t


@pytest.mark.gpu
@pytest.mark.parametrize("case", RUNS)
def test_staged_runs(B, case, lent):  # noqa: F811
    n, cin, cout, h, w, p = case
    for integer in (True, False):
        rng = np.random.default_rng(61)
        shape, gshape = (n, cin, h, w), (n, cout, h + 2 * p - 2, w + 2 * p - 2)
        x = workloads.integer_valued(shape, -3, 3, 62) if integer else rng.standard_normal(shape).astype(np.float32)
        gy = workloads.integer_valued(gshape, -3, 3, 63) if integer else rng.standard_normal(gshape).astype(np.float32)
        ref, mag = oracle.conv2d_grad_weight(x, gy, 3, 3, 1, 1, p, p)
        flat, gw = _guarded(ref.shape)
        # (the staging loads are of 16 and 8 bytes, which every tensor's alignment has to do for)
        put = to_gpu if integer else _one_float_on
        names = kernels(lambda: B.sws_conv2d_grad_weight(put(x), put(gy), 3, 3, 1, 1, p, p, gw=gw))
        assert "conv_gw_staged_kernel<%d>" % (2 if cout > 32 and case not in ONE_BLOCK else 1) in names, names
        if integer:
            assert_bit_exact(to_host(gw), ref, "gw %s" % (case,))
        else:
            # sums of up to 31680 products, by at most 1400 per run: the bound of test_parity_conv_split.py
            assert_within_tol(to_host(gw), ref, mag, "gw %s" % (case,), tol=SPLIT_TOL)
        assert _taken(lent[-1])
        assert (flat[:64] == 12345.0).all() and (flat[-64:] == 12345.0).all()
