"""Configurations of the split-operand convolution whose workgroups hold wavefronts that only stage (csrc/conv_split.hip)."""
import pytest

from tests.test_parity_conv_split import B, CASES, _check, _taken, automatic, lent  # noqa: F401

# 64 x 128 with a split contraction, and the three largest tiles
STAGED = (3, 14, 15, 16)
# one chunk, two and many; chunks of 6, 8, 9 and 12 steps and of numbers that stay in the loop; rows and images that end inside a tile; channels of
# no whole octet; more units than the multiplying wavefronts stage of the first chunk
SHAPES = [(1, 16, 128, 9, 30, 3, 3, 1, 1), (2, 32, 64, 20, 20, 3, 3, 1, 1), (2, 150, 130, 17, 19, 3, 3, 1, 1), (3, 40, 129, 40, 40, 3, 3, 2, 1),
          (1, 64, 100, 1, 700, 1, 3, 1, 0), (2, 100, 64, 12, 50, 1, 1, 1, 0), (1, 33, 70, 25, 31, 2, 3, 1, 0), (2, 24, 40, 23, 29, 5, 5, 1, 2),
          (5, 20, 36, 7, 7, 4, 3, 1, 1), (1, 9, 300, 6, 5, 3, 3, 1, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", STAGED)
@pytest.mark.parametrize("integer", [True, False])
def test_staging_wavefronts(B, cfg, integer, lent):  # noqa: F811
    B.sws_set_option("conv2d_variant", 100 + cfg)
    for i, case in enumerate(SHAPES + CASES):
        _check(B, case, 80 + i, integer, adjoint=case[7] == 1)
    taken = [_taken(t) for t in lent]
    assert sum(taken) >= 30, taken                    # (a tile that does not fit leaves a shape to the kernels without a workspace)
