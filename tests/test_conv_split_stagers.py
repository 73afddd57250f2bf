"""Configurations of the split-operand convolution whose workgroups hold wavefronts that only stage (csrc/conv_split.hip)."""
import pytest

from tests.parity_util import kernels
from tests.test_parity_conv_split import B, CASES, _check, _taken, automatic, lent  # noqa: F401

# 64 x 128 with a split contraction, and the three largest tiles
STAGED = (3, 14, 15, 16)
# one chunk, two and many; chunks of 6, 8, 9 and 12 steps and of numbers that stay in the loop; rows and images that end inside a tile; channels of
# no whole octet; more units than the multiplying wavefronts stage of the first chunk
SHAPES = [(1, 16, 128, 9, 30, 3, 3, 1, 1), (2, 32, 64, 20, 20, 3, 3, 1, 1), (2, 150, 130, 17, 19, 3, 3, 1, 1), (3, 40, 129, 40, 40, 3, 3, 2, 1),
          (1, 64, 100, 1, 700, 1, 3, 1, 0), (2, 96, 100, 20, 20, 2, 4, 1, 0), (2, 100, 64, 12, 50, 1, 1, 1, 0), (1, 33, 70, 25, 31, 2, 3, 1, 0), (2, 24, 40, 23, 29, 5, 5, 1, 2),
          (5, 20, 36, 7, 7, 4, 3, 1, 1), (1, 9, 300, 6, 5, 3, 3, 1, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", STAGED)
@pytest.mark.parametrize("integer", [True, False])
def test_staging_wavefronts(B, cfg, integer, lent):  # noqa: F811
    B.sws_set_option("conv2d_variant", 100 + cfg)
    ran = set()
    for i, case in enumerate(SHAPES + CASES):
        names = kernels(lambda: _check(B, case, 80 + i, integer, adjoint=case[7] == 1))
        ran |= {tuple(map(int, n[18:-1].split(", ")))[-2:] for n in names if n.startswith("conv_split_kernel<")}
    # (wavefronts that only stage, steps of a chunk)
    assert {s for p, s in ran if p == 4} == {6, 8, 9, 12} and {s for p, s in ran if p == 0} <= {0, 25}, ran
    taken = [_taken(t) for t in lent]
    assert sum(taken) >= 30, taken                    # (a tile that does not fit leaves a shape to the kernels without a workspace)


# n, cin, cout, h, w, k, stride: the configuration that is faster, the one that the estimate alone would take.  Times of the two, us: 82 / 96, 88 / 93, 70 / 75, 134 / 139,
# 27 / 32
FASTER = {(64, 200, 32, 41, 41, 3, 2): (5, 16), (1, 288, 320, 95, 95, 3, 1): (6, 15), (4, 384, 32, 90, 90, 3, 1): (9, 3), (1, 96, 432, 97, 97, 5, 1): (5, 16),
          (8, 320, 160, 1, 1117, 3, 1): (3, 2)}


@pytest.mark.gpu
@pytest.mark.parametrize("case", FASTER)
def test_the_faster_configuration_is_taken(B, case):  # noqa: F811
    """Told apart by the bits of the sums: the two split the contraction over different numbers of wavefronts."""
    import torch
    n, cin, cout, h, w, k, s = case
    g = torch.Generator(device="cuda").manual_seed(7)
    x, wgt = torch.randn(n, cin, h, w, generator=g, device="cuda"), torch.randn(cout, cin, k if h > 1 else 1, k, generator=g, device="cuda")
    y = {}
    for cfg in (None, *FASTER[case]):
        B.sws_set_option("conv2d_variant", 0 if cfg is None else 100 + cfg)
        y[cfg] = B.sws_conv2d(x, wgt, s, s, wgt.shape[2] // 2, k // 2)
    faster, other = (y[c] for c in FASTER[case])
    assert not torch.equal(faster, other) and torch.equal(y[None], faster)
