"""Host time of the calls that look for the best tiling anew each time.  Without a GPU the launch itself is refused, so what is timed is the checks and the
plan, in units of a call that plans nothing."""
import ctypes
import statistics
import time

import pytest
import torch


@pytest.fixture(scope="module")
def L():
    from paper_2305_16513_amd import binding
    return binding.lib()


def _ratio(f, g):
    """f's time over g's, measured in turn; the median of many, the least of five."""
    def us(h):
        t = time.perf_counter()
        for _ in range(15):
            h()
        return time.perf_counter() - t

    return min(statistics.median(us(f) / us(g) for _ in range(201)) for _ in range(5))


# n, cin, h, w, cout, k: with everything worked out for every configuration 2.4 - 2.8 and 3.3, with shapes shared by the configurations of as many
# positions and nothing for tilings that cannot be the best 2.0 and 2.6
@pytest.mark.parametrize("layer,most", [((8, 128, 56, 56, 128, 1), 2.3), ((32, 64, 30, 30, 64, 3), 3.0)])
def test_planning_of_a_convolution(L, layer, most):
    if torch.cuda.is_available():
        pytest.skip("made-up pointers")
    n, cin, h, w, cout, k = layer
    one = ctypes.c_void_p(4096)
    conv = lambda: L.sws_conv2d_ws(one, one, one, n, cin, h, w, cout, k, k, 1, 1, k // 2, k // 2, one, 1 << 40, None)
    pool = lambda: L.sws_maxpool2d_grad(one, one, one, 1, 1, 112, 112, 3, 3, 1, 1, 1, 1, None)
    assert conv() != 0 and pool() != 0
    assert _ratio(conv, pool) < most


# with every tile worked out for every block of channels, and twice where the staged kernel may be taken, 4.2 and 4.0; now 2.3
@pytest.mark.parametrize("layer", [(4, 160, 12, 12, 160), (32, 256, 14, 14, 256)])
def test_planning_of_a_weight_gradient(L, layer):
    if torch.cuda.is_available():
        pytest.skip("made-up pointers")
    n, cin, h, w, cout = layer
    one = ctypes.c_void_p(4096)
    pool = lambda: L.sws_maxpool2d_grad(one, one, one, 1, 1, 112, 112, 3, 3, 1, 1, 1, 1, None)
    assert _ratio(lambda: L.sws_conv2d_grad_weight_workspace(n, cin, h, w, cout, 3, 3, 1, 1, 1, 1), pool) < 3.2
