"""Pooling of planes of one element that every window covers (csrc/pool2d_small.hip, pool2d_spread_kernel): the adjoint of a global average."""
import pytest
import torch

from paper_2305_16513_amd import binding as B


# sizes around four, around a workgroup's share of planes, its last plane
@pytest.mark.gpu
@pytest.mark.parametrize("h,w", [(1, 1), (1, 2), (1, 3), (2, 2), (5, 1), (7, 7), (15, 17), (16, 16), (1, 257), (25, 40), (63, 65)])
@pytest.mark.parametrize("planes", [1, 3, 4, 21, 1030])
def test_one_element_planes_are_spread(h, w, planes):
    B.lib()
    g = torch.Generator(device="cuda").manual_seed(h * w + planes)
    buf = torch.randn(planes + 1, generator=g, device="cuda")
    for gy in (buf[:planes].view(1, planes, 1, 1), buf[1:].view(1, planes, 1, 1)):
        want = (gy * (1.0 / (h * w))).expand(1, planes, h, w)
        for off in (0, 1):                                                   # a result that starts on a 16-byte boundary, and one that does not
            flat = torch.full((planes * h * w + 8,), 7.0, device="cuda")
            gx = flat[4 + off:4 + off + planes * h * w].view(1, planes, h, w)
            B.sws_avgpool2d_grad(gy, h, w, h, w, 1, 1, 0, 0, 0, 1.0 / (h * w), gx=gx)
            assert torch.equal(gx, want) and (flat[:4 + off] == 7).all() and (flat[4 + off + planes * h * w:] == 7).all()
        assert torch.equal(B.sws_pool2d(B.OP_MAX, gy, h, w, 1, 1, h - 1, w - 1), gy.expand(1, planes, h, w))
        b = gy.bfloat16()
        assert torch.equal(B.sws_pool2d_16(B.OP_MIN, b, h, w, 1, 1, h - 1, w - 1), b.expand(1, planes, h, w))
