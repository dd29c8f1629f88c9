"""NCHW calls move their tensors through the library's layout conversions: a
1x1 convolution with the identity filter returns its input bit for bit, and
its gradients the output gradient, at sizes around the conversions' 8 x 8
blocks and the runs of one wave, and below the size from which blocks are used."""

import pytest
import torch

import paper_1911_07384_amd as F
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

SHAPES = [(1, 8, 1, 1), (3, 24, 5, 3), (2, 65, 7, 9), (1, 130, 16, 16), (2, 9, 31, 1),
          (4, 64, 8, 8), (1, 3, 33, 2), (2, 512, 7, 7), (1, 72, 9, 57), (5, 1, 3, 3),
          # from here on in blocks (the smaller ones element by element): all
          # blocks whole, then partial in pixels, in channels and in both
          (3, 64, 48, 48), (96, 64, 8, 8), (330, 136, 5, 5), (17, 1030, 8, 8), (3, 65, 75, 73),
          (2, 9, 241, 245), (130, 904, 3, 3),
          # 3 channels: to NHWC in blocks, back element by element
          (20, 3, 133, 137)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_identity_filter(shape):
    require_gpu()
    n, c, h, w = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x, dy, add = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    f = torch.eye(c, device="cuda").half().view(c, c, 1, 1).contiguous()
    d = F.conv_desc(n, c, h, w, c, 1, 1, 1, 0, "NCHW")
    ws = F.workspace(max(F.fp16_conv_workspace_bytes(d, p) for p in (0, 1, 2)))
    y = torch.full(shape, float("nan"), dtype=torch.float16, device="cuda")
    F.fp16_conv_fwd(d, x, f, y, ws)
    assert torch.equal(y, x)
    dx = torch.full(shape, float("nan"), dtype=torch.float16, device="cuda")
    F.fp16_conv_dgrad(d, dy, f, dx, ws)
    assert torch.equal(dx, dy)
    F.fp16_conv_dgrad_add(d, dy, f, add, dx, ws)
    assert torch.equal(dx, (dy.float() + add.float()).half())
