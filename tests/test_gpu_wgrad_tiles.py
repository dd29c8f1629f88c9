"""The weight gradient at every tile its rule picks (eight waves: 128 x 128,
256 x 128, 128 x 256; four: 64 to 256 columns), with ragged channels, pixel
counts and split counts, against float64 in plain torch.

Bound per element: one rounding to binary16 (2^-11 of the value, 2^-25 below
the normal range) plus the float32 sums' M * 2^-24 * sum |a b| over the M
pixels."""

import pytest
import torch

import paper_1911_07384_amd as F
from gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu

# (n, c, h, w, k, r, stride) and the tile ("taps": a filter tap per lane; checked
# on the host in test_kernel_choice.py)
TILES = [
    ((3, 128, 11, 13, 128, 3, 1), "128x128 8 waves"),
    ((2, 512, 7, 7, 512, 3, 1), "128x128 8 waves"),
    ((8, 384, 14, 15, 136, 5, 1), "256x128 8 waves"),
    ((32, 1000, 7, 8, 136, 3, 1), "256x128 8 waves taps"),  # ragged rows of 256, taps per lane
    ((16, 256, 11, 12, 264, 5, 1), "128x256 8 waves"),  # ragged rows
    ((32, 688, 7, 8, 72, 5, 1), "128x256 8 waves taps"),  # taps per lane
    ((2, 688, 12, 12, 384, 3, 1), "128x128 8 waves taps"),
    ((5, 72, 15, 17, 200, 3, 2), "128x128 8 waves taps"),  # channels that are multiples of 8 only: ragged tiles
    ((2, 24, 20, 21, 72, 5, 1), "128x128 8 waves taps"),  # several taps in a 64-column block, 72 of 128 output channels
    ((4, 64, 9, 9, 64, 3, 1), "64x192 4 waves"),
    ((3, 200, 8, 8, 40, 3, 1), "64x192 4 waves taps"),  # 40 output channels
    ((2, 136, 10, 10, 64, 1, 1), "64x192 4 waves taps"),
    ((2, 120, 10, 10, 64, 1, 1), "64x128 4 waves taps"),
    ((2, 56, 10, 10, 32, 1, 1), "64x64 4 waves taps"),
    ((3, 40, 9, 11, 136, 1, 1), "128x64 4 waves taps"),
    ((1, 8, 1, 1, 80, 1, 1), "128x64 4 waves taps"),  # one pixel
    ((1, 688, 7, 8, 136, 5, 1), "128x64 4 waves taps"),  # many tiles of a few k-steps
    ((1, 512, 5, 5, 1000, 3, 1), "128x64 4 waves"),  # ... with 64-channel blocks
    ((1, 96, 3, 67, 96, 3, 1), "128x128 8 waves taps"),  # rows longer than a k-step
    ((4, 64, 21, 21, 256, 3, 2), "128x128 8 waves"),
    ((2, 48, 16, 16, 64, 5, 1), "64x256 8 waves taps"),
]
SHAPES = [t[0] for t in TILES]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_wgrad_tiles(shape):
    require_gpu()
    n, c, h, w, k, r, st = shape
    pad = r // 2
    g = torch.Generator(device="cuda")
    g.manual_seed(21)
    d = F.conv_desc(n, c, h, w, k, r, r, st, pad)
    P, Q = F.fp16_conv_out_dims(d)
    x = torch.randn((n, h, w, c), generator=g, device="cuda").half()
    dy = torch.randn((n, P, Q, k), generator=g, device="cuda").half()
    xp = torch.nn.functional.pad(x.double(), (0, 0, pad, pad, pad, pad))
    flat = dy.double().reshape(-1, k).t().contiguous()
    ref = torch.zeros((k, r, r, c), dtype=torch.float64, device="cuda")
    mag = torch.zeros_like(ref)
    for i in range(r):
        for j in range(r):
            a = xp[:, i:i + st * (P - 1) + 1:st, j:j + st * (Q - 1) + 1:st, :].reshape(-1, c)
            ref[:, i, j, :] = flat @ a
            mag[:, i, j, :] = flat.abs() @ a.abs()
    bound = ref.abs() * 2.0 ** -11 + 2.0 ** -25 + (n * P * Q + 2) * 2.0 ** -24 * mag
    ws = F.workspace(F.fp16_conv_workspace_bytes(d, F.PASS_WGRAD))
    for wg in (0, 1, 100, 256, 512):
        dw = torch.full((k, r, r, c), float("nan"), dtype=torch.float16, device="cuda")
        F.fp16_conv_wgrad_ex(d, x, dy, dw, ws, workgroups=wg)
        over = ((dw.double() - ref).abs() / bound).max().item()
        assert over <= 1.0, (wg, over)
    note(f"largest error over its bound {over:.3f}")
