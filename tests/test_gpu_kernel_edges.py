"""The convolution kernels besides the wide one, at the sizes from which they are
chosen: ragged rows, channel tiles and several tiles per workgroup, with BN
statistics, addends, masks, strided addends and outputs in place.  The kernel
that each case runs on is part of its row (checked on the host in
test_kernel_choice.py).

Bounds: against float64 in plain torch as in test_gpu_wide_tiles.py; where two
calls must agree (convolution and conv + BN, the BN apply from the same
statistics, a masked or strided addend and its full form) bit for bit."""

import pytest
import torch

import paper_1911_07384_amd as F
from gpu_util import note, require_gpu
from test_gpu_wide_tiles import check, dgrad64, taps64

pytestmark = pytest.mark.gpu

# (n, c, h, w, k, r, stride), the forward's kernel, with statistics
FORWARD = [
    # pointwise over 64 channels: ragged rows, a channel tile of 8, of 8 in 256
    ((1, 64, 157, 157, 136, 1, 1), "pointwise 64 128x128", "pointwise 64 128x128"),
    ((1, 64, 129, 128, 264, 1, 1), "pointwise 64 128x256", "pointwise 64 128x128"),
    ((3, 64, 157, 161, 256, 1, 1), "pointwise 64 128x256", "pointwise 64 128x128"),  # several tiles each
    ((3, 64, 211, 223, 256, 1, 1), "pointwise 64 128x256", "pointwise 64 128x256"),  # large enough for
                                                                  # 256-channel tiles with statistics
    # over 128 and 256
    ((1, 128, 181, 181, 520, 1, 1), "pointwise 128 128x256", "pointwise 128 128x128"),
    ((1, 256, 181, 181, 520, 1, 1), "pointwise 256 128x128", "pointwise 256 128x128"),
    ((2, 256, 257, 257, 520, 1, 2), "pointwise 256 128x128", "pointwise 256 128x128"),  # strided
    # register-direct: 64-channel tiles (48 used), taps, 128-channel tiles (8 of the third used)
    ((1, 96, 212, 212, 48, 1, 1), "direct 128x64", "direct 128x64"),
    ((3, 32, 123, 125, 64, 3, 1), "direct 128x64", "direct 128x64"),
    ((1, 32, 193, 193, 200, 1, 1), "direct 128x128", "wide 160x128 taps"),
    ((1, 96, 234, 234, 264, 1, 1), "direct 128x128", "direct 128x128"),
    ((1, 96, 212, 212, 45, 1, 1), "direct 128x64", "direct 128x64"),  # odd channels: scalar stores
    # the 3x3 64-channel kernel at other widths than 56, one to several tiles an image
    ((52, 64, 40, 41, 64, 3, 1), "3x3", "3x3"),
    ((131, 64, 17, 33, 64, 3, 1), "3x3", "3x3"),
    ((260, 64, 13, 11, 64, 3, 1), "3x3", "3x3"),
]

# (n, c, h, w, k, r, stride), the data gradient's kernel, with an addend
BACKWARD = [
    ((1, 136, 157, 157, 64, 1, 1), "pointwise 64 128x128", "pointwise 64 128x128"),
    ((2, 264, 93, 95, 64, 1, 1), "pointwise 64 128x256", "pointwise 64 128x256"),
    ((1, 520, 181, 181, 128, 1, 1), "pointwise 128 128x256", "pointwise 128 128x256"),
    ((1, 520, 181, 183, 256, 1, 1), "pointwise 256 128x128", "direct 128x128"),
    ((1, 48, 212, 212, 96, 1, 1), "direct 128x64", "direct 128x64"),
    ((1, 45, 212, 212, 96, 1, 1), "direct 128x64", "direct 128x64"),
    ((1, 264, 234, 234, 96, 1, 1), "direct 128x128", "direct 128x128"),
    # stride phases: register-direct (1x1: three of the four phases empty)
    ((1, 48, 231, 233, 64, 1, 2), "direct 128x64", "direct 128x64"),
    ((1, 72, 181, 183, 128, 1, 2), "direct 128x128", "direct 128x128"),
    ((2, 72, 157, 159, 96, 3, 2), "direct 128x128", "direct 128x128"),
    # DMA-staged
    ((1, 40, 185, 183, 192, 3, 2), "dma 128x64", "dma 128x64"),
    ((1, 29, 187, 185, 192, 3, 2), "dma 128x64", "dma 128x64"),
    ((2, 64, 131, 129, 64, 5, 2), "dma 128x64", "dma 128x64"),
    ((1, 136, 157, 159, 640, 1, 2), "dma 128x128", "dma 128x128"),
    ((1, 200, 187, 189, 640, 1, 2), "dma 128x128", "dma 128x128"),
    # LDS-staged
    ((1, 40, 185, 183, 24, 1, 2), "staged 128x64", "staged 128x64"),
    ((1, 21, 185, 183, 24, 1, 2), "staged 128x64", "staged 128x64"),
    ((2, 56, 133, 131, 40, 3, 2), "staged 128x64", "staged 128x64"),
    ((1, 200, 137, 139, 24, 3, 2), "staged 128x128", "staged 128x128"),
    ((1, 72, 211, 213, 8, 3, 2), "staged 128x128", "staged 128x128"),
]


def _id(s):
    return "x".join(map(str, s))


def _bits(keep):
    w = 1 << torch.arange(8, device=keep.device, dtype=torch.int32)
    return (keep.reshape(-1, 8).int() * w).sum(1).to(torch.uint8)


@pytest.mark.parametrize("case", FORWARD, ids=[_id(c[0]) for c in FORWARD])
def test_forward(case):
    require_gpu()
    n, c, h, w, k, r, st = case[0]
    g = torch.Generator(device="cuda")
    g.manual_seed(41)
    d = F.conv_desc(n, c, h, w, k, r, r, st, r // 2)
    P, Q = F.fp16_conv_out_dims(d)
    note(f"[gpu] {case}")
    x = torch.randn((n, h, w, c), generator=g, device="cuda").half()
    f = (torch.randn((k, r, r, c), generator=g, device="cuda") * (2.0 / (c * r * r)) ** 0.5).half()
    y = torch.full((n, P, Q, k), float("nan"), dtype=torch.float16, device="cuda")
    F.fp16_conv_fwd(d, x, f, y, F.workspace(F.fp16_conv_workspace_bytes(d, F.PASS_FWD)))
    x64, f64 = x.double(), f.double()
    check(y, taps64(x64, f64, st, r // 2), taps64(x64.abs(), f64.abs(), st, r // 2), c * r * r)
    if k % 8:
        return
    gamma = (torch.randn(k, generator=g, device="cuda") * 0.3 + 1.0).half()
    beta = (torch.randn(k, generator=g, device="cuda") * 0.3).half()
    res = torch.randn(y.shape, generator=g, device="cuda").half()
    v = y.double().view(-1, k)
    mean, var = v.mean(0), v.var(0, unbiased=False)
    sd = (var + 1e-5).sqrt()
    for with_res, relu in ((True, True), (False, True), (True, False)):
        b = F.bn_desc(n, k, P, Q, "NHWC", 1e-5, 0.25, relu)
        ws = F.workspace(max(F.fp16_conv_bn_workspace_bytes(d, b), F.fp16_bn_workspace_bytes(b)))
        R = res if with_res else None
        y1, z = (torch.full_like(y, float("nan")) for _ in range(2))
        stats = torch.empty(2 * k, dtype=torch.float32, device="cuda")
        F.fp16_conv_bn_relu_fwd(d, b, x, f, gamma, beta, R, y1, z, stats, ws)
        assert torch.equal(y1, y)
        # float32 sums of a record about one of its values: well inside 2e-6 of the spread
        assert ((stats[:k].double() - mean).abs() / sd).max().item() < 2e-6
        assert ((stats[k:].double() * sd) - 1).abs().max().item() < 4e-6
        # the apply, from these statistics, as the BN's own call does it
        want = torch.empty_like(y)
        bu = F.bn_desc(n, k, P, Q, "NHWC", 1e-5, 0.25, relu, use_stats=True)
        F.fp16_bn_relu(bu, y, gamma, beta, R, want, stats, ws)
        assert torch.equal(z, want)
        # z in place of y, and of the shortcut
        F.fp16_conv_bn_relu_fwd(d, b, x, f, gamma, beta, R, y1, y1, stats, ws)
        assert torch.equal(y1, want)
        if with_res:
            z2 = res.clone()
            F.fp16_conv_bn_relu_fwd(d, b, x, f, gamma, beta, z2, y1, z2, stats, ws)
            assert torch.equal(z2, want) and torch.equal(y1, y)


@pytest.mark.parametrize("case", BACKWARD, ids=[_id(c[0]) for c in BACKWARD])
def test_data_gradient(case):
    require_gpu()
    n, c, h, w, k, r, st = case[0]
    pad = r // 2
    g = torch.Generator(device="cuda")
    g.manual_seed(42)
    d = F.conv_desc(n, c, h, w, k, r, r, st, pad)
    P, Q = F.fp16_conv_out_dims(d)
    note(f"[gpu] {case}")
    dy = torch.randn((n, P, Q, k), generator=g, device="cuda").half()
    f = (torch.randn((k, r, r, c), generator=g, device="cuda") * (2.0 / (c * r * r)) ** 0.5).half()
    add = torch.randn((n, h, w, c), generator=g, device="cuda").half()
    ws = F.workspace(F.fp16_conv_workspace_bytes(d, F.PASS_DGRAD))
    dx = torch.full(add.shape, float("nan"), dtype=torch.float16, device="cuda")
    ref = dgrad64(dy.double(), f.double(), st, pad, h, w)
    mag = dgrad64(dy.double().abs(), f.double().abs(), st, pad, h, w)
    F.fp16_conv_dgrad(d, dy, f, dx, ws)
    check(dx, ref, mag, k * r * r)
    full = torch.full_like(dx, float("nan"))
    F.fp16_conv_dgrad_add(d, dy, f, add, full, ws)
    check(full, ref + add.double(), mag + add.double().abs(), k * r * r)
    dx.copy_(add)  # in place
    F.fp16_conv_dgrad_add(d, dy, f, dx, dx, ws)
    assert torch.equal(dx, full)

    wf = torch.empty(F.fp16_conv_dgrad_filter_bytes(d) // 2, dtype=torch.float16, device="cuda")
    F.fp16_conv_dgrad_filter(d, f, wf)
    # an addend on every second row and column, against the same zero-filled
    part = add[:, ::2, ::2, :].contiguous()
    filled = torch.zeros_like(add)
    filled[:, ::2, ::2, :] = part
    F.fp16_conv_dgrad_add(d, dy, f, filled, full, ws)
    dx.fill_(float("nan"))
    F.fp16_conv_dgrad_wf_ex(d, dy, wf, part, None, 2, dx, ws)
    assert torch.equal(dx, full)
    if c % 8:
        return
    # a masked addend, whole and strided
    keep = torch.rand(add.shape, generator=g, device="cuda") < 0.5
    zero = torch.zeros((), dtype=torch.float16, device="cuda")
    F.fp16_conv_dgrad_add(d, dy, f, torch.where(keep, add, zero), full, ws)
    dx.fill_(float("nan"))
    F.fp16_conv_dgrad_wf_m(d, dy, wf, add, _bits(keep), dx, ws)
    assert torch.equal(dx, full)
    keep = torch.rand(part.shape, generator=g, device="cuda") < 0.5
    filled[:, ::2, ::2, :] = torch.where(keep, part, zero)
    F.fp16_conv_dgrad_add(d, dy, f, filled, full, ws)
    dx.fill_(float("nan"))
    F.fp16_conv_dgrad_wf_ex(d, dy, wf, part, _bits(keep), 2, dx, ws)
    assert torch.equal(dx, full)
