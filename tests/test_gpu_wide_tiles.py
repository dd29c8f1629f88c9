"""The wide implicit-GEMM kernel at every tile shape its rule picks (64 to 256
rows x 128 channels, 128 and 256 rows x 64), against float64 convolutions in
plain torch: ragged rows and channels, channel counts that are multiples of
64, of 8 or neither, strided phases, addends and masks (every tile but 128 x 64
and 64 x 128 in the form with a tap per lane and in the other), BN statistics.

Bound per element: one rounding to binary16 (2^-11 of the value, 2^-25 below
the normal range) plus the float32 sum's K * 2^-24 * sum |a b|."""

import pytest
import torch

import paper_1911_07384_amd as F
from gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


def taps64(x, w, stride, pad):
    """NHWC x, KRSC w in float64 -> (N, P, Q, K)."""
    k, r, s, c = w.shape
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    P, Q = (xp.shape[1] - r) // stride + 1, (xp.shape[2] - s) // stride + 1
    y = torch.zeros((x.shape[0] * P * Q, k), dtype=torch.float64, device=x.device)
    for i in range(r):
        for j in range(s):
            a = xp[:, i:i + stride * (P - 1) + 1:stride, j:j + stride * (Q - 1) + 1:stride, :]
            y += a.reshape(-1, c) @ w[:, i, j, :].t().contiguous()
    return y.view(x.shape[0], P, Q, k)


def dgrad64(dy, w, stride, pad, h, wd):
    k, r, s, c = w.shape
    n, P, Q, _ = dy.shape
    dx = torch.zeros((n, h + 2 * pad, wd + 2 * pad, c), dtype=torch.float64, device=dy.device)
    for i in range(r):
        for j in range(s):
            t = (dy.reshape(-1, k) @ w[:, i, j, :].contiguous()).view(n, P, Q, c)
            dx[:, i:i + stride * (P - 1) + 1:stride, j:j + stride * (Q - 1) + 1:stride, :] += t
    return dx[:, pad:pad + h, pad:pad + wd, :]


def check(got, ref, mag, K):
    # (the sums' bound doubled for the addition of an addend)
    bound = ref.abs() * 2.0 ** -11 + 2.0 ** -25 + 2 * (K + 2) * 2.0 ** -24 * mag
    over = ((got.double() - ref).abs() / bound).max().item()
    assert over <= 1.0, over
    note(f"largest error over its bound {over:.3f}")


# (n, c, h, w, k, r, stride), then the tile of the forward, of the forward with
# statistics and of the data gradient (with or without an addend); "taps": a
# filter tap per lane.  (Checked on the host in test_kernel_choice.py.)
TILES = [
    ((1, 64, 9, 7, 72, 3, 1), "64x128", "64x128", "64x128 taps"),
    ((2, 128, 90, 91, 100, 3, 1), "64x128", "64x128", "64x128 taps"),
    ((1, 64, 130, 127, 128, 3, 1), "64x128", "128x128", "128x64"),
    ((1, 72, 190, 185, 96, 3, 1), "160x128 taps", "160x128 taps", "160x128 taps"),
    ((1, 64, 211, 213, 128, 3, 1), "192x128", "192x128", "256x64"),
    ((1, 64, 237, 232, 72, 3, 1), "224x128", "224x128", "256x64 taps"),
    ((1, 24, 237, 231, 88, 3, 1), "224x128 taps", "224x128 taps", "256x64 taps"),
    ((1, 64, 255, 256, 104, 3, 1), "256x128", "256x128", "256x64 taps"),
    ((1, 136, 254, 250, 128, 3, 1), "256x128 taps", "256x128 taps", "256x128"),
    ((1, 64, 129, 131, 40, 5, 1), "128x64", "128x64", "128x64 taps"),
    ((1, 40, 131, 131, 64, 3, 1), "128x64 taps", "128x64 taps", "128x64"),
    ((1, 96, 201, 205, 64, 3, 1), "256x64 taps", "256x64 taps", "192x128"),
    ((2, 8, 33, 35, 64, 9, 2), "64x128 taps", "64x128 taps", "64x128"),
    ((3, 192, 29, 31, 320, 3, 2), "64x128", "64x128", "64x128"),
    ((1, 13, 20, 21, 21, 3, 1), "64x128 taps", "64x128 taps", "64x128 taps"),
    ((1, 128, 130, 131, 128, 3, 1), "128x128", "128x128", "128x128"),
    ((1, 104, 130, 131, 72, 3, 1), "128x128 taps", "128x128 taps", "128x128 taps"),
    ((1, 72, 181, 182, 64, 3, 1), "256x64 taps", "256x64 taps", "160x128"),
    ((1, 104, 181, 182, 72, 3, 1), "160x128 taps", "160x128 taps", "160x128 taps"),
    ((1, 72, 202, 203, 64, 3, 1), "256x64 taps", "256x64 taps", "192x128"),
    ((1, 104, 202, 203, 72, 3, 1), "192x128 taps", "192x128 taps", "192x128 taps"),
    ((1, 72, 223, 224, 64, 3, 1), "256x64 taps", "256x64 taps", "224x128"),
    ((1, 104, 223, 224, 72, 3, 1), "224x128 taps", "224x128 taps", "224x128 taps"),
    ((1, 72, 241, 242, 64, 3, 1), "256x64 taps", "256x64 taps", "256x128"),
    ((1, 104, 241, 242, 72, 3, 1), "256x128 taps", "256x128 taps", "256x128 taps"),
    ((1, 64, 180, 361, 64, 5, 1), "256x64", "256x64", "256x64"),
    ((1, 128, 181, 182, 128, 3, 1), "160x128", "160x128", "160x128"),
]
SHAPES = [t[0] for t in TILES]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_wide_tiles(shape):
    require_gpu()
    n, c, h, w, k, r, st = shape
    pad = r // 2
    g = torch.Generator(device="cuda")
    g.manual_seed(11)

    def rnd(*s, std=1.0):
        return (torch.randn(s, generator=g, device="cuda") * std).half()

    d = F.conv_desc(n, c, h, w, k, r, r, st, pad)
    P, Q = F.fp16_conv_out_dims(d)
    x, f = rnd(n, h, w, c), rnd(k, r, r, c, std=(2.0 / (c * r * r)) ** 0.5)
    dy, add = rnd(n, P, Q, k), rnd(n, h, w, c)
    ws = F.workspace(max(F.fp16_conv_workspace_bytes(d, p) for p in (0, 1, 2)))
    x64, f64, dy64 = x.double(), f.double(), dy.double()
    y = torch.full((n, P, Q, k), float("nan"), dtype=torch.float16, device="cuda")
    F.fp16_conv_fwd(d, x, f, y, ws)
    check(y, taps64(x64, f64, st, pad), taps64(x64.abs(), f64.abs(), st, pad), c * r * r)
    # data gradient: plain, with an addend, with a masked addend
    ref = dgrad64(dy64, f64, st, pad, h, w)
    mag = dgrad64(dy64.abs(), f64.abs(), st, pad, h, w)
    dx = torch.full((n, h, w, c), float("nan"), dtype=torch.float16, device="cuda")
    F.fp16_conv_dgrad(d, dy, f, dx, ws)
    check(dx, ref, mag, k * r * r)
    F.fp16_conv_dgrad_add(d, dy, f, add, dx, ws)
    check(dx, ref + add.double(), mag + add.double().abs(), k * r * r)
    if c % 8 == 0:
        keep = torch.rand(add.shape, generator=g, device="cuda") < 0.5
        bits = (keep.view(-1, 8).int() * (1 << torch.arange(8, device="cuda", dtype=torch.int32)))
        wf = torch.empty(F.fp16_conv_dgrad_filter_bytes(d) // 2, dtype=torch.float16, device="cuda")
        F.fp16_conv_dgrad_filter(d, f, wf)
        F.fp16_conv_dgrad_wf_m(d, dy, wf, add, bits.sum(1).to(torch.uint8), dx, ws)
        masked = torch.where(keep, add.double(), torch.zeros_like(ref))
        check(dx, ref + masked, mag + masked.abs(), k * r * r)


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[4] % 8 == 0],
                         ids=["x".join(map(str, s)) for s in SHAPES if s[4] % 8 == 0])
def test_wide_statistics(shape):
    """conv + BN: y bit for bit the convolution's, the statistics of y's rounded
    values (float32 sums about a shift, combined in float64)."""
    require_gpu()
    n, c, h, w, k, r, st = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(12)
    d = F.conv_desc(n, c, h, w, k, r, r, st, r // 2)
    P, Q = F.fp16_conv_out_dims(d)
    b = F.bn_desc(n, k, P, Q, "NHWC", 1e-5, 0.25, True)
    x = torch.randn((n, h, w, c), generator=g, device="cuda").half()
    f = (torch.randn((k, r, r, c), generator=g, device="cuda") * (2.0 / (c * r * r)) ** 0.5).half()
    gamma, beta = torch.ones(k, device="cuda").half(), torch.zeros(k, device="cuda").half()
    y0, y1, z = (torch.empty((n, P, Q, k), dtype=torch.float16, device="cuda") for _ in range(3))
    stats = torch.empty(2 * k, dtype=torch.float32, device="cuda")
    ws = F.workspace(max(F.fp16_conv_bn_workspace_bytes(d, b), F.fp16_conv_workspace_bytes(d, 0)))
    F.fp16_conv_fwd(d, x, f, y0, ws)
    F.fp16_conv_bn_relu_fwd(d, b, x, f, gamma, beta, None, y1, z, stats, ws)
    assert torch.equal(y0, y1)
    v = y1.double().view(-1, k)
    mean, var = v.mean(0), v.var(0, unbiased=False)
    # float32 sums of at most 256 rows per record about one of its values:
    # well inside 2e-6 of the spread
    sd = (var + 1e-5).sqrt()
    assert ((stats[:k].double() - mean).abs() / sd).max().item() < 2e-6
    assert ((stats[k:].double() * sd) - 1).abs().max().item() < 4e-6
