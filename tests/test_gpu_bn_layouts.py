"""BN at channel counts whose 8-channel chunks are not a power of two (NHWC) and
in NCHW at image sizes around the 8-value chunks: the forward bit for bit the
same in both layouts given the statistics, statistics and backward against
float64 in plain torch.

Bounds: statistics 2e-6 of the spread; dgamma and dbeta one rounding plus
M * 2^-24 of the sum of magnitudes; dx one rounding plus 1e-5 of the magnitudes
its float32 sequence adds."""

import pytest
import torch

import paper_1911_07384_amd as F
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

EPS, SCALE = 1e-5, 0.25
# (n, c, h, w)
SHAPES = [(2, 24, 5, 3), (3, 160, 9, 7), (2, 72, 14, 14), (1, 1000, 3, 5), (5, 136, 1, 1),
          (2, 2040, 2, 2), (4, 40, 33, 31), (3, 16, 7, 7), (2, 5, 4, 2), (1, 7, 61, 67),
          (40, 8, 8, 16), (3, 264, 28, 28),
          # NCHW in chunks: every remainder of a run, the smallest image and count
          (6, 9, 7, 7), (15, 3, 2, 9), (8, 4, 5, 7), (14, 6, 4, 5), (13, 3, 1, 21), (9, 5, 5, 6),
          (16, 3, 4, 4), (1, 3, 16, 16),
          # ... and one element per thread just below
          (1, 3, 15, 17), (40, 5, 3, 5)]


@pytest.mark.parametrize("form", ["plain", "residual", "stored", "norelu", "swap"])
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_layouts(shape, form):
    require_gpu()
    n, c, h, w = shape
    M = n * h * w
    relu, swap = form != "norelu", form == "swap"
    g = torch.Generator(device="cuda")
    g.manual_seed(31)

    def rnd(*s, std=1.0, mean=0.0):
        return (torch.randn(s, generator=g, device="cuda") * std + mean).half()

    x, dy = rnd(n, h, w, c, mean=0.2), rnd(n, h, w, c, std=1e-2)
    gamma, beta = rnd(c, std=0.3, mean=1.0), rnd(c, std=0.3)
    res = rnd(n, h, w, c) if form in ("residual", "stored", "swap") else None

    def run(layout):
        def put(t):
            return t if t is None or layout == "NHWC" else t.permute(0, 3, 1, 2).contiguous()

        def back(t):
            return t if layout == "NHWC" else t.permute(0, 2, 3, 1).contiguous()

        X, D, R = put(x), put(dy), put(res)
        d = F.bn_desc(n, c, h, w, layout, EPS, SCALE, relu, swap=swap)
        ws = F.workspace(F.fp16_bn_workspace_bytes(d))
        st = torch.empty(2 * c, dtype=torch.float32, device="cuda")
        y = torch.full_like(X, float("nan"))
        F.fp16_bn_relu(d, X, gamma, beta, R, y, st, ws)
        fixed = torch.cat([x.float().view(-1, c).mean(0), 1.0 / x.float().view(-1, c).std(0, unbiased=False)
                           if M > 1 else torch.ones(c, device="cuda")])
        du = F.bn_desc(n, c, h, w, layout, EPS, SCALE, relu, use_stats=True, swap=swap)
        yu = X.clone()  # in place
        F.fp16_bn_relu(du, yu, gamma, beta, R, yu, fixed, ws)
        dx, dres = torch.full_like(X, float("nan")), torch.full_like(X, float("nan"))
        dg, db = torch.empty_like(gamma), torch.empty_like(beta)
        F.fp16_bn_relu_bwd(du, X, yu if form == "stored" else None, D, gamma, beta, R, fixed, dx, dg,
                           db, dres if res is not None else None, ws)
        return st, back(yu), fixed, back(dx), dg, db, back(dres)

    a, b = run("NHWC"), run("NCHW")
    x64 = x.double().view(M, c)
    mean, var = x64.mean(0), x64.var(0, unbiased=False)
    sd = (var + EPS).sqrt()
    for st, yu, fixed, dx, dg, db, dres in (a, b):
        assert ((st[:c].double() - mean).abs() / sd).max().item() < 2e-6
        assert ((st[c:].double() * sd) - 1).abs().max().item() < 4e-6
        m, r = fixed[:c].double(), fixed[c:].double()
        mask = (yu.view(M, c) > 0) if relu else torch.ones((M, c), dtype=torch.bool, device="cuda")
        G = SCALE * dy.double().view(M, c) * mask
        xh = (x64 - m) * r
        s1, s2, mag = G.sum(0), (G * xh).sum(0), (G.abs() * (1 + xh.abs())).sum(0)
        s3 = 0.0
        if swap:
            s3 = (G * res.double().view(M, c)).sum(0)
            mag = mag + (G * res.double().view(M, c)).abs().sum(0)
        tol = (M + 4) * 2.0 ** -24 * mag + 2.0 ** -25
        assert ((db.double() - s1).abs() <= s1.abs() * 2.0 ** -11 + tol).all()
        assert ((dg.double() - (s2 + s3)).abs() <= (s2 + s3).abs() * 2.0 ** -11 + tol).all()
        A = gamma.double() * r
        ref = A * (G - s1 / M - xh * (s2 / M))
        parts = A.abs() * (G.abs() + (s1 / M).abs() + (xh * (s2 / M)).abs() + mag / M)
        err = (dx.double().view(M, c) - ref).abs()
        assert (err <= ref.abs() * 2.0 ** -11 + 1e-5 * parts + 2.0 ** -25).all()
        if swap:
            want = gamma.double() * G
            assert ((dres.double().view(M, c) - want).abs() <= want.abs() * 2.0 ** -10 + 2.0 ** -24).all()
        elif res is not None:
            assert torch.equal(dres.view(M, c), torch.where(mask, dy.view(M, c), torch.zeros_like(x.view(M, c))))
    assert torch.equal(a[1], b[1])


# tensors of over 190 MB, which with the others of a pass exceed the memory-side
# cache: many runs per workgroup, taken from the end
@pytest.mark.parametrize("form", ["plain", "residual", "stored", "swap", "mask"])
@pytest.mark.parametrize("shape", [(1, 64, 1063, 1409), (3, 40, 911, 907)],
                         ids=["64ch", "40ch"])  # a power of two of chunks, and 5
def test_beyond_the_cache(shape, form):
    """Forward and backward element by element against float64, sampled rows at
    both ends and between; sums whole."""
    require_gpu()
    n, c, h, w = shape
    M, swap, masked = n * h * w, form == "swap", form == "mask"
    g = torch.Generator(device="cuda")
    g.manual_seed(33)

    def rnd(*s, std=1.0, mean=0.0):
        return (torch.randn(s, generator=g, device="cuda") * std + mean).half()

    x, dy = rnd(n, h, w, c, mean=0.2), rnd(n, h, w, c, std=1e-2)
    gamma, beta = rnd(c, std=0.3, mean=1.0), rnd(c, std=0.3)
    res = None if form == "plain" else rnd(n, h, w, c)
    d = F.bn_desc(n, c, h, w, "NHWC", EPS, SCALE, True, swap=swap)
    if masked and not F.fp16_bn_mask_bytes(d):
        pytest.skip("no kept mask at this channel count")
    ws = F.workspace(F.fp16_bn_workspace_bytes(d))
    st = torch.empty(2 * c, dtype=torch.float32, device="cuda")
    y = torch.full_like(x, float("nan"))
    if masked:
        m = torch.zeros(F.fp16_bn_mask_bytes(d), dtype=torch.uint8, device="cuda")
        F.fp16_bn_relu_m(d, x, gamma, beta, res, y, st, m, ws)
    else:
        F.fp16_bn_relu(d, x, gamma, beta, res, y, st, ws)
    x2 = x.view(M, c)
    mean = x2.double().mean(0)
    var = (x2.double() - mean).square_().mean(0)
    sd = (var + EPS).sqrt()
    assert ((st[:c].double() - mean).abs() / sd).max().item() < 2e-6
    assert ((st[c:].double() * sd) - 1).abs().max().item() < 4e-6
    dx, dres = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
    dg, db = torch.empty_like(gamma), torch.empty_like(beta)
    if masked:
        F.fp16_bn_relu_bwd_m(d, x, m, dy, gamma, beta, st, dx, dg, db, dres, ws)
    else:
        F.fp16_bn_relu_bwd(d, x, y if form == "stored" else None, dy, gamma, beta, res, st, dx, dg,
                           db, None if res is None else dres, ws)
    keep = y.view(M, c) > 0
    A, rs = gamma.double(), st[c:].double()
    s1, s2, s3, mag = (torch.zeros(c, dtype=torch.float64, device="cuda") for _ in range(4))
    step = 1 << 18
    for i in range(0, M, step):
        b = slice(i, i + step)
        G = SCALE * dy.view(M, c)[b].double() * keep[b]
        xh = (x2[b].double() - st[:c].double()) * rs
        s1 += G.sum(0)
        s2 += (G * xh).sum(0)
        mag += (G.abs() * (1 + xh.abs())).sum(0)
        if swap:
            s3 += (G * res.view(M, c)[b].double()).sum(0)
            mag += (G * res.view(M, c)[b].double()).abs().sum(0)
    # (float32 sums at most 256 additions deep, then float64)
    tol = 2.0 ** -16 * mag + 2.0 ** -25
    assert ((db.double() - s1).abs() <= s1.abs() * 2.0 ** -11 + tol).all()
    assert ((dg.double() - (s2 + s3)).abs() <= (s2 + s3).abs() * 2.0 ** -11 + tol).all()
    for i in range(0, M, step):
        b = slice(i, i + step)
        G = SCALE * dy.view(M, c)[b].double() * keep[b]
        xh = (x2[b].double() - st[:c].double()) * rs
        ref = A * rs * (G - s1 / M - xh * (s2 / M))
        parts = (A * rs).abs() * (G.abs() + (s1 / M).abs() + (xh * (s2 / M)).abs() + mag / M)
        err = (dx.view(M, c)[b].double() - ref).abs()
        assert (err <= ref.abs() * 2.0 ** -11 + 1e-5 * parts + 2.0 ** -25).all()
        r = 0.0 if res is None else res.view(M, c)[b].double()
        v = SCALE * (A * (xh + r) + beta.double()) if swap else SCALE * (A * xh + beta.double()) + r
        fw = (y.view(M, c)[b].double() - v.clamp_min(0)).abs()
        assert (fw <= v.abs() * 2.0 ** -11 + 2e-6 * (A * xh).abs() + 1e-5).all()
        if res is not None:
            got = dres.view(M, c)[b]
            if swap:
                want = A * G
                assert ((got.double() - want).abs() <= want.abs() * 2.0 ** -10 + 2.0 ** -24).all()
            else:
                assert torch.equal(got, torch.where(keep[b], dy.view(M, c)[b], torch.zeros_like(got)))
