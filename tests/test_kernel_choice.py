"""The kernel that each case of the GPU tests runs on, asked of the library on
the host: a moved threshold must not move a test off the kernel it is for."""

import pytest

import paper_1911_07384_amd as F
import test_gpu_conv_bn
import test_gpu_kernel_edges as edges
import test_gpu_wgrad_tiles as wgrad
import test_gpu_wide_tiles as wide


def _desc(shape):
    n, c, h, w, k, r, st = shape
    return F.conv_desc(n, c, h, w, k, r, r, st, r // 2)


def _id(t):
    return "x".join(map(str, t[0]))


@pytest.mark.parametrize("case", wide.TILES, ids=_id)
def test_wide_tiles(case):
    shape, fwd, stats, dgrad = case
    d = _desc(shape)
    assert F.fp16_conv_kernel(d, F.PASS_FWD) == "wide " + fwd
    assert F.fp16_conv_kernel(d, F.PASS_FWD, stats=True) == "wide " + stats
    assert F.fp16_conv_kernel(d, F.PASS_DGRAD) == "wide " + dgrad
    assert F.fp16_conv_kernel(d, F.PASS_DGRAD, addend=True) == "wide " + dgrad


def test_every_wide_tile_is_covered():
    rows = {"64x128", "128x128", "160x128", "192x128", "224x128", "256x128", "128x64", "256x64"}
    tiles = {r + t for r in rows for t in ("", " taps")}
    assert {t[1] for t in wide.TILES} == tiles
    assert {t[2] for t in wide.TILES} == tiles
    assert {t[3] for t in wide.TILES} == tiles


@pytest.mark.parametrize("case", wgrad.TILES, ids=_id)
def test_wgrad_tiles(case):
    assert F.fp16_conv_kernel(_desc(case[0]), F.PASS_WGRAD) == case[1]


def test_every_wgrad_tile_is_covered():
    tiles = {"256x128 8 waves", "128x256 8 waves", "128x128 8 waves", "64x256 8 waves",
             "128x64 4 waves", "64x192 4 waves", "64x128 4 waves", "64x64 4 waves"}
    got = {t[1] for t in wgrad.TILES}
    assert {t.replace(" taps", "") for t in got} == tiles
    for big in ("256x128 8 waves", "128x256 8 waves", "128x128 8 waves", "128x64 4 waves",
                "64x192 4 waves"):
        assert big in got and big + " taps" in got


@pytest.mark.parametrize("case", edges.FORWARD, ids=_id)
def test_forward_kernels(case):
    d = _desc(case[0])
    assert F.fp16_conv_kernel(d, F.PASS_FWD) == case[1]
    assert F.fp16_conv_kernel(d, F.PASS_FWD, stats=True) == case[2]


@pytest.mark.parametrize("case", edges.BACKWARD, ids=_id)
def test_data_gradient_kernels(case):
    d = _desc(case[0])
    assert F.fp16_conv_kernel(d, F.PASS_DGRAD) == case[1]
    assert F.fp16_conv_kernel(d, F.PASS_DGRAD, addend=True) == case[2]


def test_in_place_case_runs_the_second_pass():
    n, c, h, k = test_gpu_conv_bn.POINTWISE_IN_PLACE
    d = F.conv_desc(n, c, h, h, k, 1, 1, 1, 0)
    assert F.fp16_conv_kernel(d, F.PASS_FWD, stats=True).startswith("pointwise 64 ")


def test_names_other_forms():
    d = F.conv_desc(128, 2048, 1, 1, 1000, 1, 1, 1, 0)
    assert F.fp16_conv_kernel(d, F.PASS_FWD) == "dense 8 splits"
    assert F.fp16_conv_kernel(F.conv_desc(2, 3, 32, 32, 64, 7, 7, 2, 3), F.PASS_FWD) == "stem"
    assert F.fp16_conv_kernel(F.conv_desc(2, 8, 9, 9, 8, 3, 3, 1, 1, accum=1), F.PASS_FWD) == "chains"
    bad = F.conv_desc(2, 8, 9, 9, 8, 3, 3, 1, 1)
    assert F.fp16_conv_kernel(bad, 3) == ""
    bad.n = 0
    assert F.fp16_conv_kernel(bad, F.PASS_FWD) == ""
