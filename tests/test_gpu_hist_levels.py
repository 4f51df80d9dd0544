"""Sliding histograms on images whose medians jump from row to row (two levels,
blocks, alternating rows, parts of such images between smooth ones), where a
work-group turns its coarse level on and off, against the CPU oracle or, for
large images, another form of the filter, bit-exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19926_amd import _lib
from paper_2507_19926_amd import workloads as wl
from paper_2507_19926_amd.ops import BatchedPlan, median_filter, median_filter_rect

pytestmark = pytest.mark.gpu


def _images(H, W, seed):
    g = np.random.default_rng(seed)
    smooth = wl.rgb30_planes(H=H, W=W, seed=seed)[2]
    two = (g.integers(0, 2, (H, W)) * 255).astype(np.uint8)
    blocks = np.repeat(np.repeat(g.integers(0, 256, (H // 8 + 1, W // 8 + 1)), 8, 0), 8, 1)[:H, :W].astype(np.uint8)
    rows = np.broadcast_to((np.arange(H) % 2 * 255).astype(np.uint8)[:, None], (H, W)).copy()
    yield two
    yield blocks
    yield rows
    for n in (1, 5, 16, 40):                       # n smooth rows, then n of two levels, and so on
        yield np.where((np.arange(H) // n % 2 == 0)[:, None], smooth, two)
    yield np.where((np.arange(W) % 100 < 50)[None, :], smooth, two)
    yield (two // 255 + 127).astype(np.uint8)      # two levels in two neighbouring groups of 16 bins
    yield np.clip(two.astype(int) // 2 + g.normal(60, 5, (H, W)), 0, 255).astype(np.uint8)


@pytest.mark.parametrize("k", [13, 15, 17, 21, 33, 75])
def test_blocks_of_64_rows(k):
    """The batched form, whose blocks have 64 rows; enough images for the
    histograms to be taken."""
    imgs = list(_images(150, 290, seed=k))
    fill = [np.zeros((1024, 1024), np.uint8)]
    xs = [torch.from_numpy(a).cuda() for a in imgs + fill]
    outs = [torch.empty_like(x) for x in xs]
    plan = BatchedPlan(xs, outs, [k] * len(xs))
    plan.launch()
    for i, (a, o) in enumerate(zip(imgs, outs)):
        assert np.array_equal(o.cpu().numpy(), oracle.median_filter(a, k)), i
    plan.close()


@pytest.mark.parametrize("k", [9, 11, 13, 21, 75])
@pytest.mark.parametrize("shape", [(37, 61), (300, 700)])
def test_short_strips(k, shape):
    for i, a in enumerate(_images(*shape, seed=k)):
        assert np.array_equal(median_filter(torch.from_numpy(a).cuda(), k).cpu().numpy(), oracle.median_filter(a, k)), i


@pytest.mark.parametrize("k", [13, 15, 17, 21])
def test_long_strips(k):
    for i, a in enumerate(_images(4001, 4100, seed=k)):
        x = torch.from_numpy(a).cuda()
        assert torch.equal(median_filter(x, k), median_filter(x, k, variant=_lib.MF_VARIANT_OBLIVIOUS)), i


@pytest.mark.parametrize("kw,kh", [(19, 3), (31, 15), (3, 29)])
def test_rectangles(kw, kh):
    for i, a in enumerate(_images(2000, 4100, seed=kw)):
        x = torch.from_numpy(a).cuda()
        assert torch.equal(median_filter_rect(x, kw, kh), median_filter_rect(x, kw, kh, variant=_lib.MF_VARIANT_DATA_AWARE)), i
