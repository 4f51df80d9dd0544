"""Calls whose grids have as many threads as a launch takes, or more: none of
them was refused by the kernels that ran them before."""
import torch
import pytest

from paper_2507_19926_amd import _lib
from paper_2507_19926_amd.ops import median_filter, median_filter_argmedian, median_filter_backward

pytestmark = pytest.mark.gpu


def test_strips_of_a_very_tall_image():
    """One column of more than 2^28 rows, k = 3: the window's three columns are
    the same, so its median is that of three rows."""
    H = (1 << 28) + 37
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randint(0, 256, (H, 1), generator=g, device="cuda", dtype=torch.uint8)
    y = median_filter(x, 3)
    a, b, c = torch.cat([x[:1], x[:-1]]), x, torch.cat([x[1:], x[-1:]])
    want = torch.maximum(torch.minimum(a, b), torch.minimum(torch.maximum(a, b), c))
    assert torch.equal(y, want)


@pytest.mark.parametrize("k", [3, 9, 31, 33])
def test_gradient_of_many_tiny_planes(k):
    """More than 2^24 planes, a work-group each, against calls of a few of
    them from either end and from the middle."""
    n = (1 << 24) + 7
    g = torch.Generator(device="cuda").manual_seed(k)
    x = torch.rand((n, 2, 3), generator=g, device="cuda")
    up = torch.rand((n, 2, 3), generator=g, device="cuda")
    y, idx = median_filter_argmedian(x, k)
    gi = median_filter_backward(up, idx, k)
    for a, b in ((0, 999), ((1 << 23) - 500, (1 << 23) + 500), (n - 999, n)):
        ys, ids = median_filter_argmedian(x[a:b].contiguous(), k)
        assert torch.equal(y[a:b], ys) and torch.equal(idx[a:b], ids)
        assert torch.equal(gi[a:b], median_filter_backward(up[a:b].contiguous(), ids, k))


def test_regions_of_a_very_wide_image():
    """2^30 columns: a region more than a launch of the ranked kernels takes."""
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.rand((1, 1 << 30), generator=g, device="cuda")
    y = median_filter(x, 21, variant=_lib.MF_VARIANT_DATA_AWARE, form=3)
    assert torch.equal(y, median_filter(x, 21, variant=_lib.MF_VARIANT_OBLIVIOUS))
