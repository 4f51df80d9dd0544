"""Calls whose grids have as many threads as a launch takes, or more: none of
them was refused by the kernels that ran them before."""
import torch
import pytest

from paper_2507_19926_amd.ops import median_filter

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
