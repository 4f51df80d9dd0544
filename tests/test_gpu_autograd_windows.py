"""Differentiable form, window sizes at the edges of its kernel variants (bit
maps with rows of 8, 16 and 32 bits, comparisons beyond) on shapes narrower
than the window, one block, and ragged blocks; an index tensor of another
window names pixels outside the window, which do not count."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19926_amd import workloads as wl
from paper_2507_19926_amd.ops import median_filter_argmedian, median_filter_backward

pytestmark = pytest.mark.gpu


def _same(a, b):
    return a.tobytes() == b.tobytes()


@pytest.mark.parametrize("k", [3, 5, 7, 9, 15, 17, 31, 33])
@pytest.mark.parametrize("shape", [(1, 1), (1, 70), (70, 1), (16, 64), (17, 65), (8, 130), (35, 200)])
def test_shapes(k, shape):
    for x in (wl.autograd_tensor(shape=shape), np.zeros(shape, np.float32),
              wl.tie_heavy_plane(*shape, np.float32, levels=2, seed=k)):
        g = wl.grad_out_like(shape, seed=k)
        y, idx = median_filter_argmedian(torch.from_numpy(x).cuda(), k)
        gi = median_filter_backward(torch.from_numpy(g).cuda(), idx, k)
        v, i = oracle.argmedian_f32(x, k)
        assert _same(y.cpu().numpy(), v) and np.array_equal(idx.cpu().numpy(), i)
        assert _same(gi.cpu().numpy(), oracle.grad_f32(g, i))


@pytest.mark.parametrize("k", [5, 15, 31])
def test_names_outside_the_window_do_not_count(k):
    shape = (40, 90)
    g = wl.grad_out_like(shape, seed=k)
    _, idx = median_filter_argmedian(torch.from_numpy(wl.autograd_tensor(shape=shape)).cuda(), k + 10)
    idx[3, 4], idx[5, 6] = -1, 40 * 90
    got = median_filter_backward(torch.from_numpy(g).cuda(), idx, k).cpu().numpy()
    ii, r = idx.cpu().numpy(), (k - 1) // 2
    py, px = np.mgrid[0:40, 0:90]
    keep = (ii >= 0) & (ii < 40 * 90) & (abs(ii // 90 - py) <= r) & (abs(ii % 90 - px) <= r)
    want = np.zeros(shape, np.float32)
    for y, x in zip(*np.nonzero(keep)):
        want.flat[ii[y, x]] += g[y, x]
    assert _same(got, want)
