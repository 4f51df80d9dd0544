"""The differentiable form on images of few levels, where a wave stops looking
for the medians' places early, and of few work-groups: the places are the first
ones in their windows, and the gradient is that of a scatter by them."""
import numpy as np
import pytest
import torch

from paper_2507_19926_amd.ops import median_filter, median_filter_argmedian, median_filter_backward

pytestmark = pytest.mark.gpu


def _first_places(x, y, k):
    H, W = x.shape
    r = (k - 1) // 2
    rows = np.clip(np.arange(-r, H + r), 0, H - 1)
    cols = np.clip(np.arange(-r, W + r), 0, W - 1)
    u = np.lib.stride_tricks.sliding_window_view(x[rows][:, cols], (k, k)).reshape(H, W, k * k)
    first = (u == y[..., None]).argmax(-1)
    qy = np.clip(np.arange(H)[:, None] - r + first // k, 0, H - 1)
    qx = np.clip(np.arange(W)[None, :] - r + first % k, 0, W - 1)
    return (qy * W + qx).astype(np.int32)


@pytest.mark.parametrize("k", [3, 7, 9, 15, 17, 33])
@pytest.mark.parametrize("shape", [(1, 7, 5), (1, 33, 70), (3, 65, 130), (40, 8, 9), (300, 20, 66)])
def test_places_and_gradient(k, shape):
    g = np.random.default_rng(k)
    for levels in (1, 2, 5):
        x = g.integers(0, levels, shape).astype(np.float32)
        t = torch.from_numpy(x).cuda()
        y, idx = median_filter_argmedian(t, k)
        assert torch.equal(y, median_filter(t, k))
        up = g.standard_normal(shape).astype(np.float32)
        gi = median_filter_backward(torch.from_numpy(up).cuda(), idx, k).cpu().numpy()
        for p in (0, shape[0] - 1):
            want = _first_places(x[p], y[p].cpu().numpy(), k)
            assert np.array_equal(idx[p].cpu().numpy(), want), (levels, p)
            acc = np.zeros(x[p].size, np.float32)
            for q, v in zip(want.ravel(), up[p].ravel()):          # ascending outputs, in binary32
                acc[q] += v
            assert gi[p].tobytes() == acc.reshape(x[p].shape).tobytes(), (levels, p)
