"""Narrow images and many tiny planes, whose calls choose between the
histograms and the schedules by the shape: the choice, either form asked for and
the oracle agree, bit-exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19926_amd import _lib
from paper_2507_19926_amd import workloads as wl
from paper_2507_19926_amd.ops import BatchedPlan, median_filter, median_filter_3d, median_filter_rect

pytestmark = pytest.mark.gpu

SHAPES = [(1, 9000, 24), (1, 30000, 8), (1, 24, 9000), (1, 2100, 64), (600, 16, 16), (200, 28, 28), (90, 40, 40), (3000, 7, 7)]


def _planes(dt, n, H, W, seed):
    img = wl.float_specials_plane(n * H, W, seed) if dt == np.float32 else wl.uniform_plane(n * H, W, dt, seed)
    return img.reshape(n, H, W)


def _sampled(img, kw, kh, got):
    g = np.random.default_rng(kw)
    for p in g.integers(0, len(img), 3):
        want = oracle.median_filter(img[p], kw) if kw == kh else oracle.median_filter_rect(img[p], kw, kh)
        assert got[p].tobytes() == want.tobytes(), (img.shape, kw, kh)


@pytest.mark.parametrize("dtype,k", [(np.uint8, 9), (np.uint8, 11), (np.uint8, 23), (np.uint8, 35), (np.uint16, 21), (np.uint16, 23),
                                     (np.uint16, 35), (np.uint32, 25), (np.float32, 21), (np.float32, 33)])
@pytest.mark.parametrize("shape", SHAPES)
def test_squares(dtype, k, shape):
    img = _planes(dtype, *shape, seed=k)
    x = torch.from_numpy(img).cuda()
    got = median_filter(x, k).cpu().numpy()
    _sampled(img, k, k, got)
    assert got.tobytes() == median_filter(x, k, variant=_lib.MF_VARIANT_DATA_AWARE).cpu().numpy().tobytes()
    if not (dtype == np.uint8 and k < 13) and not (dtype == np.uint16 and k < 23):
        assert got.tobytes() == median_filter(x, k, variant=_lib.MF_VARIANT_DATA_AWARE, form=3).cpu().numpy().tobytes()


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16, np.float32])
@pytest.mark.parametrize("kw,kh", [(19, 3), (3, 23), (19, 11), (13, 29), (31, 29)])
@pytest.mark.parametrize("shape", [(1, 20000, 24), (1, 24, 20000), (1200, 20, 20), (1, 730, 740)])
def test_rectangles(dtype, kw, kh, shape):
    img = _planes(dtype, *shape, seed=kw)
    x = torch.from_numpy(img).cuda()
    got = median_filter_rect(x, kw, kh).cpu().numpy()
    _sampled(img, kw, kh, got)
    assert got.tobytes() == median_filter_rect(x, kw, kh, variant=_lib.MF_VARIANT_DATA_AWARE).cpu().numpy().tobytes()


@pytest.mark.parametrize("k", [3, 5, 9, 15])
@pytest.mark.parametrize("shape", [(64, 4, 48), (4, 8, 200), (20, 30, 70)])
def test_boxes_of_few_voxels(k, shape):
    D, H, W = shape
    vol = wl.uniform_plane(D * H, W, np.uint8, seed=k).reshape(shape)
    got = median_filter_3d(torch.from_numpy(vol).cuda(), k).cpu().numpy()
    assert np.array_equal(got, oracle.median_filter_3d(vol, k))


@pytest.mark.parametrize("dtype,k,n,H,W", [(np.uint8, 13, 8, 260, 500), (np.uint8, 13, 130, 70, 250), (np.uint8, 21, 200, 60, 64),
                                           (np.uint8, 23, 16, 64, 64), (np.uint8, 35, 70, 65, 66), (np.uint8, 25, 1100, 16, 16),
                                           (np.uint16, 25, 2100, 16, 16), (np.uint16, 23, 36, 130, 130), (np.float32, 25, 900, 16, 40)])
def test_batches_of_small_images(dtype, k, n, H, W):
    img = _planes(dtype, n, H, W, seed=k)
    xs = [torch.from_numpy(a).cuda() for a in img]
    outs = [torch.empty_like(x) for x in xs]
    plan = BatchedPlan(xs, outs, [k] * n)
    plan.launch()
    got = torch.stack([o.view(torch.uint8) for o in outs]).cpu().numpy()
    plan.close()
    want = median_filter(torch.from_numpy(img).cuda(), k).cpu().numpy()
    assert got.tobytes() == want.tobytes()
    _sampled(img, k, k, want)
