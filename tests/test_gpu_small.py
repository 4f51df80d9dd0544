"""Images around the sizes at which a call changes its kernel (8-bit k = 9 and
11, 16-bit k = 17 to 23, 32-bit k = 17 to 21 and 23), and the k = 3 strips on
images of one to a few work-groups, against the CPU oracle, bit-exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19926_amd import workloads as wl
from paper_2507_19926_amd.ops import BatchedPlan, median_filter, median_filter_3d, median_filter_rect

pytestmark = pytest.mark.gpu


def _img(dt, H, W, seed):
    return wl.float_specials_plane(H, W, seed) if dt == np.float32 else wl.uniform_plane(H, W, dt, seed)


@pytest.mark.parametrize("dtype,k,line", [(np.uint8, 9, 1 << 18), (np.uint8, 11, 1 << 20), (np.uint16, 17, 1 << 17),
                                          (np.uint16, 19, 1 << 18), (np.uint16, 21, 1 << 17), (np.uint16, 21, 1 << 20),
                                          (np.uint16, 23, 1 << 17), (np.uint32, 19, 1 << 16), (np.float32, 17, 1 << 16),
                                          (np.float32, 21, 1 << 17), (np.float32, 23, 1 << 17)])
def test_both_sides_of_a_line(dtype, k, line):
    W = 509
    for H in (line // W, line // W + 1):
        img = _img(dtype, H, W, seed=k)
        got = median_filter(torch.from_numpy(img).cuda(), k).cpu().numpy()
        g = np.random.default_rng(k)
        ys, xs = g.integers(0, H, 4000), g.integers(0, W, 4000)
        assert got[ys, xs].tobytes() == oracle.median_points(img, k, ys, xs).tobytes(), (H, W)
    tiny = _img(dtype, 33, 41, seed=k)
    assert median_filter(torch.from_numpy(tiny).cuda(), k).cpu().numpy().tobytes() == oracle.median_filter(tiny, k).tobytes()


def test_rectangle_line():
    for H in (257, 258):
        img = _img(np.uint16, H, 509, seed=H)
        got = median_filter_rect(torch.from_numpy(img).cuda(), 21, 13).cpu().numpy()
        assert np.array_equal(got, oracle.median_filter_rect(img, 21, 13))


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16, np.uint32, np.float32])
@pytest.mark.parametrize("shape", [(1, 1), (3, 5), (4, 512), (5, 511), (15, 513), (16, 1024), (17, 1025), (33, 4100)])
def test_strips(dtype, shape):
    img = _img(dtype, *shape, seed=shape[1])
    assert median_filter(torch.from_numpy(img).cuda(), 3).cpu().numpy().tobytes() == oracle.median_filter(img, 3).tobytes()


def test_strips_of_either_chunk():
    for H in (2047, 2049):               # 8-bit images below and above 2^22 pixels
        img = wl.uniform_plane(H, 2048, np.uint8, seed=H)
        got = median_filter(torch.from_numpy(img).cuda(), 3).cpu().numpy()
        assert np.array_equal(got, oracle.median_filter(img, 3))


@pytest.mark.parametrize("k,line", [(3, 64), (5, 16), (7, 8), (9, 8)])
def test_narrow_volumes(k, line):
    for W in (line, line + 1):
        vol = wl.uniform_plane(6 * 9, W, np.uint8, seed=W).reshape(6, 9, W)
        got = median_filter_3d(torch.from_numpy(vol).cuda(), k).cpu().numpy()
        assert np.array_equal(got, oracle.median_filter_3d(vol, k)), W


@pytest.mark.parametrize("dtype,k,line", [(np.uint8, 13, 1 << 20), (np.uint8, 21, 1 << 20), (np.uint8, 23, 1 << 20),
                                          (np.uint16, 23, 1 << 19), (np.float32, 21, 1 << 19)])
def test_batches_at_a_line(dtype, k, line):
    """Two images whose pixels are together just below and at the line."""
    for H in (line // 1024 - 33, line // 1024 - 32):
        imgs = [_img(dtype, H, 1024, seed=k), _img(dtype, 32, 1024, seed=k + 1)]
        xs = [torch.from_numpy(a).cuda() for a in imgs]
        outs = [torch.empty_like(x) for x in xs]
        plan = BatchedPlan(xs, outs, [k, k])
        plan.launch()
        g = np.random.default_rng(k)
        for a, o in zip(imgs, outs):
            ys, xx = g.integers(0, a.shape[0], 2000), g.integers(0, 1024, 2000)
            assert o.cpu().numpy()[ys, xx].tobytes() == oracle.median_points(a, k, ys, xx).tobytes(), (H, a.shape)
        plan.close()
