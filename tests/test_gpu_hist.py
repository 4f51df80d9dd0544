"""Sliding-histogram form (8-bit data: square windows from k = 13 on, and
rectangular windows without a network) against the CPU oracle, bit-exact: one
and two counter words, edges of the column blocks and of the row strips,
windows beyond the image, 3-D boxes, the fullest counters (constant and two-valued
images), pitched rows, planes, the batched form and stream capture."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19926_amd import _lib
from paper_2507_19926_amd import workloads as wl
from paper_2507_19926_amd.ops import BatchedPlan, median_filter, median_filter_3d, median_filter_rect

pytestmark = pytest.mark.gpu


def _images(H, W, seed):
    two = wl.tie_heavy_plane(H, W, np.uint8, levels=2, seed=seed) * 255
    return {"noise": wl.uniform_plane(H, W, np.uint8, seed=seed), "two": two.astype(np.uint8),
            "full": np.full((H, W), 255, np.uint8), "zero": np.zeros((H, W), np.uint8),
            "rgb": wl.rgb30_planes(H=H, W=W, seed=seed)[2]}


def _check(img, kw, kh, got):
    want = oracle.median_filter_rect(img, kw, kh) if kw != kh else oracle.median_filter(img, kw)
    assert np.array_equal(got, want), int((got != want).sum())


@pytest.mark.parametrize("k", list(range(13, 76, 2)))
def test_every_k(k):
    for name, img in _images(37 + k // 2, 150 + k, seed=k).items():
        x = torch.from_numpy(img).cuda()
        _check(img, k, k, median_filter(x, k).cpu().numpy())
        _check(img, k, k, median_filter(x, k, variant=_lib.MF_VARIANT_DATA_AWARE, tile=(1, 1), group=1,
                                        form=3).cpu().numpy())


@pytest.mark.parametrize("k", [15, 17, 75])
@pytest.mark.parametrize("shape", [(1, 1), (1, 300), (300, 1), (2, 3), (3, 127), (5, 128), (4, 129), (7, 255),
                                   (6, 256), (9, 257), (64, 131), (65, 64), (67, 63)])
def test_block_edges(k, shape):
    for name, img in _images(*shape, seed=shape[1]).items():
        _check(img, k, k, median_filter(torch.from_numpy(img).cuda(), k).cpu().numpy())


@pytest.mark.parametrize("kw,kh", [(3, 19), (19, 3), (19, 5), (21, 13), (31, 15), (19, 15), (13, 21), (31, 29), (3, 29),
                                   (29, 31), (25, 11)])
def test_rectangular(kw, kh):
    for name, img in _images(61, 277, seed=kw * 64 + kh).items():
        _check(img, kw, kh, median_filter_rect(torch.from_numpy(img).cuda(), kw, kh).cpu().numpy())


@pytest.mark.parametrize("k", [13, 35])
def test_pitched_planes_in_place_of_a_view(k):
    """Rows and planes with gaps, source and destination at odd addresses;
    nothing is written between the rows."""
    base = wl.uniform_plane(3 * 50, 400, np.uint8, seed=k).reshape(3, 50, 400)
    buf = torch.from_numpy(base).cuda()
    out = torch.full_like(buf, 77)
    x, y = buf[:, 3:47, 5:338], out[:, 3:47, 5:338]
    median_filter(x, k, out=y)
    got = out.cpu().numpy()
    for p in range(3):
        want = np.full((50, 400), 77, np.uint8)
        want[3:47, 5:338] = oracle.median_filter(np.ascontiguousarray(base[p, 3:47, 5:338]), k)
        assert np.array_equal(got[p], want)


def test_tall_image_several_strips_and_stream():
    img = wl.uniform_plane(3000, 70, np.uint8, seed=3)
    s = torch.cuda.Stream()
    x = torch.from_numpy(img).cuda()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        y = median_filter(x, 21)
    s.synchronize()
    _check(img, 21, 21, y.cpu().numpy())


def test_batched_and_graph():
    """Images of every size class in one plan, one launch and replays of a
    captured graph of plain calls, eager work between them."""
    shapes = [(64, 64, 13), (63, 257, 15), (200, 128, 17), (129, 130, 25), (31, 300, 25), (1, 5, 13)]
    imgs = [wl.uniform_plane(h, w, np.uint8, seed=h + w) for h, w, _ in shapes]
    xs = [torch.from_numpy(a).cuda() for a in imgs]
    outs = [torch.empty_like(x) for x in xs]
    plan = BatchedPlan(xs, outs, [k for _, _, k in shapes])
    for _ in range(3):
        for o in outs:
            o.zero_()
        plan.launch()
        for a, o, (_, _, k) in zip(imgs, outs, shapes):
            _check(a, k, k, o.cpu().numpy())
    plan.close()
    x, y = xs[3], torch.empty_like(xs[3])
    median_filter(x, 25, out=y)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        median_filter(x, 25, out=y)
    for r in range(3):
        x.copy_(torch.from_numpy(np.roll(imgs[3], r + 1, axis=0)))
        g.replay()
        torch.cuda.synchronize()
        _check(np.roll(imgs[3], r + 1, axis=0), 25, 25, y.cpu().numpy())


@pytest.mark.parametrize("k", [3, 5, 9, 15])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 17, 129), (9, 1, 23), (7, 8, 1), (5, 33, 260)])
def test_boxes(k, shape):
    D, H, W = shape
    for seed in range(5):
        vol = np.stack([list(_images(H, W, seed=z).values())[seed] for z in range(D)])
        got = median_filter_3d(torch.from_numpy(vol).cuda(), k).cpu().numpy()
        assert np.array_equal(got, oracle.median_filter_3d(vol, k)), seed
