"""Ranked sliding-histogram form (16- and 32-bit data from the window where the
networks end on, and rectangular windows without a network) against the CPU
oracle, bit-exact: region edges, ties of every multiplicity, the largest value
(which the sort's fillers share), NaNs and signed zeros, pitched rows, planes,
the batched form and stream capture."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19926_amd import _lib
from paper_2507_19926_amd import workloads as wl
from paper_2507_19926_amd.ops import BatchedPlan, median_filter, median_filter_rect

pytestmark = pytest.mark.gpu
DTYPES = (np.uint16, np.uint32, np.float32)


def _images(dt, H, W, seed):
    yield wl.float_specials_plane(H, W, seed) if dt == np.float32 else wl.uniform_plane(H, W, dt, seed)
    two = wl.tie_heavy_plane(H, W, np.uint8, levels=2, seed=seed).astype(bool)
    top = np.uint32(0x7FFFFFFF).view(np.float32) if dt == np.float32 else np.iinfo(dt).max   # largest key
    yield np.where(two, np.full((H, W), top, dt), np.zeros((H, W), dt))
    yield np.full((H, W), top, dt)
    yield (wl.rgb30_planes(H=H, W=W, seed=seed)[2].astype(dt) * dt(3))       # a few hundred levels
    yield np.where(two, wl.uniform_plane(H, W, np.uint16, seed) % 16, 9).astype(dt)


def _check(img, kw, kh, got):
    want = oracle.median_filter_rect(img, kw, kh) if kw != kh else oracle.median_filter(img, kw)
    assert got.tobytes() == want.tobytes(), (img.dtype, kw, kh, img.shape)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("k", list(range(19, 76, 4)) + [21, 25, 33, 73])
def test_windows(k, dtype):
    for img in _images(dtype, 67 + k // 2, 150 + k, seed=k):
        x = torch.from_numpy(img).cuda()
        _check(img, k, k, median_filter(x, k).cpu().numpy())


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape", [(1, 1), (1, 300), (300, 1), (2, 3), (8, 127), (9, 128), (63, 129), (64, 64), (65, 257)])
def test_region_edges(shape, dtype):
    for k in (25, 75):
        for img in _images(dtype, *shape, seed=shape[1]):
            _check(img, k, k, median_filter(torch.from_numpy(img).cuda(), k).cpu().numpy())


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kw,kh", [(3, 19), (19, 3), (19, 5), (21, 13), (13, 21), (31, 29), (29, 31), (31, 11)])
def test_rectangular(kw, kh, dtype):
    for img in _images(dtype, 70, 277, seed=kw * 64 + kh):
        _check(img, kw, kh, median_filter_rect(torch.from_numpy(img).cuda(), kw, kh).cpu().numpy())


@pytest.mark.parametrize("dtype", [np.uint16, np.float32])
def test_pitched_planes(dtype):
    """Rows and planes with gaps; nothing is written between the rows."""
    base = next(_images(dtype, 3 * 90, 400, seed=4)).reshape(3, 90, 400)
    buf = torch.from_numpy(base).cuda()
    fill = np.full(base.shape, 77, dtype)
    out = torch.from_numpy(fill).cuda()
    median_filter(buf[:, 3:87, 5:338], 27, out=out[:, 3:87, 5:338])
    got = out.cpu().numpy()
    for p in range(3):
        want = fill[p].copy()
        want[3:87, 5:338] = oracle.median_filter(np.ascontiguousarray(base[p, 3:87, 5:338]), 27)
        assert got[p].tobytes() == want.tobytes()


@pytest.mark.parametrize("k", [21, 31, 33, 51, 75])
@pytest.mark.parametrize("dtype", [np.uint32, np.float32])
def test_tall_regions(k, dtype):
    """32-bit images large enough that the launch takes regions of more than
    64 rows (where the window leaves room for them), the last one ragged."""
    img = next(_images(dtype, 1211, 2100, seed=k))
    got = median_filter(torch.from_numpy(img).cuda(), k).cpu().numpy()
    g = np.random.default_rng(k)
    ys = np.concatenate([g.integers(0, 1211, 1500), np.arange(1211), np.full(64, 1210)])
    xs = np.concatenate([g.integers(0, 2100, 1500), np.full(1211, 2099), g.integers(0, 2100, 64)])
    assert got[ys, xs].tobytes() == oracle.median_points(img, k, ys, xs).tobytes()


def test_many_regions_sampled():
    """Several rounds of regions over the chip, in strips of the rows the
    launch chooses, against sampled pixels of the oracle."""
    img = wl.uniform_plane(2300, 3100, np.float32, seed=8)
    got = median_filter(torch.from_numpy(img).cuda(), 31).cpu().numpy()
    g = np.random.default_rng(1)
    ys, xs = g.integers(0, 2300, 3000), g.integers(0, 3100, 3000)
    assert np.array_equal(got[ys, xs], oracle.median_points(img, 31, ys, xs))


@pytest.mark.parametrize("dtype", [np.uint16, np.float32])
def test_ragged_regions(dtype):
    """Regions whose columns end in their first half and whose rows do not
    fill the threads' share, many of them at once: no thread may take the
    intermediate result of an output that another has finished."""
    for H, W in ((1003, 128 * 7 + 5), (517, 128 * 9 + 60), (65, 128 * 30 + 1), (301, 33)):
        img = next(_images(dtype, H, W, seed=H))
        x = torch.from_numpy(img).cuda()
        a = median_filter(x, 23, variant=_lib.MF_VARIANT_DATA_AWARE, form=3)
        b = median_filter(x, 23, variant=_lib.MF_VARIANT_DATA_AWARE)
        assert a.cpu().numpy().tobytes() == b.cpu().numpy().tobytes(), (H, W)


def test_batched_and_graph():
    shapes = [(64, 64, 25, np.uint16), (63, 257, 25, np.uint16), (200, 128, 27, np.float32), (65, 130, 27, np.uint32),
              (1, 5, 25, np.uint16), (40, 300, 25, np.uint8)]
    imgs = [next(_images(dt, h, w, seed=h + w)) if dt != np.uint8 else wl.uniform_plane(h, w, dt, 3)
            for h, w, _, dt in shapes]
    xs = [torch.from_numpy(a).cuda() for a in imgs]
    outs = [torch.empty_like(x) for x in xs]
    plan = BatchedPlan(xs, outs, [k for _, _, k, _ in shapes])
    for _ in range(3):
        plan.launch()
        for a, o, (_, _, k, _) in zip(imgs, outs, shapes):
            _check(a, k, k, o.cpu().numpy())
    plan.close()
    x, y = xs[2], torch.empty_like(xs[2])
    median_filter(x, 27, out=y)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        median_filter(x, 27, out=y)
    for r in range(3):
        x.copy_(torch.from_numpy(np.roll(imgs[2], r + 1, axis=0)))
        g.replay()
        torch.cuda.synchronize()
        _check(np.roll(imgs[2], r + 1, axis=0), 27, 27, y.cpu().numpy())


@pytest.mark.parametrize("dtype", DTYPES)
def test_variants_agree(dtype):
    code = {np.uint16: _lib.MF_U16, np.uint32: _lib.MF_U32, np.float32: _lib.MF_F32}[dtype]
    img = next(_images(dtype, 131, 517, seed=9))
    x = torch.from_numpy(img).cuda()
    for k in (23, 41):
        v, tw, th, g, f, _ = _lib.query_options(code, k)
        assert f == 3
        a = median_filter(x, k, variant=v, tile=(tw, th), group=g, form=f)
        b = median_filter(x, k, variant=_lib.MF_VARIANT_DATA_AWARE)
        assert a.cpu().numpy().tobytes() == b.cpu().numpy().tobytes()
