"""Ranked sliding histograms, asked for by form (a call of few pixels takes the
schedule by itself) or, for rectangles and batches, on enough pixels to be the
library's choice: every window against the schedule, and against the CPU oracle,
bit-exact, with ties of every multiplicity, the largest key (which the sort's fillers
share), NaNs and signed zeros, pitched rows, planes and stream capture."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19926_amd import _lib
from paper_2507_19926_amd import workloads as wl
from paper_2507_19926_amd.ops import BatchedPlan, median_filter, median_filter_rect

pytestmark = pytest.mark.gpu
DTYPES = (np.uint16, np.uint32, np.float32)
SCHEDULE = dict(variant=_lib.MF_VARIANT_DATA_AWARE)
RANKED = dict(variant=_lib.MF_VARIANT_DATA_AWARE, form=3)


def _images(dt, H, W, seed):
    yield wl.float_specials_plane(H, W, seed) if dt == np.float32 else wl.uniform_plane(H, W, dt, seed)
    two = wl.tie_heavy_plane(H, W, np.uint8, levels=2, seed=seed).astype(bool)
    top = np.uint32(0x7FFFFFFF).view(np.float32) if dt == np.float32 else np.iinfo(dt).max   # largest key
    yield np.where(two, np.full((H, W), top, dt), np.zeros((H, W), dt))
    yield np.full((H, W), top, dt)
    yield (wl.rgb30_planes(H=H, W=W, seed=seed)[2].astype(dt) * dt(3))       # a few hundred levels
    yield np.where(two, wl.uniform_plane(H, W, np.uint16, seed) % 16, 9).astype(dt)


def _kernels(call):
    """Names of the kernels that a call launches."""
    call()
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return " ".join(e.name for e in p.events())


def _bytes(t):
    return t.cpu().numpy().tobytes()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("k", list(range(23, 76, 2)))
def test_windows(k, dtype):
    for i, img in enumerate(_images(dtype, 67 + k // 2, 150 + k, seed=k)):
        x = torch.from_numpy(img).cuda()
        got = _bytes(median_filter(x, k, **RANKED))
        assert got == _bytes(median_filter(x, k, **SCHEDULE)), i
        if i == k % 5:
            assert got == oracle.median_filter(img, k).tobytes(), i


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape", [(1, 1), (1, 300), (300, 1), (2, 3), (8, 127), (9, 128), (63, 129), (64, 64), (65, 257),
                                   (128, 128), (129, 127)])
def test_region_edges(shape, dtype):
    for k in (25, 75):
        for i, img in enumerate(_images(dtype, *shape, seed=shape[1])):
            got = _bytes(median_filter(torch.from_numpy(img).cuda(), k, **RANKED))
            assert got == oracle.median_filter(img, k).tobytes(), (k, i)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kw,kh", [(3, 19), (19, 3), (5, 23), (19, 5), (21, 13), (13, 21), (31, 29), (29, 31), (31, 11), (23, 17)])
def test_rectangles(kw, kh, dtype):
    """1100 columns by 520 rows: above every line of the choice."""
    for i, img in enumerate(_images(dtype, 520, 1100, seed=kw * 64 + kh)):
        x = torch.from_numpy(img).cuda()
        got = median_filter_rect(x, kw, kh)
        assert _bytes(got) == _bytes(median_filter_rect(x, kw, kh, **SCHEDULE)), i
    if kw * kh >= 200:
        assert "mf_rank_kernel" in _kernels(lambda: median_filter_rect(x, kw, kh))
    corner = img[:40, :60]
    assert got.cpu().numpy()[:40 - kh // 2, :60 - kw // 2].tobytes() == \
        oracle.median_filter_rect(corner, kw, kh)[:40 - kh // 2, :60 - kw // 2].tobytes()


@pytest.mark.parametrize("dtype", DTYPES)
def test_pitched_planes(dtype):
    """Rows and planes with gaps; nothing is written between the rows."""
    base = next(_images(dtype, 3 * 90, 400, seed=4)).reshape(3, 90, 400)
    buf = torch.from_numpy(base).cuda()
    fill = np.full(base.shape, 77, dtype)
    out = torch.from_numpy(fill).cuda()
    median_filter(buf[:, 3:87, 5:338], 27, out=out[:, 3:87, 5:338], **RANKED)
    got = out.cpu().numpy()
    for p in range(3):
        want = fill[p].copy()
        want[3:87, 5:338] = oracle.median_filter(np.ascontiguousarray(base[p, 3:87, 5:338]), 27)
        assert got[p].tobytes() == want.tobytes()


@pytest.mark.parametrize("dtype", DTYPES)
def test_capture(dtype):
    imgs = list(_images(dtype, 130, 300, seed=6))
    x = torch.from_numpy(imgs[0]).cuda()
    y = torch.empty_like(x)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        median_filter(x, 35, out=y, **RANKED)
    for img in imgs:
        x.copy_(torch.from_numpy(img))
        g.replay()
        torch.cuda.synchronize()
        assert _bytes(y) == oracle.median_filter(img, 35).tobytes()


@pytest.mark.parametrize("dtype,k", [(np.uint16, 23), (np.uint16, 51), (np.uint32, 21), (np.float32, 25), (np.float32, 75)])
def test_batches(dtype, k):
    """Images of several sizes, 2^19 pixels and more together."""
    shapes = [(700, 600), (64, 128), (65, 129), (1, 5), (300, 40), (500, 260)]
    imgs = [img for h, w in shapes for img in list(_images(dtype, h, w, seed=h + w))[:2]]
    xs = [torch.from_numpy(a).cuda() for a in imgs]
    outs = [torch.empty_like(x) for x in xs]
    plan = BatchedPlan(xs, outs, [k] * len(xs))
    assert "mf_rank_kernel" in _kernels(plan.launch)
    for _ in range(2):
        plan.launch()
        for i, (x, o) in enumerate(zip(xs, outs)):
            assert _bytes(o) == _bytes(median_filter(x, k, **SCHEDULE)), i
    plan.close()
    for a, o in zip(imgs[2:8], outs[2:8]):
        assert _bytes(o) == oracle.median_filter(a, k).tobytes()


@pytest.mark.parametrize("dtype,k,H,W", [(np.uint8, 9, 512, 512), (np.uint8, 9, 513, 512), (np.uint8, 11, 768, 512),
                                         (np.uint8, 11, 769, 512), (np.uint8, 11, 513, 513)])
def test_lines_of_8_bit_squares(dtype, k, H, W):
    img = wl.uniform_plane(H, W, dtype, seed=k)
    x = torch.from_numpy(img).cuda()
    got = median_filter(x, k)
    assert torch.equal(got, median_filter(x, k, variant=_lib.MF_VARIANT_OBLIVIOUS))
    histograms = H * ((W + 255) // 256 * 256) <= (1 << 18 if k == 9 else 3 << 17)
    assert ("mf_hist_kernel" in _kernels(lambda: median_filter(x, k))) == histograms
    g = np.random.default_rng(k)
    ys, xs = g.integers(0, H, 2000), g.integers(0, W, 2000)
    assert np.array_equal(got.cpu().numpy()[ys, xs], oracle.median_points(img, k, ys, xs))


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kw,kh,H", [(21, 13, 511), (21, 13, 512), (25, 13, 383), (25, 13, 384), (31, 29, 255), (31, 29, 256)])
def test_lines_of_rectangles(dtype, kw, kh, H):
    for i, img in enumerate(_images(dtype, H, 512, seed=H)):
        x = torch.from_numpy(img).cuda()
        assert _bytes(median_filter_rect(x, kw, kh)) == _bytes(median_filter_rect(x, kw, kh, **SCHEDULE)), i
    ranked = "mf_rank_kernel" in _kernels(lambda: median_filter_rect(x, kw, kh))
    # (16-bit data at 2^17 pixels of this shape: the schedule's estimate is the lower one)
    assert ranked == (H in (512, 384, 256) and (H, dtype) != (256, np.uint16))
