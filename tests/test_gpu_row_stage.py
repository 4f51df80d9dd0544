"""Small networks' tile kernels at the edges of their blocks, against the CPU
oracle, bit-exact: footprints just inside and just outside the image, the last
columns of a block, tile rows past the last image row, and rows stored in one
piece from and to every alignment, with nothing written between the rows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19926_amd import _lib
from paper_2507_19926_amd import workloads as wl
from paper_2507_19926_amd.ops import median_filter, median_filter_rect

pytestmark = pytest.mark.gpu

DTYPES = [np.uint8, np.uint16, np.uint32, np.float32]


def _img(dt, H, W, seed):
    return wl.float_specials_plane(H, W, seed) if dt == np.float32 else wl.uniform_plane(H, W, dt, seed)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("k", [5, 7, 9, 11])
def test_block_edges(dtype, k):
    for H, W in ((1, 255), (2, 256), (7, 257), (8, 261), (9, 511), (15, 513), (17, 520), (33, 770), (5, 1030)):
        img = _img(dtype, H, W, seed=W)
        x = torch.from_numpy(img).cuda()
        want = oracle.median_filter(img, k).tobytes()
        assert median_filter(x, k).cpu().numpy().tobytes() == want, (H, W)
        assert median_filter(x, k, variant=_lib.MF_VARIANT_OBLIVIOUS).cpu().numpy().tobytes() == want, (H, W)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("k,tile", [(3, (2, 2)), (5, (2, 2)), (5, (4, 2)), (7, (2, 2)), (7, (4, 2))])
def test_rows_of_any_alignment(dtype, k, tile):
    base = _img(dtype, 2 * 21, 801, seed=k).reshape(2, 21, 801)
    for x0, W in ((1, 530), (2, 517), (3, 258)):
        want = np.stack([oracle.median_filter(np.ascontiguousarray(p[:, x0:x0 + W]), k) for p in base])
        src = torch.from_numpy(base).cuda()
        out = src.clone()
        median_filter(src[:, :, x0:x0 + W], k, out=out[:, :, x0:x0 + W], variant=_lib.MF_VARIANT_OBLIVIOUS, tile=tile)
        got = out.cpu().numpy()
        assert np.ascontiguousarray(got[:, :, x0:x0 + W]).tobytes() == want.tobytes(), (x0, W)
        got[:, :, x0:x0 + W] = base[:, :, x0:x0 + W]
        assert got.tobytes() == base.tobytes()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kw,kh", [(5, 3), (31, 1), (1, 31), (31, 3), (1, 7), (17, 9)])
def test_rectangles(dtype, kw, kh):
    for H, W in ((3, 540), (37, 513), (40, 1100)):
        img = _img(dtype, H, W, seed=W)
        got = median_filter_rect(torch.from_numpy(img).cuda(), kw, kh).cpu().numpy()
        assert got.tobytes() == oracle.median_filter_rect(img, kw, kh).tobytes(), (H, W)
