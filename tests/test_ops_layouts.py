"""Layout rules of the torch entry point: which tensors take the short way
(packed planes), and that the others are treated as before."""
import numpy as np
import pytest
import torch

from paper_2507_19926_amd import ops


def test_packed():
    t = torch.zeros((3, 4, 5))
    assert ops._packed(t) and ops._packed(t[1]) and ops._packed(t[:1])
    assert not ops._packed(t[:, :, :4]) and not ops._packed(t[:, ::2]) and not ops._packed(t.transpose(1, 2))
    assert not ops._packed(torch.zeros((0, 4, 5))) and not ops._packed(torch.zeros((4, 0)))
    # strides of dimensions of size 1 count, as they do in the comparison with out
    assert not ops._packed(torch.zeros((4, 7)).as_strided((1, 4), (1, 1)))
    assert not ops._packed(torch.zeros((4, 8))[:, :1])


@pytest.mark.gpu
def test_layouts_on_gpu():
    import oracle
    a = np.random.default_rng(0).integers(0, 256, (3, 40, 50), dtype=np.uint8)
    x = torch.from_numpy(a).cuda()
    want = np.stack([oracle.median_filter(p, 5) for p in a])
    assert np.array_equal(ops.median_filter(x, 5).cpu().numpy(), want)
    assert np.array_equal(ops.median_filter(x, 5, out=torch.empty_like(x)).cpu().numpy(), want)
    assert np.array_equal(ops.median_filter(x[0], 5).cpu().numpy(), want[0])
    assert np.array_equal(ops.median_filter(x[None], 5).cpu().numpy(), want[None])
    v = x[:, 3:30, 4:41]        # pitched: out has other strides, refused as ever
    with pytest.raises(ValueError):
        ops.median_filter(v, 5)
    out = torch.empty_like(x)[:, 3:30, 4:41]
    ops.median_filter(v, 5, out=out)
    assert np.array_equal(out.cpu().numpy(), np.stack([oracle.median_filter(np.ascontiguousarray(p[3:30, 4:41]), 5) for p in a]))
    assert ops.median_filter(x[:0], 5).shape == (0, 40, 50)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        y = ops.median_filter(x, 5)
    s.synchronize()
    assert np.array_equal(y.cpu().numpy(), want)
