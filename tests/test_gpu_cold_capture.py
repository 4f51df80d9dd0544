"""The first call of a process captured into a graph: whatever kernel it takes,
it has nothing to prepare that a capture does not let pass. Each case is a
process of its own."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

_ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_CODE = r"""
import sys
import torch
from paper_2507_19926_amd import _lib
from paper_2507_19926_amd.ops import median_filter, median_filter_rect
dtype, H, W, kw, kh = getattr(torch, sys.argv[1]), *map(int, sys.argv[2:])
g = torch.Generator(device="cuda").manual_seed(1)
def image():
    v = torch.randint(0, 200, (H, W), generator=g, device="cuda")
    return v.to(torch.int16).view(torch.uint16) if dtype == torch.uint16 else v.to(dtype)
x = image()
out = torch.empty_like(x)
def call(y, **kw_):
    if kw == kh:
        median_filter(x, kw, out=y, **kw_)
    else:
        median_filter_rect(x, kw, kh, out=y, **kw_)
torch.cuda.synchronize()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph):
    call(out)
for _ in range(3):
    x.copy_(image())
    graph.replay()
    torch.cuda.synchronize()
    want = torch.empty_like(x)
    call(want)                                                  # the same choice, not captured
    general = torch.empty_like(x)
    call(general, variant=_lib.MF_VARIANT_DATA_AWARE)           # the schedule
    assert out.cpu().numpy().tobytes() == want.cpu().numpy().tobytes() == general.cpu().numpy().tobytes()
print("ok")
"""


@pytest.mark.parametrize("dtype,H,W,kw,kh", [
    ("uint16", 64, 96, 17, 17), ("uint16", 64, 96, 19, 19), ("float32", 64, 96, 17, 17),    # small: the schedule
    ("float32", 96, 64, 25, 25),
    ("uint8", 64, 96, 13, 13), ("float32", 400, 700, 21, 21), ("uint8", 64, 96, 21, 13),    # histograms
    ("uint8", 64, 96, 7, 7), ("float32", 64, 96, 5, 5)])                                    # networks
def test_first_call_captured(dtype, H, W, kw, kh):
    r = subprocess.run([sys.executable, "-c", _CODE, dtype] + [str(v) for v in (H, W, kw, kh)], cwd=_ROOT,
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stderr[-2000:]
