"""Model of the sliding-histogram search (the walk of a wave's lanes from one
median's bin to the next): it ends at the median, and every counter that it
reads lies inside the kernel's counters or the room left around them."""
import os
import re

import numpy as np
import pytest

_HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_19926_amd", "csrc",
                       "mf_hist_kernel.h")
BINS, BIN_BYTES = 256, 256


def _constant(name):
    with open(_HEADER) as f:
        return int(re.search(r"constexpr uint32_t %s = (\d+);" % name, f.read()).group(1))


def _walk(hist, start, rank):
    """Bins of the medians of a wave's lanes, and the first and last bin read:
    hist (lanes, 256) counts, start the bin of each lane's last median, rank the
    number of values below its next one. All lanes probe while any walks."""
    lanes = len(hist)
    below = np.array([hist[i, :start[i]].sum() for i in range(lanes)])
    n = rank - below
    step = np.where(n < 0, -1, 1)
    at = np.where(n < 0, start - 1, start)
    n = np.where(n < 0, ~n, n)
    first, last = BINS, -1
    probe = 4
    while True:
        walks = False
        for i in range(lanes):
            found = False
            for j in range(probe):
                b = at[i] + step[i] * j
                first, last = min(first, b), max(last, b)
                if not found:
                    count = hist[i, b] if 0 <= b < BINS else 0
                    if n[i] < count:
                        found, to = True, b
                    else:
                        n[i] -= count
            if found:
                at[i] = to
            else:
                at[i] += step[i] * probe
                walks = True
        if not walks:
            return at, first, last
        probe = 8


def _cases():
    g = np.random.default_rng(7)
    for lanes in (1, 64):
        for size in (9, 169, 5625):
            yield np.stack([np.bincount(g.integers(0, 256, size), minlength=256) for _ in range(lanes)])
            # dark, bright and two-valued windows beside each other
            lo = np.stack([np.bincount(g.integers(0, 2, size) * (255 if i % 2 else 0) if i % 4 < 2 else
                                       g.integers(0, 3, size) + (253 if i % 2 else 0), minlength=256)
                           for i in range(lanes)])
            yield lo


def test_walk_ends_at_the_median_inside_the_counters():
    pad = _constant("kPad")
    assert _constant("kCounters") == BINS * BIN_BYTES
    g = np.random.default_rng(3)
    reach = [0, 0]
    for hist in _cases():
        lanes = len(hist)
        size = int(hist[0].sum())
        rank = np.full(lanes, (size - 1) // 2)
        want = np.array([np.searchsorted(np.cumsum(h), (size - 1) // 2, side="right") for h in hist])
        for start in (np.zeros(lanes, int), np.full(lanes, 255), g.integers(0, 256, lanes), want):
            got, first, last = _walk(hist, start.copy(), rank)
            assert np.array_equal(got, want)
            assert pad + first * BIN_BYTES >= 0
            assert last * BIN_BYTES + BIN_BYTES <= BINS * BIN_BYTES + pad
            reach = [min(reach[0], first), max(reach[1], last)]
    assert reach == [-7, 262]           # the cases do go to either limit


@pytest.mark.parametrize("bins", [-7, 262])
def test_room_holds_the_farthest_bin(bins):
    pad = _constant("kPad")
    lo = pad + bins * BIN_BYTES
    assert 0 <= lo and lo + BIN_BYTES <= 2 * pad + BINS * BIN_BYTES
