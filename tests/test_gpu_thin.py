"""Thin sets whose extreme slots are two points (the filter polygon is a
segment): the refinement rounds work on both sides of it, on the general path
and the one-block path.  Hulls against the oracle; hardly any candidates are
left where the set has few hull vertices, and all survive the filter.
"""
import numpy as np
import pytest

import oracle
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu


def _thin(n, seed, width):
    """Points along a diagonal segment, `width` grid units across it, that
    no fixed direction sees past the segment's ends."""
    r = np.random.default_rng(seed)
    t = r.integers(0, 1 << 22, size=n)
    w = r.integers(-width, width + 1, size=n) * (np.minimum(t, (1 << 22) - t) > 1 << 12)
    kx, ky = 1000 + 3 * t - w, 2000 + 1 * t + 3 * w
    kx[:2], ky[:2] = (1000, 1000 + 3 * (1 << 22)), (2000, 2000 + (1 << 22))
    return inputs.to_float(kx), inputs.to_float(ky)


@pytest.mark.parametrize("n", [500, 8000, 20000, 300001])
@pytest.mark.parametrize("width", [0, 1, 200])
def test_thin(n, width):
    import torch
    from paper_1405_3454_amd.api import Hull, as_u32
    H = Hull(0)
    x, y = _thin(n, n + width, width)
    slots, _ = oracle.extremes(x, y)
    assert len(oracle.polygon(x, y, slots)) == 2
    xt, yt = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0")
    want = oracle.hull_subset(x, y)
    assert np.array_equal(as_u32(H.compute(xt, yt)), want)
    counts = H.candidate_counts()
    assert counts[0] == n
    if width == 200:
        assert counts[-1] < n // 4
    # several sets: the thin one, one point, the thin one again
    off = np.array([0, n, n + 1, 2 * n + 1], np.int64)
    xb, yb = torch.cat([xt, xt[:1], xt]), torch.cat([yt, yt[:1], yt])
    hull, ho = H.compute_batched(xb, yb, torch.from_numpy(off).to("cuda:0"))
    hv, ho = as_u32(hull), ho.cpu().numpy()
    assert np.array_equal(hv[: ho[1]], want)
    assert list(hv[ho[1]:ho[2]]) == [n]
    assert np.array_equal(hv[ho[2]:ho[3]], want + n + 1)
    H.close()
