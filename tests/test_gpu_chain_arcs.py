"""Chains whose joins walk long arcs back: convex arcs of a parabola, each cut
off by one point far below its end, with arcs and sets that end inside, at and
beyond the pieces of 32 points, the chunks of 256 and the 4096 keys that a wave
takes; one set and several, as all points and as survivors; and the same with
repeated points.  Against the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu


def _arcs(n, teeth, seed, step=1):
    """n points on `teeth` equal arcs, a point far below after each; step > 1 repeats points."""
    i = np.arange(n) // step * step
    t = i / max(n, 1)
    u = t * teeth % 1.0
    kx, ky = np.rint(t * (2.0 ** 24 - 2)), np.rint(1000 + u * u * 1.4e7 + t * 1000)
    for k in range(1, teeth + 1):
        ky[min(n - 1, k * n // teeth)] = k % 2
    p = np.random.default_rng(seed).permutation(n)
    return inputs.to_float(kx[p].astype(np.int64)), inputs.to_float(ky[p].astype(np.int64))


@pytest.fixture(scope="module")
def H():
    import torch
    from paper_1405_3454_amd.api import Hull
    h = Hull(0)
    yield h
    torch.cuda.synchronize()
    h.close()


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("n", [33, 300, 1025, 2049, 8192, 8193, 70001, 400000])
@pytest.mark.parametrize("teeth,step", [(1, 1), (1, 3), (7, 1), (40, 2)])
def test_one_set(H, n, teeth, step):
    from paper_1405_3454_amd.api import as_u32
    x, y = _arcs(n, teeth, n, step)
    want = oracle.hull_subset(x, y)
    for kw in ({"nofilter": True}, {"refine": False}, {}):
        assert np.array_equal(as_u32(H.compute(_dev(x), _dev(y), **kw)), want), (n, teeth, step, kw)


@pytest.mark.parametrize("sizes", [(300,) * 2100, (2000,) * 150, (4096, 4097, 5, 4000) * 20, (30000, 9000) * 9])
@pytest.mark.parametrize("teeth", [1, 8])
def test_several(H, sizes, teeth):
    from paper_1405_3454_amd.api import as_u32
    sets = [_arcs(n, teeth, i, 1 + i % 2) for i, n in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    x, y = (np.concatenate([s[k] for s in sets]) for k in (0, 1))
    for kw in ({"nofilter": True}, {"refine": False}):
        hull, ho = H.compute_batched(_dev(x), _dev(y), _dev(off), **kw)
        hv, ho = as_u32(hull), ho.cpu().numpy()
        for i, (px, py) in enumerate(sets):
            assert np.array_equal(hv[ho[i]:ho[i + 1]], oracle.hull_subset(px, py) + off[i]), (i, sizes[i], kw)
