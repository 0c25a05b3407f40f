"""The one-block-per-set path at the sizes where its storage changes: empty
and tiny sets, the side-by-side LDS lists (2048), the LDS lists (8192), more
survivors and more candidates than LDS holds (points on a circle: nothing is
discarded), ties and duplicates, sets on a line; one set, batches, with and
without the filter and the refinement.  Hulls and candidate counts against
the oracle and, above the path's sizes, the general path on the same points.
"""
import numpy as np
import pytest

import oracle
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu


def _circle(n, seed):
    """About n distinct grid points close to a circle (most are hull vertices)."""
    t = np.sort(np.random.default_rng(seed).random(n)) * 2 * np.pi
    kx = np.rint((0.5 + 0.49 * np.cos(t)) * 2.0 ** 24).astype(np.int64)
    ky = np.rint((0.5 + 0.49 * np.sin(t)) * 2.0 ** 24).astype(np.int64)
    return inputs.to_float(kx), inputs.to_float(ky)


def _line(n, seed):
    t = np.random.default_rng(seed).integers(0, 3000, size=n)
    return inputs.to_float(100 + 3 * t), inputs.to_float(7000 - 2 * t)


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
    return torch.from_numpy(a).to("cuda:0")


ONE = [("square", 0), ("square", 1), ("square", 2), ("square", 3), ("disk", 63), ("disk", 257), ("annulus", 1000),
       ("annulus", 4095), ("annulus", 8191), ("gaussian", 8192), ("circle", 2048), ("circle", 2049),
       ("circle", 8192), ("circle", 8193), ("line", 900), ("lattice", 3000), ("same", 500)]


def _set(kind, n, seed):
    if kind == "circle":
        return _circle(n, seed)
    if kind == "line":
        return _line(n, seed)
    if kind == "lattice":
        return inputs.small_grid(n, 12, seed)
    if kind == "same":
        return inputs.small_grid(n, 1, seed)
    return inputs.DISTRIBUTIONS[kind](n, seed)


@pytest.mark.parametrize("kind,n", ONE)
@pytest.mark.parametrize("preset", [0, 1, 2, 7])
def test_one_set(H, kind, n, preset):
    from paper_1405_3454_amd.api import as_u32
    x, y = _set(kind, n, 3 + n)
    H.set_directions(preset)
    want = oracle.hull_subset(x, y)
    for kw in ({}, {"refine": False}, {"nofilter": True}):
        got = as_u32(H.compute(_dev(x), _dev(y), **kw))
        assert np.array_equal(got, want), (kind, n, preset, kw)
        if kw == {"nofilter": True}:
            assert H.candidate_counts() == [n] + [-1] * 4
    H.compute(_dev(x), _dev(y))
    counts = H.candidate_counts()
    slots, _ = H.extremes(_dev(x), _dev(y))
    assert counts[0] == H.discard(_dev(x), _dev(y), slots).numel()
    assert all(0 <= b <= a for a, b in zip(counts, counts[1:]))
    H.set_directions(0)


BATCHES = [
    [("square", 10), ("square", 0), ("disk", 5000), ("line", 40), ("same", 9), ("annulus", 8193)],
    [("circle", 20000), ("annulus", 60001)] + [("square", 1 + i) for i in range(20)],
    [("circle", 8193), ("circle", 8192), ("circle", 12001), ("disk", 100000)] + [("same", 3)] * 30,
    [("disk", 20 + 4 * i) for i in range(300)],
]


@pytest.mark.parametrize("sets", BATCHES)
def test_batches(H, sets):
    from paper_1405_3454_amd.api import as_u32
    pts = [_set(k, n, 11 + i) for i, (k, n) in enumerate(sets)]
    off = np.zeros(len(pts) + 1, np.int64)
    off[1:] = np.cumsum([len(p[0]) for p in pts])
    x, y = np.concatenate([p[0] for p in pts]), np.concatenate([p[1] for p in pts])
    assert len(x) <= min(1 << 18, 8192 + 4096 * len(sets))      # one block per set
    for kw in ({}, {"refine": False}, {"nofilter": True}):
        hull, ho = H.compute_batched(_dev(x), _dev(y), _dev(off), **kw)
        hv, ho = as_u32(hull).astype(np.int64), ho.cpu().numpy()
        for s, (px, py) in enumerate(pts):
            want = oracle.hull_subset(px, py).astype(np.int64) + off[s]
            assert np.array_equal(hv[ho[s]:ho[s + 1]], want), (s, sets[s], kw)
    # the counts are the general path's: the same sets with one more that
    # takes the batch past the small path, less that set's own counts
    H.compute_batched(_dev(x), _dev(y), _dev(off))
    small = np.array(H.candidate_counts())
    bx, by = inputs.DISTRIBUTIONS["disk"](1 << 18, 5)
    H.compute(_dev(bx), _dev(by))
    big = np.array(H.candidate_counts())
    off2 = np.append(off, off[-1] + len(bx))
    H.compute_batched(_dev(np.concatenate([x, bx])), _dev(np.concatenate([y, by])), _dev(off2))
    both = np.array(H.candidate_counts())
    assert np.array_equal(small + big, both), (small, big, both)
