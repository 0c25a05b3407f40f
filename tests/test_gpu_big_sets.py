"""Small batches with sets too large for one block, which several blocks share:
sizes about the parts of 4096 points, the 8192 survivors and the 16384 points
that one block takes, and the largest batch of that path; points that the
filter drops nearly all of and points on a circle, a line, one column and one
place, of which every point goes on, so that the parts' chains are merged in
LDS or by ranks and slices.  Hulls against the oracle, the candidate counts
against the general path's; new points in the same buffers, replays of a graph,
and calls of several contexts at once.
"""
import numpy as np
import pytest

import oracle
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu
G = 2.0 ** 24


def _points(kind, n, seed):
    r = np.random.default_rng(seed)
    if kind == "circle":
        t = r.random(n) * 2 * np.pi
        kx, ky = np.rint((0.5 + 0.49 * np.cos(t)) * G), np.rint((0.5 + 0.49 * np.sin(t)) * G)
    elif kind == "ring":                     # a coarse circle: repeated points, equal x
        t = r.random(n) * 2 * np.pi
        kx, ky = np.rint(2000 + 1990 * np.cos(t)), np.rint(2000 + 1990 * np.sin(t))
    elif kind == "line":
        t = r.integers(0, 1 << 20, n)
        kx, ky = 100 + 3 * t, (1 << 23) - 2 * t
    elif kind == "column":
        kx, ky = np.full(n, 77), r.integers(0, 1 << 24, n)
    elif kind == "same":
        kx, ky = np.full(n, 9), np.full(n, 8)
    elif kind == "parabola":
        t = r.random(n)
        kx, ky = np.rint(t * (G - 2)), np.rint(t * t * (G - 2))
    else:
        return inputs.DISTRIBUTIONS[kind](n, seed)
    return inputs.to_float(kx.astype(np.int64)), inputs.to_float(ky.astype(np.int64))


def _batch(sets, seed):
    pts = [_points(k, n, seed + i) for i, (k, n) in enumerate(sets)]
    off = np.concatenate([[0], np.cumsum([n for _, n in sets])]).astype(np.int64)
    x, y = (np.concatenate([p[k] for p in pts]) for k in (0, 1))
    assert 8192 < len(x) <= min(1 << 18, 8192 + 4096 * len(sets))
    want = [oracle.hull_subset(px, py) + off[i] for i, (px, py) in enumerate(pts)]
    return x, y, off, np.concatenate(want), np.concatenate([[0], np.cumsum([len(w) for w in want])])


def _dev(*arrays):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in arrays]


def _check(hull, ho, want, want_off, what):
    from paper_1405_3454_amd.api import as_u32
    assert np.array_equal(ho.cpu().numpy(), want_off), what
    assert np.array_equal(as_u32(hull)[:len(want)], want), what


TINY = [("square", 7), ("disk", 300), ("same", 4)]
SIZES = [(8193, 8192), (8200, 12288, 12289), (16384, 16385, 3), (20479, 20480, 20481), (60000,)]
KINDS = ["square", "disk", "annulus", "circle", "ring", "line", "column", "same", "parabola"]


@pytest.fixture(scope="module")
def H():
    import torch
    from paper_1405_3454_amd.api import Hull
    h = Hull(0)
    yield h
    torch.cuda.synchronize()
    h.close()


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("kind", KINDS)
def test_sizes(H, kind, sizes):
    sets = TINY + [(kind, n) for n in sizes] + TINY * 4
    for preset in (0, 1, 7):
        H.set_directions(preset)
        x, y, off, want, want_off = _batch(sets, 10 * preset)
        _check(*H.compute_batched(*_dev(x, y, off)), want, want_off, (kind, sizes, preset))
    H.set_directions(0)


@pytest.mark.parametrize("sets", [
    [("circle", 240000)] + TINY * 20, TINY * 20 + [("annulus", 250000)], [("ring", 130000), ("circle", 120000)] + TINY * 20,
    [("circle", 8193), ("annulus", 8300)] * 15 + [("disk", 100)] * 33, [("column", 90000), ("same", 70000), ("line", 80000)] + TINY * 20])
def test_largest(H, sets):
    x, y, off, want, want_off = _batch(sets, 5)
    _check(*H.compute_batched(*_dev(x, y, off)), want, want_off, sets[0])
    counts = np.array(H.candidate_counts())
    # the general path's counts: the same sets and one more, less that set's own
    bx, by = inputs.DISTRIBUTIONS["disk"](1 << 18, 5)
    H.compute(*_dev(bx, by))
    one = np.array(H.candidate_counts())
    H.compute_batched(*_dev(np.concatenate([x, bx]), np.concatenate([y, by]), np.append(off, off[-1] + len(bx))))
    assert np.array_equal(counts + one, np.array(H.candidate_counts())), sets[0]


def test_new_points_in_the_same_buffers(H):
    import torch
    for kind, n in (("circle", 30000), ("disk", 50000), ("circle", 30001), ("same", 9000), ("annulus", 40000)):
        x, y, off, want, want_off = _batch(TINY * 5 + [(kind, n)], n)
        dx, dy, do = _dev(x, y, off)
        hull, ho = H.compute_batched(dx, dy, do)
        _check(hull, ho, want, want_off, (kind, n))
        torch.cuda.synchronize()


def test_graph(H):
    import torch
    sets = TINY * 6 + [("circle", 20000), ("disk", 40000), ("annulus", 18000)]
    x, y, off, want, want_off = _batch(sets, 1)
    dx, dy, do = _dev(x, y, off)
    hull = torch.empty(len(x), dtype=torch.int32, device="cuda:0")
    ho = torch.empty(len(off), dtype=torch.int64, device="cuda:0")
    H.graph_capture(dx, dy, do, hull, ho)
    for seed in (1, 2, 3, 4):
        x, y, off, want, want_off = _batch(sets, seed)
        for d, a in ((dx, x), (dy, y)):
            d.copy_(torch.from_numpy(a))
        hull.fill_(-1)
        H.graph_launch()
        torch.cuda.synchronize()
        _check(hull, ho, want, want_off, seed)
        _check(*H.compute_batched(dx, dy, do), want, want_off, seed)


def test_several_contexts_at_once():
    import torch
    from paper_1405_3454_amd.api import Hull
    jobs = []
    for c in range(4):
        b = _batch(TINY * 15 + [("circle" if c % 2 else "annulus", 150000 + 1000 * c)], 50 + c)
        dx, dy, do = _dev(*b[:3])
        h = Hull(0)
        hull, ho = h.compute_batched(dx, dy, do)
        jobs.append((h, torch.cuda.Stream(), dx, dy, do, hull.new_empty(len(b[0])), torch.empty_like(ho), b))
    torch.cuda.synchronize()
    for _ in range(5):
        for h, st, dx, dy, do, hull, ho, _b in jobs:
            h.compute_batched_into(dx, dy, do, hull, ho, stream=st)
    torch.cuda.synchronize()
    for h, _st, _x, _y, _o, hull, ho, b in jobs:
        _check(hull, ho, b[3], b[4], len(b[0]))
        h.close()
