"""3D sets whose survivors are many enough for the reduction before the
rounds (2^16 and more): sets where it drops nearly all of them (ball, shell),
where the far points of few cells exist (two clusters), where thousands of
points on a sphere surround the others, and repeated points.  Against the
oracle; the survivors, which the reduction must not change, too.
"""
import numpy as np
import pytest

from oracle import hull3d as o3
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu


def _grid(v):
    return [inputs.to_float(np.clip(np.rint(c * 2.0 ** 24), 0, 2 ** 24 - 1).astype(np.int64)) for c in v]


def _sphere(n, seed):
    r = np.random.default_rng(seed)
    v = r.standard_normal((3, n))
    rad = np.where(np.arange(n) % 40 == 0, 0.49, 0.46 * r.random(n) ** 0.05)
    return _grid(0.5 + rad * v / np.linalg.norm(v, axis=0))


def _clusters(n, seed):
    """Two small balls far apart and points along a coarse octahedron."""
    r = np.random.default_rng(seed)
    v = r.standard_normal((3, n))
    v *= 0.05 * r.random(n) ** (1 / 3) / np.linalg.norm(v, axis=0)
    v[:, : n // 2] += np.array([[0.1], [0.1], [0.1]])
    v[:, n // 2:] += np.array([[0.9], [0.9], [0.8]])
    return _grid(v)


def _twice(n, seed):
    x, y, z = inputs.shell3(n // 2, seed)
    return [np.concatenate([c, c]) for c in (x, y, z)]


SETS = {"ball": lambda: inputs.ball3(400003, 1), "shell": lambda: inputs.shell3(150001, 2),
        "sphere": lambda: _sphere(200000, 3), "clusters": lambda: _clusters(500000, 4),
        "twice": lambda: _twice(160000, 5)}


@pytest.mark.parametrize("name", list(SETS))
def test_many_survivors(name):
    import torch
    from paper_1405_3454_amd.api import Hull, as_u32
    H = Hull(0)
    x, y, z = SETS[name]()
    slots, surv, hull = H.compute3(*[torch.from_numpy(np.ascontiguousarray(c)).to("cuda:0") for c in (x, y, z)])
    want, want_surv = o3.compute(x, y, z, 0, want_survivors=True)
    print(name, len(x), len(want_surv), len(want), flush=True)
    assert np.array_equal(as_u32(surv), want_surv)
    assert np.array_equal(as_u32(hull), want)
    H.close()
