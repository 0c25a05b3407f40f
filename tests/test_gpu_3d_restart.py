"""3D hulls that outgrow their first face room: the stage starts again with
twice the room, as often as it takes, while the round launched after the full
one must leave the mesh alone.  Against the oracle, and against the default
room, for room that is gone in the first round, in a later one, and for the
one-block insertion.
"""
import numpy as np
import pytest

from oracle import hull3d as o3
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu


def _sphere(n, every, seed):
    """Every so many points on a sphere, nearly all of them vertices; the others near it."""
    v = np.random.default_rng(seed).standard_normal((3, n))
    rad = np.where(np.arange(n) % every == 0, 0.49, 0.47)
    k = np.rint((0.5 + rad * v / np.linalg.norm(v, axis=0)) * 2.0 ** 24).astype(np.int64)
    return [inputs.to_float(c) for c in k]


def check(n, every, room, **kw):
    import torch
    from paper_1405_3454_amd._lib import check as ok, lib
    from paper_1405_3454_amd.api import Hull, as_u32
    p = _sphere(n, every, n)
    want = o3.compute(*p)
    assert len(want) > 0.9 * n / every      # about 5.6 faces are made for each
    d = [torch.from_numpy(c).to("cuda:0") for c in p]
    H = Hull(0)
    ok(lib().hull3_face_room(H._h, room), "hull3_face_room")
    print(n, room, kw, len(want), flush=True)
    hull = H.compute3(*d, **kw)[2]
    assert np.array_equal(as_u32(hull), want)
    ok(lib().hull3_face_room(H._h, 0), "hull3_face_room")      # the larger buffers stay
    assert np.array_equal(as_u32(H.compute3(*d, **kw)[2]), want)
    H.close()


# over 2^16 survivors: reduced before the rounds
@pytest.mark.parametrize("serial", [False, True])
@pytest.mark.parametrize("room", [4, 500, 4000, 12000])
def test_reduced(room, serial):
    check(120000, 40, room, serial=serial)


# fewer survivors, and no filter: the rounds start from the survivor list,
# which every turn copies anew
@pytest.mark.parametrize("kw", [{}, {"nofilter": True}, {"nofilter": True, "serial": True}])
@pytest.mark.parametrize("room", [4, 3000])
def test_from_the_list(room, kw):
    check(20000, 10, room, **kw)
