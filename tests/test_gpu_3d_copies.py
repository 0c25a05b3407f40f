"""3D sets of many copies of few points, enough of them for the reduction
before the rounds (2^16 survivors and more), which leaves the candidates in any
order: a repeated vertex is still named by its lowest index.  Against the
oracle; one point alone, the corners of a cube and of a tetrahedron, a segment
and a flat square.
"""
import numpy as np
import pytest

from oracle import hull3d as o3
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu

CORNERS = {
    "point": [(5, 6, 7)],
    "segment": [(1, 2, 3), (11, 22, 33)],
    "square": [(0, 0, 9), (0, 8, 9), (8, 0, 9), (8, 8, 9)],
    "tetrahedron": [(0, 0, 0), (1000, 0, 0), (0, 1000, 0), (0, 0, 1000)],
    "cube": [(a, b, c) for a in (3, 900) for b in (3, 900) for c in (3, 900)],
}


@pytest.mark.parametrize("n", [65535, 65536, 200003])
@pytest.mark.parametrize("name", list(CORNERS))
def test_lowest_index_of_copies(name, n):
    import torch
    from paper_1405_3454_amd.api import Hull, as_u32
    c = np.array(CORNERS[name], np.int64)
    c = c[np.random.default_rng(n).integers(0, len(c), size=n)]
    p = [inputs.to_float(np.ascontiguousarray(c[:, k])) for k in range(3)]
    want = o3.compute(*p)
    H = Hull(0)
    for kw in ({}, {"serial": True}, {"nofilter": True}):
        hull = H.compute3(*[torch.from_numpy(v).to("cuda:0") for v in p], **kw)[2]
        assert np.array_equal(as_u32(hull), want), (kw, as_u32(hull), want)
    H.close()
