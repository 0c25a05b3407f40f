"""The sort of the hull stage by (set, x) where runs of equal x change hands:
runs of up to 256 keys (a thread), up to 4096 (a wave), up to 2^18 (a block),
longer (every block), mixed with distinct x, at counts below and above the
tile sizes.  All points go to the sort (no filter), and the hull is compared
with the oracle's.
"""
import numpy as np
import pytest

import oracle
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu


def _columns(runs, seed):
    """Points in columns: runs = [(points per column, columns)], in random order."""
    r = np.random.default_rng(seed)
    kx, ky, x = [], [], 1000
    for per, cols in runs:
        for _ in range(cols):
            kx.append(np.full(per, x))
            ky.append(r.integers(0, 1 << 24, size=per))
            x += int(r.integers(1, 200))
    kx, ky = np.concatenate(kx), np.concatenate(ky)
    p = r.permutation(len(kx))
    return inputs.to_float(kx[p]), inputs.to_float(ky[p])


CASES = [
    [(1, 4097)], [(16, 300), (17, 300)], [(4096, 3), (4097, 3), (1, 5000)], [(40000, 2), (2, 40000), (1, 1000)],
    [(255, 70), (256, 70), (257, 70), (258, 70)], [(30, 3000), (2, 9)],
    [(1 << 18, 1), ((1 << 18) + 1, 2), (300000, 1), (5, 5000)], [(700001, 1)], [(1, 20000), (3, 2500), (100, 20)],
]


@pytest.mark.parametrize("runs", CASES)
def test_columns(runs):
    import torch
    from paper_1405_3454_amd.api import Hull, as_u32
    H = Hull(0)
    x, y = _columns(runs, 5)
    xt, yt = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0")
    want = oracle.hull_subset(x, y)
    assert np.array_equal(as_u32(H.compute(xt, yt, nofilter=True)), want)
    # two sets: the same points and a square, set digits in the keys
    sx, sy = inputs.square(30000, 6)
    off = np.array([0, len(x), len(x) + len(sx)], np.int64)
    hull, ho = H.compute_batched(torch.cat([xt, torch.from_numpy(sx).to("cuda:0")]),
                                 torch.cat([yt, torch.from_numpy(sy).to("cuda:0")]),
                                 torch.from_numpy(off).to("cuda:0"), nofilter=True)
    hv, ho = as_u32(hull), ho.cpu().numpy()
    assert np.array_equal(hv[: ho[1]], want)
    assert np.array_equal(hv[ho[1]:ho[2]], oracle.hull_subset(sx, sy) + len(x))
    H.close()
