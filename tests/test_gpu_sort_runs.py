"""Runs of equal x that a wave takes (33 to 256 keys) and that all blocks share
(above 2^18 keys, in parts of 2^15): lengths where either ends and where a
wave's steps and the parts end, several such runs, more parts than blocks,
among shorter runs and alone, and runs of one repeated point.  All points go to
the sort (no filter); hulls against the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu

B, P = 1 << 18, 1 << 15
CASES = [[B], [B + 1], [B + P - 1], [B + P, 3], [B + P + 1, B, 1], [B + 1] * 9 + [5000], [300 * P + 7, 2],
         [2 * B, 70, 3 * B - 1, 4097, B + 9 * P],
         [32, 33] * 100, [63, 64, 65, 66] * 40, [127, 128, 129, 1] * 30, [191, 192, 193] * 20, [256, 257] * 10,
         list(range(1, 270))]


@pytest.mark.parametrize("runs", CASES)
@pytest.mark.parametrize("same", [False, True])
def test_runs(runs, same):
    import torch
    from paper_1405_3454_amd.api import Hull, as_u32
    r = np.random.default_rng(len(runs))
    kx = np.repeat(1000 + 77 * np.arange(len(runs)), runs)
    ky = np.repeat(r.integers(0, 1 << 24, len(runs)), runs) if same else r.integers(0, 1 << 24, len(kx))
    p = r.permutation(len(kx))
    x, y = inputs.to_float(kx[p]), inputs.to_float(ky[p])
    H = Hull(0)
    got = H.compute(torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0"), nofilter=True)
    assert np.array_equal(as_u32(got), oracle.hull_subset(x, y))
    H.close()
