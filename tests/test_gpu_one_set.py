"""One set's tile map in a single launch: sizes around a tile and around 256
tiles, starting at each position of a 16-byte block, as one set and as a batch
of one; Step 1, Step 3 and the hull against the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 1021, 1024, 1025, 256 * 1024 - 1, 256 * 1024 + 2])
@pytest.mark.parametrize("phase", [0, 1, 2, 3])
def test_one_set(n, phase):
    import torch
    from paper_1405_3454_amd.api import Hull, as_u32
    x, y = inputs.disk(n + phase, 11 * n + phase)
    xt, yt = (torch.from_numpy(a).to("cuda:0")[phase:] for a in (x, y))
    x, y = x[phase:], y[phase:]
    H = Hull(0)
    slots, _ = oracle.extremes(x, y, 0)
    got = H.extremes(xt, yt)
    got = got[0] if isinstance(got, tuple) else got
    assert np.array_equal(as_u32(got), slots)
    surv = oracle.discard(x, y, oracle.polygon(x, y, slots))
    assert np.array_equal(as_u32(H.discard(xt, yt, got)), surv)
    want = oracle.hull_subset(x, y, surv)
    assert np.array_equal(as_u32(H.compute(xt, yt)), want)
    hull, ho = H.compute_batched(xt, yt, torch.tensor([0, n], dtype=torch.int64, device="cuda:0"))
    assert np.array_equal(as_u32(hull)[: int(ho[1])], want)
    H.close()
