"""Several sets' candidates sorted set by set: sizes around the runs of 64 keys
that a wave ranks, the 1024 keys that a block takes one per thread, the range
that the network takes and the one that goes to the radix passes; points close
to circles, which the filter keeps, distinct and with equal points and equal x.
"""
import numpy as np
import pytest

import oracle
from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu


def _ring(n, bits, seed):
    """n points of a 2^bits grid close to a circle: few bits, many equal ones."""
    t = np.random.default_rng(seed).random(n) * 2 * np.pi
    half = 1 << (bits - 1)
    kx, ky = (np.rint(half + 0.98 * half * f(t)).astype(np.int64) << (24 - bits) for f in (np.cos, np.sin))
    return inputs.to_float(kx), inputs.to_float(ky)


@pytest.mark.parametrize("sizes", [
    (1, 63, 64, 65, 1000), (255, 256, 257, 300, 511), (1023, 1024, 1025, 2), (2048, 8192, 3, 700),
    (8193, 5, 1024, 64), (600,) * 40])
@pytest.mark.parametrize("bits", [7, 24])
def test_sets_sorted_one_by_one(sizes, bits):
    import torch
    from paper_1405_3454_amd.api import Hull, as_u32
    sets = [_ring(n, bits, 7 * i + n) for i, n in enumerate(sizes)]
    sets.append(inputs.square(300000, 3))          # too many points in all for a block per set
    off = np.concatenate([[0], np.cumsum([len(s[0]) for s in sets])]).astype(np.int64)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
           for a in (*(np.concatenate([s[k] for s in sets]) for k in (0, 1)), off)]
    H = Hull(0)
    for refine in (False, True):
        hull, ho = H.compute_batched(*dev, refine=refine)
        hv, ho = as_u32(hull), ho.cpu().numpy()
        for i, (x, y) in enumerate(sets):
            assert np.array_equal(hv[ho[i]:ho[i + 1]], oracle.hull_subset(x, y) + off[i]), (i, len(x), refine)
    H.close()
