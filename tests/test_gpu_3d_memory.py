"""Device memory of a 3D call with millions of survivors: the reduction before
the rounds works in the workspace, and the hull stage's own buffers are sized
from what it leaves, so a call takes less beyond the workspace than the 36
bytes a survivor that a separate buffer would.
"""
import numpy as np
import pytest

from paper_1405_3454_amd import inputs

pytestmark = pytest.mark.gpu


def test_reduction_needs_no_memory_of_its_own():
    import torch
    from paper_1405_3454_amd.api import Hull
    d = [torch.from_numpy(c).to("cuda:0") for c in inputs.shell3(1 << 23, 3)]
    H = Hull(0)
    H.compute(d[0], d[1])                     # the workspace for this many points
    out = H.compute3(d[0][:1000].clone(), d[1][:1000].clone(), d[2][:1000].clone())
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    held = torch.cuda.memory_reserved()
    out = H.compute3(*d)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0] - (torch.cuda.memory_reserved() - held)
    survivors = out[1].numel()
    print("survivors", survivors, "bytes", used, flush=True)
    assert survivors > 1 << 21
    assert used < 36 * survivors
    H.close()
