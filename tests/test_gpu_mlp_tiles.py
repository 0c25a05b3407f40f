"""The network's products tile by tile: every 16 x 16 tile of the scores and of
the weight gradients, and every 16 entries of the bias gradients, so that one
tile left out, repeated or misplaced shows; at batches whose products take
tiles of 32, 64 and 128 rows a block.

The reference rounds where the kernels do (bf16 weights, activations, hidden
and output gradients), in binary64 otherwise.  What is left between them is
the float32 sums, which may turn single roundings over: at most 2^-8 of a
value at each of the four roundings on the way to the first layer's gradient.
A tile's error, in its Frobenius norm, therefore stays below four times 2^-8 of
its size, taken as its own norm plus that of an average tile (sums of mixed
signs may cancel); a wrong tile is off by the size itself.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

T = 16


def _bf16(t):
    import torch
    return t.to(torch.float32).to(torch.bfloat16).double()


def _tiles(a):
    """Norms of the T x T tiles (a vector: of T entries)."""
    import torch
    a = a.reshape(a.shape[0], -1)
    r, c = -a.shape[0] % T, -a.shape[1] % T if a.shape[1] > 1 else 0
    a = torch.nn.functional.pad(a, (0, c, 0, r))
    w = T if a.shape[1] > 1 else 1
    return (a * a).reshape(a.shape[0] // T, T, a.shape[1] // w, w).sum((1, 3)).sqrt()


def _check(got, want, what):
    size = _tiles(want)
    size = size + (size * size).mean().sqrt()
    bad = _tiles(got - want) > 4 * 2.0 ** -8 * size
    assert not bad.any(), (what, bad.nonzero()[:8].tolist(), int(bad.sum()))


@pytest.mark.parametrize("B", [1, 31, 64, 65, 200, 512, 2049, 4097, 8200])
def test_every_tile(B):
    import torch
    from paper_1405_3454_amd import train
    from paper_1405_3454_amd.api import Hull
    r = np.random.default_rng(100 + B)
    p = train.init_params(7)
    shapes = ((512, 1024), (512, 512), (64, 512))
    w, bias, at = [], [], 0
    for o, i in shapes:
        p[at + o * i:at + o * i + o] = r.standard_normal(o) * 0.1
        w.append(_bf16(torch.from_numpy(p[at:at + o * i].copy()).view(o, i)))
        bias.append(torch.from_numpy(p[at + o * i:at + o * i + o].copy()).double())
        at += o * i + o
    x = torch.from_numpy(r.random((B, 1024)) * (r.random((B, 1024)) < 0.3) * 4).to(torch.bfloat16)
    d = torch.from_numpy((r.standard_normal((B, 64)) / B).astype(np.float32))
    H = Hull(0)
    H.mlp_set_params(p)
    hist = x.view(torch.int16).to("cuda:0")
    scores = H.mlp_forward(hist).cpu().double()
    grads = H.mlp_backward(hist, d.to("cuda:0")).cpu().double()
    H.close()
    x, dd = x.double(), _bf16(d)
    a1 = _bf16(torch.relu(x @ w[0].t() + bias[0]))
    a2 = _bf16(torch.relu(a1 @ w[1].t() + bias[1]))
    _check(scores, a2 @ w[2].t() + bias[2], "scores")
    d2 = _bf16(dd @ w[2]) * (a2 > 0)
    d1 = _bf16(d2 @ w[1]) * (a1 > 0)
    at = 0
    for name, g in (("W1", d1.t() @ x), ("b1", d1.sum(0)), ("W2", d2.t() @ a1), ("b2", d2.sum(0)),
                    ("W3", dd.t() @ a2), ("b3", dd.sum(0))):
        _check(grads[at:at + g.numel()].view(g.shape), g, name)
        at += g.numel()
