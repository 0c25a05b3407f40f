"""The workloads this library is timed on, through the entry points of
``paper_1405_3454_amd.api.Hull`` as a program calls them.

A case is a dict of plain values; ``path`` names the call:

  compute   one set in device memory, the whole method (``compute_into``),
            or the hull of all its points without the filter
  filter    Step 1 and Step 3 as separate calls: ``extremes`` then
            ``discard_into``
  sets      many sets in one call (``compute_batched_into``), optionally with
            the learned direction proposal
  labels    what a training loop asks per batch of sets: marginal gains of the
            64 candidate directions and the occupancy histograms
  mlp       the proposal network, forward and backward
  solid     the 3D method (``hull3_compute`` of the C interface)

Results go to buffers that the caller keeps, as long as the calls ask for
(one entry per point) and zero past the count that comes with them.

``listed()`` gives the fixed cases, ``draw(rng)`` one more of the same ranges.
"""
import ctypes
import math

import torch

from paper_1405_3454_amd import inputs, train
from paper_1405_3454_amd._lib import HULL3_SLOTS, check, lib
from paper_1405_3454_amd.api import HULL_DIRS_CUMULATIVE, HULL_DIRS_EVEN, HULL_DIRS_PAPER, Hull

DEV = "cuda:0"
KINDS = ("square", "disk", "gaussian", "annulus")
N_BINS, N_HIDDEN, N_DIRS = 1024, 512, 64

# One context per direction preset, as a serving program keeps it: contexts
# hold the device workspace and the network's weights.
_handles = {}


def _handle(preset):
    if preset not in _handles:
        h = Hull(0, preset)
        if preset == HULL_DIRS_PAPER:
            h.mlp_set_params(train.init_params(0))
        _handles[preset] = h
    return _handles[preset]


def listed():
    return [
        # the smallest request a service sees: latency and launches
        dict(name="one_1k", path="compute", kind="square", n=1_000, preset=HULL_DIRS_PAPER, nofilter=False),
        # the latency line of the benchmark
        dict(name="one_100k", path="compute", kind="disk", n=100_000, preset=HULL_DIRS_PAPER, nofilter=False),
        # an ordinary set of odd size, the other direction table, many survivors
        dict(name="one_3m", path="compute", kind="annulus", n=3_000_017, preset=HULL_DIRS_CUMULATIVE,
             nofilter=False),
        # a program that wants the survivors and not the hull; 16 even directions
        dict(name="filter_16m", path="filter", kind="disk", n=16_000_003, preset=HULL_DIRS_EVEN(4)),
        # the comparison arm without the filter: sort and chain of every point
        dict(name="all_points_8m", path="compute", kind="disk", n=1 << 23, preset=HULL_DIRS_PAPER,
             nofilter=True),
        # a small batch of small sets (clusters, contours): latency again
        dict(name="sets_64", path="sets", mix="plain", S=64, lo=500, hi=8_000, preset=HULL_DIRS_PAPER,
             learned=False),
        # the batched line of the benchmark: sizes over three decades
        dict(name="sets_4096", path="sets", mix="plain", S=4096, lo=1_000, hi=1_000_000,
             preset=HULL_DIRS_PAPER, learned=False),
        # the main line of the benchmark: one set of each kind, the largest inputs
        dict(name="sets_4x2p27", path="sets", mix="plain", S=4, lo=1 << 27, hi=1 << 27,
             preset=HULL_DIRS_PAPER, learned=False),
        # the learned proposal on the sets it is meant for
        dict(name="learned_256", path="sets", mix="mixture", S=256, lo=1 << 17, hi=1 << 17,
             preset=HULL_DIRS_PAPER, learned=True),
        # training targets of one batch
        dict(name="labels_256", path="labels", S=256, n=1 << 16),
        # the training batch size
        dict(name="mlp_512", path="mlp", B=512),
        # the 3D line of the benchmark
        dict(name="solid_16m", path="solid", kind="ball", n=1 << 24),
    ]


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi], odd as often as even."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choice(("compute", "compute", "compute", "filter", "sets", "sets", "learned", "labels", "mlp",
                       "solid"))
    preset = rng.choice((HULL_DIRS_PAPER, HULL_DIRS_CUMULATIVE, HULL_DIRS_EVEN(4)))
    kind = rng.choice(KINDS)
    if path == "compute":
        nofilter = rng.random() < 0.2
        return dict(path="compute", kind=kind, n=_log_int(rng, 1_000, 1 << (23 if nofilter else 27)),
                    preset=preset, nofilter=nofilter)
    if path == "filter":
        return dict(path="filter", kind=kind, n=_log_int(rng, 1_000, 1 << 27), preset=preset)
    if path == "sets":
        S = _log_int(rng, 2, 4096)
        lo = _log_int(rng, 500, 20_000)
        hi = _log_int(rng, lo, min(1 << 22, (1 << 28) // S))
        return dict(path="sets", mix="plain", S=S, lo=lo, hi=hi, preset=preset, learned=False)
    if path == "learned":
        n = _log_int(rng, 4_000, 1 << 17)
        return dict(path="sets", mix="mixture", S=_log_int(rng, 16, min(512, (1 << 25) // n)), lo=n, hi=n,
                    preset=HULL_DIRS_PAPER, learned=True)
    if path == "labels":
        n = _log_int(rng, 4_000, 1 << 16)
        return dict(path="labels", S=_log_int(rng, 16, 256), n=n)
    if path == "mlp":
        return dict(path="mlp", B=_log_int(rng, 16, 2048))
    kind = rng.choice(("cube", "ball", "gaussian", "shell"))
    return dict(path="solid", kind=kind, n=_log_int(rng, 10_000, 1 << (20 if kind == "shell" else 23)))


def _sets(case, seed):
    """(x, y, offsets) of a "sets" case on the device."""
    if case["mix"] == "mixture":
        S, n = case["S"], case["lo"]
        x, y = inputs.mixture_batch_torch(S, n, seed, device=DEV)
        return x, y, torch.arange(S + 1, dtype=torch.int64, device=DEV) * n
    # the set sizes go with the case (buffers are laid out once), the points with the seed
    sizes = inputs.batch_sizes(case["S"], 2024, case["lo"], case["hi"])
    if case["S"] <= len(KINDS):     # a few large sets: one of each kind
        x, y, off, _ = inputs.batch_torch(sizes, seed + 1, device=DEV, pick=lambda i: KINDS[i])
    else:
        x, y, off, _ = inputs.batch_torch(sizes, seed + 1, device=DEV)
    return x, y, off


def _mlp_inputs(case, seed):
    """Occupancy histograms (bf16 bits) of Gaussian blobs and output gradients."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    B = case["B"]
    u = (torch.arange(32, device=DEV) + 0.5) / 32
    mean = 0.25 + 0.5 * torch.rand((B, 2), generator=g, device=DEV)
    sig = 0.04 + 0.2 * torch.rand((B, 2), generator=g, device=DEV)
    dx = torch.exp(-0.5 * ((u[None] - mean[:, :1]) / sig[:, :1]) ** 2)
    dy = torch.exp(-0.5 * ((u[None] - mean[:, 1:]) / sig[:, 1:]) ** 2)
    h = (dy[:, :, None] * dx[:, None, :]).reshape(B, N_BINS)
    h = h * (0.5 + torch.rand((B, N_BINS), generator=g, device=DEV))
    h = torch.round(h / h.sum(1, keepdim=True) * 16384) * (N_BINS / 16384)
    d = torch.randn((B, N_DIRS), generator=g, device=DEV) / (B * N_DIRS)
    return h.to(torch.bfloat16).contiguous(), d


def prepare(case, seed):
    path = case["path"]
    s = dict(case, H=_handle(case.get("preset", HULL_DIRS_PAPER)))
    if path in ("compute", "filter"):
        s["x"], s["y"] = inputs.set_torch(case["kind"], case["n"], seed, device=DEV)
    elif path == "sets":
        s["x"], s["y"], s["off"] = _sets(case, seed)
        s["hoff"] = torch.zeros(case["S"] + 1, dtype=torch.int64, device=DEV)
    elif path == "labels":
        s["x"], s["y"], s["off"] = train.batch_tensors(case["S"], case["n"], seed, DEV)
    elif path == "mlp":
        h, s["d"] = _mlp_inputs(case, seed)
        s["hist"] = h.view(torch.int16)
    else:
        s["x"], s["y"], s["z"] = inputs.set3_torch(case["kind"], case["n"], seed, device=DEV)
        s["slots"] = torch.zeros(HULL3_SLOTS, dtype=torch.int32, device=DEV)
    if path in ("filter", "solid"):
        s["surv"] = torch.zeros(case["n"], dtype=torch.int32, device=DEV)
        s["n_surv"] = torch.zeros(1, dtype=torch.int64, device=DEV)
    if path in ("compute", "sets", "solid"):
        s["hull"] = torch.zeros(s["x"].numel(), dtype=torch.int32, device=DEV)
        s["h"] = torch.zeros(1, dtype=torch.int64, device=DEV)
    return s


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def run(s):
    H, path = s["H"], s["path"]
    if path == "compute":
        H.compute_into(s["x"], s["y"], s["hull"], s["h"], nofilter=s["nofilter"])
        return s["hull"], s["h"]
    if path == "filter":
        slots, vals = H.extremes(s["x"], s["y"])
        H.discard_into(s["x"], s["y"], slots, s["surv"], s["n_surv"])
        return slots, vals, s["surv"], s["n_surv"]
    if path == "sets":
        H.compute_batched_into(s["x"], s["y"], s["off"], s["hull"], s["hoff"], learned=s["learned"])
        return s["hull"], s["hoff"]
    if path == "labels":
        gain = H.labels_batched(s["x"], s["y"], s["off"])
        bits, hist = H.histogram_batched(s["x"], s["y"], s["off"])
        return gain, bits, hist
    if path == "mlp":
        return H.mlp_forward(s["hist"]), H.mlp_backward(s["hist"], s["d"])
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    check(lib().hull3_compute(H._h, _ptr(s["x"]), _ptr(s["y"]), _ptr(s["z"]), s["n"], _ptr(s["slots"]),
                              _ptr(s["surv"]), _ptr(s["n_surv"]), _ptr(s["hull"]), _ptr(s["h"]), 0, stream),
          "hull3_compute")
    return s["slots"], s["surv"], s["n_surv"], s["hull"], s["h"]


def _kept(kind, preset):
    """About what fraction of a large set the sixteen directions keep."""
    disk = {HULL_DIRS_PAPER: 0.034, HULL_DIRS_CUMULATIVE: 0.067}.get(preset, 0.026)
    return {"disk": disk, "annulus": disk / 0.19}.get(kind, 0.0)


def work(case):
    path = case["path"]
    if path in ("compute", "filter"):
        out = 4 * case["n"] * _kept(case["kind"], case["preset"]) if path == "filter" else 0
        return {"bytes": 8 * case["n"] + out, "flops": 0}
    if path == "sets":
        lo, hi = case["lo"], case["hi"]
        mean = lo if hi == lo else (hi - lo) / math.log(hi / lo)
        return {"bytes": case["S"] * (8 * mean + 16), "flops": 0}
    if path == "labels":
        return {"bytes": case["S"] * (8 * case["n"] + 4 * N_DIRS + 6 * N_BINS), "flops": 0}
    if path == "mlp":
        B, p = case["B"], N_BINS * N_HIDDEN + N_HIDDEN * N_HIDDEN + N_HIDDEN * N_DIRS
        # forward for the scores, then forward and backward (no gradient of the input)
        flops = 2 * B * (2 * p + p + N_HIDDEN * N_HIDDEN + N_HIDDEN * N_DIRS)
        return {"bytes": 2 * B * N_BINS + 8 * B * N_DIRS + 2 * p + 4 * p, "flops": flops}
    return {"bytes": 12 * case["n"], "flops": 0}


def _exact_mlp(case, seed):
    h, d = _mlp_inputs(case, seed)
    p = torch.from_numpy(train.init_params(0)).to(DEV).double()
    parts, at = [], 0
    for o, i in ((N_HIDDEN, N_BINS), (N_HIDDEN, N_HIDDEN), (N_DIRS, N_HIDDEN)):
        parts.append((p[at:at + o * i].view(o, i), p[at + o * i:at + o * i + o]))
        at += o * i + o
    (w1, b1), (w2, b2), (w3, b3) = parts
    x, d = h.double(), d.double()
    a1 = torch.relu(x @ w1.t() + b1)
    a2 = torch.relu(a1 @ w2.t() + b2)
    d2 = (d @ w3) * (a2 > 0)
    d1 = (d2 @ w2) * (a1 > 0)
    grads = (d1.t() @ x, d1.sum(0), d2.t() @ a1, d2.sum(0), d.t() @ a2, d.sum(0))
    return a2 @ w3.t() + b3, torch.cat([g.reshape(-1) for g in grads])


def _exact_extremes(case, seed):
    """The extreme values of Step 1 in 64 bits; None for the chosen indices."""
    x, y = (t.double() for t in inputs.set_torch(case["kind"], case["n"], seed, device=DEV))
    if case["preset"] == HULL_DIRS_PAPER:
        angles = (0.0, 30.0, 45.0, 60.0)
    elif case["preset"] == HULL_DIRS_CUMULATIVE:
        angles = (0.0, 30.0, 75.0, 120.0)
    else:
        angles = (0.0, 22.5, 45.0, 67.5)
    vals = []
    for a in angles:
        c, s = math.cos(math.radians(a)), math.sin(math.radians(a))
        for v in (c * x - s * y, s * x + c * y):
            vals += [v.min(), v.max()]
    return None, torch.stack(vals), None, None


def exact(case, seed):
    """Outputs that are computed numbers, in 64 bits: the network's scores and
    gradients, and Step 1's extreme values.  Everything else is indices,
    offsets and counts; the labels' fractions are counts over sizes."""
    if case["path"] == "mlp":
        return _exact_mlp(case, seed)
    if case["path"] == "filter":
        return _exact_extremes(case, seed)
    return None
