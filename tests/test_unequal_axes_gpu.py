"""Gradients where one axis has many more frequencies than the other, so that the two contractions of a launch have K loops
of very different length: either may be the longer one, with few and with many blocks, and (bf16) with workgroups of both sizes.

The problem with its axes exchanged has the same contractions in the other order: its gy is this one's gx to the bit.  Against
the FP64 oracle at sampled blocks; bars: the precisions' own."""
import sys

import numpy as np
import pytest

import oracle
from workloads import make_random

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-10, "fp32": 1e-5, "bf16x3": 1e-3, "bf16mix": 1e-3, "bf16": 3e-2}


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("prec,n,Mu,Mp", [("fp64", 90, 700, 40), ("fp64", 9000, 900, 63), ("fp32", 300, 1100, 30),
                                          ("fp32", 40000, 1030, 100), ("bf16x3", 30344, 1200, 132), ("bf16x3", 700, 60, 1500),
                                          ("bf16", 33100, 1300, 17), ("bf16mix", 53629, 1175, 33), ("bf16mix", 13200, 257, 1600)])
def test_either_axis_the_longer_one(prec, n, Mu, Mp):
    W, H = 700.0, 500.0
    wl = make_random(n, W, H, Mu, Mp, seed=n)
    print(f"[unequal] {prec} n={n} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n)
    a = rng.standard_normal((Mu, Mp)) / (1.0 + np.arange(Mu)[:, None] ** 2 + np.arange(Mp)[None, :] ** 2)
    x, y, w, h = (torch.as_tensor(np.ascontiguousarray(v), device="cuda:0") for v in wl.arrays())
    at = torch.as_tensor(a, device="cuda:0")
    gx, gy = pp.field(x, y, w, h, at, W=W, H=H, precision=prec)
    hy, hx = pp.field(y, x, h, w, at.t().contiguous(), W=H, H=W, precision=prec)
    assert torch.equal(gx, hx) and torch.equal(gy, hy)
    idx = np.unique(np.concatenate([[0, n - 1, n - 2], rng.integers(0, n, 150)]))
    gxo, gyo = oracle.grad_sampled(W, H, *wl.arrays(), a, idx)
    assert rel(gx.cpu().numpy()[idx], gxo) <= TOL[prec] and rel(gy.cpu().numpy()[idx], gyo) <= TOL[prec]
