"""The FP32 coefficient contraction on both sides of its 256 x 256 tiles (an even number of tiles of 128 each way, at least 12 chunks
of 32 blocks a split, nearly full rounds of workgroups): sizes that end inside a tile and inside either run of a thread, and the
same sizes with fewer blocks, an odd number of tiles or rounds left half empty.

Against the FP64 oracle at sampled coefficients, the last rows and columns among them, scaled by the sum of magnitudes (bar 1e-6:
FP32 rounding of each product, 6e-8, and of the sums of at most 1600 of them), and against the FP64 path in the norm (1e-5, the
FP32 path's own bar)."""
import sys

import numpy as np
import pytest

import oracle
from workloads import make_random

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,Mu,Mp", [(49200, 500, 390), (49100, 500, 390), (49200, 512, 511), (100000, 250, 510), (100000, 250, 385),
                                     (16385, 250, 255), (4100, 500, 390), (13000, 1000, 900), (12200, 1500, 1410), (200100, 130, 129)])
def test_ragged_sizes(n, Mu, Mp):
    wl = make_random(n, 900.0, 700.0, Mu, Mp, seed=n)
    print(f"[fp32 wide] n={n} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    x, y, w, h = (torch.as_tensor(np.ascontiguousarray(v), device="cuda:0") for v in wl.arrays())
    E, a = pp.energy(x, y, w, h, W=wl.W, H=wl.H, Mu=Mu, Mp=Mp, precision="fp32")
    E64, a64 = pp.energy(x, y, w, h, W=wl.W, H=wl.H, Mu=Mu, Mp=Mp, precision="fp64")
    assert float((a - a64).norm()) <= 1e-5 * float(a64.norm()) and abs(float(E) - float(E64)) <= 1e-5 * float(E64)
    rng = np.random.default_rng(n)
    us = np.concatenate([[0, Mu - 1, Mu - 1, 0, Mu // 2, 127, 128], rng.integers(0, Mu, 25)])
    ps = np.concatenate([[Mp - 1, Mp - 1, 0, 1, Mp - 1, 128, 127], rng.integers(0, Mp, 25)])
    ao, _, Rabs = oracle.coeffs_sampled_full(wl.W, wl.H, *wl.arrays(), us, ps)
    scale = np.abs(oracle.coef_factors(wl.W, wl.H, Mu, Mp)[us, ps]) * Rabs
    e = np.abs(a.cpu().numpy()[us, ps] - ao)
    assert (e <= 1e-6 * scale).all(), float((e / np.where(scale > 0, scale, 1)).max())
