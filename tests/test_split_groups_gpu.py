"""The bf16 forward that adds its splits on the way, at the edges of its 128 x 128 tiles, with one, two and three chunks of
32 blocks per split, even and odd numbers of chunks in a group and a short last group, against the FP64 oracle and against the
store mode, which writes every split's FP32 partials and reduces them.

Bars: the oracle's, the precision's own (1e-3 with three products, 3e-2 with one, as in the parity tests). The store mode's,
1e-12: the splits' FP32 sums are the same bits there and only the order of at most 2048 FP64 additions differs
(2 * 2048 * 2^-53 = 4.5e-13 of the sum of magnitudes)."""
import sys

import numpy as np
import pytest

import oracle
from workloads import make_random

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu
TOL = {"bf16x3": 1e-3, "bf16": 3e-2}


@pytest.mark.parametrize("prec", ["bf16x3", "bf16"])
@pytest.mark.parametrize("n,Mu,Mp", [(33, 1, 2), (64, 127, 128), (65, 128, 129), (97, 129, 127), (1000, 64, 300), (2017, 257, 255),
                                     (20000, 257, 130), (66000, 40, 33), (70001, 128, 1), (131100, 130, 36), (65536, 1, 129)])
def test_groups_of_splits(prec, n, Mu, Mp):
    wl = make_random(n, 500.0, 300.0, Mu, Mp, seed=n)
    print(f"[split groups] {prec} n={n} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    x, y, w, h = (torch.as_tensor(np.ascontiguousarray(v), device="cuda:0") for v in wl.arrays())
    size = dict(W=wl.W, H=wl.H, Mu=Mu, Mp=Mp, precision=prec)
    E, a = pp.energy(x, y, w, h, **size)
    Es, as_ = pp.energy(x, y, w, h, basis="store", **size)
    Eo, ao, _ = oracle.energy(wl.W, wl.H, *wl.arrays(), Mu, Mp)
    a, as_ = a.cpu().numpy(), as_.cpu().numpy()
    assert a[0, 0] == 0.0
    assert np.linalg.norm(a - as_) <= 1e-12 * np.linalg.norm(as_)
    assert np.linalg.norm(a - ao) <= TOL[prec] * np.linalg.norm(ao)
    assert abs(float(E) - Eo) <= 2 * TOL[prec] * abs(Eo)


@pytest.mark.parametrize("n,Mu,Mp", [(65, 128, 129), (997, 256, 40), (70001, 33, 256)])
def test_mixed_split_of_one_tile_per_axis(n, Mu, Mp):
    """Up to 256 frequencies per axis the mixed split contracts everything with three products: bf16x3's coefficients."""
    wl = make_random(n, 500.0, 300.0, Mu, Mp, seed=n)
    x, y, w, h = (torch.as_tensor(np.ascontiguousarray(v), device="cuda:0") for v in wl.arrays())
    size = dict(W=wl.W, H=wl.H, Mu=Mu, Mp=Mp)
    assert torch.equal(pp.coeffs(x, y, w, h, precision="bf16mix", **size), pp.coeffs(x, y, w, h, precision="bf16x3", **size))
