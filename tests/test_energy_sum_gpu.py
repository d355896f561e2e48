"""The ends of the coefficient reduction: planes of one to three coefficients with many splits (one coefficient a lane), and the
final energy sum at the partial counts where its waves and its loop of four change (one partial per 256 coefficients: 64, 65,
1024, 1025, more than 4096).

Bars: FP64 sums of n = 65,500 terms, 1e-11; FP32's own, 1e-5."""
import sys

import numpy as np
import pytest

import oracle
from workloads import make_random

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-11), ("fp32", 1e-5)])
@pytest.mark.parametrize("n,Mu,Mp", [(65500, 1, 1), (65500, 1, 2), (65000, 3, 1), (500, 1, 3), (40, 128, 128), (40, 129, 128),
                                     (40, 512, 512), (40, 513, 512), (40, 1100, 1000)])
def test_few_coefficients_and_many(n, Mu, Mp, prec, tol):
    wl = make_random(n, 90.0, 70.0, Mu, Mp, seed=n + Mp)
    print(f"[energy sum] {prec} n={n} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    x, y, w, h = (torch.as_tensor(np.ascontiguousarray(v), device="cuda:0") for v in wl.arrays())
    E, a = pp.energy(x, y, w, h, W=wl.W, H=wl.H, Mu=Mu, Mp=Mp, precision=prec)
    Eo, ao, _ = oracle.energy(wl.W, wl.H, *wl.arrays(), Mu, Mp)
    a = a.cpu().numpy()
    assert a[0, 0] == 0.0
    if Mu * Mp == 1:
        assert float(E) == 0.0
        return
    scale = np.linalg.norm(oracle.coeffs_sampled_full(wl.W, wl.H, *wl.arrays(), [Mu - 1], [Mp - 1])[2] * oracle.coef_factors(wl.W, wl.H, Mu, Mp)[-1, -1])
    assert np.linalg.norm(a - ao) <= tol * max(np.linalg.norm(ao), scale if Mu * Mp < 4 else 0.0)
    if Mu * Mp >= 4:
        assert abs(float(E) - Eo) <= tol * abs(Eo)
    else:   # a coefficient's own terms cancel; the energy is its square times a factor
        assert abs(float(E) - Eo) <= 2 * tol * max(np.linalg.norm(ao), scale) / np.linalg.norm(ao) * abs(Eo)
