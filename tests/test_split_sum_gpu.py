"""The split-K reduction of the coefficient contraction, through pp.energy in FP64 and FP32, at the split counts where its
loops change (fewer splits than the 16 FP32 or 8 FP64 loads in flight, one and several batches of them, remainders), at
coefficient counts around its blocks of 256 and where its four coefficients a lane leave a rest.  Up to 2048 splits a split is one chunk of 32 blocks here, so n = 32 s - r
gives s splits.

Bar: the FP64 oracle; n eps = 1e-11 relative in the worst case at n = 65,000 in FP64, 1e-5 in FP32 (the FP32 path's own bar)."""
import sys

import numpy as np
import pytest

import oracle
from workloads import make_random

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-11), ("fp32", 1e-5)])
@pytest.mark.parametrize("splits,r,Mu,Mp", [(1, 31, 1, 1), (2, 0, 16, 16), (3, 5, 17, 15), (4, 0, 64, 64), (28, 1, 5, 7),
                                            (7, 4, 1, 3), (8, 0, 2, 2), (9, 9, 37, 7), (15, 1, 3, 3), (16, 0, 51, 5),
                                            (17, 8, 257, 1), (29, 0, 16, 17), (31, 2, 3, 85), (32, 0, 8, 32), (33, 0, 9, 57), (67, 7, 6, 6),
                                            (2031, 3, 4, 5)])
def test_split_counts_and_block_edges(splits, r, Mu, Mp, prec, tol):
    wl = make_random(32 * splits - r, 90.0, 70.0, Mu, Mp, seed=splits)
    print(f"[split sum] {prec} n={wl.n} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    x, y, w, h = (torch.as_tensor(np.ascontiguousarray(v), device="cuda:0") for v in wl.arrays())
    E, a = pp.energy(x, y, w, h, W=wl.W, H=wl.H, Mu=Mu, Mp=Mp, precision=prec)
    Eo, ao, _ = oracle.energy(wl.W, wl.H, *wl.arrays(), Mu, Mp)
    a = a.cpu().numpy()
    assert a[0, 0] == 0.0
    if Mu * Mp > 1:
        assert np.linalg.norm(a - ao) <= tol * np.linalg.norm(ao)
        assert abs(float(E) - Eo) <= tol * abs(Eo)
    else:
        assert float(E) == 0.0
