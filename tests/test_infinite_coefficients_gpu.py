"""One infinite coefficient in the FP64 and FP32 row forms, at the highest frequency of an axis that ends inside a chunk of 32:
the rest of that chunk holds no coefficient, and every result is the infinity that a plain sum gives, not NaN.  At each tile
of the dispatch: 32 and 128 blocks, 64, 128 and (FP32) 256 frequencies, operand rows with and without 16-byte alignment.

Expected: the FP64 oracle's sums, equal in sign and kind; the finite remainder of the coefficients is held by the parity tests."""
import sys

import numpy as np
import pytest

import oracle
from workloads import make_random

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu


def gpu(*arrs):
    return [torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0") for a in arrs]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,Mu,Mp", [(40, 33, 35), (40, 70, 75), (15001, 130, 130), (15001, 131, 129), (28700, 50, 61),
                                     (66001, 252, 252), (66001, 251, 253)])
def test_infinity_at_the_last_frequency(prec, n, Mu, Mp):
    W, H = 500.0, 350.0
    wl = make_random(n, W, H, Mu, Mp, seed=n)
    print(f"[inf] {prec} n={n} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    idx = np.unique(np.concatenate([[0, n - 1], np.random.default_rng(n).integers(0, n, 40)]))
    at = torch.as_tensor(idx, device="cuda:0")
    for (u, p), v in (((2, Mp - 1), np.inf), ((Mu - 1, 3), -np.inf)):
        a = np.random.default_rng(1).standard_normal((Mu, Mp))
        a[u, p] = v
        gx, gy = pp.field(*gpu(*wl.arrays()), gpu(a)[0], W=W, H=H, precision=prec)
        got = [gx, gy, *pp.point_field(*gpu(wl.x, wl.y), gpu(a)[0], W=W, H=H, precision=prec),
               pp.block_potential(*gpu(*wl.arrays()), gpu(a)[0], W=W, H=H, precision=prec)]
        sub = [c[idx] for c in wl.arrays()]
        with np.errstate(invalid="ignore"):
            ref = [*oracle.grad(W, H, *sub, a), *oracle.point_field(W, H, a, *sub[:2]), oracle.block_potential(W, H, *sub, a)]
        for name, g, r in zip(("gx", "gy", "psi", "xix", "xiy", "N"), got, ref):
            assert np.isinf(r).all(), name
            assert np.array_equal(g[at].cpu().numpy(), r), name
