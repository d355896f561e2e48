"""The bf16 row forms with one and with two 32-block subtiles per wave, on both sides of the lines between them: few blocks take
one, n = 16,385 and more at two N tiles take two, n = 33,100 there and n = 13,200 at five N tiles take whole rounds of two and
the rest of the blocks with one.  A block's results do not depend on the other blocks, so the first and the last
blocks of a large launch are compared with a launch of them alone (the other kernel), and both with the FP64 oracle.

Bars: the precision's own against the oracle (1e-3, 3e-2); 1e-12 between the kernels (the FP32 run sums are the same bits, the
FP64 sum over at most nine runs per tile and the tiles is in another order)."""
import sys

import numpy as np
import pytest

import oracle
from workloads import make_random

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu
TOL = {"bf16x3": 1e-3, "bf16": 3e-2}


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("prec", ["bf16x3", "bf16"])
@pytest.mark.parametrize("n,part,Mu,Mp", [(16384, 127, 40, 33), (16385, 128, 40, 33), (17001, 129, 33, 255), (16513, 257, 65, 256),
                                          (9000, 255, 257, 300), (33100, 400, 16, 130), (13200, 150, 257, 600), (20000, 1, 2, 1)])
def test_one_and_two_subtiles(prec, n, part, Mu, Mp):
    W, H = 500.0, 350.0
    wl = make_random(n, W, H, Mu, Mp, seed=n)
    print(f"[bwd rows] {prec} n={n} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n)
    a = rng.standard_normal((Mu, Mp)) / (1.0 + np.arange(Mu)[:, None] ** 2 + np.arange(Mp)[None, :] ** 2)
    at = torch.as_tensor(a, device="cuda:0")

    def forms(arrs):
        x, y, w, h = (torch.as_tensor(np.ascontiguousarray(v), device="cuda:0") for v in arrs)
        out = [*pp.field(x, y, w, h, at, W=W, H=H, precision=prec), *pp.point_field(x, y, at, W=W, H=H, precision=prec),
               pp.block_potential(x, y, w, h, at, W=W, H=H, precision=prec)]
        return [o.cpu().numpy() for o in out]

    full = forms(wl.arrays())
    for sl in (slice(0, part), slice(n - part, n)):
        arrs = [v[sl] for v in wl.arrays()]
        gxo, gyo = oracle.grad(W, H, *arrs, a)
        ref = [gxo, gyo, *oracle.point_field(W, H, a, *arrs[:2]), oracle.block_potential(W, H, *arrs, a)]
        for name, f, o, r in zip(("gx", "gy", "psi", "xix", "xiy", "N"), full, forms(arrs), ref):
            assert rel(f[sl], o) <= 1e-12 if np.any(o) else not np.any(f[sl]), name
            if np.linalg.norm(r) > 1e-9 * np.linalg.norm(a) and part >= 33 and max(Mu, Mp) > 2:
                assert rel(o, r) <= TOL[prec], name
