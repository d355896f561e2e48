"""The bin scheme's transforms on both sides of the lines between fast transforms and matrix products: few and many frequencies
of many bins, each choice of outputs, and the small lengths where the coefficients' line depends on the truncation.

Bar: 1e-12 of the largest magnitude, as for the fast transforms at every length; the products here sum at most 1100 terms of
random signs per axis, or 63 of one sign (63 * 2^-53 * 63 * 1.5 / 0.2 of the largest coefficient: 3e-12 at the very worst, a
hundredth of it at random)."""
import sys

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu
TOL = 1e-12


def gpu(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


@pytest.mark.parametrize("m,Mu,Mp", [(4, 4, 4), (5, 5, 5), (8, 1, 8), (31, 31, 31), (32, 32, 32), (33, 16, 33), (33, 17, 17), (33, 33, 16), (40, 33, 4), (40, 33, 5),
                                     (63, 16, 63), (63, 63, 17), (63, 63, 16), (64, 5, 64), (65, 1, 65)])
def test_coeffs(m, Mu, Mp):
    W, H = 40.0, 25.0
    P = np.random.default_rng(m).uniform(0.0, 1.5, (m, m))
    a = pp.bin_coeffs(gpu(P), W=W, H=H, Mu=Mu, Mp=Mp).cpu().numpy()
    u, p = (v.ravel() for v in np.meshgrid(np.arange(Mu), np.arange(Mp), indexing="ij"))
    ref = oracle.bin_coeffs_at(W, H, P, u, p).reshape(Mu, Mp)
    assert a[0, 0] == 0.0 and np.abs(a - ref).max() <= TOL * np.abs(ref).max()


@pytest.mark.parametrize("m,Mu,Mp", [(100, 1, 16), (100, 64, 16), (200, 33, 200), (300, 64, 16), (400, 65, 65), (512, 8, 8), (640, 64, 64),
                                     (1000, 96, 96), (1000, 160, 40), (1024, 33, 33), (1500, 128, 128), (2047, 160, 160),
                                     (2048, 33, 33), (2048, 64, 128), (2049, 300, 64), (2049, 640, 64), (4095, 16, 1100), (4096, 96, 64)])
def test_field(m, Mu, Mp):
    W, H = 13.0, 29.0
    rng = np.random.default_rng(m + Mu)
    print(f"[bins routes] field m={m} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    a = rng.standard_normal((Mu, Mp))
    ls, js = (np.concatenate([[0, m - 1, m // 2], rng.integers(0, m, 40)]) for _ in range(2))
    tu, tp = ((np.arange(M)[:, None] * (2 * s[None, :] + 1)) % (4 * m) * (np.pi / (2 * m)) for M, s in ((Mu, ls), (Mp, js)))
    wu, vp = np.arange(Mu)[:, None] * np.pi / W, np.arange(Mp)[:, None] * np.pi / H
    ref = [((x.T @ a) * y.T).sum(1) for x, y in ((np.cos(tu), np.cos(tp)), (wu * np.sin(tu), np.cos(tp)), (np.cos(tu), vp * np.sin(tp)))]
    names = ("psi", "xix", "xiy")
    full = pp.bin_field(gpu(a), W=W, H=H, m=m)
    for want in (names, ("psi",), ("xix",), ("xiy",), ("xix", "xiy"), ("psi", "xiy")):
        got = pp.bin_field(gpu(a), W=W, H=H, m=m, want=want)
        for name, g, f, r in zip(names, got, full, ref):
            assert (g is None) == (name not in want)
            if g is not None:
                assert torch.equal(g, f), (name, want)
                g = g.cpu().numpy()
                assert np.isfinite(g).all() and np.abs(g[ls, js] - r).max() <= TOL * np.abs(g).max(), (name, want)
