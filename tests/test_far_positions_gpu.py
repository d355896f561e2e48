"""Blocks and points far outside the region in FP64 and FP32: the series continues periodically, so a centre of t L lies at
phase k (t mod 2) half turns for every frequency k, up to the largest finite t (an even number of half turns from 2^54 on).

Expected values from exact arithmetic: t = c / L is a double here (L is a power of two), k t mod 2 a fraction of integers.
Bars: 1e-10 and 1e-5, the precisions' own."""
import sys
from fractions import Fraction

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-10, "fp32": 1e-5}
W, H = 64.0, 128.0
TX = [0.28125, -3.4, 2.0**38 + 0.28125, 2.0**48 + 0.3125, -(2.0**50) - 0.75, 2.0**51 + 0.5, 2.0**52 - 1.5, 2.0**53 - 1.0, 2.0**54, 3e40, 1e300]
TY = [1e290, 0.59, -(2.0**45) - 0.875, 2.0**51 + 1.5, 2.0**50 + 0.25, 2.0**49 - 0.125, 0.40625, -(2.0**52) - 1.0, 2.0**53 + 2.0, 0.71875, -7e60]


def turns(t, M):
    """k t mod 2 in [-1, 1], k < M: [len(t), M]."""
    out = np.empty((len(t), M))
    for i, v in enumerate(t):
        for k in range(M):
            r = (k * Fraction(v)) % 2
            out[i, k] = float(r - 2 if r > 1 else r)
    return out


def factors(t, size, L, M):
    a, b = np.pi * turns(t, M), np.pi * turns([s / (2 * L) for s in size], M)
    S, K = 2.0 * np.cos(a) * np.sin(b), -2.0 * np.sin(a) * np.sin(b)
    S[:, 0], K[:, 0] = size, 0.0
    return np.cos(a), np.sin(a), S, K


def rel(got, ref):
    return np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("Mu,Mp,far_size", [(40, 37, False), (130, 70, False), (33, 260, True)])
def test_far_blocks(prec, Mu, Mp, far_size):
    rng = np.random.default_rng(Mu)
    w, h = rng.uniform(1.0, 8.0, len(TX)), rng.uniform(1.0, 8.0, len(TX))
    if far_size:   # and sizes of many periods: 2^50 + 1/4 and 2^52 + 1 half turns of the size's own phase
        w[2], h[4] = 2 * W * (2.0**50 + 0.25), 2 * H * (2.0**52 + 1.0)
    print(f"[far] {prec} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    x, y, wt, ht = (torch.as_tensor(v, device="cuda:0") for v in (np.array(TX) * W, np.array(TY) * H, w, h))
    cx, sx, S, K = factors(TX, w, W, Mu)
    cy, sy, T, L = factors(TY, h, H, Mp)
    size = dict(W=W, H=H, precision=prec)

    a = pp.coeffs(x, y, wt, ht, Mu=Mu, Mp=Mp, **size)
    raw, f = S.T @ T, oracle.coef_factors(W, H, Mu, Mp)
    assert rel(a, f * raw) <= TOL[prec]
    if not far_size:   # the raw sums: every frequency weighs alike
        got = a.cpu().numpy() / np.where(f == 0.0, 1.0, f)
        raw[0, 0] = 0.0
        assert np.linalg.norm(got[1:, 1:] - raw[1:, 1:]) <= TOL[prec] * np.linalg.norm(raw[1:, 1:])

    g = rng.standard_normal((Mu, Mp))
    gt = torch.as_tensor(g, device="cuda:0")
    wu, vp = np.arange(Mu) * np.pi / W, np.arange(Mp) * np.pi / H
    wt_, vt_ = np.where(wu == 0, 1.0, wu), np.where(vp == 0, 1.0, vp)
    gx, gy = pp.field(x, y, wt, ht, gt, **size)
    assert rel(gx, (K * (T @ (g / vt_).T)).sum(1)) <= TOL[prec]
    assert rel(gy, (L * (S @ (g / wt_[:, None]))).sum(1)) <= TOL[prec]
    psi, xix, xiy = pp.point_field(x, y, gt, **size)
    assert rel(psi, (cx * (cy @ g.T)).sum(1)) <= TOL[prec]
    assert rel(xix, (sx * wu * (cy @ g.T)).sum(1)) <= TOL[prec]
    assert rel(xiy, (sy * vp * (cx @ g)).sum(1)) <= TOL[prec]
    N = pp.block_potential(x, y, wt, ht, gt, **size)
    assert rel(N, (S * (T @ (g / (wt_[:, None] * vt_)).T)).sum(1)) <= TOL[prec]
