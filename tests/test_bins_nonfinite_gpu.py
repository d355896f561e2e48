"""Infinite and NaN bins and coefficients in the bin scheme's transforms: every result is what the separable sums give, an
infinity of the right sign, or NaN where a factor is zero or infinities of both signs meet.  At lengths of every form of the
fast transforms and at one left to the matrix products, which have always summed so.

Expected: the terms of the elements that are not finite, by the definitions; the finite rest cannot change them.  Equality."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu
W, H = 40.0, 25.0
LENGTHS = [1, 2, 3, 7, 12, 64, 100, 128, 200, 512, 600, 1024, 1500, 2048, 2100, 4096, 4100]


def trig(f, m):
    """cos and sin of f (2s + 1) pi / (2m) over s, with exact zeros."""
    q = f * (2 * np.arange(m) + 1)
    c, s = np.cos(q % (4 * m) * (np.pi / (2 * m))), np.sin(q % (4 * m) * (np.pi / (2 * m)))
    c[q % (2 * m) == m], s[q % (2 * m) == 0] = 0.0, 0.0
    return c, s


def cos_of(n, M, m):
    """cos(f (2n + 1) pi / (2m)) over f < M."""
    q = np.arange(M) * (2 * n + 1)
    c = np.cos(q % (4 * m) * (np.pi / (2 * m)))
    c[q % (2 * m) == m] = 0.0
    return c


def same(got, ref):
    got = got.cpu().numpy()
    return np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[~np.isnan(ref)], ref[~np.isnan(ref)])


def sets(m, rng):
    k = [int(v) for v in rng.integers(0, m, 8)]
    return [[(k[0], k[1], np.inf)], [(0, 0, -np.inf)], [(m - 1, k[2], np.nan)], [(k[3], m - 1, -np.inf), (k[3], k[4], -np.inf)],
            [(k[5], k[6], np.inf), (min(k[5] + 1, m - 1), k[7], -np.inf)]]


@pytest.mark.parametrize("m", LENGTHS)
def test_coeffs(m):
    rng = np.random.default_rng(m)
    Mu, Mp = max(1, m - m // 3), m
    if m > 1024:
        Mu, Mp = 70, 61
    print(f"[bins nonfinite] coeffs m={m}", file=sys.stderr, flush=True)
    for bad in sets(m, rng):
        P = torch.rand((m, m), dtype=torch.float64, device="cuda:0")
        for l, j, v in bad:
            P[l, j] = v
        a = pp.bin_coeffs(P, W=W, H=H, Mu=Mu, Mp=Mp)
        with np.errstate(invalid="ignore"):
            Q = {}
            for l, j, v in dict(((l, j), (l, j, v)) for l, j, v in bad).values():
                Q[l] = Q.get(l, 0.0) + v * cos_of(j, Mp, m)
            ref = sum(np.outer(cos_of(l, Mu, m), q) for l, q in Q.items())
            ref[0, 0] *= 0.0
        assert same(a, ref), bad


@pytest.mark.parametrize("m", LENGTHS)
def test_field(m):
    rng = np.random.default_rng(50 + m)
    M = m if m <= 1024 else 300
    print(f"[bins nonfinite] field m={m}", file=sys.stderr, flush=True)
    for bad in sets(M, rng):
        a = torch.randn((M, M), dtype=torch.float64, device="cuda:0")
        for u, p, v in bad:
            a[u, p] = v
        got = pp.bin_field(a, W=W, H=H, m=m)
        with np.errstate(invalid="ignore"):
            R, Rs = {}, {}
            for u, p, v in dict(((u, p), (u, p, v)) for u, p, v in bad).values():
                c, s = trig(p, m)
                R[u] = R.get(u, 0.0) + v * c
                Rs[u] = Rs.get(u, 0.0) + v * (s * (p * np.pi / H))
            psi = sum(np.outer(trig(u, m)[0], r) for u, r in R.items())
            xix = sum(np.outer(trig(u, m)[1] * (u * np.pi / W), r) for u, r in R.items())
            xiy = sum(np.outer(trig(u, m)[0], r) for u, r in Rs.items())
        for name, g, r in zip(("psi", "xix", "xiy"), got, (psi, xix, xiy)):
            assert same(g, r), (name, bad)
        one = pp.bin_field(a, W=W, H=H, m=m, want=("xiy",))
        assert same(one[2], xiy)
