"""The bin scheme's fast transforms on the GPU against the FP64 oracle, at the lengths where their form changes: powers
of two from 64 to 8192 (one complex transform of the length itself, 0, 1 or 2 modulo 3 radix-2 steps), every other length up
to 4096 (Bluestein's form, whose convolution length doubles where 2 m - 1 passes a power of two), and the lengths left to
the matrix products (4097).

Bar: 1e-12 of the largest magnitude.  A transform of length L in FP64 is off by at most about 3 log2(L) 2^-53 in the
2-norm, 4e-15 at L = 8192; an entry passes two of them (four in Bluestein's form) and the frequency factors weight the
lowest frequencies by up to m, spread over the m entries of a row: 1e-14 relative to the largest magnitude in the norm, with
room of a hundred for single entries."""
import sys

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-12
LENGTHS = [2, 3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 256, 257, 513, 1024, 1025, 2048, 2049, 4095, 4096, 8192]


def gpu(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device=DEV)


@pytest.mark.parametrize("m", LENGTHS)
def test_fast_coeffs_at_every_form(m):
    W, H = 40.0, 25.0
    Mu, Mp = min(m, 37), min(m, 34 + m % 2)
    rng = np.random.default_rng(m)
    P = rng.uniform(0.0, 1.5, (m, m))
    print(f"[bins fft] coeffs m={m}", file=sys.stderr, flush=True)
    a = pp.bin_coeffs(gpu(P), W=W, H=H, Mu=Mu, Mp=Mp).cpu().numpy()
    us = np.concatenate([[0, 0, 1, min(1, Mu - 1), Mu - 1], rng.integers(0, Mu, 6)]) % Mu
    ps = np.concatenate([[1, Mp - 1, 0, min(1, Mp - 1), Mp - 1], rng.integers(0, Mp, 6)]) % Mp
    ref = oracle.bin_coeffs_at(W, H, P, us, ps)
    assert np.isfinite(a).all() and a[0, 0] == 0.0
    assert np.abs(a[us, ps] - ref).max() <= TOL * np.abs(ref).max()
    # the whole axes: all frequencies of one, few of the other
    full = pp.bin_coeffs(gpu(P), W=W, H=H, Mu=m, Mp=2).cpu().numpy()
    us = np.unique(np.concatenate([[1, m - 1, m // 2], rng.integers(0, m, 4)]))
    ref = oracle.bin_coeffs_at(W, H, P, us, np.ones_like(us))
    assert np.abs(full[us, 1] - ref).max() <= TOL * np.abs(full[:, 1]).max()


@pytest.mark.parametrize("m", LENGTHS)
def test_fast_field_at_every_form(m):
    W, H = 13.0, 29.0
    rng = np.random.default_rng(1000 + m)
    print(f"[bins fft] field m={m}", file=sys.stderr, flush=True)
    # few terms at the lowest and at the highest frequencies, each summed directly at sampled bins
    us, ps = np.unique([0, 1, m // 2, m - 1]), np.unique([0, 1, (m + 1) // 3, m - 1])
    a = np.zeros((m, m))
    a[np.ix_(us, ps)] = rng.normal(size=(len(us), len(ps)))
    got = [t.cpu().numpy() for t in pp.bin_field(gpu(a), W=W, H=H, m=m)]
    ls, js = (np.concatenate([[0, m - 1, m // 2], rng.integers(0, m, 30)]) for _ in range(2))
    tu, tp = ((f[:, None] * (2 * s[None, :] + 1)) % (4 * m) * (np.pi / (2 * m)) for f, s in ((us, ls), (ps, js)))
    b = a[np.ix_(us, ps)]
    wu, vp = us[:, None] * np.pi / W, ps[:, None] * np.pi / H
    ref = [np.einsum("us,up,ps->s", x, b, y) for x, y in ((np.cos(tu), np.cos(tp)), (wu * np.sin(tu), np.cos(tp)),
                                                           (np.cos(tu), vp * np.sin(tp)))]
    for g, r in zip(got, ref):
        assert np.isfinite(g).all()
        assert np.abs(g[ls, js] - r).max() <= TOL * np.abs(g).max()


def test_first_length_left_to_the_matrix_products():
    """m = 4097: the same sums as matrix products.  Their rounding follows the partial sums, which the mean of P drives to
    0.75 m^2 / pi = 4e6 in the transform of the row sums: 2^-53 of that over m steps at random, 3e-8, against a result of
    0.43 m 2^-1/2 = 1.2e3, 2.4e-11; bar 1e-10."""
    m, W, H = 4097, 40.0, 25.0
    P = np.random.default_rng(m).uniform(0.0, 1.5, (m, m))
    a = pp.bin_coeffs(gpu(P), W=W, H=H, Mu=5, Mp=4).cpu().numpy()
    us, ps = np.array([0, 1, 1, 4]), np.array([1, 0, 1, 3])
    ref = oracle.bin_coeffs_at(W, H, P, us, ps)
    assert a[0, 0] == 0.0 and np.abs(a[us, ps] - ref).max() <= 1e-10 * np.abs(ref).max()
