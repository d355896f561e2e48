"""The gradient's and the evaluation rows' launches: both contractions of a gradient in one launch, N axes of one tile
that write results themselves (128 frequencies in FP64 and FP32, 256 in the bf16 types) beside axes that leave partial sums,
few blocks and many (one workgroup per axis, ragged block tiles), and FP64 outputs that share memory with the inputs.

Bars: each precision's own, against the FP64 oracle (as in the parity tests): 1e-10, 1e-5, 1e-3."""
import sys

import numpy as np
import pytest

import oracle
from workloads import make_random

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-10, "fp32": 1e-5, "bf16x3": 1e-3, "bf16mix": 1e-3}


def gpu(*arrs):
    return [torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0") for a in arrs]


def rel(a, b):
    return np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3", "bf16mix"])
@pytest.mark.parametrize("n,Mu,Mp", [(1, 3, 2), (31, 64, 65), (33, 128, 129), (129, 129, 128), (257, 128, 128), (600, 256, 257),
                                     (255, 257, 256), (1030, 256, 40)])
def test_one_and_several_tiles_per_axis(prec, n, Mu, Mp):
    W, H = 120.0, 75.0
    wl = make_random(n, W, H, Mu, Mp, seed=n)
    print(f"[rows] {prec} n={n} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    x, y, w, h = gpu(*wl.arrays())
    _, ao, _ = oracle.energy(W, H, *wl.arrays(), Mu, Mp)
    a, dE = gpu(ao)[0], torch.tensor(-0.5, dtype=torch.float64, device="cuda:0")
    gxo, gyo = oracle.grad(W, H, *wl.arrays(), ao)
    for scale, arg in ((1.0, None), (-0.5, dE)):
        gx, gy = pp.field(x, y, w, h, a, W=W, H=H, precision=prec, dE=arg)
        assert rel(gx, scale * gxo) <= TOL[prec] and rel(gy, scale * gyo) <= TOL[prec]
    if prec == "bf16mix":
        return
    psi, xix, xiy = pp.point_field(x, y, a, W=W, H=H, precision=prec)
    po, xo, yo = oracle.point_field(W, H, ao, *wl.arrays()[:2])
    assert rel(psi, po) <= TOL[prec] and rel(xix, xo) <= TOL[prec] and rel(xiy, yo) <= TOL[prec]
    for want in (("psi",), ("xix",), ("xiy",), ("xix", "xiy")):
        got = pp.point_field(x, y, a, W=W, H=H, precision=prec, want=want)
        for name, g, o in zip(("psi", "xix", "xiy"), got, (po, xo, yo)):
            assert (g is None) == (name not in want) and (g is None or rel(g, o) <= TOL[prec])
    N = pp.block_potential(x, y, w, h, a, W=W, H=H, precision=prec)
    assert rel(N, oracle.block_potential(W, H, *wl.arrays(), ao)) <= TOL[prec]


@pytest.mark.parametrize("prec,n,Mu,Mp", [("fp64", 15001, 128, 128), ("fp64", 15001, 130, 129), ("fp64", 28700, 50, 64),
                                          ("fp32", 15001, 128, 128), ("fp32", 15001, 131, 127), ("fp32", 28700, 50, 64),
                                          ("fp32", 65500, 256, 256), ("fp32", 66001, 250, 255)])
def test_tiles_of_128_blocks_and_wide_tiles(prec, n, Mu, Mp):
    """Enough blocks for the full block tile (below, tiles of 32 blocks), half N tiles, rows of the operand that are not
    16-byte aligned, and FP32's N tiles of 256; sampled blocks, any coefficients (the gradient is linear in them)."""
    W, H = 500.0, 350.0
    wl = make_random(n, W, H, Mu, Mp, seed=n)
    print(f"[rows] {prec} n={n} M={Mu}x{Mp}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n)
    a = rng.standard_normal((Mu, Mp)) / (1.0 + np.arange(Mu)[:, None] ** 2 + np.arange(Mp)[None, :] ** 2)
    idx = np.unique(np.concatenate([[0, 127, 128, n - 1], rng.integers(0, n, 150)]))
    gx, gy = pp.field(*gpu(*wl.arrays()), gpu(a)[0], W=W, H=H, precision=prec)
    gxo, gyo = oracle.grad_sampled(W, H, *wl.arrays(), a, idx)
    assert rel(gx[torch.as_tensor(idx, device="cuda:0")], gxo) <= TOL[prec]
    assert rel(gy[torch.as_tensor(idx, device="cuda:0")], gyo) <= TOL[prec]
    psi, xix, xiy = pp.point_field(*gpu(wl.x, wl.y), gpu(a)[0], W=W, H=H, precision=prec)
    po, xo, yo = oracle.point_field(W, H, a, wl.x[idx], wl.y[idx])
    at = torch.as_tensor(idx, device="cuda:0")
    assert rel(psi[at], po) <= TOL[prec] and rel(xix[at], xo) <= TOL[prec] and rel(xiy[at], yo) <= TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_outputs_in_the_memory_of_the_inputs(prec):
    """gx and gy over x and y, psi and xi over the points: the results are those of separate outputs, bit for bit."""
    import ctypes
    W, H, Mu, Mp = 120.0, 75.0, 60, 50
    wl = make_random(700, W, H, Mu, Mp, seed=3)
    x, y, w, h = gpu(*wl.arrays())
    a = pp.coeffs(x, y, w, h, W=W, H=H, Mu=Mu, Mp=Mp, precision=prec)
    gx, gy = pp.field(x, y, w, h, a, W=W, H=H, precision=prec)
    psi, xix, xiy = pp.point_field(x, y, a, W=W, H=H, precision=prec)
    N = pp.block_potential(x, y, w, h, a, W=W, H=H, precision=prec)
    P = pp.PPProblem(W, H, wl.n, Mu, Mp, pp.PRECISIONS[prec], 0)
    need = pp.workspace_size(W, H, wl.n, Mu, Mp, precision=prec)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    lib, st = pp.load(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def vp(t):
        return ctypes.c_void_p(t.data_ptr())
    x2, y2, w2, h2 = (t.clone() for t in (x, y, w, h))
    assert lib.pp_field(ctypes.byref(P), vp(x2), vp(y2), vp(w2), vp(h2), vp(a), None, vp(y2), vp(x2), vp(ws), need, st) == 0
    assert torch.equal(y2, gx) and torch.equal(x2, gy)
    x2, y2 = x.clone(), y.clone()
    assert lib.pp_point_field(ctypes.byref(P), vp(x2), vp(y2), vp(a), vp(x2), vp(y2), vp(w2), vp(ws), need, st) == 0
    assert torch.equal(x2, psi) and torch.equal(y2, xix) and torch.equal(w2, xiy)
    x2, w2 = x.clone(), w.clone()
    assert lib.pp_block_potential(ctypes.byref(P), vp(x2), vp(y), vp(w2), vp(h), vp(a), vp(w2), vp(ws), need, st) == 0
    assert torch.equal(w2, N)
