"""The work that users of the library have it do, as cases that can be timed and compared.

Four kinds of work, each through the Python entry points:

  step      one placement iteration: energy and coefficients, then the per-block gradient (pp.energy, pp.field),
            with a workspace that the program keeps.  FP64 is the plain form, FP32 the reference form of the split
            precisions, bf16x3 the form that placement runs, bf16mix and fp8x3 its cheaper variants.
  autograd  the same through the differentiable energy: forward, then backward (pp.energy_autograd), without a kept
            workspace.
  eval      pictures and reports: psi and xi at every block centre (pp.point_field), and the block potentials
            (pp.block_potential), from given coefficients.
  bins      the bin scheme: bin densities, binned coefficients, potential and field at the bin centres, and block
            values weighted back from the bins.

Blocks are standard cells (width U[1, 8], height 1) with a few macros, or small blocks in a small region, centres
uniform or in Gaussian clusters, clamped into the region: the distributions of the benchmark workloads.
"""
import math

import numpy as np
import torch

import paper_2307_12041_amd as pp

DEV = "cuda:0"

# Cost of one (block, u, p) triple of a step relative to bf16x3, for keeping drawn cases below the largest listed one.
COST = {"fp64": 8.0, "fp32": 4.5, "bf16x3": 1.0, "bf16mix": 0.6, "fp8x3": 0.75}


def _case(kind, name, precision, n, W, H, Mu, Mp, macros=0, side=200.0, clusters=0):
    """clusters: 0 for uniform centres; side: the largest side of a macro (the smallest is a tenth)."""
    return {"name": name, "kind": kind, "precision": precision, "n": n, "W": float(W), "H": float(H), "Mu": Mu, "Mp": Mp,
            "macros": macros, "side": float(side), "clusters": clusters}


def listed():
    return [
        # A toy or a unit test of a placer, and the smallest call: launches and host time are what it costs.
        _case("step", "step_fp64_1k_m64", "fp64", 1000, 1024, 1024, 64, 64),
        # A block-level floorplan with a truncation that is no multiple of anything, on a region that is not square.
        _case("step", "step_bf16x3_5k_257x513", "bf16x3", 5000, 300, 900, 257, 513),
        # A small circuit (200 thousand cells, 50 macros) in the precision that placement runs ...
        _case("step", "step_bf16x3_200k_m512", "bf16x3", 200050, 8192, 8192, 512, 512, macros=50),
        # ... in FP32 ...
        _case("step", "step_fp32_200k_m512", "fp32", 200050, 8192, 8192, 512, 512, macros=50),
        # ... and in plain FP64, against which results are checked.
        _case("step", "step_fp64_200k_m512", "fp64", 200050, 8192, 8192, 512, 512, macros=50),
        # Gradient-based placement of a million clustered cells through autograd.
        _case("autograd", "autograd_bf16x3_1m_m1024", "bf16x3", 1000000, 16384, 16384, 1024, 1024, clusters=16),
        # The same size in the FP8 split.
        _case("step", "step_fp8x3_1m_m1024", "fp8x3", 1000000, 16384, 16384, 1024, 1024, clusters=16),
        # The benchmark workload: two million cells and 500 macros.  The largest.
        _case("step", "step_bf16x3_2m_m2048", "bf16x3", 2000500, 16384, 16384, 2048, 2048, macros=500, side=400),
        # Potential and field at every block centre and the block potentials of a small circuit.
        _case("eval", "eval_bf16x3_200k_m512", "bf16x3", 200050, 8192, 8192, 512, 512, macros=50),
        # The bin scheme on a coarse grid of no particular size, on that of a small circuit, and at the benchmark's size.
        _case("bins", "bins_20k_m200", "fp64", 20000, 3000, 1700, 200, 200, macros=12),
        _case("bins", "bins_200k_m512", "fp64", 200050, 8192, 8192, 512, 512, macros=50),
        _case("bins", "bins_2m_m2048", "fp64", 2000500, 16384, 16384, 2048, 2048, macros=500, side=400),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "autograd", "eval", "bins", "bins"])
    aspect = rng.choice([1.0, 1.0, 0.5, 2.0, 0.37])
    clusters = rng.choice([0, 0, 16])
    macros = rng.choice([0, 12, 50, 500])
    if kind == "bins":
        n, m = _log(rng, 1000, 2000000), _log(rng, 48, 2048)
        Mu = m if rng.random() < 0.6 else rng.randint((m + 1) // 2, m)
        Mp = m if rng.random() < 0.6 else rng.randint((m + 1) // 2, m)
        precision = "fp64"
    else:
        precision = rng.choice({"step": ["fp64", "fp32", "bf16x3", "bf16x3", "bf16mix", "fp8x3"], "autograd": ["fp64", "bf16x3"],
                                "eval": ["fp64", "fp32", "bf16x3"]}[kind])
        n, Mu = _log(rng, 300, 2000000), _log(rng, 24, 2048)
        Mp = Mu if rng.random() < 0.5 else max(24, min(2048, _log(rng, Mu / 2, Mu * 2)))
        # at most half of the benchmark workload's work
        n = max(300, min(n, int(0.5 * 2000500 * 2048 * 2048 / (COST[precision] * Mu * Mp))))
    W = 8.0 * max(m if kind == "bins" else max(Mu, Mp), math.sqrt(8.0 * n))
    macros = min(macros, n // 20)
    case = _case(kind, "", precision, n, W, W * aspect, Mu, Mp, macros=macros, side=min(400.0, W * aspect / 8), clusters=clusters)
    del case["name"]
    return case


def _blocks(case, seed):
    """x, y, w, h in the order of the benchmark's workloads: sizes, then centres, then the clamp into the region."""
    rng = np.random.default_rng([int(seed), case["n"]])
    n, W, H, k = case["n"], case["W"], case["H"], case["macros"]
    w = rng.uniform(1.0, 8.0, n)
    h = np.ones(n)
    if k:
        w[n - k:] = rng.uniform(case["side"] / 10, case["side"], k)
        h[n - k:] = rng.uniform(case["side"] / 10, case["side"], k)
    x, y = rng.uniform(0.0, W, n), rng.uniform(0.0, H, n)
    c = case["clusters"]
    if c:
        cx, cy = rng.uniform(0.0, W, c), rng.uniform(0.0, H, c)
        at = rng.integers(0, c, n)
        sigma = W / 20
        x = cx[at] + sigma * rng.standard_normal(n)
        y = cy[at] + sigma * rng.standard_normal(n)
    x = np.clip(x, np.minimum(w, W) / 2, W - np.minimum(w, W) / 2)
    y = np.clip(y, np.minimum(h, H) / 2, H - np.minimum(h, H) / 2)
    return [torch.as_tensor(v, device=DEV) for v in (x, y, w, h)]


def _given_coeffs(case, seed):
    """Coefficients that an evaluation is handed: they fall like those of a density."""
    rng = np.random.default_rng([int(seed), 77])
    u, p = np.arange(case["Mu"])[:, None], np.arange(case["Mp"])[None, :]
    s = (u / case["W"]) ** 2 + (p / case["H"]) ** 2
    s[0, 0] = 1.0
    a = rng.standard_normal((case["Mu"], case["Mp"])) / (s * case["W"] * case["H"])
    a[0, 0] = 0.0
    return torch.as_tensor(a, device=DEV)


def prepare(case, seed):
    W, H = case["W"], case["H"]
    blocks = _blocks(case, seed)
    state = {"case": case, "blocks": blocks}
    if case["kind"] == "bins":
        size = pp.bin_workspace_size(W, H, case["n"], case["Mu"] if case["Mu"] > case["Mp"] else case["Mp"], case["Mu"], case["Mp"])
        state["ws"] = torch.empty(size, dtype=torch.uint8, device=DEV)
    elif case["kind"] != "autograd":
        size = pp.workspace_size(W, H, case["n"], case["Mu"], case["Mp"], precision=case["precision"])
        state["ws"] = torch.empty(size, dtype=torch.uint8, device=DEV)
    if case["kind"] == "autograd":
        state["x"], state["y"] = blocks[0].clone().requires_grad_(True), blocks[1].clone().requires_grad_(True)
    if case["kind"] == "eval":
        state["a"] = _given_coeffs(case, seed)
    return state


def run(state):
    case, (x, y, w, h) = state["case"], state["blocks"]
    W, H, Mu, Mp, prec = case["W"], case["H"], case["Mu"], case["Mp"], case["precision"]
    if case["kind"] == "step":
        E, a = pp.energy(x, y, w, h, W=W, H=H, Mu=Mu, Mp=Mp, precision=prec, workspace=state["ws"])
        gx, gy = pp.field(x, y, w, h, a, W=W, H=H, precision=prec, workspace=state["ws"])
        return {"E": E, "a": a, "gx": gx, "gy": gy}
    if case["kind"] == "autograd":
        xr, yr = state["x"], state["y"]
        xr.grad = yr.grad = None
        E = pp.energy_autograd(xr, yr, w, h, W=W, H=H, Mu=Mu, Mp=Mp, precision=prec)
        E.backward()
        return {"E": E.detach(), "gx": xr.grad, "gy": yr.grad}
    if case["kind"] == "eval":
        psi, xix, xiy = pp.point_field(x, y, state["a"], W=W, H=H, precision=prec, workspace=state["ws"])
        N = pp.block_potential(x, y, w, h, state["a"], W=W, H=H, precision=prec, workspace=state["ws"])
        return {"psi": psi, "xix": xix, "xiy": xiy, "N": N}
    m, ws = max(Mu, Mp), state["ws"]
    P = pp.bin_density(x, y, w, h, W=W, H=H, m=m, workspace=ws)
    a = pp.bin_coeffs(P, W=W, H=H, Mu=Mu, Mp=Mp, workspace=ws)
    psi, xix, xiy = pp.bin_field(a, W=W, H=H, m=m, workspace=ws)
    N, gx, gy = pp.bin_interp(x, y, w, h, psi, xix, xiy, W=W, H=H, workspace=ws)
    return {"P": P, "a": a, "psi": psi, "xix": xix, "xiy": xiy, "N": N, "gx": gx, "gy": gy}


def work(case):
    """Blocks read once, outputs written once, coefficients written and read once; two operations per (block, u, p)
    and contraction.  The bin scheme: fast cosine transforms of the m x m arrays, and the block arrays twice."""
    n, MM = float(case["n"]), float(case["Mu"]) * case["Mp"]
    if case["kind"] == "bins":
        m = max(case["Mu"], case["Mp"])
        return {"bytes": 2 * 32 * n + 24 * n + 8.0 * (2 * m * m + 2 * MM + 2 * 3 * m * m), "flops": 4 * 5.0 * m * m * math.log2(max(2, m))}
    if case["kind"] == "eval":
        return {"bytes": (16 + 32) * n + 32 * n + 2 * 8 * MM, "flops": 3 * 2 * n * MM}
    return {"bytes": 2 * 32 * n + 16 * n + 2 * 8 * MM, "flops": 3 * 2 * n * MM}


# ----------------------------------------------------------------------------------------------------------------
# The same in 64 bits from the definitions: tables of the trigonometric factors and plain matrix products.
# ----------------------------------------------------------------------------------------------------------------
def _phase(c, L, M):
    """cos and sin of k pi c / L, [n, M]: k c / L is reduced to (-1, 1] half turns, its leading part exactly."""
    t = c / L
    hi = torch.round(t * 2.0 ** 38) / 2.0 ** 38
    k = torch.arange(M, dtype=torch.float64, device=c.device)
    r = torch.outer(hi, k)
    r = (r - 2.0 * torch.round(0.5 * r)) + torch.outer(t - hi, k)
    r = r * math.pi
    return torch.cos(r), torch.sin(r)


def _tables(c, s, L, M):
    """Per block and frequency: the cosine integrated over the block, and its derivative by the centre."""
    ca, sa = _phase(c, L, M)
    _, sb = _phase(0.5 * s, L, M)
    f = torch.arange(M, dtype=torch.float64, device=c.device) * (math.pi / L)
    f[0] = 1.0
    X, K = 2.0 * ca * sb / f, -2.0 * sa * sb
    X[:, 0], K[:, 0] = s, 0.0
    return X, K


def _chunks(n, M):
    step = max(1, int(2 ** 28 // max(1, M)))
    return [slice(i, min(n, i + step)) for i in range(0, n, step)]


def _exact_coeffs(case, x, y, w, h):
    W, H, Mu, Mp = case["W"], case["H"], case["Mu"], case["Mp"]
    A = torch.zeros((Mu, Mp), dtype=torch.float64, device=DEV)
    for c in _chunks(case["n"], Mu + Mp):
        A += _tables(x[c], w[c], W, Mu)[0].T.contiguous() @ _tables(y[c], h[c], H, Mp)[0]
    u = torch.arange(Mu, dtype=torch.float64, device=DEV)[:, None] * (math.pi / W)
    v = torch.arange(Mp, dtype=torch.float64, device=DEV)[None, :] * (math.pi / H)
    eps = torch.where(u > 0, 2.0, 1.0) * torch.where(v > 0, 2.0, 1.0)
    s = W * H * (u * u + v * v)
    s[0, 0] = math.inf
    a = eps.double() / s * A
    return 0.5 * (a * A).sum(), a


def _exact_rows(case, x, y, w, h, a):
    """Per block: sum_up a_up of (dX/dx Y, X dY/dy, X Y)."""
    n = case["n"]
    gx, gy, N = (torch.empty(n, dtype=torch.float64, device=DEV) for _ in range(3))
    for c in _chunks(n, 3 * (case["Mu"] + case["Mp"])):
        X, K = _tables(x[c], w[c], case["W"], case["Mu"])
        Y, L = _tables(y[c], h[c], case["H"], case["Mp"])
        Z = Y @ a.T.contiguous()
        gx[c], N[c] = (K * Z).sum(1), (X * Z).sum(1)
        gy[c] = (L * (X @ a)).sum(1)
    return gx, gy, N


def _exact_points(case, x, y, a):
    n = case["n"]
    wu = torch.arange(case["Mu"], dtype=torch.float64, device=DEV) * (math.pi / case["W"])
    vp = torch.arange(case["Mp"], dtype=torch.float64, device=DEV) * (math.pi / case["H"])
    psi, xix, xiy = (torch.empty(n, dtype=torch.float64, device=DEV) for _ in range(3))
    for c in _chunks(n, 3 * (case["Mu"] + case["Mp"])):
        cx, sx = _phase(x[c], case["W"], case["Mu"])
        cy, sy = _phase(y[c], case["H"], case["Mp"])
        Z = cy @ a.T.contiguous()
        psi[c], xix[c] = (cx * Z).sum(1), (sx * wu * Z).sum(1)
        xiy[c] = (sy * vp * (cx @ a)).sum(1)
    return psi, xix, xiy


def _overlaps(c, s, L, m):
    """[n, m]: the length of each block inside each bin along one axis."""
    edge = torch.arange(m + 1, dtype=torch.float64, device=DEV) * (L / m)
    lo, hi = (c - 0.5 * s)[:, None], (c + 0.5 * s)[:, None]
    return (torch.minimum(hi, edge[1:]) - torch.maximum(lo, edge[:-1])).clamp_(min=0.0)


def _bin_trig(M, m):
    """cos and sin of f (2 s + 1) pi / (2 m), [M, m]."""
    f = torch.arange(M, device=DEV)[:, None]
    q = (f * (2 * torch.arange(m, device=DEV)[None, :] + 1)) % (4 * m)
    t = q.double() * (math.pi / (2 * m))
    return torch.cos(t), torch.sin(t)


def _exact_bins(case, x, y, w, h):
    W, H, Mu, Mp, n = case["W"], case["H"], case["Mu"], case["Mp"], case["n"]
    m = max(Mu, Mp)
    P = torch.zeros((m, m), dtype=torch.float64, device=DEV)
    for c in _chunks(n, 2 * m):
        P += _overlaps(x[c], w[c], W, m).T.contiguous() @ _overlaps(y[c], h[c], H, m)
    P /= (W / m) * (H / m)
    Cu, Su = _bin_trig(Mu, m)
    Cp, Sp = _bin_trig(Mp, m)
    R = Cu @ (P @ Cp.T.contiguous())
    # each bin's cosine integral over its width, 2 sin(f pi / 2m) / (f pi / L) (its width at f = 0), along both axes,
    # and the scale of the series
    wu = torch.arange(Mu, dtype=torch.float64, device=DEV) * (math.pi / W)
    vp = torch.arange(Mp, dtype=torch.float64, device=DEV) * (math.pi / H)
    bu, bp = 2.0 * torch.sin(wu * (0.5 * W / m)) / wu, 2.0 * torch.sin(vp * (0.5 * H / m)) / vp
    bu[0], bp[0] = W / m, H / m
    s = W * H * (wu[:, None] ** 2 + vp[None, :] ** 2)
    s[0, 0] = math.inf
    eu, ep = torch.full((Mu, 1), 2.0, dtype=torch.float64, device=DEV), torch.full((1, Mp), 2.0, dtype=torch.float64, device=DEV)
    eu[0], ep[0, 0] = 1.0, 1.0
    a = R * bu[:, None] * bp[None, :] * eu * ep / s
    Cut, Sut = Cu.T.contiguous(), (Su * wu[:, None]).T.contiguous()
    Z = a @ Cp
    psi, xix, xiy = Cut @ Z, Sut @ Z, Cut @ (a @ (Sp * vp[:, None]))
    N, gx, gy = (torch.empty(n, dtype=torch.float64, device=DEV) for _ in range(3))
    for c in _chunks(n, 4 * m):
        ox, oy = _overlaps(x[c], w[c], W, m), _overlaps(y[c], h[c], H, m)
        N[c], gx[c], gy[c] = ((ox @ psi) * oy).sum(1), -((ox @ xix) * oy).sum(1), -((ox @ xiy) * oy).sum(1)
    return {"P": P, "a": a, "psi": psi, "xix": xix, "xiy": xiy, "N": N, "gx": gx, "gy": gy}


def exact(case, seed):
    x, y, w, h = _blocks(case, seed)
    if case["kind"] == "bins":
        return _exact_bins(case, x, y, w, h)
    if case["kind"] == "eval":
        a = _given_coeffs(case, seed)
        psi, xix, xiy = _exact_points(case, x, y, a)
        return {"psi": psi, "xix": xix, "xiy": xiy, "N": _exact_rows(case, x, y, w, h, a)[2]}
    E, a = _exact_coeffs(case, x, y, w, h)
    gx, gy, _ = _exact_rows(case, x, y, w, h, a)
    return {"E": E, "a": a, "gx": gx, "gy": gy} if case["kind"] == "step" else {"E": E, "gx": gx, "gy": gy}
