"""The timing hooks' records: each stage of a call has the records that callers have always divided by, also where one launch
does the work of several stages, and the times of the stages are not negative."""
import numpy as np
import pytest

from workloads import make_random

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2307_12041_amd")

pytestmark = pytest.mark.gpu
STAGES = ("tables", "seeds", "build", "fwd", "reduce", "energy", "prep", "bwd", "final", "point", "potential")


def records(call):
    pp.timing_enable(True)
    try:
        call()
        got = {s: pp.timing_query(s) for s in STAGES}
    finally:
        pp.timing_enable(False)
    assert all(ms >= 0.0 for ms, _ in got.values())
    assert all(got[s][0] > 0.0 for s in ("fwd", "bwd", "point", "potential") if got[s][1])
    return {s: c for s, (_, c) in got.items() if c}


@pytest.mark.parametrize("Mu,Mp", [(40, 33), (300, 20), (600, 530)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3", "bf16", "bf16mix", "fp8x3", "fp8", "store"])
def test_records_of_each_stage(prec, Mu, Mp):
    wl = make_random(700, 300.0, 200.0, Mu, Mp, seed=5)
    x, y, w, h = (torch.as_tensor(np.ascontiguousarray(v), device="cuda:0") for v in wl.arrays())
    basis = "store" if prec == "store" else "recompute"
    prec = "bf16x3" if prec == "store" else prec
    gen = prec not in ("fp64", "fp32")
    ws = torch.empty(pp.workspace_size(wl.W, wl.H, wl.n, Mu, Mp, precision=prec, basis=basis), dtype=torch.uint8, device="cuda:0")
    size = dict(W=wl.W, H=wl.H, precision=prec, workspace=ws)
    out = []
    want = {"fwd": 1, "reduce": 1, "energy": 1, **({"tables": 1, "seeds": 1} if gen else {}), **({"build": 1} if basis == "store" else {})}
    assert records(lambda: out.append(pp.energy(x, y, w, h, Mu=Mu, Mp=Mp, basis=basis, **size))) == want
    a = out[0][1]
    rows = {"prep": 1, "final": 1, **({"tables": 1} if gen else {})}
    assert records(lambda: pp.field(x, y, w, h, a, basis=basis, **size)) == {**rows, "bwd": 2}
    if basis == "store" or prec in ("bf16mix", "fp8x3", "fp8"):
        return
    assert records(lambda: pp.point_field(x, y, a, **size)) == {**rows, "point": 2}
    assert records(lambda: pp.point_field(x, y, a, want=("xix",), **size)) == {**rows, "point": 1}
    assert records(lambda: pp.block_potential(x, y, w, h, a, **size)) == {**rows, "potential": 1}
