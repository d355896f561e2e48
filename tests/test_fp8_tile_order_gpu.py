"""The order of the FP8 forward's workgroups at every kind of grid: fewer than eight splits, whole eights and a rest, with workgroup
counts that are and are not multiples of eight (the last splits are dealt differently then), against the FP64 oracle per output
tile.  A split is one chunk of 64 blocks here, so n = 64 s gives s splits.

Bar: that of the FP8X3 parity tests, 1e-2."""
import pytest

from tests import gpu_parity
from workloads import make_random

pytest.importorskip("torch")
pytest.importorskip("paper_2307_12041_amd")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("splits,Mu,Mp", [(1, 600, 300), (3, 500, 1000), (4, 257, 200), (5, 300, 500), (7, 256, 300), (8, 257, 256),
                                          (11, 512, 900), (12, 260, 250), (19, 40, 300)])
def test_every_tile_of_every_split(splits, Mu, Mp):
    gpu_parity.check(make_random(64 * splits - 5, 900.0, 700.0, Mu, Mp, seed=splits), "fp8x3", 1e-2)
