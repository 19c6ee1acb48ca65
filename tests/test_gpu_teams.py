"""Teams of wavefronts: every launch shape of the spin and force kernels gives
the oracle's step. The classes end inside a team (108 and 172 atoms per class
or so, teams of 8, 16 and 64 atoms), the rows inside a round (14 entries on 1,
2, 4 or 8 lanes), with and without the bath (its noise is drawn by other
wavefronts than the one that rotates). FP64: 20 steps of roundoff, so 1e-12."""
import numpy as np
import pytest

from paper_1801_10233_amd import workloads as W
from tests.common import make_gpu, make_oracle

pytestmark = pytest.mark.gpu

SHAPES = [(0, 0, 0, 0), (1, 1, -1, -1), (2, 2, -1, 1), (4, 4, -1, -1), (8, 8, -1, 1),
          (8, 4, 128, -1), (4, 8, 4096, 1)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("physics", ["langevin", "nve", "soc", "eam"])
def test_shapes_match_the_oracle(physics, shape):
    w = {"langevin": lambda: W.large_langevin(n=7), "nve": lambda: W.coupled_nve(n=6),
         "soc": lambda: W.soc_coupled(n=6, lam=0.01), "eam": lambda: W.eam_coupled(n=6, lam=0.01)}[physics]()
    w.r = w.r + W.thermal_displacements(w.N, 0.05, 11)   # uneven classes, rows of 13 to 16
    o, g = make_oracle(w), make_gpu(w)
    g.set_tuning(*shape)
    o.step(20, w.dt)
    g.step(20, w.dt)
    ro, vo, so = o.get_state()
    rg, vg, sg = g.get_state()
    assert np.abs(rg - ro).max() < 1e-12 * w.box[0]
    assert np.abs(sg - so).max() < 1e-12
    assert np.abs(vg - vo).max() < 1e-12 * np.abs(vo).max()
