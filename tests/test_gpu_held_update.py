"""The first class's last update of a step and its first of the next in one launch, which
holds the boundary state aside for the force launch and its energy samples: under launch
shapes and at a size where the spins do not run in one workgroup. A rebuild at such a
boundary undoes the held update."""
import numpy as np
import pytest

from paper_1801_10233_amd import workloads as W
from tests.common import make_gpu, make_oracle, parity

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2, 0, -1), (1, 1, 0, 1), (4, 0, 0, 1), (8, 8, 0, -1)]


@pytest.mark.parametrize("shape", SHAPES)
def test_held_update_through_rebuilds_and_samples(shape):
    w = W.coupled_nve(n=8, T=1500.0)           # four classes of 256 atoms at first
    o, g = make_oracle(w), make_gpu(w, thermo_every=10)
    g.set_tuning(*shape)
    Es = []
    for _ in range(20):
        o.step(10, 2e-4)
        Es.append(o.energy()["total"])
    g.step(200, 2e-4)
    assert o.num_rebuilds >= 2 and g.stats()["rebuilds"] == o.num_rebuilds
    steps, Eg, _ = g.thermo()
    assert list(steps) == list(range(10, 201, 10))
    assert np.allclose(Eg, Es, rtol=1e-11, atol=1e-9)
    p = parity(w, o, g, rtol_r=1e-10, tol_s=1e-9, rtol_v=1e-9)
    assert p["ok"], p


@pytest.mark.parametrize("n,shape", [(8, s) for s in SHAPES] + [(14, (0, 0, 0, 0))])
def test_one_call_equals_many(n, shape):
    # one step per call holds nothing back, and between rebuilds it must give the
    # same state bit for bit
    w = W.coupled_nve(n=n)
    runs = []
    for calls in (1, 40):
        g = make_gpu(w, thermo_every=10)
        g.set_tuning(*shape)
        for _ in range(calls):
            g.step(40 // calls, w.dt)
        assert g.stats()["rebuilds"] <= 1      # the initial build only
        runs.append(g)
    for a, b in zip(runs[0].get_state(), runs[1].get_state()):
        assert np.array_equal(a, b)
    assert np.array_equal(runs[0].thermo()[1], runs[1].thermo()[1])
