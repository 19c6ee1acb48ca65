"""Small systems whose spin half-steps run in one workgroup (the default
launch shape), and runs of small classes that fetch ahead (small_class 4096):
classes of less than a team of 64 atoms, of a whole number of teams and of more
than one piece of 512 atoms, few and many classes, rows longer than the 16 entries
of the first round, frozen runs past one chunk of 64 steps. FP64: 20 steps of
roundoff, so 1e-12 (70 frozen steps: 4e-12). FP32: at most 280 updates, each off by
2e-7 or less, so 6e-5 against the FP64 oracle."""
import numpy as np
import pytest

from paper_1801_10233_amd import spinlat as sl
from paper_1801_10233_amd import workloads as W
from tests.common import make_gpu, make_oracle

pytestmark = pytest.mark.gpu


def _run(w, steps, precision, shape=None):
    o, g = make_oracle(w), make_gpu(w, precision=precision)
    if shape:
        g.set_tuning(*shape)
    o.step(steps, w.dt)
    g.step(steps, w.dt)
    return np.abs(g.get_state()[2] - o.get_state()[2]).max()


@pytest.mark.parametrize("precision,tol", [(sl.SL_FP64, 4e-12), (sl.SL_FP32, 6e-5)])
@pytest.mark.parametrize("n,rc", [(4, None), (5, None), (8, None), (8, 4.2), (11, None)])
def test_frozen(n, rc, precision, tol):
    w = W.spin_frozen(n=n)
    if rc:
        w.pot["ex_rc"] = rc
    assert _run(w, 70, precision) < tol


@pytest.mark.parametrize("precision,tol", [(sl.SL_FP64, 1e-12), (sl.SL_FP32, 6e-5)])
@pytest.mark.parametrize("shape", [None, (2, 2, 4096, -1), (4, 1, 4096, 1)])
@pytest.mark.parametrize("physics,n,rc", [("nve", 5, None), ("nve", 6, 4.2), ("nve", 12, None),
                                          ("langevin", 4, None), ("langevin", 6, 4.2), ("langevin", 12, None)])
def test_moving(physics, n, rc, shape, precision, tol):
    w = W.large_langevin(n=n) if physics == "langevin" else W.coupled_nve(n=n)
    w.r = w.r + W.thermal_displacements(w.N, 0.05, 11)
    if rc:
        w.pot["ex_rc"] = rc
    assert _run(w, 20, precision, shape) < tol
