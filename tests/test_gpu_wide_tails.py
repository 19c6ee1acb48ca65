"""Runs of classes in one workgroup with classes of more atoms than its four-wavefront
teams take in a pass (128): on teams of two, and with more successive updates of a class
than those draw noise for (a single class: no neighbours within the cutoff) on teams of
four. FP64: 20 steps of roundoff, so 1e-12; FP32: at most 160 updates, each off by 2e-7
or less, so 4e-5 against the FP64 oracle."""
import numpy as np
import pytest

from paper_1801_10233_amd import spinlat as sl
from paper_1801_10233_amd import workloads as W
from tests.common import make_gpu, make_oracle

pytestmark = pytest.mark.gpu

TOL = {sl.SL_FP64: 1e-12, sl.SL_FP32: 4e-5}


def _spins(w, precision, shape, steps):
    o, g = make_oracle(w), make_gpu(w, precision=precision)
    g.set_tuning(*shape)
    o.step(steps, w.dt)
    g.step(steps, w.dt)
    return np.abs(g.get_state()[2] - o.get_state()[2]).max()


@pytest.mark.parametrize("precision", [sl.SL_FP64, sl.SL_FP32])
@pytest.mark.parametrize("jcache", [-1, 1])
@pytest.mark.parametrize("physics,n", [("langevin", 7), ("langevin", 9), ("nve", 8), ("nve", 13)])
def test_classes_about_the_limit(physics, n, jcache, precision):
    # 686 to 4394 atoms in 9 to 11 classes of 2 to 600 atoms
    w = W.large_langevin(n=n) if physics == "langevin" else W.coupled_nve(n=n)
    w.r = w.r + W.thermal_displacements(w.N, 0.05, 11)
    assert _spins(w, precision, (2, 2, 4096, jcache), 20) < TOL[precision]


@pytest.mark.parametrize("precision", [sl.SL_FP64, sl.SL_FP32])
@pytest.mark.parametrize("frozen", [True, False])
def test_one_class_with_the_bath(frozen, precision):
    w = W.large_langevin(n=6)
    w.pot = dict(w.pot, ex_rc=2.0)             # nearest neighbours are 2.48 A apart
    w.frozen = frozen
    assert _spins(w, precision, (2, 2, 4096, -1), 20) < TOL[precision]
