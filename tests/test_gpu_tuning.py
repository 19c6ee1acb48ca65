"""The launch shape that is reported is the one that runs: set again, on the same
system or on a fresh one, it gives the same launches, so the same bits."""
import itertools

import numpy as np
import pytest

from paper_1801_10233_amd import spinlat as sl
from paper_1801_10233_amd import workloads as W
from tests.common import make_gpu

pytestmark = pytest.mark.gpu

KEYS = ("spin_lanes", "force_lanes", "jcache")


def test_reported_tuning_is_a_fixed_point():
    g = make_gpu(W.coupled_nve(n=4))
    seen = set()
    for s, f, j in itertools.product((0, 1, 2, 4, 8), (0, 1, 2, 4, 8), (0, -1, 1)):
        g.set_tuning(s, f, 0, j)
        t = g.tuning()
        default = (s, f, j) in ((0, 0, 0), (2, 1, 0))
        assert tuple(t[k] for k in KEYS) == ((2, 1, 0) if default else (s, f, j))
        g.set_tuning(**t)
        assert g.tuning() == t
        seen.add(tuple(t[k] for k in KEYS))
    assert len(seen) == 5 * 5 * 3 - 1


@pytest.mark.parametrize("precision", [sl.SL_FP64, sl.SL_FP32])
@pytest.mark.parametrize("shape", [(0, 0, 0), (0, 2, 0), (0, 0, 1), (4, 0, 0), (2, 2, 0), (2, 1, 1), (2, 1, -1)])
@pytest.mark.parametrize("n", [6, 14])     # with and without the one-workgroup form
def test_set_tuning_of_the_reported_one_changes_no_bit(n, shape, precision):
    w = W.coupled_nve(n=n)
    w.r = w.r + W.thermal_displacements(w.N, 0.05, 11)
    spin, force, jc = shape
    runs = []
    for again in (False, True):
        g = make_gpu(w, precision=precision)
        if shape != (0, 0, 0):
            g.set_tuning(spin, force, 0, jc)
        if again:
            t = g.tuning()
            g = make_gpu(w, precision=precision)
            g.set_tuning(**t)
        g.step(10, w.dt)
        runs.append(g.get_state())
    for a, b in zip(*runs):
        assert np.array_equal(a, b)
