"""A list capacity far above the rows it holds (the caller's choice, which also
bounds the launches over slots) changes nothing: the learned potential's pairs and
the exchange cache of a caller's list, 128 atoms, bit for bit as with the default."""
import os

import numpy as np
import pytest

from paper_1801_10233_amd import spinlat as sl
from paper_1801_10233_amd import workloads as W
from tests.common import make_gpu

pytestmark = pytest.mark.gpu


def _states_equal(a, b):
    for x, y in zip(a.get_state(), b.get_state()):
        assert np.array_equal(x, y)


def test_pairs_of_the_learned_potential():
    w = W.coupled_nve(n=4)
    w.r = w.r + W.thermal_displacements(w.N, 0.05, 11)
    mlp = sl.Mlp()
    mlp.set_weights(np.load(os.path.join(os.path.dirname(sl.__file__), "data", "mlp_bj_weights.npy")))
    runs = []
    for cap in (0, 70000):
        g = make_gpu(w, precision=sl.SL_FP32, max_nbr=cap)
        g.set_mlp(mlp)
        g.set_mlp_mode(sl.SL_MLP_PAIRWISE)
        g.step(5, w.dt)
        runs.append(g)
    _states_equal(*runs)


@pytest.mark.parametrize("precision", [sl.SL_FP64, sl.SL_FP32])
def test_exchange_cache_of_a_callers_list(precision):
    w = W.coupled_nve(n=4)
    g0 = make_gpu(w, precision=precision)
    g0.step(0, w.dt)
    _, na, rows = g0.neighbor_list()
    off = np.concatenate([[0], np.cumsum(na)])
    runs = []
    for cap in (0, 400000):
        g = make_gpu(w, precision=precision, max_nbr=cap)
        g.set_neighbor_list(off, np.concatenate(rows))
        g.set_tuning(2, 2, -1, 1)
        g.step(5, w.dt)
        runs.append(g)
    _states_equal(*runs)
