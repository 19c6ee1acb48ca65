"""List capacities. One far above the rows it holds (the caller's choice, which also
bounds the launches over slots) changes nothing: the learned potential's pairs and
the exchange cache of a caller's list, 128 atoms, bit for bit as with the default. The
cache is sized by the spin segment, down to fewer slots than a first round reads."""
import ctypes
import os

import numpy as np
import pytest

from paper_1801_10233_amd import spinlat as sl
from paper_1801_10233_amd import workloads as W
from tests.common import make_gpu, make_oracle

pytestmark = pytest.mark.gpu


def _free_bytes():
    hip = ctypes.CDLL("libamdhip64.so.7")
    free, total = ctypes.c_size_t(), ctypes.c_size_t()
    assert hip.hipMemGetInfo(ctypes.byref(free), ctypes.byref(total)) == 0
    return free.value


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


@pytest.mark.parametrize("precision", [sl.SL_FP64, sl.SL_FP32])
def test_exchange_cache_is_sized_by_the_spin_segment(precision):
    # 8192 atoms, rows of up to 4000 slots, at most 32 of them in the spin segment:
    # two caches of 32 slots are 4.2 MB in FP64, of 4000 slots 524 MB
    w = W.large_langevin(n=16)
    g = make_gpu(w, precision=precision, max_nbr=4000)
    g.set_tuning(2, 2, -1, 1)
    g.step(0, w.dt)
    free0 = _free_bytes()
    g.step(2, w.dt)
    g.synchronize()
    assert free0 - _free_bytes() < 64 << 20


def test_exchange_cache_follows_a_callers_longer_rows():
    # the spin segment of a caller's list may be longer than max_spin_nbr: the caches
    # of the built list (16 slots) grow for it, and the run
    # is the one of a system that held the list from the start
    w = W.coupled_nve(n=6)
    w.pot = dict(w.pot, ex_rc=4.2)
    full = make_gpu(w)
    full.step(0, w.dt)
    _, na, rows = full.neighbor_list()
    off, idx = np.concatenate([[0], np.cumsum(na)]), np.concatenate(rows)
    runs = []
    for first in (True, False):
        g = make_gpu(w, max_spin_nbr=16)
        g.set_tuning(2, 2, -1, 1)
        if first:                              # caches of 16 slots, at both positions
            short = dict(w.pot, ex_rc=3.5)
            g.set_potential(short)
            g.step(3, w.dt)
            g.set_potential(w.pot)
            g.set_state(w.r, w.v, w.s)
            g.set_step(0)
        g.set_neighbor_list(off, idx)
        g.step(5, w.dt)
        runs.append(g)
    for x, y in zip(runs[0].get_state(), runs[1].get_state()):
        assert np.abs(x - y).max() < 1e-12 * max(1.0, np.abs(y).max())


@pytest.mark.parametrize("shape", [(0, 0, 0, 0), (1, 1, -1, 1), (2, 2, 4096, 1), (4, 4, -1, 1), (8, 8, -1, 1)])
@pytest.mark.parametrize("physics", ["nve", "langevin"])
def test_fewer_slots_than_a_first_round(physics, shape):
    # eight nearest neighbours, and room for no more
    w = W.coupled_nve(n=6) if physics == "nve" else W.large_langevin(n=6)
    w.pot = dict(w.pot, ex_rc=2.55)
    w.skin = 0.2
    o, g = make_oracle(w), make_gpu(w, max_spin_nbr=8)
    g.set_tuning(*shape)
    o.step(10, w.dt)
    g.step(10, w.dt)
    assert g.stats()["max_spin_nbr_seen"] == 8
    assert np.abs(g.get_state()[2] - o.get_state()[2]).max() < 1e-12
