"""The list and the colouring at the sizes where their kernels change (states of
the colouring in LDS up to 57 344 atoms, 8 threads or one per row in the row
order), and batched replicas whose classes straddle the 256 atoms below which a
replica's classes run in its tail. Lists and colours are whole numbers: exactly
the oracle's. Batched: FP64 as the other batch tests, 1e-10 after 20 steps; in FP32
against the persistent mode, which draws the same noise, so at most 80 updates that
differ by the summation order, 2e-7 or less each: 2e-5."""
import numpy as np
import pytest

from paper_1801_10233_amd import spinlat as sl
from paper_1801_10233_amd import workloads as W
from tests.common import make_gpu, make_oracle, row_sets

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 16, 30, 31])
def test_list_and_colouring_exact(n):
    w = W.coupled_nve(n=n)
    w.r = w.r + W.thermal_displacements(w.N, 0.12, 77)
    o, g = make_oracle(w), make_gpu(w)
    o.build()
    g.step(0, w.dt)
    nso, _, ro = o.neighbor_list()
    nsg, _, rg = g.neighbor_list()
    assert row_sets(ro, nso, "spin") == row_sets(rg, nsg, "spin")
    co, Ko = o.coloring()
    cg, Kg = g.coloring()
    assert Ko == Kg and np.array_equal(co, cg)


def _batch(lo, hi):
    ws = W.batched_replicas(R=3, seed=31, n_lo=lo, n_hi=hi)
    for k, w in enumerate(ws):
        w.r = w.r + W.thermal_displacements(w.N, 0.05, 11 + k)
    return ws


SIZES = pytest.mark.parametrize("lo,hi", [(4, 5), (7, 9), (11, 13)])


@SIZES
def test_batch_tails_and_phases_fp64(lo, hi):
    ws = _batch(lo, hi)
    b = sl.Batch(ws, precision=sl.SL_FP64)
    b.set_mode(sl.SL_BATCH_PHASED)
    b.step(20, 1e-4)
    for k, w in enumerate(ws):
        o = make_oracle(w)
        o.step(20, 1e-4)
        assert np.abs(b.get_state(k)[2] - o.get_state()[2]).max() < 1e-10


@SIZES
def test_batch_tails_and_phases_fp32(lo, hi):
    spins = []
    for mode in (sl.SL_BATCH_PHASED, sl.SL_BATCH_PERSISTENT):
        b = sl.Batch(_batch(lo, hi), precision=sl.SL_FP32)
        b.set_mode(mode)
        b.step(20, 1e-4)
        spins.append([b.get_state(k)[2] for k in range(3)])
    for x, y in zip(*spins):
        assert np.abs(x - y).max() < 2e-5
