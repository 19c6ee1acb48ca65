"""Rows with more conflicting neighbours than the 16 that a packed colouring row
holds (an exchange cutoff of 4.2 A: 26 in bcc iron). The colours are whole numbers:
exactly the oracle's, with the state of the colouring in LDS (up to 57 344 atoms)
and in memory. A long row is shared by the lanes of its atom: twice the neighbours
cost a build about twice the time, so less than six times is asked (one lane per
long row took 17 times)."""
import time

import numpy as np
import pytest

from paper_1801_10233_amd import workloads as W
from tests.common import make_gpu, make_oracle

pytestmark = pytest.mark.gpu


def _thermal(n, rc):
    w = W.coupled_nve(n=n)
    w.r = w.r + W.thermal_displacements(w.N, 0.05, 11)
    w.pot = dict(w.pot, ex_rc=rc)
    return w


@pytest.mark.parametrize("n", [5, 31])
def test_long_rows_colour_exactly(n):
    w = _thermal(n, 4.2)
    o, g = make_oracle(w), make_gpu(w)
    o.build()
    g.step(0, w.dt)
    co, Ko = o.coloring()
    cg, Kg = g.coloring()
    assert Ko == Kg and np.array_equal(co, cg)


def test_long_rows_cost_what_their_length_does():
    best = {}
    for rc in (3.5, 4.2):
        w = _thermal(40, rc)
        g = make_gpu(w)
        times = []
        for _ in range(6):
            g.set_state(r=w.r)
            g.synchronize()
            t = time.perf_counter()
            g.step(0, w.dt)
            g.synchronize()
            times.append(time.perf_counter() - t)
        best[rc] = min(times)
        g.close()
    print("build seconds", best, flush=True)
    assert best[4.2] < 6.0 * best[3.5]
