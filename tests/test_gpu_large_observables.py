"""Fields, temperatures and the loss where their kernels change with the size: fields on
one wavefront per 64 atoms (above 120 000 atoms; eight below), sums in two passes
(above 8192 terms). Tolerances are those of the same comparisons at small sizes: the
terms are the same and only the order of FP64 sums differs."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1801_10233_amd import spinlat as sl
from paper_1801_10233_amd import workloads as W
from tests.common import make_gpu, make_oracle
from tests.test_gpu_mlp import _blocks, _small_weights

pytestmark = pytest.mark.gpu


def _thermal(n):
    w = W.coupled_nve(n=n)
    w.r = w.r + W.thermal_displacements(w.N, 0.08, 5)
    return w


@pytest.mark.parametrize("n", [39, 40])        # 118 638 and 128 000 atoms
def test_fields_about_the_change_of_shape(n):
    w = _thermal(n)
    F, hw = make_gpu(w).fields()
    o = make_oracle(w)
    Fo, Wo = o.forces(), o.omega() * O.HBAR
    assert np.abs(F - Fo).max() <= 1e-11 * np.abs(Fo).max()
    assert np.abs(hw - Wo).max() <= 1e-13


@pytest.mark.parametrize("n", [15, 16, 17])    # 6750, 8192 and 9826 atoms
def test_temperatures_about_two_passes(n):
    w = _thermal(n)
    TLo, TSo = make_oracle(w).temperatures()
    TLg, TSg = make_gpu(w).temperatures()
    assert TLg == pytest.approx(TLo, rel=1e-10)
    assert TSg == pytest.approx(TSo, rel=1e-9)


def _snapshot(n, p):
    """Snapshot of n^3 cells with references that are off, and the fields there."""
    w = _thermal(n)
    g = make_gpu(w, precision=sl.SL_FP32)
    m = sl.Mlp()
    m.set_weights(p.astype(np.float32))
    g.set_mlp(m)
    g.set_mlp_mode(sl.SL_MLP_PAIRWISE)
    F, hw = g.fields()
    rng = np.random.default_rng(n)
    Fref, Wref = F + 0.1 * rng.standard_normal(F.shape), hw + 0.01 * rng.standard_normal(hw.shape)
    return w, m, F, hw, Fref, Wref


@pytest.mark.parametrize("n", [16, 17])
def test_loss_sum_in_two_passes(n):
    w, m, F, hw, Fref, Wref = _snapshot(n, _small_weights(7))
    ds = sl.Dataset(w.box, w.r[None], w.s[None], np.zeros(1), Fref[None], Wref[None])
    loss, _ = sl.mlp_loss_grad(m, ds, 0, (0.0, 1.0, 30.0))
    want = (((F - Fref) ** 2).sum() + 30.0 * ((hw - Wref) ** 2).sum()) / (3 * w.N)
    assert loss == pytest.approx(want, rel=1e-10)


def test_gradient_of_more_than_8192_pairs():
    # a snapshot of 128 atoms (3712 pairs: sums in one pass) and eight copies of it (two
    # passes) have the same loss and gradient: every term is a mean over atoms, and 8 is a
    # power of two, so the copies' products are the same numbers scaled. What differs is
    # the order of FP32 sums over 512 partial sums at most per thread: 512 x 2^-24 = 3e-5
    # of the sum of absolute terms, allowed to be 300 times a block's largest component.
    # (c3 is left out: its second component is an exact zero, a difference of large sums.)
    p = _small_weights(7)
    w, m, F, hw, Fref, Wref = _snapshot(4, p)
    shift = np.array([[x, y, z] for x in (0, 1) for y in (0, 1) for z in (0, 1)]) * w.box
    tile = lambda a: np.concatenate([a] * 8)
    one = sl.Dataset(w.box, w.r[None], w.s[None], np.array([3.0]), Fref[None], Wref[None])
    r8 = np.concatenate([w.r + d for d in shift])
    eight = sl.Dataset(2 * w.box, r8[None], tile(w.s)[None], np.array([24.0]), tile(Fref)[None],
                       tile(Wref)[None])
    l1, g1 = sl.mlp_loss_grad(m, one, 0, (1.0, 0.5, 30.0))
    l8, g8 = sl.mlp_loss_grad(m, eight, 0, (1.0, 0.5, 30.0))
    assert l8 == pytest.approx(l1, rel=1e-6)
    b1, b8 = _blocks(g1.astype(np.float64)), _blocks(g8.astype(np.float64))
    for name in ("W1", "c1", "W2", "c2", "W3"):
        err = np.abs(b8[name] - b1[name]).max() / np.abs(b1[name]).max()
        print(name, err, flush=True)
        assert err < 1e-2, name
