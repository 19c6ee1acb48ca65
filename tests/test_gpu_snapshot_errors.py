"""A snapshot too dense for the list: the loss names the rows it met, and the
handle goes on with the next snapshot."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1801_10233_amd import spinlat as sl
from paper_1801_10233_amd import workloads as W

pytestmark = pytest.mark.gpu


def _dense(n, a):
    r, _ = W.bcc_lattice(n, a)
    return r + 0.02 * np.random.default_rng(3).standard_normal(r.shape), np.array([n * a] * 3)


def test_row_overflow_of_a_loss_names_the_rows():
    r, box = _dense(6, 2.0)                    # some 130 neighbours within 5 A
    s = W.random_unit_spins(len(r), 5)
    z = np.zeros((1,) + r.shape)
    m = sl.Mlp()
    m.set_weights((np.random.default_rng(7).standard_normal(sl.SL_MLP_NPARAM) * 0.2).astype(np.float32))
    ds = sl.Dataset(box, r[None], s[None], np.zeros(1), z, z)

    def longest(rc):
        return np.bincount(O.brute_pairs(r, box, rc)[0], minlength=len(r)).max()

    rows, spin = longest(5.0), longest(3.5)
    assert rows > 80
    with pytest.raises(sl.SpinLatError) as e:
        sl.mlp_loss_grad(m, ds, 0)
    assert e.value.code == sl.SL_E_NBR_OVERFLOW
    assert f"seen {rows} (spin {spin})" in str(e.value)
    r, box = _dense(6, W.BCC_A)                # the next snapshot fits
    loss, grad = sl.mlp_loss_grad(m, sl.Dataset(box, r[None], s[None], np.zeros(1), z, z), 0)
    assert np.isfinite(loss) and np.isfinite(grad).all()
