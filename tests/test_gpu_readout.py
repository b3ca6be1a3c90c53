"""Reading spins from the packed layout: row fields of 2 to 32 sites per colour,
one to several fields per word, against the int8 layout's plain copy."""
import numpy as np
import pytest

from paper_2003_04621_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,L", [(2, 4), (2, 6), (2, 10), (2, 18), (2, 26), (2, 32), (2, 50), (2, 62), (2, 64),
                                 (3, 4), (3, 6), (3, 10), (3, 12), (3, 14), (3, 24)])
def test_packed_spins_read_as_int8(d, L):
    from paper_2003_04621_amd import pt
    J, b = W.couplings_pm_j(2, L, d, 3), W.geometric_betas(0.5, 2.0, 3)
    a = pt.pt_init(2, 3, L, d, J, b, 9, layout=pt.PT_LAYOUT_INT8)
    p = pt.pt_init(2, 3, L, d, J, b, 9, layout=pt.PT_LAYOUT_PACKED)
    for job in (a, p):
        pt.pt_sweep(job, 2)
    assert (pt.pt_get_spins(a) == pt.pt_get_spins(p)).all()
    x = np.random.default_rng(L).choice(np.array([-1, 1], np.int8), pt.pt_get_spins(p).shape)
    pt.pt_set_spins(p, x)
    assert (pt.pt_get_spins(p) == x).all()
