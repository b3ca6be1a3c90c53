"""Single-cluster Houdayer moves inside the fused steps at the sizes where the
in-register cluster can go wrong: rows of 2 to 32 sites per colour, one to
several row fields per word, lattices that fill the wavefront's lanes and
lattices that leave lanes empty.  Ladders start cold, so that clusters wrap
around the lattice.  Everything is exact: spins, energies, maps and moments
equal the oracle's (+-J) or the per-step kernels' (Gaussian couplings)."""
import numpy as np
import pytest

import oracle
from paper_2003_04621_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pt():
    import torch
    assert torch.cuda.is_available()
    from paper_2003_04621_amd import pt as _pt
    _pt.lib()
    return _pt


# (dim, L, samples, replicas, layout, steps)
CASES = [(2, L, 2, nt, lay, 30) for L, nt, lay in
         [(4, 2, 0), (8, 3, 1), (12, 5, 0), (16, 4, 0), (18, 3, 1), (22, 4, 0), (28, 2, 1), (32, 20, 0),
          (34, 3, 0), (46, 3, 1), (48, 4, 0), (50, 17, 1), (62, 3, 0), (64, 4, 0)]]


@pytest.mark.parametrize("d,L,S,NT,layout,steps", CASES)
def test_fused_clusters_match_oracle(pt, d, L, S, NT, layout, steps):
    J = W.couplings_pm_j(S, L, d, 40 + L)
    betas = W.geometric_betas(0.3 if d == 2 else 0.7, 2.5, NT)
    job = pt.pt_init(S, NT, L, d, J, betas, 77 + L, layout=layout)
    assert pt.pt_get_plan(job, houdayer=True, measure=True)["mode"] == 1
    ref = oracle.OracleJob(S, NT, L, d, J, betas, 77 + L)
    for n in (1, steps):
        pt.pt_mcs(job, n, houdayer=True, measure=True)
        ref.mcs(n, houdayer=True, measure=True)
        assert (pt.pt_get_energies(job) == ref.energies()).all()
        for a, b in zip(pt.pt_get_maps(job), ref.maps()):
            assert (a == b).all()
        assert (pt.pt_get_spins(job) == ref.spins()).all()
        gm, rm = pt.pt_get_moments(job), ref.moments()
        for k in rm:
            assert (np.asarray(gm[k]) == np.asarray(rm[k]).astype(np.asarray(gm[k]).dtype)).all(), k
    pt.pt_destroy(job)


@pytest.mark.parametrize("d,L,S,NT,layout,steps", CASES)
def test_fused_clusters_match_steps_gauss(pt, d, L, S, NT, layout, steps):
    J = W.couplings_gauss(S, L, d, 60 + L)
    betas = W.geometric_betas(0.3 if d == 2 else 0.7, 2.5, NT)
    a = pt.pt_init_gauss(S, NT, L, d, J, betas, 99 + L, layout=layout)
    b = pt.pt_init_gauss(S, NT, L, d, J, betas, 99 + L, layout=layout)
    assert pt.pt_get_plan(a, houdayer=True)["mode"] == 0
    pt.pt_mcs(a, steps, houdayer=True, measure=True)
    pt.pt_mcs(b, steps, houdayer=True, measure=True, plain=True)
    assert (pt.pt_get_energies64(a) == pt.pt_get_energies64(b)).all()
    for x, y in zip(pt.pt_get_maps(a), pt.pt_get_maps(b)):
        assert (x == y).all()
    assert (pt.pt_get_spins(a) == pt.pt_get_spins(b)).all()
    assert (pt.pt_get_moments8(a) == pt.pt_get_moments8(b)).all()
    pt.pt_destroy(a)
    pt.pt_destroy(b)
