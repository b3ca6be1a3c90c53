"""Fused Gaussian steps over the launch shapes: one and several teams per
workgroup, workgroups of 512 and 1024 threads (more and fewer samples than
CUs), lattices with fewer groups than a wavefront and more than a team, the
serial exchange of ladders above 64 temperatures, and samples that nearly fill
the LDS.  Spins, 64-bit energies, maps and moments equal the oracle's."""
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


# (dim, L, samples, replicas, layout, houdayer)
SHAPES = [(2, 6, 300, 2, 0, True), (2, 14, 3, 5, 1, True), (2, 26, 2, 64, 0, False), (2, 8, 2, 65, 1, True),
          (2, 64, 1, 140, 0, False), (2, 62, 257, 2, 0, True), (3, 4, 257, 2, 1, True), (3, 8, 2, 9, 0, True),
          (3, 10, 2, 3, 1, False), (3, 6, 1, 70, 0, True), (3, 22, 1, 12, 0, True)]


@pytest.mark.parametrize("d,L,S,NT,layout,hou", SHAPES)
def test_gauss_fused_shapes(pt, d, L, S, NT, layout, hou):
    Jf = W.couplings_gauss(S, L, d, 500 + L)
    betas = W.geometric_betas(0.4, 2.0, NT)
    job = pt.pt_init_gauss(S, NT, L, d, Jf, betas, 4000 + NT, layout=layout)
    plan = pt.pt_get_plan(job, houdayer=hou, measure=True)
    assert plan["mode"] == 0 and plan["lds_bytes"] <= 160 * 1024
    ref = oracle.OracleGaussJob(S, NT, L, d, W.gauss_units(Jf), betas, 4000 + NT)
    for n in (1, 4):
        pt.pt_mcs(job, n, houdayer=hou, measure=True)
        ref.mcs(n, houdayer=hou, measure=True)
        assert (pt.pt_get_energies64(job) == ref.energies()).all()
        for a, b in zip(pt.pt_get_maps(job), ref.maps()):
            assert (a == b).all()
        assert (pt.pt_get_spins(job) == ref.spins()).all()
    m = ref.moments()
    got = pt.pt_get_moments8(job)
    assert (got[..., 0] == m["E"]).all() and (got[..., 4] == m["Q2"]).all()
    assert (got[..., 1] == m["E2"][..., 0].astype(np.int64)).all()
    assert (got[..., 7] == m["E2"][..., 1].astype(np.int64)).all()
    pt.pt_destroy(job)
