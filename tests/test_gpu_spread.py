"""Jobs with few samples run each sample on several workgroups (pt_mcs): bit
identical to the oracle with and without measurements, modes, the replica walk
and measurement intervals; and to one workgroup per sample where another stream
holds a split launch, through pt_mcs_noalloc and through per-step kernels."""
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


def make(pt, d, L, S, NT, layout, **kw):
    J = W.couplings_pm_j(S, L, d, 7 * L + NT)
    b = W.geometric_betas(0.8 if d == 3 else 0.4, 2.2, NT)
    return (pt.pt_init(S, NT, L, d, J, b, 600 + L, layout=layout, **kw),
            oracle.OracleJob(S, NT, L, d, J, b, 600 + L))


def same(pt, job, ref):
    assert (pt.pt_get_energies(job) == ref.energies()).all()
    for a, b in zip(pt.pt_get_maps(job), ref.maps()):
        assert (a == b).all()
    assert (pt.pt_get_spins(job) == ref.spins()).all()
    assert pt.pt_get_counters(job) == ref.counters()
    gm, rm = pt.pt_get_moments(job), ref.moments()
    for k in rm:
        assert (np.asarray(gm[k]) == np.asarray(rm[k]).astype(np.asarray(gm[k]).dtype)).all(), k


# (dim, L, samples, replicas, layout, walk, modes): parts of one to several
# configurations, a last part that is shorter, both sets inside one part
SHAPES = [(3, 16, 1, 16, 0, False, False), (3, 16, 3, 9, 1, True, False), (3, 14, 2, 13, 0, False, True),
          (3, 20, 2, 5, 1, True, True), (3, 24, 1, 3, 0, False, False), (3, 26, 1, 9, 1, False, False),
          (3, 32, 1, 24, 0, True, False), (2, 64, 2, 12, 0, False, True), (2, 62, 1, 20, 1, True, False),
          (3, 12, 2, 40, 0, False, False)]


@pytest.mark.parametrize("d,L,S,NT,layout,walk,modes", SHAPES)
def test_spread_matches_oracle(pt, d, L, S, NT, layout, walk, modes):
    job, ref = make(pt, d, L, S, NT, layout, walk=walk, modes=modes)
    if modes:
        ref.enable_modes()
    for n, meas, every in ((1, False, 1), (3, True, 1), (5, True, 3), (2, False, 1)):
        pt.pt_set_measure_interval(job, every)
        ref.set_measure_every(every)
        pt.pt_mcs(job, n, measure=meas)
        ref.mcs(n, measure=meas)
        same(pt, job, ref)
    if modes:
        assert (pt.pt_get_modes(job) == ref.modes()).all()
    if walk:
        for a, b in zip(pt.pt_get_walk(job), ref.walk()):
            assert (a == b).all()
    pt.pt_mcs_noalloc(job, 2, measure=True)
    pt.pt_mcs(job, 1, measure=True, plain=True)
    pt.pt_mcs(job, 2, measure=True)
    ref.mcs(5, measure=True)
    same(pt, job, ref)
    pt.pt_destroy(job)


def test_spread_on_two_streams(pt):
    import torch
    streams = [torch.cuda.Stream() for _ in range(2)]
    pairs = [make(pt, 3, 16, 2, 16, 0) for _ in streams]
    for (job, _), st in zip(pairs, streams):
        pt.pt_set_stream(job, st)
    torch.cuda.synchronize()
    for _ in range(4):
        for job, ref in pairs:
            pt.pt_mcs(job, 6, measure=True)
            ref.mcs(6, measure=True)
    for job, ref in pairs:
        same(pt, job, ref)
        pt.pt_destroy(job)
