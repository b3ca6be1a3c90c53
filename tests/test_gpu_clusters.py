"""Single-cluster Houdayer moves at the sizes where a cluster can go wrong: in
registers, rows of 2 to 32 sites per colour, one to several row fields per word,
lattices that fill the wavefront's lanes and lattices that leave lanes empty;
in LDS, lattices of more words than lanes; and the per-step kernels.  Ladders
start cold, so that clusters wrap around the lattice.  Everything is exact:
spins, energies, maps and moments equal the oracle's."""
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


CASES += [(3, L, 2, nt, lay, 12) for L, nt, lay in
          [(4, 3, 0), (6, 2, 1), (8, 5, 0), (10, 18, 0), (12, 4, 1), (14, 3, 0), (16, 4, 0), (16, 17, 1), (18, 2, 0),
           (20, 3, 1), (24, 2, 0)]]


def same(pt, job, ref):
    for a, b in zip(pt.pt_get_maps(job), ref.maps()):
        assert (a == b).all()
    assert (pt.pt_get_spins(job) == ref.spins()).all()


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
        same(pt, job, ref)
        gm, rm = pt.pt_get_moments(job), ref.moments()
        for k in rm:
            assert (np.asarray(gm[k]) == np.asarray(rm[k]).astype(np.asarray(gm[k]).dtype)).all(), k
    pt.pt_destroy(job)


@pytest.mark.parametrize("plain", [False, True])
@pytest.mark.parametrize("d,L,S,NT,layout,steps", CASES)
def test_gauss_clusters_match_oracle(pt, d, L, S, NT, layout, steps, plain):
    J = W.couplings_gauss(S, L, d, 60 + L)
    betas = W.geometric_betas(0.3 if d == 2 else 0.7, 2.5, NT)
    job = pt.pt_init_gauss(S, NT, L, d, J, betas, 99 + L, layout=layout)
    assert pt.pt_get_plan(job, houdayer=True, plain=plain)["mode"] == (-1 if plain else 0)
    ref = oracle.OracleGaussJob(S, NT, L, d, W.gauss_units(J), betas, 99 + L)
    pt.pt_mcs(job, steps, houdayer=True, measure=True, plain=plain)
    ref.mcs(steps, houdayer=True, measure=True)
    assert (pt.pt_get_energies64(job) == ref.energies()).all()
    same(pt, job, ref)
    pt.pt_destroy(job)


@pytest.mark.parametrize("d,L,S,NT,layout,steps", CASES + [(3, 28, 1, 2, 0, 3), (3, 32, 1, 2, 1, 3), (3, 36, 1, 2, 0, 2)])
def test_step_clusters_match_oracle(pt, d, L, S, NT, layout, steps):
    J = W.couplings_pm_j(S, L, d, 20 + L)
    betas = W.geometric_betas(0.3 if d == 2 else 0.7, 2.5, NT)
    job = pt.pt_init(S, NT, L, d, J, betas, 55 + L, layout=layout, stats=True)
    ref = oracle.OracleJob(S, NT, L, d, J, betas, 55 + L)
    pt.pt_mcs(job, steps, houdayer=True, measure=True)
    ref.mcs(steps, houdayer=True, measure=True)
    assert (pt.pt_get_energies(job) == ref.energies()).all()
    same(pt, job, ref)
    pt.pt_destroy(job)


# rows with the most runs a row can hold (alternating sites), whole-row and
# wrapping runs, row counts that are no multiple of the wavefront, and
# workgroups with fewer wavefronts than scratch areas
@pytest.mark.parametrize("threads", [0, 256])
@pytest.mark.parametrize("d,L,S,NT", [(2, 4, 2, 3), (2, 10, 2, 2), (2, 26, 2, 3), (2, 50, 1, 12), (2, 64, 1, 9),
                                      (3, 4, 2, 2), (3, 10, 1, 3), (3, 12, 1, 6), (3, 14, 1, 2), (3, 20, 1, 2)])
def test_multi_clusters_match_oracle(pt, d, L, S, NT, threads):
    J = W.couplings_pm_j(S, L, d, 30 + L)
    betas = W.geometric_betas(0.3 if d == 2 else 0.7, 2.5, NT)
    job = pt.pt_init(S, NT, L, d, J, betas, 45 + L)
    ref = oracle.OracleJob(S, NT, L, d, J, betas, 45 + L)
    x = np.indices((L,) * d).sum(axis=0).reshape(-1)
    spins = pt.pt_get_spins(job)
    spins[:, 0] = spins[:, NT] * np.where(x % 2 == 0, -1, 1)  # checkerboard overlap
    if NT > 2:
        spins[:, 1] = -spins[:, NT + 1]                       # q = -1 everywhere
        cols = (np.arange(L ** d) % L)                        # whole columns, one wrapping
        spins[:, 2] = spins[:, NT + 2] * np.where((cols % 4 == 0) | (cols == L - 1), -1, 1)
    pt.pt_set_spins(job, spins)
    ref.set_spins(spins)
    pt.pt_houdayer_multi(job)  # on those overlaps
    ref.houdayer(multi=True)
    assert (pt.pt_get_energies(job) == ref.energies()).all()
    same(pt, job, ref)
    batch = pt.pt_batch_create([job])
    pt.pt_batch_set_config(batch, threads, 2, 0)
    pt.pt_batch_run(batch, 6, houdayer=True, multi=True, measure=True)
    ref.mcs(6, houdayer=True, multi=True, measure=True)
    assert (pt.pt_get_energies(job) == ref.energies()).all()
    same(pt, job, ref)
    pt.pt_batch_destroy(batch)
    pt.pt_destroy(job)


# per-step exchange and measurement: ladders of one and two decision words and
# of more than a wavefront, lattices of 16-byte and 4-byte rows of loads
@pytest.mark.parametrize("d,L,S,NT,layout", [(3, 8, 3, 32, 0), (2, 6, 3, 33, 0), (2, 10, 2, 64, 1), (2, 6, 2, 70, 1),
                                             (3, 6, 300, 2, 0), (3, 32, 1, 3, 0), (2, 64, 2, 17, 1)])
def test_per_step_exchange_and_measure_match_oracle(pt, d, L, S, NT, layout):
    J = W.couplings_pm_j(S, L, d, 70 + L)
    betas = W.geometric_betas(0.6, 2.0, NT)
    job = pt.pt_init(S, NT, L, d, J, betas, 13 + L, layout=layout, walk=True, modes=True)
    ref = oracle.OracleJob(S, NT, L, d, J, betas, 13 + L)
    ref.enable_modes()
    for n, meas, every in ((4, True, 1), (3, False, 1), (5, True, 2), (1, True, 3)):
        pt.pt_set_measure_interval(job, every)
        ref.set_measure_every(every)
        pt.pt_mcs(job, n, measure=meas, plain=True)
        ref.mcs(n, measure=meas)
        assert pt.pt_get_counters(job) == ref.counters()
        same(pt, job, ref)
    pt.pt_exchange(job)
    pt.pt_measure(job)
    ref.exchange()
    ref.measure()
    assert pt.pt_get_counters(job) == ref.counters()
    same(pt, job, ref)
    gm, rm = pt.pt_get_moments(job), ref.moments()
    for k in rm:
        assert (np.asarray(gm[k]) == np.asarray(rm[k]).astype(np.asarray(gm[k]).dtype)).all(), k
    for a, b in zip(pt.pt_get_walk(job), ref.walk()):
        assert (a == b).all()
    assert (pt.pt_get_modes(job) == ref.modes()).all()
    pt.pt_destroy(job)


# the spins of an int8 job between the steps of one call: sizes whose packed
# words fill their int8 bytes, whose lattices do and do not start 16-byte
# aligned, one and several words per thread
@pytest.mark.parametrize("d,L,S,NT,multi", [(2, 4, 3, 3, False), (2, 6, 5, 3, True), (2, 14, 3, 4, False),
                                            (2, 50, 2, 3, True), (2, 64, 2, 3, False), (3, 4, 3, 3, True),
                                            (3, 6, 3, 3, False), (3, 16, 2, 3, True), (3, 28, 1, 2, False)])
def test_int8_jobs_step_as_packed_ones(pt, d, L, S, NT, multi):
    J = W.couplings_pm_j(S, L, d, 80 + L)
    betas = W.geometric_betas(0.5, 2.0, NT)
    job = pt.pt_init(S, NT, L, d, J, betas, 17 + L, layout=0, modes=True)
    ref = oracle.OracleJob(S, NT, L, d, J, betas, 17 + L)
    ref.enable_modes()
    for n, hou in ((2, False), (1, True), (4, True), (3, False)):
        pt.pt_mcs(job, n, houdayer=hou, measure=True, plain=True, multi=multi and hou)
        ref.mcs(n, houdayer=hou, measure=True, multi=multi and hou)
        assert (pt.pt_get_energies(job) == ref.energies()).all()
        same(pt, job, ref)
        assert (pt.pt_get_modes(job) == ref.modes()).all()
        gm, rm = pt.pt_get_moments(job), ref.moments()
        for k in rm:
            assert (np.asarray(gm[k]) == np.asarray(rm[k]).astype(np.asarray(gm[k]).dtype)).all(), k
    pt.pt_destroy(job)
