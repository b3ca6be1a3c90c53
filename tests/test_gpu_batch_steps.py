"""Batches whose calls differ only in their number of steps, with a job that has
no fused plan for the flags (its steps run through the per-step kernels): every
job matches the oracle after each call."""
import pytest

import oracle
from paper_2003_04621_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [False, True])
def test_step_count_changes_beside_an_unplanned_job(graph):
    from paper_2003_04621_amd import pt
    jobs, refs = [], []
    for n, (L, S, NT, layout) in enumerate([(8, 2, 4, 1), (32, 1, 4, 0), (12, 1, 3, 0)]):
        J = W.couplings_pm_j(S, L, 3, 230 + n)
        b = W.geometric_betas(0.5, 2.2, NT)
        jobs.append(pt.pt_init(S, NT, L, 3, J, b, 900 + n, layout=layout))
        refs.append(oracle.OracleJob(S, NT, L, 3, J, b, 900 + n))
    assert pt.pt_get_plan(jobs[1], houdayer=True)["mode"] == -1
    batch = pt.pt_batch_create(jobs)
    for steps in (2, 3, 1):
        pt.pt_batch_run(batch, steps, houdayer=True, measure=True, graph=graph)
        for job, ref in zip(jobs, refs):
            ref.mcs(steps, houdayer=True, measure=True)
            assert pt.pt_get_counters(job) == ref.counters(), steps
            assert (pt.pt_get_spins(job) == ref.spins()).all(), steps
            assert (pt.pt_get_energies(job) == ref.energies()).all(), steps
            for x, y in zip(pt.pt_get_maps(job), ref.maps()):
                assert (x == y).all(), steps
    pt.pt_batch_destroy(batch)
    for job in jobs:
        pt.pt_destroy(job)
