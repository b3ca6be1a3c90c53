"""Allocator hooks set by pt_set_allocator belong to the jobs created under them
until those jobs are destroyed."""
import gc

import pytest

from paper_2003_04621_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_a_job_keeps_its_hooks():
    import torch
    from paper_2003_04621_amd import pt
    held = set()

    def alloc(n, ctx):
        p = torch.cuda.caching_allocator_alloc(int(n))
        held.add(p)
        return p

    def free(p, ctx):
        if p:
            held.remove(p)
            torch.cuda.caching_allocator_delete(int(p))

    pt.pt_set_allocator(alloc, free)
    try:
        job = pt.pt_init(2, 3, 4, 2, W.couplings_pm_j(2, 4, 2, 1), W.geometric_betas(0.5, 2.0, 3), 1)
        other = pt.pt_init_gauss(2, 3, 4, 2, W.couplings_gauss(2, 4, 2, 1), W.geometric_betas(0.5, 2.0, 3), 1)
    finally:
        pt.use_torch_memory()
    gc.collect()
    assert held
    pt.pt_mcs(job, 2)
    pt.pt_mcs(other, 2)
    pt.pt_destroy(job)
    pt.pt_destroy(other)
    assert not held
