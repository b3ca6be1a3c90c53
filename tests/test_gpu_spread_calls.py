"""What a pt_mcs call that spreads a job's few samples over more workgroups does
besides its steps: memory, waiting, capture and other streams."""
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


def make(pt, d, L, S, NT, seed=600, **kw):
    J = W.couplings_pm_j(S, L, d, 7 * L + NT)
    b = W.geometric_betas(0.8 if d == 3 else 0.4, 2.2, NT)
    return pt.pt_init(S, NT, L, d, J, b, seed, **kw), oracle.OracleJob(S, NT, L, d, J, b, seed)


def same(pt, job, ref):
    assert pt.pt_get_counters(job) == ref.counters()
    assert (pt.pt_get_energies(job) == ref.energies()).all()
    assert (pt.pt_get_spins(job) == ref.spins()).all()
    for a, b in zip(pt.pt_get_maps(job), ref.maps()):
        assert (a == b).all()
    gm, rm = pt.pt_get_moments(job), ref.moments()
    for k in rm:
        assert (np.asarray(gm[k]) == np.asarray(rm[k]).astype(np.asarray(gm[k]).dtype)).all(), k


def test_first_call_only_enqueues(pt):
    """The first pt_mcs of a spread job waits for no other stream and asks the
    allocator hooks for nothing."""
    import torch
    warm, _ = make(pt, 3, 16, 3, 16)        # code and per-process memory in place
    pt.pt_mcs(warm, 1, measure=True)
    pt.pt_get_energies(warm)
    sizes = []

    def alloc(n, ctx):
        sizes.append(int(n))
        return torch.cuda.caching_allocator_alloc(int(n))

    pt.pt_set_allocator(alloc, lambda p, ctx: torch.cuda.caching_allocator_delete(int(p)) if p else None)
    try:
        job, ref = make(pt, 3, 16, 3, 16)
    finally:
        pt.use_torch_memory()
    held = sum(sizes)
    assert held <= pt.pt_job_bytes(3, 16, 16, 3, W.geometric_betas(0.8, 2.2, 16))
    busy, own = torch.cuda.Stream(), torch.cuda.Stream()
    pt.pt_set_stream(job, own)
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        torch.cuda._sleep(500_000_000)      # some 0.2 s
        done = torch.cuda.Event()
        done.record(busy)
    pt.pt_mcs(job, 4, measure=True)
    assert not done.query()
    torch.cuda.synchronize()
    assert sum(sizes) == held
    ref.mcs(4, measure=True)
    same(pt, job, ref)
    pt.pt_destroy(job)
    pt.pt_destroy(warm)
