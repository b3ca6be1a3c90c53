"""What a pt_mcs call that spreads a job's few samples over more workgroups does
besides its steps: memory, waiting, capture and other streams."""
import gc

import numpy as np
import pytest

import oracle
from paper_2003_04621_amd import workloads as W
from test_gpu_spread import SHAPES

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pt():
    import torch
    assert torch.cuda.is_available()
    from paper_2003_04621_amd import pt as _pt
    _pt.lib()
    return _pt


@pytest.fixture(autouse=True)
def no_other_jobs():
    gc.collect()                            # those that earlier tests dropped


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
    pt.pt_destroy(warm)
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
    assert pt.pt_get_launch(job)["parts"] > 1
    pt.pt_destroy(job)


def cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("d,L,S,NT,layout,walk,modes", SHAPES)
@pytest.mark.parametrize("meas", [False, True])
def test_the_shapes_of_the_spread_tests_spread(pt, d, L, S, NT, layout, walk, modes, meas):
    job, _ = make(pt, d, L, S, NT, layout=layout, walk=walk, modes=modes)
    assert pt.pt_get_launch(job)["mode"] == -2
    plan = pt.pt_get_plan(job, measure=meas)
    pt.pt_mcs(job, 3, measure=meas)
    ran = pt.pt_get_launch(job)
    assert ran["mode"] == 3 and ran["parts"] > plan["parts"] and S * ran["parts"] <= cus(), (plan, ran)
    assert ran["parts"] * ran["per_part"] >= 2 * NT > (ran["parts"] - 1) * ran["per_part"]
    pt.pt_mcs_noalloc(job, 3, measure=meas)
    assert pt.pt_get_launch(job) == plan
    pt.pt_mcs(job, 3, measure=meas, plain=True)
    assert pt.pt_get_launch(job)["mode"] == -1
    pt.pt_destroy(job)


# just outside the rule: too few attempted flips per step, too few words for two
# parts or to fill one workgroup's wavefronts, samples on more than half the CUs,
# Houdayer moves, too few steps in the call; and just inside it
@pytest.mark.parametrize("d,L,samples,NT,steps,houdayer,parts", [
    (3, 8, 8, 31, 300, False, 1), (3, 8, 8, 32, 300, False, 2), (2, 16, 8, 96, 300, False, 1),
    (2, 64, 4, 4, 300, False, 1), (2, 64, 4, 8, 2, False, 1), (2, 64, 4, 8, 3, False, 8),
    (3, 16, "half", 32, 1, False, 2),
    (3, 16, "more", 32, 20, False, 1), (3, 16, 4, 32, 20, True, 1), (3, 8, 8, 32, 10, False, 1),
    (3, 8, 8, 32, 11, False, 4), (3, 16, 2, 10, 1, False, 1), (3, 16, 2, 10, 2, False, 10),
    (3, 14, 1, 24, 1, False, 16)])
def test_where_spreading_begins(pt, d, L, samples, NT, steps, houdayer, parts):
    S = {"half": cus() // 2, "more": cus() // 2 + 1}.get(samples, samples)
    job, _ = make(pt, d, L, S, NT)
    for _ in range(2):
        pt.pt_mcs(job, steps, measure=True, houdayer=houdayer)
        ran, plan = pt.pt_get_launch(job), pt.pt_get_plan(job, measure=True, houdayer=houdayer)
        if parts == 1:
            assert ran == plan
        else:
            assert ran["parts"] >= parts
        pt.pt_mcs(job, 1)                   # another form and other flags between
    pt.pt_destroy(job)


def test_calls_of_few_and_many_steps_mix(pt):
    """One job's calls take either form by their steps, against the oracle."""
    job, ref = make(pt, 3, 16, 3, 9, layout=1)
    plan = pt.pt_get_plan(job, measure=True)
    for n in (1, 1, 4, 1, 2, 3, 7, 7, 1, 30):
        pt.pt_mcs(job, n, measure=True)
        ref.mcs(n, measure=True)
        ran = pt.pt_get_launch(job)
        assert ran == plan if n < 3 else ran["parts"] > 1, n
        same(pt, job, ref)
    pt.pt_destroy(job)


@pytest.mark.parametrize("d,L,S,NT,measure", [(3, 16, 3, 16, True), (2, 64, 2, 12, False)])
def test_capture_of_a_warmed_up_job(pt, d, L, S, NT, measure):
    """pt_mcs with its memory in place records into a caller's graph: replayed
    between the program's own calls, all steps match the oracle."""
    import torch
    st = torch.cuda.Stream()
    job, ref = make(pt, d, L, S, NT)
    pt.pt_set_stream(job, st)
    torch.cuda.synchronize()
    plan = pt.pt_get_plan(job, measure=measure)
    for n in (2, 3):
        pt.pt_mcs(job, n, measure=measure)
    assert pt.pt_get_launch(job)["parts"] > plan["parts"]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        pt.pt_mcs(job, 3, measure=measure)
    assert pt.pt_get_launch(job) == plan
    ref.mcs(5, measure=measure)
    same(pt, job, ref)              # nothing has run yet
    for _ in range(3):
        with torch.cuda.stream(st):
            graph.replay()
        ref.mcs(3, measure=measure)
        same(pt, job, ref)
        pt.pt_mcs(job, 3, measure=measure)
        assert pt.pt_get_launch(job)["parts"] > plan["parts"]
        ref.mcs(3, measure=measure)
        same(pt, job, ref)
    del graph
    pt.pt_mcs(job, 2, measure=measure)
    ref.mcs(2, measure=measure)
    same(pt, job, ref)
    pt.pt_destroy(job)


def test_streams_side_by_side_keep_to_the_plan(pt):
    """Jobs spread only while the process's jobs and batches share one stream;
    each call decides anew, whatever ran before."""
    import torch
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    job, ref = make(pt, 3, 16, 3, 16)
    plan = pt.pt_get_plan(job, measure=True)

    def step(spread):
        pt.pt_mcs(job, 2, measure=True)
        ref.mcs(2, measure=True)
        ran = pt.pt_get_launch(job)
        assert ran["parts"] > plan["parts"] if spread else ran == plan

    pt.pt_set_stream(job, a)
    torch.cuda.synchronize()
    step(True)
    other, oref = make(pt, 3, 16, 2, 16, seed=9)
    pt.pt_set_stream(other, b)
    torch.cuda.synchronize()
    for _ in range(3):                      # side by side
        step(False)
        pt.pt_mcs(other, 3, measure=True)
        oref.mcs(3, measure=True)
        assert pt.pt_get_launch(other) == plan
    torch.cuda.synchronize()
    pt.pt_set_stream(other, a)              # one stream for both
    step(True)
    pt.pt_mcs(other, 3, measure=True)
    oref.mcs(3, measure=True)
    assert pt.pt_get_launch(other)["parts"] > 1
    batch = pt.pt_batch_create([other])
    step(True)
    assert pt.lib().pt_batch_set_stream(batch.h, b.cuda_stream) == pt.PT_OK
    torch.cuda.synchronize()
    step(False)
    pt.pt_batch_run(batch, 2, measure=True)
    oref.mcs(2, measure=True)
    torch.cuda.synchronize()
    pt.pt_batch_destroy(batch)
    step(True)
    same(pt, other, oref)
    pt.pt_destroy(other)
    # a job that began beside another stream's spreads once that is gone
    late, lref = make(pt, 3, 16, 3, 16, seed=11)
    pt.pt_set_stream(late, b)
    torch.cuda.synchronize()
    pt.pt_mcs(late, 2, measure=True)
    assert pt.pt_get_launch(late) == plan
    same(pt, job, ref)
    pt.pt_destroy(job)
    pt.pt_mcs(late, 2, measure=True)
    assert pt.pt_get_launch(late)["parts"] > 1
    lref.mcs(4, measure=True)
    same(pt, late, lref)
    pt.pt_destroy(late)
