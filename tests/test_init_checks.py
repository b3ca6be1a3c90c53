"""Couplings that pt_init takes (host only: an accepted job then fails for want of
a device), and spins that pt_set_spins takes."""
import ctypes as C

import numpy as np
import pytest


@pytest.mark.parametrize("at", [0, 17, 31])
def test_only_unit_couplings_pass(at):
    import torch
    from paper_2003_04621_amd import pt
    L = pt.lib()
    b = np.array([1.0, 0.5])
    for c in range(-128, 128):
        if c in (1, -1) and torch.cuda.is_available():
            continue
        J = np.where(np.arange(32) % 3 == 0, 1, -1).astype(np.int8)
        J[at] = c
        h = C.c_void_p()
        rc = L.pt_init_ex(C.byref(h), 1, 2, 4, 2, pt._p(J), pt._p(b), C.c_uint64(1), 0)
        assert (rc == pt.PT_EINVAL) == (c not in (1, -1)), c
        assert not h.value


@pytest.mark.gpu
@pytest.mark.parametrize("layout", [0, 1])
def test_only_unit_spins_pass(layout):
    from paper_2003_04621_amd import pt, workloads as W
    job = pt.pt_init(1, 3, 6, 3, W.couplings_pm_j(1, 6, 3, 1), W.geometric_betas(0.8, 2.0, 3), 5, layout=layout)
    old = pt.pt_get_spins(job)
    n = old.size
    for at in (0, 65, n - 1):
        for c in range(-128, 128):
            s = old.copy()
            s.reshape(-1)[at] = c
            rc = pt.lib().pt_set_spins(job.h, pt._p(s))
            assert (rc == pt.PT_EINVAL) == (c not in (1, -1)), c
            assert (pt.pt_get_spins(job) == (s if rc == 0 else old)).all()
            if rc == 0:
                old = s
    pt.pt_destroy(job)
