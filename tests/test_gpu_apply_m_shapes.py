"""M and M^dag at the thread counts of their kernels, with workgroups whose
last wavefronts are full, partly filled and empty of cells, against the oracle
(1e-12 in FP64, 3e-6 in FP32, the bounds of the other operator tests)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2508_16298_amd import inputs
from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Nt", [(2, 2), (16, 3), (18, 1), (32, 2), (34, 2), (48, 2), (50, 2), (62, 2), (64, 3), (66, 2)])
@pytest.mark.parametrize("prec,dt,tol", [("fp64", torch.complex128, 1e-12), ("fp32", torch.complex64, 3e-6)])
def test_apply_m_at_thread_counts(L, Nt, prec, dt, tol):
    th = inputs.hot_start_theta(L, Nt, 19 + L)
    v = inputs.gauss_cvec(L, Nt, 20 + L)
    thd, vd = torch.from_numpy(th).cuda(), torch.from_numpy(v).cuda().to(dt)
    with Q.Lattice(L, Nt) as lat:
        for dagger in (False, True):
            got = lat.apply_M(thd, vd, dagger=dagger, prec=prec).cpu().numpy().reshape(-1)
            ref = O.apply_M(O.lat(L, Nt), th, v, dagger=dagger).reshape(-1)
            assert np.linalg.norm(got - ref) / np.linalg.norm(ref) < tol, dagger
