"""M^dag M at theta with the phases formed in the kernel: one thread to a
workgroup of cells, the last sizes of each thread count, the first sizes that
rebuild the phase cache instead, a single slice and two (both neighbours the
same slice), against the oracle (1e-12 in FP64, 3e-6 in FP32, the bounds of the
other operator tests); large angles; and a call at one theta after a call at
another (nothing is kept)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2508_16298_amd import inputs
from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(np.asarray(a).reshape(-1) - b.reshape(-1)) / np.linalg.norm(b)


@pytest.mark.parametrize("L,Nt", [(2, 1), (2, 2), (4, 1), (16, 3), (18, 2), (44, 3), (46, 2), (48, 2), (50, 2)])
@pytest.mark.parametrize("prec,dt,tol", [("fp64", torch.complex128, 1e-12), ("fp32", torch.complex64, 3e-6)])
def test_apply_at_thread_counts(L, Nt, prec, dt, tol):
    th = inputs.hot_start_theta(L, Nt, 9 + L)
    th[0, 0, 0, 0] = 1e6
    th[1, -1, -1, -1] = -3e9
    v = inputs.gauss_cvec(L, Nt, 10 + L)
    ref = O.apply_MdagM(O.lat(L, Nt), th, v)
    with Q.Lattice(L, Nt) as lat:
        thd, vd = torch.from_numpy(th).cuda(), torch.from_numpy(v).cuda().to(dt)
        a = lat.apply_MdagM(thd, vd, prec=prec)
        other = lat.apply_MdagM(torch.zeros_like(thd), vd, prec=prec)
        b = lat.apply_MdagM(thd, vd, prec=prec)
    assert _rel(a.cpu().numpy(), ref) < tol
    assert torch.equal(a, b) and not torch.equal(a, other)
