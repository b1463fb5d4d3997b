"""Plain CG on slices of 513 to 1024 cells, one workgroup of more than 512
threads each: odd and even budgets (the solution takes two steps at a time)
against textbook CG with the FP64 operator.  The same iterates up to rounding,
1e-16 (FP32 recursion: 1e-7) growing by the condition of at most 8 steps."""
import numpy as np
import pytest
import torch

from paper_2508_16298_amd import inputs
from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Nt", [(46, 5), (48, 2), (64, 3)])
@pytest.mark.parametrize("prec,close", [("fp64", 1e-11), ("fp32", 1e-5)])
def test_budgets(L, Nt, prec, close):
    th = torch.from_numpy(inputs.noisy_pi_flux_theta(L, Nt, 0.3, 7 + L)).cuda()
    b = torch.from_numpy(np.ascontiguousarray(inputs.gauss_cvec(L, Nt, 8 + L).reshape(Nt, L, L))).cuda()
    with Q.Lattice(L, Nt) as lat:
        x, r = torch.zeros_like(b), b.clone()
        p, rr = r.clone(), torch.sum(r.abs() ** 2)
        want = {}
        for k in range(1, 9):
            s = lat.apply_MdagM(th, p, prec="fp64")
            alpha = rr / torch.sum((p.conj() * s).real)
            x, r = x + alpha * p, r - alpha * s
            rn = torch.sum(r.abs() ** 2)
            p, rr = r + (rn / rr) * p, rn
            want[k] = x
        for k in (1, 2, 7, 8):
            got, st, it, _ = lat.cg_solve(th, b, tol=1e-12, maxit=k, prec=prec)
            err = float(torch.linalg.vector_norm(got - want[k]) / torch.linalg.vector_norm(want[k]))
            assert st == Q.ENOCONV and it == k and err < close, (L, k, err)
