"""Batched CG at the edges of its iteration kernel: workgroups of several
slices that share their neighbours (a last workgroup with one slice, cells that
do not fill a group, a chain inside one workgroup) and, with one chain too large
for two slices per workgroup, the form that reads them; odd and even budgets,
since the solution is brought up to date every second iteration.  Against the
single-lattice solver after the same few iterations: the two differ by the
order of their sums, 1e-16 (FP32 recursion: 1e-7) growing by the condition of
a few steps, so 1e-11 and 1e-5 after at most 8; and the true residual of whole
solves, recomputed, which differs from the solver's by rounding alone."""
import numpy as np
import pytest
import torch

from paper_2508_16298_amd import inputs
from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu

SHARED = [(2, 2), (6, 5), (8, 17), (12, 9), (16, 5), (20, 7), (22, 2)]


def _cat(arrs):
    return torch.from_numpy(np.concatenate([np.ascontiguousarray(a).reshape(-1) for a in arrs])).cuda()


@pytest.mark.parametrize("sizes", [SHARED, SHARED[:4] + [(34, 3)]], ids=["shared", "own"])
@pytest.mark.parametrize("prec,close", [("fp64", 1e-11), ("fp32", 1e-5)])
def test_batch_iteration_edges(sizes, prec, close):
    ths = [inputs.noisy_pi_flux_theta(L, Nt, 0.3, 70 + c) for c, (L, Nt) in enumerate(sizes)]
    rhs = [inputs.gauss_cvec(L, Nt, 90 + c).reshape(Nt, L, L) for c, (L, Nt) in enumerate(sizes)]
    with Q.Batch(sizes) as b:
        for maxit in (1, 2, 7, 8, 10_000):
            x, st, it, rel = b.cg_solve(_cat(ths), _cat(rhs), tol=1e-9, maxit=maxit, prec=prec)
            for c, (L, Nt) in enumerate(sizes):
                xc = b.vec_view(x, c).reshape(Nt, L, L).contiguous()
                th, v = torch.from_numpy(ths[c]).cuda(), torch.from_numpy(rhs[c]).cuda()
                with Q.Lattice(L, Nt) as lat:
                    if maxit < 10:
                        ref, _, it1, rel1 = lat.cg_solve(th, v, tol=1e-9, maxit=maxit, prec=prec)
                        err = float(torch.linalg.vector_norm(xc - ref) / torch.linalg.vector_norm(ref))
                        assert it[c] == it1 and err <= close, (L, Nt, maxit, it[c], it1, err)
                    else:
                        r = v - lat.apply_MdagM(th, xc, prec="fp64")
                        true = float(torch.linalg.vector_norm(r) / torch.linalg.vector_norm(v))
                        print(L, Nt, it[c], rel[c], true, flush=True)
                        assert st == Q.OK and rel[c] <= 1e-9 and true <= 1.02e-9, (L, Nt)
