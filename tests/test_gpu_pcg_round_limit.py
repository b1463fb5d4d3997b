"""A preconditioned solve that its round limit ends returns what it has: the
solution it reached, its iterations and its last true residual, and no
convergence.  The limit lies beyond every solve's rounds; here it is two (20
triples of launches), which a solve to 1e-12 outlasts."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2508_16298_amd import inputs
from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [Q.FP64, Q.FP32])
def test_outputs_at_the_limit(prec):
    L, Nt = 8, 24
    th = torch.from_numpy(inputs.noisy_pi_flux_theta(L, Nt, 0.3, 61)).cuda()
    rhs = torch.from_numpy(np.ascontiguousarray(inputs.gauss_cvec(L, Nt, 62).reshape(Nt, L, L))).cuda()
    fn = Q.load()._ZN2qh14pcg_solve_implEP10qedhmc_ctxPKdPddi16qedhmc_precisionPiS4_S6_bl
    fn.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_double, C.c_int, C.c_int, C.c_void_p, C.c_void_p,
                   C.c_void_p, C.c_bool, C.c_long]
    with Q.Lattice(L, Nt) as lat:
        _, st, full, _ = lat.cg_solve(th, rhs, tol=1e-12, prec=prec, precond="paper")  # leaves the phases of th
        assert st == Q.OK and full > 20
        x = torch.full_like(rhs, 3.0)
        it, nrel, rel = C.c_int(-1), C.c_int(-1), C.c_double(-1.0)
        st = fn(lat.h, rhs.data_ptr(), x.data_ptr(), 1e-12, 10_000, prec, C.byref(it), C.byref(rel), C.byref(nrel),
                False, 2)
        r = rhs - lat.apply_MdagM(th, x, prec="fp64")
        true = float(torch.linalg.vector_norm(r) / torch.linalg.vector_norm(rhs))
        print(it.value, rel.value, nrel.value, true, flush=True)
        assert st == Q.ENOCONV and "did not end" in Q.last_error()
        assert 10 <= it.value <= 20 and nrel.value >= 0 and 1e-12 < rel.value <= 1.0
        assert true < 0.5 and not bool((x == 3.0).any())
