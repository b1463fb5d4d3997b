"""The preconditioner's launches behind a solver's stop flag: with the flag set
they are no-ops for every thread of every workgroup, those without a momentum
(L^2 / 2 is no whole number of wavefronts at L = 2, 6, 10, 24, 30) among them,
so a vector they would write stays as it was; with the flag clear they give
what the public call gives.  The sizes take the tau sum fused into the inverse
transform, its separate form (L = 60) and the stencil passes (N_tau = 12)."""
import ctypes as C

import pytest
import torch

from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu

PREC = {"fp64": (0, torch.complex128), "fp32": (1, torch.complex64)}


def _apply(lat, prec, v, out, stop):
    fn = Q.load()._ZN2qh20launch_apply_precondEP10qedhmc_ctx16qedhmc_precisionPKvPvPKd
    fn.argtypes = [C.c_void_p, C.c_int, C.c_void_p, C.c_void_p, C.c_void_p]
    assert fn(lat.h, PREC[prec][0], v.data_ptr(), out.data_ptr(), stop.data_ptr()) == Q.OK
    torch.cuda.synchronize()


@pytest.mark.parametrize("L,Nt", [(2, 13), (6, 14), (10, 13), (24, 17), (30, 13), (44, 13), (60, 13), (8, 12)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_stopped_launches_write_nothing(L, Nt, prec):
    g = torch.Generator(device="cuda").manual_seed(L)
    v = torch.randn((Nt, L, L), dtype=torch.complex128, device="cuda", generator=g).to(PREC[prec][1])
    with Q.Lattice(L, Nt) as lat:
        want = lat.apply_precond(v, prec=prec)
        out = torch.full_like(v, 7.0 - 3.0j)
        for flag in (1.0, 2.0, 5.0):
            _apply(lat, prec, v, out, torch.full((1,), flag, dtype=torch.float64, device="cuda"))
            assert bool((out == 7.0 - 3.0j).all()), (L, Nt, prec, flag)
        _apply(lat, prec, v, out, torch.zeros(1, dtype=torch.float64, device="cuda"))
        assert torch.equal(out, want)
