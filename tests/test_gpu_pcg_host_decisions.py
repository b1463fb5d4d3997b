"""QEDHMC_NO_GRAPH with the paper's preconditioner: the host launches every
iteration and takes every decision (stop, reliable update, budget, stall), and
the results are those of the solve that decides on the device, bit for bit.
That the host decides shows in the launches: it makes none past the budget,
where rounds of ten triples would run on."""
import numpy as np
import pytest
import torch

from paper_2508_16298_amd import inputs
from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu


def _case(L, Nt):
    th = torch.from_numpy(inputs.noisy_pi_flux_theta(L, Nt, 0.3, 80 + L)).cuda()
    return th, torch.from_numpy(np.ascontiguousarray(inputs.gauss_cvec(L, Nt, 81 + L).reshape(Nt, L, L))).cuda()


@pytest.mark.parametrize("L,Nt", [(4, 12), (8, 20), (44, 13)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_launches_end_with_the_budget(L, Nt, prec, monkeypatch):
    th, rhs = _case(L, Nt)
    monkeypatch.setenv("QEDHMC_NO_GRAPH", "1")
    with Q.Lattice(L, Nt) as lat:
        lat.profile(1)
        _, st, it, _ = lat.cg_solve(th, rhs, tol=1e-12, maxit=3, prec=prec, precond="paper")
        count = lat.profile_read(Q.K_PCG_MV_FP64 if prec == "fp64" else Q.K_PCG_MV_FP32)[0]
        assert st == Q.ENOCONV and it == 3 and 3 <= count <= 6, count


@pytest.mark.parametrize("L,Nt", [(4, 12), (8, 40), (24, 24)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_stall_and_odd_ends(L, Nt, prec, monkeypatch):
    """Tolerances that no solve reaches (the updates stop making progress), a
    budget of one, and a right-hand side at the edge of what squares hold."""
    th, rhs = _case(L, Nt)
    cases = [(rhs, 1e-18, 10_000), (rhs, 1e-15, 400), (rhs, 1e-9, 1), (rhs * 1e150, 1e-9, 10_000), (rhs * 0, 1e-9, 5)]
    with Q.Lattice(L, Nt) as lat:
        dev = [lat.cg_solve(th, b, tol=t, maxit=m, prec=prec, precond="paper") for b, t, m in cases]
        monkeypatch.setenv("QEDHMC_NO_GRAPH", "1")
        for (b, t, m), d in zip(cases, dev):
            x, *rest = lat.cg_solve(th, b, tol=t, maxit=m, prec=prec, precond="paper")
            print(L, prec, t, m, rest, d[1:], flush=True)
            assert np.array_equal(np.array(rest), np.array(d[1:]), equal_nan=True)
            assert torch.equal(torch.view_as_real(x).nan_to_num(1.0), torch.view_as_real(d[0]).nan_to_num(1.0))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_warm_starts_of_a_trajectory(prec, monkeypatch):
    L, Nt = 8, 40
    th, _ = _case(L, Nt)
    out = []
    for direct in (False, True):
        if direct:
            monkeypatch.setenv("QEDHMC_NO_GRAPH", "1")
        with Q.Lattice(L, Nt, seed=5) as lat:
            t = th.clone()
            out.append((t, lat.hmc_trajectory(t, 0, 3, 0.06, tol=1e-9, prec=prec, precond="paper")))
    assert torch.equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]
