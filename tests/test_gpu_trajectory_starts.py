"""What a trajectory reports of warm starts that do not iterate, the same with
and without the paper's preconditioner: angles that are no numbers leave no
finite residual, so the proposal is rejected with an infinite one and only the
first solve counts; steps so short that the previous solution still meets the
target add no iterations and no reliable updates (FP64: one, the first
solve's check)."""
import math

import pytest
import torch

from paper_2508_16298_amd import inputs
from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu
L, NT = 6, 16


def _run(theta, precond, prec, length, direct, monkeypatch):
    if direct:
        monkeypatch.setenv("QEDHMC_NO_GRAPH", "1")
    with Q.Lattice(L, NT, seed=2) as lat:
        return lat.hmc_trajectory(theta, 0, 3, length, tol=1e-6, prec=prec, precond=precond)


@pytest.mark.parametrize("bad", [math.nan, math.inf])
@pytest.mark.parametrize("precond,direct", [(None, False), ("paper", False), ("paper", True)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_angles_that_are_no_numbers(bad, precond, direct, prec, monkeypatch):
    th = torch.from_numpy(inputs.noisy_pi_flux_theta(L, NT, 0.3, 3)).cuda()
    th.view(-1)[7] = bad
    r = _run(th, precond, prec, 0.06, direct, monkeypatch)
    assert r["status"] == 2 and r["accepted"] == 0 and r["max_true_resid"] == math.inf
    assert (r["n_solves"], r["cg_iters_total"], r["reliable_updates"]) == (1, 0, 0)


@pytest.mark.parametrize("precond,direct", [(None, False), ("paper", False), ("paper", True)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_starts_that_meet_the_target(precond, direct, prec, monkeypatch):
    th = torch.from_numpy(inputs.noisy_pi_flux_theta(L, NT, 0.3, 3)).cuda()
    with Q.Lattice(L, NT, seed=2) as lat:
        _, R = lat.heatbath(0)
        eta = lat.apply_M(th, R, dagger=True)
        it = lat.cg_solve(th, eta, tol=1e-6, prec=prec, precond=precond)[2]
    r = _run(th, precond, prec, 1e-9, direct, monkeypatch)
    assert r["status"] == 0 and r["n_solves"] == 4 and r["cg_iters_total"] == it == r["cg_iters_max"]
    if prec == "fp64":
        assert r["reliable_updates"] == 1
