"""The paper preconditioner's spectral form at the sizes where its kernels
change: one to five blocks of 16 DFT outputs per axis with full and nearly
empty last blocks, even and odd L/2, tables in LDS and in memory, the tau sum
fused and separate, against the oracle's stencil.  Tolerances: the oracle's
own sums are FP64; an output adds about 50 blocks and two transforms of at
most 128 points of values of order one, so 1e-12 in FP64 and 5e-6 in FP32 (the
bounds of the other preconditioner tests)."""
import functools

import numpy as np
import pytest
import torch

import oracle as O
from oracle import precond as PC
from paper_2508_16298_amd import inputs
from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=1)
def _taps():
    return PC.build_stencil(8, 24, cap=Q.PC_TAU_REACH)[0]


def _rel(a, b):
    a, b = np.asarray(a).reshape(-1), np.asarray(b).reshape(-1)
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("L,Nt", [(2, 13), (6, 27), (30, 14), (32, 13), (58, 13), (62, 15), (64, 13), (66, 14), (94, 13),
                                  (96, 13), (128, 13)])
def test_apply_at_block_edges(L, Nt, monkeypatch):
    v = inputs.gauss_cvec(L, Nt, 51 + L)
    ref = PC.apply_P(_taps(), v)
    with Q.Lattice(L, Nt) as lat:
        for prec, dt, tol in (("fp64", torch.complex128, 1e-12), ("fp32", torch.complex64, 5e-6)):
            if prec == "fp64" and L > 90:  # the stencil kernels take these
                continue
            for fuse in ("0", "1"):
                monkeypatch.setenv("QEDHMC_PC_FUSE", fuse)
                out = lat.apply_precond(torch.from_numpy(v).cuda().to(dt), prec=prec).cpu().numpy()
                assert _rel(out, ref) < tol, (L, Nt, prec, fuse)


@pytest.mark.parametrize("prec,dt,tol", [("fp64", torch.complex128, 1e-12), ("fp32", torch.complex64, 5e-6)])
@pytest.mark.parametrize("fuse", ["0", "1"])
def test_apply_takes_element_aligned_vectors(prec, dt, tol, fuse, monkeypatch):
    """in and out one element past an aligned address."""
    monkeypatch.setenv("QEDHMC_PC_FUSE", fuse)
    L, Nt = 10, 16
    v = inputs.gauss_cvec(L, Nt, 5)
    a = torch.zeros(v.size + 1, dtype=dt, device="cuda")
    b = torch.zeros(v.size + 2, dtype=dt, device="cuda")
    a[1:] = torch.from_numpy(v).cuda().to(dt).reshape(-1)
    with Q.Lattice(L, Nt) as lat:
        lat.apply_precond(a[1:].view(Nt, L, L), prec=prec, out=b[1:-1].view(Nt, L, L))
    assert _rel(b[1:-1].cpu().numpy(), PC.apply_P(_taps(), v)) < tol
    assert b[0] == 0 and b[-1] == 0


@pytest.mark.parametrize("L", [6, 34, 66, 96])
def test_solve_with_the_update_kernels_transform(L):
    """The PCG's update kernel transforms r itself: mixed solves at one size
    per instantiation, by the oracle's true residual."""
    Nt, tol = 14, 1e-9
    p = O.lat(L, Nt)
    th = inputs.noisy_pi_flux_theta(L, Nt, 0.3, 3)
    eta = O.apply_M(p, th, inputs.gauss_cvec(L, Nt, 4), dagger=True).reshape(Nt, L, L)
    with Q.Lattice(L, Nt) as lat:
        x, st, it, rel = lat.cg_solve(torch.from_numpy(th).cuda(), torch.from_numpy(eta).cuda(), tol=tol, prec="fp32",
                                      precond="paper")
        _, _, it0, _ = lat.cg_solve(torch.from_numpy(th).cuda(), torch.from_numpy(eta).cuda(), tol=tol, prec="fp32")
    assert st == Q.OK and rel <= tol and it < it0
    r = eta.reshape(-1) - O.apply_MdagM(p, th, x.cpu().numpy()).reshape(-1)
    assert np.linalg.norm(r) <= 1.05 * tol * np.linalg.norm(eta)
