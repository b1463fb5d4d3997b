"""The spectral preconditioner on both sides of the line between its two forms
(the tau sum fused into the inverse transform or separate), which lies at
different slices in FP32 and FP64: the form taken by itself is one of the two
that can be forced, and they agree up to the order of the same sums, a few
roundings of terms that add up to at most about ten times the result."""
import pytest
import torch

from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Nt", [(24, 25), (26, 25), (48, 13), (50, 13), (58, 14), (60, 14)])
@pytest.mark.parametrize("prec,eps", [("fp64", 2.0**-53), ("fp32", 2.0**-24)])
def test_both_forms(L, Nt, prec, eps, monkeypatch):
    g = torch.Generator(device="cuda").manual_seed(L)
    v = torch.randn((Nt, L, L), dtype=torch.complex128, device="cuda", generator=g)
    v = v if prec == "fp64" else v.to(torch.complex64)
    out = {}
    with Q.Lattice(L, Nt) as lat:
        for f in (None, "1", "0"):
            if f is not None:
                monkeypatch.setenv("QEDHMC_PC_FUSE", f)
            out[f] = lat.apply_precond(v, prec=prec)
    diff = float(torch.linalg.vector_norm(out["1"] - out["0"]) / torch.linalg.vector_norm(out["0"]))
    fused = L <= (24 if prec == "fp64" else 48)
    print(L, prec, diff, flush=True)
    assert torch.equal(out[None], out["1" if fused else "0"]) and diff <= 50 * eps
