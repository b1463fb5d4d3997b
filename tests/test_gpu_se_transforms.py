"""The spin correlator's transforms at the sizes where their kernels change:
one and two blocks of 16 spatial frequencies, one to many blocks of tau
frequencies, four, two and one tile of a pair in LDS (N_tau 254 | 255, 510 |
511), odd N_tau, the largest N_tau, single pairs and ragged chunks of pairs,
against numpy's FFTs.  Bound 1e-12 of max |C|, as for the other correlator
tests: FP64 sums of at most 1137 terms of equal size, twice."""
import numpy as np
import pytest
import torch

import oracle as O
from oracle import se as SE
from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Nt,n_rv", [(2, 1, 2), (2, 3, 2), (6, 31, 3), (8, 33, 9), (30, 5, 3), (32, 6, 3), (44, 7, 2),
                                       (6, 254, 4), (4, 255, 3), (4, 256, 5), (4, 510, 2), (4, 511, 3), (2, 1137, 3)])
def test_correlator_at_block_edges(L, Nt, n_rv):
    rng = np.random.default_rng(1000 * L + Nt)
    xi, X = rng.normal(size=(2, n_rv, Nt, L, L)) + 1j * rng.normal(size=(2, n_rv, Nt, L, L))
    ref = SE.spin_correlator_se(O.lat(L, Nt), xi, X)
    with Q.Stochastic(L, Nt, n_rv) as se:
        C = se.spin_correlator(torch.from_numpy(xi).cuda(), torch.from_numpy(X).cuda()).cpu().numpy()
        again = se.spin_correlator(torch.from_numpy(xi).cuda(), torch.from_numpy(X).cuda()).cpu().numpy()
    assert np.abs(C - ref).max() < 1e-12 * np.abs(ref).max()
    assert np.array_equal(C, again)
