"""One training step at the sizes where the matrix-core training kernels
change: a single slice (every tau tap wraps), bricks of the weight gradient
that are ragged in y (14 = 5 + 5 + 4), in x (50 = 17 + 17 + 16) or split in x
(26 = 13 + 13), tiles of 16 sites that end ragged (N = 4, 12), and workgroups
that walk several tiles and bricks (24 x 60), against the oracle.  Bounds as
for the other training tests (1e-5 of the loss, 1e-4 of each gradient: FP32
sums of at most a few thousand terms of either sign)."""
import numpy as np
import pytest
import torch

import oracle as O
from oracle import net as NN
from paper_2508_16298_amd import inputs
from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu


def _rel(a, b):
    a, b = np.asarray(a, float).reshape(-1), np.asarray(b, float).reshape(-1)
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("L,Nt", [(2, 1), (2, 3), (6, 1), (14, 2), (26, 2), (50, 2), (24, 60)])
def test_train_step_at_tile_edges(L, Nt):
    th = inputs.noisy_pi_flux_theta(L, Nt, 0.3, 70 + L)
    r = inputs.gauss_cvec(L, Nt, 71 + L)
    p = O.lat(L, Nt)
    rng = np.random.default_rng(5)
    params = [(W.astype(np.float32).astype(float), rng.normal(0, 0.1, b.shape).astype(np.float32).astype(float))
              for W, b in inputs.net_init_weights(3)]
    loss_o, grads_o = NN.loss_and_grads_residual(params, th, r, lambda v: O.apply_MdagM(p, th, v).reshape(Nt, L, L))
    with Q.Lattice(L, Nt) as lat, Q.Net(lat) as net:
        net.set_params(params)
        loss, g = net.train_step_residual(torch.from_numpy(th).cuda(), torch.from_numpy(r).cuda(), lr=1e-3,
                                          want_grad=True)
        back = net.get_params()
        net.set_params(params)
        assert np.array_equal(net.get_params(), Q.Net.pack(params))
    assert abs(loss - loss_o) <= 1e-5 * loss_o
    for (gW, gb), (oW, ob) in zip(Q.Net.unpack(g), grads_o):
        assert _rel(gW, oW) <= 1e-4 and _rel(gb, ob) <= 1e-4
    assert back.shape == g.shape and not np.array_equal(back, Q.Net.pack(params))
