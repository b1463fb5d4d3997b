"""Rounding of the weight gradients' FP32 sums on a lattice of 2^19 sites.

With hidden weights zero the activations are one constant per channel, so every
tap of the last layer's dW is that constant times one and the same sum of the
output gradient over the lattice, known in FP64; with one channel per output
that enters by +-1/8 at two taps, the sums of the hidden layer before it are
zero.  What is left is the rounding of the sums.  A running sum of n terms of
random sign is rounded at every term by at most half a unit of 2^-24 / sqrt(3)
RMS of its size, which grows as the root of the terms: sqrt(n / 2) 2^-24 /
sqrt(3) of the final size.  The sums hold at most 288 sites here before they
are added in FP64: 4.13e-7."""
import numpy as np
import pytest
import torch

from paper_2508_16298_amd import qedhmc as Q

pytestmark = pytest.mark.gpu

CH = (6, 32, 32, 32, 32, 32, 2)
BOUND = np.sqrt(288 / 2) * 2.0**-24 / np.sqrt(3)


def _rounding(L, Nt, seed):
    """Mean squares of the hidden and the last layer's errors in units of the sums' random size."""
    N = L * L * Nt
    g = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    r, e = (torch.randn((Nt, L, L), dtype=torch.complex128, device="cuda", generator=g) for _ in range(2))
    W = [np.zeros((CH[l + 1], CH[l], 27), np.float32) for l in range(6)]
    b = [rng.uniform(0.5, 1.5, CH[l + 1]).astype(np.float32) for l in range(5)] + [np.zeros(2, np.float32)]
    for o, c in enumerate((3, 17)):
        W[5][o, c, 0], W[5][o, c, 26] = 0.125, -0.125  # the outputs are exactly zero
    with Q.Lattice(L, Nt) as lat, Q.Net(lat) as n:
        n.set_params(list(zip(W, b)))
        _, grad = n.train_step(torch.zeros((2, Nt, L, L), dtype=torch.float64, device="cuda"), r, e, lr=0.0,
                               want_grad=True)
    G = Q.Net.unpack(grad.astype(np.float64))
    sig = [1 / (1 + np.exp(-x.astype(np.float64))) for x in b]
    act = [x * s for x, s in zip(b, sig)]
    d4 = sig[4] * (1 + b[4] * (1 - sig[4]))
    c = 2 * float(torch.sqrt(r.abs().square().sum() / N)) / float(e.abs().square().sum())
    out = [(-c * t).to(torch.float32).to(torch.float64) for t in (e.real, e.imag)]
    size = [float(t.square().sum().sqrt()) for t in out]
    last = [(G[5][0][o] - act[4][:, None] * float(out[o].sum())) / (act[4][:, None] * size[o]) for o in range(2)]
    hidden = [G[4][0][ch] / (act[3][:, None] * d4[ch] * 0.125 * np.sqrt(2) * size[o]) for o, ch in enumerate((3, 17))]
    return [float(np.mean(np.square(x))) for x in (hidden, last)]


def test_sums_are_no_longer_than_stated():
    rms = np.sqrt(np.mean([_rounding(64, 128, s) for s in range(1, 7)], axis=0))
    print(rms, BOUND, flush=True)
    assert (rms <= BOUND).all()
