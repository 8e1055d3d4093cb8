"""The species networks (float32 form) hold every bit of their weights: networks
whose weights all need the last of their 24 bits, all rounded the same way if
it is dropped, on atoms whose terms are all positive.

Tolerance: each of the three layers may err by half the unit roundoff of
float32 (2^-25 of the value) in the mean over atoms.  Weights without their last
bit are too large by 2^-23 / 1.5 in the mean, 2.4e-7 over three layers."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2405_01491_amd as nnp
from tests.gpu_helpers import dev

pytestmark = pytest.mark.gpu
TOL = 3 * 2.0 ** -25


def last_bits(rng, shape, exponent):
    """2^exponent m, m in [2^23, 2^24) whole: 11 bits, and a remainder that is
    odd, above 2^11, and 3 mod 4 (nearest-even of its upper 11 bits: up)."""
    m = rng.integers(2 ** 10, 2 ** 11, shape) * 2 ** 13 + 2 ** 11 + 4 * rng.integers(0, 2 ** 9, shape) + 3
    return np.ldexp(m.astype(np.float64), exponent - 24).astype(np.float32)


@pytest.mark.parametrize("seed", [1, 2])
def test_means_over_atoms(spec, seed):
    rng = np.random.default_rng(seed)
    w, net = list(spec.widths), []
    for _ in range(spec.n_species):
        net.append([(last_bits(rng, (w[k + 1], w[k]), (-9, -7, -7)[k]),
                     rng.uniform(0.0, 0.1, w[k + 1]).astype(np.float32)) for k in range(3)] +
                   [(rng.uniform(0.5, 1.0, (1, w[3])).astype(np.float32), np.zeros(1, np.float32))])
    m = nnp.Model(dataclasses.replace(spec, weights=net), "fp32")
    n, dim = 700, w[0]
    a = np.zeros((n, m.aev_stride), np.float32)
    a[:, :dim] = rng.uniform(0.1, 1.0, (n, dim))
    species = np.arange(n, dtype=np.int32) % spec.n_species
    E, G = nnp.nnp_mlp(m, torch.from_numpy(species).to(dev()), torch.from_numpy(a).to(dev()))
    E, G = E.cpu().numpy().astype(np.float64), G.cpu().numpy().astype(np.float64)
    for k in range(spec.n_species):
        at = species == k
        W = [x.astype(np.float64) for x, _ in net[k]]
        h, g = a[at, :dim].astype(np.float64), W[3][0]
        for layer in range(3):   # every value is positive: CELU leaves it
            h = h @ W[layer].T + net[k][layer][1].astype(np.float64)
        for layer in (2, 1, 0):
            g = g @ W[layer]
        e = (E[at] / (h @ W[3][0]) - 1).mean()
        d = (G[at, :dim] / g - 1).mean()
        print("species %d: energies %.1e, dE/dAEV %.1e" % (k, e, d))
        assert abs(e) <= TOL and abs(d) <= TOL
