"""The float32 networks against float64, with a bound that operands of 11 bits
(the first halves of the float16 pairs alone) do not meet.

Bound: 64 times each output's spread when every operand of every product, every
product and every CELU errs independently by up to 2^-24 of itself.  16 of it
hold the largest of a million such errors, whose tails are longer than a normal
distribution's; 4 hold the accumulators' own roundings (four per 32 terms, within
one unit in the last place of a partial sum: 4.2 times the spread of 1,024 terms
of either sign).  An operand of 11 bits errs by up to 2^-12."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2405_01491_amd as nnp
from tests.gpu_helpers import dev
from tests.test_gpu_networks import features

TRIALS = 8


def exact(x):
    return x


def spread(rng):
    return lambda x: x * (1.0 + 2.0 ** -24 * rng.uniform(-1, 1, x.shape))


def eleven_bits(x):
    """The nearest number with 11 bits."""
    m, e = np.frexp(x)
    return np.ldexp(np.round(m * 2.0 ** 11) / 2.0 ** 11, e)


def networks(a, species, spec, act=exact, weight=exact, out=exact):
    """Energies and dE/dAEV in float64, with each product's operands passed
    through act and weight and every layer's results through out."""
    al = float(np.float32(spec.celu_alpha))
    E, G = np.zeros(len(a)), np.zeros((len(a), spec.aev_dim))
    for s in np.unique(species):
        at = species == s
        W = [np.asarray(w, np.float64) for w, _ in spec.weights[s]]
        h, D = a[at, :spec.aev_dim].astype(np.float64), []
        for k in range(3):
            z = out(act(h) @ weight(W[k]).T) + np.asarray(spec.weights[s][k][1], np.float64)
            e = out(np.exp(np.minimum(z, 0.0) / al))
            h = np.maximum(z, 0.0) + al * (e - 1.0)
            D.append(e)
        E[at] = out(out(h) @ W[3][0] + float(spec.weights[s][3][1][0]))
        d = np.broadcast_to(W[3][0], h.shape)
        for k in (2, 1, 0):
            d = out(act(out(d * D[k])) @ weight(W[k]))
        G[at] = d
    return E, G


def bounds(a, species, spec):
    E, G = networks(a, species, spec)
    vE, vG = np.zeros_like(E), np.zeros_like(G)
    for t in range(TRIALS):
        s = spread(np.random.default_rng(100 + t))
        e, g = networks(a, species, spec, s, s, s)
        vE += (e - E) ** 2 / TRIALS
        vG += (g - G) ** 2 / TRIALS
    # a few trials see an element's own spread only roughly
    sG = np.maximum(np.sqrt(vG), 0.5 * np.sqrt(vG.mean(1))[:, None])
    sE = np.maximum(np.sqrt(vE), 0.5 * np.sqrt(np.median(vE)) * np.minimum(1.0, np.abs(E) / np.median(np.abs(E))))
    return E, G, 64 * sE, 64 * sG


def beyond(e, g, ref):
    E, G, tE, tG = ref
    return np.abs(e - E) / tE, (np.abs(g - G) / tG).max(1)


def inputs(spec, n):
    a, species = features(n, n, -(-spec.aev_dim // 64) * 64, spec.aev_dim)
    return a, species


@pytest.mark.parametrize("n", [33, 250])
@pytest.mark.parametrize("dropped", ["activations", "weights"])
def test_eleven_bits_are_seen(spec_bias, n, dropped):
    a, species = inputs(spec_bias, n)
    ref = bounds(a, species, spec_bias)
    e, g = networks(a, species, spec_bias, **{"act" if dropped == "activations" else "weight": eleven_bits})
    xE, xG = beyond(e, g, ref)
    print("n %d, %s of 11 bits: energies %.3g, dE/dAEV %.3g of the bound (medians)" %
          (n, dropped, np.median(xE), np.median(xG)))
    assert np.mean(xG > 1) > 0.9 and np.mean(xE > 1) > 0.5


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 33, 250, 4113])
def test_networks_within_the_spread(spec_bias, n):
    a, species = inputs(spec_bias, n)
    # the atomic energies as the networks give them: no self energy in their float
    m = nnp.Model(dataclasses.replace(spec_bias, self_energy=np.zeros(spec_bias.n_species)), "fp32")
    e, g = nnp.nnp_mlp(m, torch.from_numpy(species).to(dev()), torch.from_numpy(a).to(dev()))
    xE, xG = beyond(e.cpu().numpy().astype(np.float64), g.cpu().numpy()[:, :spec_bias.aev_dim],
                    bounds(a, species, spec_bias))
    print("n %d: energies %.3g, dE/dAEV %.3g of the bound" % (n, xE.max(), xG.max()))
    assert xE.max() <= 1 and xG.max() <= 1
