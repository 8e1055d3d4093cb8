"""The forces' mean error over many pairs where only the cutoff function acts.
An error that is the same for every pair adds up in a box's virial.

The radial Gaussians are flat (eta = 1e-9) and the networks linear with weights
that are powers of two, so that a pair's force is its cutoff's slope times a
known number.  Tolerance of the mean, relative: the sine of these angles (0.45 to
0.71) is the hardware's, within one unit in the last place below 1/2 to 1 (at
most 2^-24 over 0.45: 1.3e-7); every other rounding is to nearest and leaves no
mean."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2405_01491_amd as nnp
from tests.gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rc", [5.1, 3.5, 5.2, 4.0])
def test_mean_over_distances(spec, rc):
    n, w = 20000, spec.widths
    rng = np.random.default_rng(7)
    net = [(np.full((w[k + 1], w[k]), 2.0 ** e, np.float32), np.full(w[k + 1], b, np.float32))
           for k, (e, b) in enumerate([(-10, 0.125), (-8, 0.125), (-8, 0.125), (-7, 0.0)])]
    g = float(w[1] * w[2] * w[3]) * 2.0 ** -33
    flat = dataclasses.replace(spec, rc_r=rc, rc_a=min(rc, spec.rc_a) / 4, eta_r=1e-9, weights=[net] * spec.n_species)
    pos = rng.uniform(-3, 3, (n, 2, 3))
    d = rng.normal(size=(n, 3))
    pos[:, 1] = pos[:, 0] + d * (rng.uniform(0.75, 0.85, n) * rc / np.linalg.norm(d, axis=1))[:, None]
    pos = pos.astype(np.float32)
    m = nnp.Model(flat, "fp32")
    x = torch.from_numpy(pos.reshape(-1, 3)).to(dev())
    species = torch.zeros(2 * n, dtype=torch.int32, device=dev())
    mol = torch.arange(2 * n, dtype=torch.int32, device=dev()) // 2
    _, _, F = nnp.nnp_energy_forces(m, x, species, mol, n, None)
    F = F.cpu().numpy().reshape(n, 2, 3).astype(np.float64)
    v = pos[:, 1].astype(np.float64) - pos[:, 0]
    r = np.linalg.norm(v, axis=1)
    t = np.pi / float(np.float32(rc))
    away = np.float64(r[:, None]) - spec.shf_r.astype(np.float64)
    e = np.exp(-1e-9 * away ** 2)
    slope = spec.radial_prefactor * (e * (-0.5 * t * np.sin(t * r)[:, None]
                                          - 2e-9 * away * (0.5 * np.cos(t * r) + 0.5)[:, None])).sum(1)
    # the force on the first atom along the pair: both atoms' energies pull
    err = (F[:, 0] * v).sum(1) / r / (2 * g * slope) - 1
    print("rc %.1f: mean relative error of the forces %.1e, rms %.1e" % (rc, err.mean(), err.std()))
    assert abs(err.mean()) <= 2.0 ** -24 / 0.45
