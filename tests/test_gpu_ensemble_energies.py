"""Every network's structure energies, from the kernels that sum all networks
in one launch, against the networks evaluated one by one.

Tolerance: both sides add float32 atomic energies in float64; an atomic energy
is the same but for the rounding of its network's value, 2^-20 of the sum of
the magnitudes that enter it (bounded by 16 times the largest atomic energy
here, biases and weights being of order one)."""
import numpy as np
import pytest
import torch

import paper_2405_01491_amd as nnp
import synthetic
from tests.gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


# one workgroup's structure (the largest, 8,192 atoms, and one atom in a box), a
# structure summed in chunks, and structures side by side, short and long
@pytest.mark.parametrize("n,n_mol", [(1, 1), (8192, 1), (8193, 1), (9000, 3), (4000, 1000)])
@pytest.mark.parametrize("nets", [2, 5])
def test_structure_energies_of_every_network(n, n_mol, nets):
    whole = synthetic.ani2x_like_ensemble(n_nets=nets, weight_seed=7, bias_scale=0.05)
    w = synthetic.geometry.water_box(-(-n // 3))
    mol = np.sort(np.arange(n) % n_mol).astype(np.int32)
    w.pos, w.species, w.mol, w.n_mol = w.pos[:n], w.species[:n], mol, n_mol
    w.box = w.box if n > 100 else np.array([14.0, 14.0, 14.0], np.float32)
    pos, sp, mo = to_dev(w)
    m = nnp.Model(whole, "fp32")
    mo = mo if n_mol > 1 else None
    nl = nnp.nnp_neighbors(m, pos, mo, n_mol, w.box, 5.1)
    e_mol, e_net, e_atom, _ = nnp.nnp_energy_forces_ensemble(m, pos, sp, mo, n_mol, w.box, nl, e_atom=True)
    size = n / n_mol * e_atom.abs().max().item() * 16 * 2.0 ** -20
    assert (e_mol - e_net.mean(0)).abs().max().item() <= size
    per_atom = torch.zeros(n_mol, dtype=torch.float64, device=pos.device)
    per_atom.index_add_(0, torch.from_numpy(mol.astype(np.int64)).to(pos.device), e_atom.double())
    assert (e_mol - per_atom).abs().max().item() <= size
    for k in range(nets):
        one = nnp.Model(synthetic.ani2x_like_spec(7 + k, 0.05), "fp32")
        e, _, _ = nnp.nnp_energy_forces(one, pos, sp, mo, n_mol, w.box, nl, forces=False)
        assert (e - e_net[k]).abs().max().item() <= size, k
