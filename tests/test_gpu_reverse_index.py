"""The list's reverse index on both sides of the size from which rows are
searched by four lanes: structures of m atoms that are all neighbours (rows of
m - 1 entries, 16 a block, four blocks at once and one at a time beyond 64)."""
import numpy as np
import pytest
import torch

import paper_2405_01491_amd as nnp
from tests.gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def model(spec):
    return nnp.Model(spec, "fp32")


@pytest.mark.parametrize("m", [2, 16, 17, 18, 33, 64, 65, 66, 81, 129, 256, 257])
@pytest.mark.parametrize("least", [4900, 5000])
def test_reverse_index_at_row_lengths(model, m, least):
    n_mol = least // m if least < 5000 else -(-least // m)
    rng = np.random.default_rng(m)
    pos = rng.normal(size=(n_mol, m, 3))
    pos *= (2.5 * rng.random((n_mol, m, 1)) ** (1 / 3)) / np.linalg.norm(pos, axis=2, keepdims=True)
    x = torch.from_numpy(pos.reshape(-1, 3).astype(np.float32)).to(dev())
    mol = torch.arange(n_mol * m, dtype=torch.int32, device=dev()) // m
    nl = nnp.nnp_neighbors(model, x, mol, n_mol, None, 5.1)
    # row a of a structure holds its other atoms in order
    a, b = np.nonzero(~np.eye(m, dtype=bool))
    first = (np.arange(n_mol) * m * (m - 1))[:, None]
    j = (np.arange(n_mol) * m)[:, None] + b
    rev = first + b * (m - 1) + a - (a > b)
    assert nl.n_pairs == n_mol * m * (m - 1)
    assert np.array_equal(nl.col[:nl.n_pairs].cpu().numpy(), j.ravel())
    assert np.array_equal(nl.rev[:nl.n_pairs].cpu().numpy(), rev.ravel())
    nnp.nnp_check(model)
