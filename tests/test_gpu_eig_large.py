"""The full decomposition of matrices whose eigenvalues' products leave the range of float64 upwards
(above about 2^512): the same bounds as at the scale of one, the decomposition being invariant under
scaling by powers of two."""
import numpy as np
import pytest
import torch

import paper_2308_01480_amd as ttr
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exponent", [500, 520, 700, 900, 1005])
@pytest.mark.parametrize("n,rank", [(2, 1), (2, 2), (16, 16), (17, 5), (33, 33), (65, 64), (129, 40)])
def test_large_values(n, rank, exponent):
    announce(f"sym_eig n={n} rank={rank} 2^{exponent}")
    b = np.random.default_rng(n + rank).standard_normal((n, rank))
    g = b @ b.T
    vecs, vals = ttr.sym_eig(torch.from_numpy(np.ldexp(g, exponent)).cuda())
    v, lam = vecs.cpu().numpy(), np.ldexp(vals.cpu().numpy(), -exponent)
    ref = np.maximum(np.linalg.eigvalsh(g)[::-1], 0.0)
    # the bounds of the decomposition: 1e-12 between vectors, 4e-12 sqrt(n) of the largest value for the pairs
    tol = 4e-12 * np.sqrt(n) * ref[0]
    assert np.abs(lam - ref).max() <= tol
    assert np.all(lam[rank:] <= tol)
    kept = lam > tol
    assert kept.sum() == rank
    assert np.abs(v[:, kept].T @ v[:, kept] - np.eye(rank)).max() <= 1e-12
    assert np.abs(g @ v[:, kept] - v[:, kept] * lam[kept]).max() <= tol
