"""One or two leading pairs, where the Cholesky-QR's compiled width is much more than its columns:
the smallest matrices, and both sides of the size where the matrix leaves the registers."""
import numpy as np
import pytest
import torch

import paper_2308_01480_amd as ttr
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r", [(1, 1), (2, 1), (2, 2), (3, 1), (3, 2), (3, 3), (4, 1), (16, 2), (128, 1), (128, 2),
                                 (129, 2), (130, 1), (200, 3), (256, 1), (256, 2)])
def test_few_pairs(n, r):
    announce(f"eig_top n={n} r={r}")
    q = np.linalg.qr(np.random.default_rng(n).standard_normal((n, n)))[0]
    a = (q / np.arange(1, n + 1)) @ q.T
    a = 0.5 * (a + a.T)
    vecs, vals = ttr.sym_eig_top(torch.from_numpy(a).cuda(), r)
    v, lam = vecs.cpu().numpy(), vals.cpu().numpy()
    # Householder and bisection: backward error a small multiple of n eps ||A||, ||A|| = 1
    tol = 16 * n * np.finfo(np.float64).eps
    assert np.abs(lam - np.linalg.eigvalsh(a)[::-1][:r]).max() <= tol
    assert np.abs(v.T @ v - np.eye(r)).max() <= tol
    assert np.abs(a @ v - v * lam).max() <= tol
