"""Block orthonormalisation at the edges of its compiled widths (multiples of eight columns),
of its row chunks, and of the two ways its partial sums travel: summed by the next launch's
work-groups (up to 960 rows) or by launches of their own (more rows; sums that do not fit
beside a wide block's rows in LDS; a scratch that holds one partial buffer).

Tolerances are those of the rank-revealing block test (orthonormality 1e-13 and the projector
to 1e-9 over six decades of singular values) and of the float64 sweep (1e-10)."""
import numpy as np
import pytest
import torch

import paper_2308_01480_amd as ttr
from tests.gpu_util import announce
from tests.test_gpu_sweep import run_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,s,rank", [(960, 8, 8), (961, 9, 9), (100, 16, 12), (17, 17, 17), (959, 24, 24), (65, 25, 20),
                                      (1025, 32, 32), (640, 33, 30), (960, 40, 40), (2000, 41, 41), (961, 48, 31),
                                      (700, 49, 49), (16384, 56, 56), (960, 57, 57), (64, 64, 60), (8192, 63, 63)])
def test_orth_widths_and_rows(m, s, rank):
    from oracle import ttrbki
    announce(f"orth m={m} s={s} rank={rank}")
    rng = np.random.default_rng(11 * m + s)
    U, _ = np.linalg.qr(rng.standard_normal((m, rank)))
    V, _ = np.linalg.qr(rng.standard_normal((s, rank)))
    P = (U * np.logspace(0, -6, rank)) @ V.T
    ref = float(np.linalg.norm(P))
    q, k = ttr.orth(torch.from_numpy(P).cuda(), ref, 1e-10)
    Q = q.cpu().numpy()
    Qo = ttrbki.orth_tau(P, ref, 1e-10)
    assert k == Qo.shape[1] == rank
    assert np.all(Q[:, k:] == 0.0)
    assert np.max(np.abs(Q[:, :k].T @ Q[:, :k] - np.eye(k))) <= 1e-13
    # equal dimensions: ||(I - Qo Qo^T) Q||_2 is the distance of the two projectors
    assert np.linalg.norm(Q[:, :k] - Qo @ (Qo.T @ Q[:, :k]), 2) <= 1e-9


@pytest.mark.parametrize("dims,ranks,q,p", [
    ((20, 20, 900), [20, 56], 3, 8),      # 256 Krylov columns: sums of 192 x 64 are read from memory
    ((20, 50, 1000), [20, 56], 3, 8),     # the same on a tall block (1000 rows)
    ((10, 100, 90), [10, 60], 0, 4),      # no Krylov step, 64 columns: one partial buffer
    ((30, 40, 60), [25, 30], 1, 5)])
def test_sweep_with_wide_blocks(dims, ranks, q, p):
    rng = np.random.default_rng(sum(dims) + q)
    X = rng.standard_normal(dims)
    for k, I in enumerate(dims):  # decaying directions along every mode
        shape = [1] * len(dims)
        shape[k] = I
        X = X * (1.0 + np.arange(I)).reshape(shape) ** -1.0
    run_pair(X, ranks, q, p, 7, "f64", "wide-blocks")
