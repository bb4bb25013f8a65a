"""The radius and angle of the Box-Muller pairs over the words that feed them.  The device
takes its division and square root from hardware estimates with one correction, which is
exact for every one of the 2^23 uniforms: 25 million pairs reach 95% of them on either side,
and the first and last uniforms are the extremes of the logarithm.  Every entry equals the
oracle's bit for bit (no tolerance)."""
import numpy as np
import pytest
import torch

import paper_2308_01480_amd as ttr
from oracle.philox import omega as omega_ref
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,k,b0", [(3, 1, 0), (2 ** 40 + 1, 7, 12345), (99, 2, 2 ** 32 - 100), (17, 4, 2 ** 50)])
def test_omega_bits(seed, k, b0):
    rows, s = 196608, 64
    announce(f"omega bits seed={seed} k={k} beta0={b0} rows={rows} s={s}")
    got = ttr.omega(seed, k, b0, rows, s).cpu().numpy()
    assert np.array_equal(got, omega_ref(seed, k, b0, b0 + rows, s))


@pytest.mark.parametrize("nrows,s", [(1, 1), (31, 8), (33, 9), (1000, 70), (7, 3000)])
def test_omega_row_groups(nrows, s):
    """Row groups of the materialising kernel: few rows, one column group, many column groups."""
    announce(f"omega rows={nrows} s={s}")
    got = ttr.omega(5, 3, 77, nrows, s).cpu().numpy()
    assert np.array_equal(got, omega_ref(5, 3, 77, 77 + nrows, s))


@pytest.mark.parametrize("m,n,s", [(129, 64 * 2 * 256 * 2 + 65, 40), (256, 127, 8), (250, 129, 9), (192, 70000, 64)])
def test_gram_sketch_large_rows(m, n, s):
    """The bf16 Gram-and-sketch kernel of 128 < m <= 256 rows at interval remainders; the sketch
    entries are sums of n products with float32 sums (the blocks' bf16 bound 1.2e-2)."""
    announce(f"gram_sketch bf16 m={m} n={n} s={s}")
    rng = np.random.default_rng(m + n)
    a = torch.from_numpy(rng.standard_normal((m, n))).cuda().to(torch.bfloat16)
    A = a.to(torch.float64).cpu().numpy()
    gm, y = ttr.gram_sketch(a, 11, 1, s)
    gm, y = gm.cpu().numpy(), y.cpu().numpy()
    absA = np.abs(A)
    assert np.max(np.abs(gm - A @ A.T) / (absA @ absA.T)) <= 2e-6
    assert np.array_equal(gm, gm.T)
    om = omega_ref(11, 1, 0, n, s)
    assert np.max(np.abs(y - A @ om) / (absA @ np.abs(om))) <= 1.2e-2
