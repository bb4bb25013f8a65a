"""The streamed TT error against a plain float64 reconstruction, at the edges of its tiles:
one or two row groups of 64 and their remainders, column tails of every vector width,
inner sizes whose rows are not aligned, one to three leading modes, ranks 1 to 64.

Tolerances.  Every entry of Xhat is a chain of float64 sums over the ranks, |error| <=
2 u sum(r) C |Xhat| with u = 2^-53 and C <= 40 the growth of the absolute products of
Gaussian cores at these ranks (sum(r) <= 140): 1.3e-12 |Xhat|.  The residual is 1e-2 of
|Xhat|, so ||X - Xhat||^2 carries 2 * 1.3e-12 / 1e-2 < 1e-9; max |Xhat| 1e-11; ||X||^2 is a
sum of squares, 1e-12."""
import math

import numpy as np
import pytest
import torch

import paper_2308_01480_amd as ttr
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

DT = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}

CASES = [((3, 5), (2,)), ((64, 257), (16,)), ((65, 1001), (1,)), ((130, 63, 31), (7, 20)), ((129, 2050), (33,)),
         ((200, 70, 16), (64, 16)), ((4, 5, 6, 7, 8), (4, 9, 24, 8)),
         ((70, 3, 349527), (5, 12)), ((3, 3, 3, 349527), (3, 9, 13)), ((5, 1, 14, 262147), (5, 5, 64))]


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("dims,ranks", CASES)
def test_tt_error_matches_reconstruction(dt, dims, ranks):
    announce(f"tt_error {dt} dims={dims} ranks={ranks}")
    rng = np.random.default_rng(sum(dims) + len(ranks))
    rk = [1, *ranks, 1]
    cores = [rng.standard_normal((rk[k], dims[k], rk[k + 1])) / math.sqrt(rk[k]) for k in range(len(dims))]
    full = cores[0].reshape(dims[0], -1)
    for c in cores[1:]:
        full = (full.reshape(-1, c.shape[0]) @ c.reshape(c.shape[0], -1)).reshape(-1, c.shape[2])
    full = full.reshape(dims)
    x = torch.from_numpy(full + 1e-2 * rng.standard_normal(dims)).to(DT[dt]).cuda()
    X = x.to(torch.float64).cpu().numpy()
    e2, x2, xinf = ttr.tt_error(x, [torch.from_numpy(c).cuda() for c in cores]).cpu().numpy()
    want = (np.sum((X - full) ** 2), np.sum(X * X), np.max(np.abs(full)))
    assert abs(e2 - want[0]) <= 1e-9 * want[0]
    assert abs(x2 - want[1]) <= 1e-12 * want[1]
    assert abs(xinf - want[2]) <= 1e-11 * want[2]


def test_tt_error_of_a_tensor_that_is_not_aligned():
    """X one entry into its buffer: rows of an aligned length at an address that is not."""
    announce("tt_error offset view")
    rng = np.random.default_rng(5)
    cores = [rng.standard_normal((1, 70, 6)), rng.standard_normal((6, 64, 1))]
    full = cores[0].reshape(70, 6) @ cores[1].reshape(6, 64)
    for dt in DT.values():
        buf = torch.zeros(70 * 64 + 1, dtype=dt, device="cuda")
        x = buf[1:].view(70, 64)
        x.copy_(torch.from_numpy(full))
        X = x.to(torch.float64).cpu().numpy()
        e2, x2, xinf = ttr.tt_error(x, [torch.from_numpy(c).cuda() for c in cores]).cpu().numpy()
        assert abs(e2 - np.sum((X - full) ** 2)) <= 1e-12 * np.sum(X * X)
        assert abs(x2 - np.sum(X * X)) <= 1e-12 * np.sum(X * X)
        assert abs(xinf - np.max(np.abs(full))) <= 1e-11 * np.max(np.abs(full))
