"""The streamed TT error with entries of a core that are infinite, undefined, or overflow in a
product: positive cores, so that every entry of Xhat is a sum of positive terms and the results
are what plain float64 sums give (an infinite squared error, not an undefined one), at ragged
last rows and columns of a tile as at whole ones."""
import math

import numpy as np
import pytest
import torch

import paper_2308_01480_amd as ttr
from tests.gpu_util import DT, announce

pytestmark = pytest.mark.gpu

DIMS = [((64, 64), (4,)), ((3, 5), (2,)), ((65, 1001), (1,)), ((130, 63, 31), (7, 20)), ((70, 3, 349527), (5, 12))]


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("dims,ranks", DIMS)
@pytest.mark.parametrize("kind", ["inf", "overflow", "nan"])
def test_nonfinite_core(dt, dims, ranks, kind):
    announce(f"tt_error {kind} {dt} dims={dims}")
    rng = np.random.default_rng(sum(dims))
    rk = [1, *ranks, 1]
    x = torch.from_numpy(rng.uniform(0.5, 1.5, dims)).to(DT[dt]).cuda()
    x2 = float((x.double() ** 2).sum())
    for where in range(len(dims)):
        cores = [rng.uniform(0.5, 1.0, (rk[k], dims[k], rk[k + 1])) for k in range(len(dims))]
        if kind == "overflow":
            cores[where][0, dims[where] // 2, 0] = 1e200
            cores[where - 1][:, dims[where - 1] // 2, :] = 1e200
        else:
            cores[where][0, dims[where] // 2, 0] = {"inf": math.inf, "nan": math.nan}[kind]
        got = ttr.tt_error(x, [torch.from_numpy(c).cuda() for c in cores]).cpu().numpy()
        assert abs(got[1] - x2) <= 1e-12 * x2
        if kind == "nan":
            assert math.isnan(got[0])
        else:
            assert got[0] == math.inf and got[2] == math.inf, got
