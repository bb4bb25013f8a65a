"""A tall saturated mode (n < m, more than 960 rows) behind a tall regular mode of few columns: the
orthonormalisation of its r columns shares the partial sums' region that the plan sizes for the
regular mode's blocks, which are smaller."""
import numpy as np
import pytest

import paper_2308_01480_amd as ttr
from tests.test_gpu_sweep import run_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,ranks,q,p", [((961, 481, 24), [2, 24], 0, 0), ((1000, 500, 30), [2, 28], 0, 4),
                                            ((970, 490, 20), [2, 18], 1, 3), ((500, 481, 24), [2, 24], 0, 0)])
def test_tall_saturated_mode(dims, ranks, q, p):
    pl = ttr.plan(list(dims), ranks, q, p)
    assert pl.kinds == ["regular", "saturated"]
    X = np.random.default_rng(sum(dims)).standard_normal(dims)
    for k, I in enumerate(dims):  # decaying directions along every mode
        shape = [1] * len(dims)
        shape[k] = I
        X = X * (1.0 + np.arange(I)).reshape(shape) ** -1.0
    run_pair(X, ranks, q, p, 7, "f64", "tall-saturated")
