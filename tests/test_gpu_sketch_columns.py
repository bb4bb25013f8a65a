"""A sketch's columns do not depend on how many are drawn beside them: float32 sketches of 17 to 48
columns take the same number of column groups, so the sums of a column are formed in the same order
at either padded width (32 or 48) and its bits are the same."""
import pytest
import torch

import paper_2308_01480_amd as ttr
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(12, 16884), (30, 20001), (100, 50000), (256, 40003)])
def test_same_columns_at_both_widths(m, n):
    announce(f"sketch columns {m}x{n}")
    g = torch.Generator(device="cuda").manual_seed(m)
    a = torch.randn(m, n, generator=g, device="cuda", dtype=torch.float32)
    few = ttr.sketch(a, 5, 2, 24)
    for s in (33, 40, 48):
        assert torch.equal(ttr.sketch(a, 5, 2, s)[:, :24], few)
        assert torch.equal(ttr.gram_sketch(a, 5, 2, s)[1][:, :24], few)
