"""The one-pass Krylov product Y = A (A^T Z) at the edges of its register form: row counts
around its compiled k-step counts (multiples of 16 and 32 rows up to 320, then 64), the rows
where the form with Z in LDS takes over, every padded width, ragged column tails and rows that
are not aligned.  Bounds as for the product's own test: |error| <= 4 * 2e-5 (float32) or 1e-13
(float64) of |A| (|A|^T |Z|), rounding of sums of products."""
import numpy as np
import pytest
import torch

import paper_2308_01480_amd as ttr
from tests.gpu_util import announce, bound_check, stored_f64, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(64, 4096, 16), (65, 1001, 16), (80, 640, 17), (96, 3333, 32), (97, 500, 33), (161, 2049, 48), (176, 31, 49),
          (208, 1000, 64), (272, 4099, 20), (288, 2048, 18), (289, 700, 30), (321, 650, 40), (384, 515, 64),
          (385, 600, 50), (449, 1000, 32), (512, 33, 16), (512, 640, 64), (2, 100, 2), (33, 70000, 10)]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("m,n,s", SHAPES)
def test_krylov_rows(dt, m, n, s):
    announce(f"krylov rows {dt} m={m} n={n} s={s}")
    rng = np.random.default_rng(13 * m + n + s)
    a = to_dev(rng.standard_normal((m, n)), dt)
    A = stored_f64(a)
    s = min(s, m)
    Z = np.linalg.qr(rng.standard_normal((m, s)))[0]
    y = ttr.krylov(a, torch.from_numpy(np.ascontiguousarray(Z)).cuda()).cpu().numpy()
    bound_check(y, A @ (A.T @ Z), np.abs(A) @ (np.abs(A).T @ np.abs(Z)), 1e-13 if dt == "f64" else 8e-5)
