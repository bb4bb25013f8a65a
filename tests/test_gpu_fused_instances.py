"""The one-pass Krylov product Y = A (A^T Z) at every row count it takes: each multiple of sixteen
rows up to 512 (so every compiled instance of the register form and of the form with Z in LDS, on
both sides of every limit), each padded width, both types, with a ragged last row block and column
tile.  Which row counts are one-pass is part of the test: the timed entry refuses the others.

Few columns of Gaussian entries (one column tile per work-group): a sum of k products in
arithmetic of unit roundoff u is within (k + 4) u of the sum of the absolute products; Y sums n
products of sums of m.  Many columns (two and three tiles per work-group) of entries -1, 0, 1:
every sum is a whole number below 2^24, so Y is exact in either type."""
import pytest
import torch

import paper_2308_01480_amd as ttr
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

LDS = 160 * 1024


def one_pass(rows, width, size):
    """Tile (odd pitch), Z and the four partials of W in LDS; float32 beyond 512 rows is another kernel."""
    tile = 16 if size == 8 else 32
    return size * (rows * (tile + 1) + rows * width + 4 * tile * width) <= LDS


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("width", [16, 32, 48, 64])
def test_every_row_count(dtype, width):
    size = 8 if dtype == torch.float64 else 4
    u = 2.0**-53 if dtype == torch.float64 else 2.0**-24
    taken = 0
    for rows in range(16, 513, 16):
        m, s = rows - rows // 16 % 3, width - rows // 16 % 5
        s = min(s, m)
        if (s + 15) // 16 * 16 != width:
            continue
        n = 5 * 32 + 7 + rows // 16  # at least six column tiles, the last one ragged
        announce(f"one-pass krylov {dtype} m={m} n={n} s={s}")
        g = torch.Generator(device="cuda").manual_seed(rows + width)
        a = torch.randn(m, n, generator=g, device="cuda", dtype=torch.float64).to(dtype)
        z = torch.linalg.qr(torch.randn(m, s, generator=g, device="cuda", dtype=torch.float64))[0].contiguous()
        A, Z = a.double(), z.to(dtype).double()
        ref, bound = A @ (A.t() @ Z), (m + n + 4) * u * (A.abs() @ (A.abs().t() @ Z.abs()))
        assert not (ref.abs() <= bound).all()
        assert ((ttr.krylov(a, z) - ref).abs() <= bound).all()
        if one_pass(rows, width, size):
            y, _ = ttr.krylov_timed(a, z, 1)
            assert torch.equal(y, ttr.krylov(a, z))
            taken += 1
            n = 2 * 1024 * (32 if size == 4 else 16) + 37
            a = torch.randint(-1, 2, (m, n), generator=g, device="cuda").to(dtype)
            z = torch.randint(-1, 2, (m, s), generator=g, device="cuda").double()
            w = a.double().t() @ z
            assert int((a.double().abs() @ w.abs()).max()) < 2**24
            assert torch.equal(ttr.krylov(a, z), a.double() @ w)
        else:
            with pytest.raises(ttr.TTRError):
                ttr.krylov_timed(a, z, 1)
    assert taken >= 9
