"""Rows of odd length and tensors that start between two vectors, through every streaming kernel.
Aligned and offset storage of an odd row length take the same kernels, whose answers are the same
bits; each agrees with float64 products of the operands as the kernel stores them.

Bounds: a sum of k products in arithmetic of unit roundoff u is within (k + 4) u of the sum of the
absolute products (u = 2^-53 or 2^-24; the four cover the operands' own rounding and the last
one).  bfloat16 rounds Z, Omega and the intermediate W = A^T Z to eight bits (2^-9 of an entry) and
multiplies and adds in float32.  Each bound is also held against a result of zeros, which has to
miss it."""
import pytest
import torch

import paper_2308_01480_amd as ttr
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


def unaligned(a):
    """The same matrix, one element off any vector boundary."""
    flat = torch.empty(a.numel() + 1, dtype=a.dtype, device=a.device)
    flat[1:] = a.reshape(-1)
    return flat[1:].view(a.shape)


def within(got, ref, bound):
    assert not (ref.abs() <= bound).all()
    assert ((got.double() - ref).abs() <= bound).all()


# rows up to 16, 32, 64 (no LDS), one staged chunk, more than one, and above 512; columns of one
# element more or less than whole tiles of 16 to 128
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,n,s", [(5, 1023, 3), (24, 4097, 10), (60, 2049, 12), (100, 1021, 20), (129, 513, 40),
                                   (250, 3073, 30), (320, 511, 17), (513, 2047, 64), (700, 1025, 40)])
def test_same_bits_and_products(m, n, s, dtype):
    announce(f"unaligned rows {dtype} m={m} n={n} s={s}")
    g = torch.Generator().manual_seed(m + s)
    a = torch.randn(m, n, generator=g).to(dtype).cuda()
    z = torch.randn(m, s, generator=g, dtype=torch.float64).cuda()
    b = unaligned(a)
    assert b.data_ptr() % 16 != 0 and torch.equal(a, b)
    u = 2.0**-53 if dtype == torch.float64 else 2.0**-24
    A = a.double()
    Z = z.to(dtype).double()  # as stored for the product
    om = ttr.omega(7, 2, 0, n, s).to(dtype).double()
    W = A.t() @ Z
    absW = A.abs().t() @ Z.abs()
    w_rounding = 1.01 * 2.0**-9 * (A.abs() @ W.abs()) if dtype == torch.bfloat16 else 0.0
    runs = []
    for x in (a, b):
        r = {"carry": ttr.carry(x, z), "krylov": ttr.krylov(x, z), "sketch": ttr.sketch(x, 7, 2, s)}
        if m <= 256:
            r["gram"] = ttr.gram(x)
            r["gram of both"], r["sketch of both"] = ttr.gram_sketch(x, 7, 2, s)
        runs.append(r)
    for key, got in runs[0].items():
        assert torch.equal(got, runs[1][key]), key
        if key == "carry":
            within(got, W.t(), (m + 4) * u * absW.t())
        elif key == "krylov":
            within(got, A @ W, (m + n + 4) * u * (A.abs() @ absW) + w_rounding)
        elif key.startswith("sketch"):
            within(got, A @ om, (n + 4) * u * (A.abs() @ om.abs()))
        else:
            within(got, A @ A.t(), (n + 4) * u * (A.abs() @ A.abs().t()))
