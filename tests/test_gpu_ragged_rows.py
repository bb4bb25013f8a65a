"""Rows of odd length, and tensors that start between two vectors, through every streaming kernel:
each answer is that of the same numbers in aligned storage."""
import pytest
import torch

import paper_2308_01480_amd as tt

pytestmark = pytest.mark.gpu


def unaligned(a):
    """The same matrix, one element off any vector boundary."""
    flat = torch.empty(a.numel() + 1, dtype=a.dtype, device=a.device)
    flat[1:] = a.reshape(-1)
    return flat[1:].view(a.shape)


# rows up to 16, 32, 64 (no LDS), one staged chunk, more than one, and above 512; columns of one
# element more or less than whole tiles of 16 to 128
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,n,s", [(5, 1023, 3), (24, 4097, 10), (60, 2049, 12), (100, 1021, 20), (250, 3073, 30),
                                   (320, 511, 17), (700, 1025, 40)])
def test_offset_and_odd_rows(m, n, s, dtype):
    g = torch.Generator().manual_seed(m)
    a = torch.randn(m, n, generator=g).to(dtype).cuda()
    z = torch.randn(m, s, generator=g, dtype=torch.float64).cuda()
    b = unaligned(a)
    assert b.data_ptr() % 16 != 0 and torch.equal(a, b)
    ref = a.double()
    # products of m or n terms in the kernel's own precision, sums of |a||z| as the scale; bfloat16
    # rounds z (and the carry) to eight bits
    eps = {torch.float64: 2.0**-52, torch.float32: 2.0**-23, torch.bfloat16: 2.0**-8}[dtype]
    zd = z.to(dtype).double() if dtype != torch.bfloat16 else z
    for x in (a, b):
        c = tt.carry(x, z).double()
        assert ((c - zd.t() @ ref).abs() <= 4 * eps * m**0.5 * (z.abs().t() @ ref.abs())).all()
        y = tt.krylov(x, z).double()
        w = ref.abs() @ (ref.abs().t() @ z.abs())
        assert ((y - ref @ (ref.t() @ zd)).abs() <= 4 * eps * (m + n)**0.5 * w).all()
        if m <= 256:
            q = tt.gram(x).double()
            assert ((q - ref @ ref.t()).abs() <= 4 * eps * n**0.5 * (ref.abs() @ ref.abs().t())).all()
    assert torch.equal(tt.carry(a, z), tt.carry(b, z))
