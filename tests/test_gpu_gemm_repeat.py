"""The same GEMM gives the same bits every time: its sums have a fixed order, and
no operand of a K step may be replaced before it was used."""

import pytest
import torch

from paper_2607_00501_amd import binding as B

pytestmark = pytest.mark.gpu


# 704 and 1,200 workgroups of 64-row tiles (more than one round on the chip), with
# and without split-K, and the 64 x 128 and 128 x 256 tiles.
@pytest.mark.parametrize("m,n,k", [(700, 4096, 960), (700, 4096, 480), (1200, 4096, 960), (300, 2048, 8192),
                                   (300, 16384, 2048)])
@pytest.mark.parametrize("fmt", [B.Q4_G32, B.Q8_G32, B.F16])
def test_gemm_repeats_bits(fmt, m, n, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n + k)
    w = B.qm_repack(B.qm_quantise(torch.randn(n, k, generator=g, device="cuda") * 0.02, fmt), B.LAYOUT_DEVICE)
    xs = [torch.randn(m, k, generator=g, device="cuda").half() for _ in range(3)]
    refs = [B.qmatmul_gemm(w, x) for x in xs]
    for _ in range(20):
        for x, ref in zip(xs, refs):
            assert torch.equal(B.qmatmul_gemm(w, x), ref)
