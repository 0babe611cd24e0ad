"""The same GEMM gives the same bits every time, and the right ones: its sums have
a fixed order, and no operand of a K step may be replaced before it was used."""

import numpy as np
import pytest
import torch

from oracle import qmatmul_oracle as O
from paper_2607_00501_amd import binding as B
from tests.helpers import MFMA_TOL, fewrow_plan, gemm_plan, rel_err

pytestmark = pytest.mark.gpu


# Every tile with K slices or several panels: one-wavefront slices over more
# than one round of workgroups and in one, 64 x 256 over more than one round,
# 128 x 256, and the 2-way split-K of 64 x 128 and of 64 x 256 (eight wavefronts).
@pytest.mark.parametrize("m,n,k,tile", [
    (700, 4096, 960, (64, 1, 2)), (700, 4096, 480, (64, 1, 2)), (300, 2048, 8192, (64, 1, 8)),
    (300, 1001, 2048, (32, 1, 4)), (1200, 4096, 960, (64, 4, 1)), (300, 16384, 2048, (128, 4, 1)),
    (512, 3072, 2048, (64, 2, 2)), (512, 8192, 2048, (64, 4, 2)), (2048, 2048, 8192, (64, 4, 2)),
])
@pytest.mark.parametrize("fmt", [(O.Q4, B.Q4_G32), (O.Q8, B.Q8_G32), (O.F16, B.F16)], ids=["q4", "q8", "f16"])
def test_gemm_repeats_bits(fmt, m, n, k, tile):
    assert fewrow_plan(fmt[1], m, n, k) is None and gemm_plan(m, n, k) == tile
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n + k)
    w_host = torch.randn(n, k, generator=g, device="cuda") * 0.02
    w = B.qm_repack(B.qm_quantise(w_host, fmt[1]), B.LAYOUT_DEVICE)
    xs = [torch.randn(m, k, generator=g, device="cuda").half() for _ in range(3)]
    refs = [B.qmatmul_gemm(w, x) for x in xs]
    rng = np.random.default_rng(m + k)
    rows, cols = (np.unique(np.r_[rng.choice(e, 24, replace=False), 0, e - 1]) for e in (m, n))
    q, s = O.quantise(w_host.cpu().numpy()[cols], fmt[0])
    for x, ref in zip(xs, refs):
        exact = O.gemm(O.pack(q, fmt[0]), s, fmt[0], x.cpu().numpy()[rows])
        assert rel_err(ref.cpu().numpy()[np.ix_(rows, cols)], exact) <= MFMA_TOL
    for _ in range(20):
        for x, ref in zip(xs, refs):
            assert torch.equal(B.qmatmul_gemm(w, x), ref)
