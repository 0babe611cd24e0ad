"""GPU parity of the 64 x 256 tiles with 2-way split-K: ragged rows, a last
column block with one panel short, a K whose first slice is a step short, every
format; dense and with the SwiGLU epilogue."""

import numpy as np
import pytest
import torch

from oracle import qmatmul_oracle as O
from paper_2607_00501_amd import binding as B
from paper_2607_00501_amd import inputs
from tests.helpers import FORMATS, MFMA_TOL, rel_err

pytestmark = pytest.mark.gpu


def _case(seed, n, k, fmt):
    w = inputs.weights_np(seed, (n, k))
    q, s = O.quantise(w, fmt[0])
    dev = B.qm_repack(B.qm_quantise(torch.from_numpy(w).cuda(), fmt[1]), B.LAYOUT_DEVICE)
    return (O.pack(q, fmt[0]), s), dev


@pytest.mark.parametrize("fmt", FORMATS, ids=lambda f: str(f[1]))
def test_wide_splitk_parity(fmt):
    m, n, k = 1000, 4001, 2080                   # 16 x 16 workgroups, 33 K steps
    (packed, scales), w = _case(m + k, n, k, fmt)
    x = inputs.activations_np(m + n, (m, k))
    y = B.qmatmul_gemm(w, torch.from_numpy(x).cuda(), out=torch.full((m, n), float("nan"), device="cuda"))
    assert rel_err(y.cpu().numpy(), O.gemm(packed, scales, fmt[0], x)) <= MFMA_TOL


@pytest.mark.parametrize("fmt", [FORMATS[0], FORMATS[1], FORMATS[6]], ids=lambda f: str(f[1]))
def test_wide_splitk_swiglu_parity(fmt):
    m, n, k = 260, 6211, 2048                    # 5 x 49 workgroups, an odd number of panels
    (g, wg), (u, wu) = _case(3, n, k, fmt), _case(4, n, k, fmt)
    x = inputs.activations_np(m, (m, k))
    y = B.qmatmul_gemm_swiglu_f16(wg, wu, torch.from_numpy(x).cuda()).cpu().numpy()
    G, U = O.gemm(*g, fmt[0], x), O.gemm(*u, fmt[0], x)
    assert rel_err(y, O.silu(G) * U) <= MFMA_TOL
