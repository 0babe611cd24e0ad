"""GPU parity of the few-row matmul kernel: edges of its 16-row weight and
activation tiles, K with a partial last step (K % 128 != 0), every tile of its
plan, each format, and groups."""

import numpy as np
import pytest
import torch

from oracle import qmatmul_oracle as O
from paper_2607_00501_amd import binding as B
from paper_2607_00501_amd import inputs
from tests.helpers import FORMATS, MFMA_TOL, fewrow_plan, rel_err

pytestmark = pytest.mark.gpu


def _case(seed, n, k, fmt):
    w = inputs.weights_np(seed, (n, k))
    q, s = O.quantise(w, fmt[0])
    dev = B.qm_repack(B.qm_quantise(torch.from_numpy(w).cuda(), fmt[1]), B.LAYOUT_DEVICE)
    return (O.pack(q, fmt[0]), s), dev


@pytest.mark.parametrize("fmt", FORMATS, ids=lambda f: str(f[1]))
@pytest.mark.parametrize("m,n,k", [
    (2, 70, 32),           # less than one step, ragged columns
    (8, 64, 160),          # one full step and a partial one
    (9, 1000, 1056),       # 16-row tile, 33 groups
    (17, 130, 4128),       # two row blocks, two steps in flight, partial last step
    (40, 3072, 224),       # 32-row sub-panels, three row blocks
    (77, 3072, 192),       # whole panels (the wide formats take other tiles)
    (128, 3072, 128),      # 32-row blocks of whole panels
    (5, 16448, 96),        # more panels than CUs
    (31, 16448, 64),       # as many, K too short for 32 rows: the tiles
])
def test_fewrow_parity(fmt, m, n, k):
    (packed, scales), w = _case(7 * m + k, n, k, fmt)
    x = inputs.activations_np(11 * m + n, (m, k))
    y = B.qmatmul_gemm(w, torch.from_numpy(x).cuda(), out=torch.full((m, n), float("nan"), device="cuda"))
    assert rel_err(y.cpu().numpy(), O.gemm(packed, scales, fmt[0], x)) <= MFMA_TOL


@pytest.mark.parametrize("fmt", FORMATS, ids=lambda f: str(f[1]))
def test_fewrow_wide_matrix_sampled(fmt):
    """32-row blocks of more panels than CUs, K with a partial last step."""
    m, n, k = 29, 16440, 1056
    assert fewrow_plan(fmt[1], m, n, k) == (4, 8, 1)
    w, x = inputs.weights_np(51, (n, k)), inputs.activations_np(52, (m, k))
    dev = B.qm_repack(B.qm_quantise(torch.from_numpy(w).cuda(), fmt[1]), B.LAYOUT_DEVICE)
    y = B.qmatmul_gemm(dev, torch.from_numpy(x).cuda()).cpu().numpy()
    cols = np.unique(np.concatenate([np.random.default_rng(53).choice(n, 300, replace=False), [0, 63, 64, n - 1]]))
    q, s = O.quantise(w[cols], fmt[0])
    assert rel_err(y[:, cols], O.gemm(O.pack(q, fmt[0]), s, fmt[0], x)) <= MFMA_TOL


def test_fewrow_group_and_unaligned_output():
    """A group with odd column counts, outputs at 4-byte alignment, and
    neighbours of the output left alone."""
    m, k, ns = 12, 416, (65, 130, 64)
    x = inputs.activations_np(3, (m, k))
    cases = [_case(100 + i, n, k, (O.Q4, B.Q4_G32)) for i, n in enumerate(ns)]
    bufs = [torch.full((m * n + 2,), 7.0, device="cuda") for n in ns]
    B.qmatmul_gemm_grouped([c[1] for c in cases], torch.from_numpy(x).cuda(),
                           outs=[b[1:-1].view(m, n) for b, n in zip(bufs, ns)])
    for ((packed, scales), _), b, n in zip(cases, bufs, ns):
        b = b.cpu().numpy()
        assert b[0] == 7.0 and b[-1] == 7.0
        assert rel_err(b[1:-1].reshape(m, n), O.gemm(packed, scales, O.Q4, x)) <= MFMA_TOL


def test_fewrow_infinities_stay_in_their_row():
    """An infinite activation in the last groups of a partial step gives
    infinities of the weight's sign, and only in its own row."""
    m, n, k = 6, 64, 160
    (packed, scales), w = _case(5, n, k, (O.Q4, B.Q4_G32))
    x = inputs.activations_np(6, (m, k))
    x[3, k - 1] = np.inf
    y = B.qmatmul_gemm(w, torch.from_numpy(x).cuda()).cpu().numpy()
    col = O.dequantise(packed, scales, O.Q4)[:, k - 1]
    nz = col != 0
    assert nz.any() and np.isfinite(np.delete(y, 3, 0)).all()
    assert np.array_equal(y[3, nz], np.sign(col[nz]) * np.inf)
