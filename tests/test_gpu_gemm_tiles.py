"""GPU parity of every MFMA tile of qmatmul_gemm outside the few-row kernel's
sizes, each format: ragged rows, columns and K, exact integers and the fp16
rounding of the weights, with the weights through registers and through LDS."""

import numpy as np
import pytest
import torch

from oracle import qmatmul_oracle as O
from paper_2607_00501_amd import binding as B
from paper_2607_00501_amd import inputs
from tests.helpers import FORMATS, fewrow_plan, gemm_plan, rel_err

pytestmark = pytest.mark.gpu


def _run(w, x, fmt, tile):
    """The call's output, with the tile it is meant for."""
    shape = (x.shape[0],) + w.shape
    assert fewrow_plan(fmt[1], *shape) is None and gemm_plan(*shape) == tile
    dev = B.qm_repack(B.qm_quantise(torch.from_numpy(w).cuda(), fmt[1]), B.LAYOUT_DEVICE)
    out = torch.full((x.shape[0], w.shape[0]), float("nan"), device="cuda")
    return B.qmatmul_gemm(dev, torch.from_numpy(x).cuda(), out=out).cpu().numpy()


def _cols(n, count=200):
    return np.unique(np.r_[np.random.default_rng(n).choice(n, count, replace=False), 0, 63, 64, n - 1])


@pytest.mark.parametrize("fmt", FORMATS, ids=lambda f: str(f[1]))
@pytest.mark.parametrize("m,n,k,tile", [
    (300, 1000, 96, (32, 1, 1)), (300, 1000, 544, (32, 1, 2)), (300, 1001, 2080, (32, 1, 4)),
    (200, 1010, 8224, (32, 1, 8)), (700, 4090, 928, (64, 1, 2)), (500, 2040, 2080, (64, 1, 4)),
    (290, 2040, 8224, (64, 1, 8)), (500, 3000, 2080, (64, 2, 2)), (2040, 2040, 96, (64, 4, 1)),
    (1000, 4001, 2080, (64, 4, 2)), (2000, 8000, 96, (128, 4, 1)),
])
def test_gemm_tile_parity(fmt, m, n, k, tile):
    w, x = inputs.weights_np(m + k, (n, k)), inputs.activations_np(m + n, (m, k))
    y = _run(w, x, fmt, tile)
    assert np.isfinite(y).all()
    rows, cols = np.unique(np.r_[np.random.default_rng(m).choice(m, 40, replace=False), 0, 63, 64, m - 1]), _cols(n)
    q, s = O.quantise(w[cols], fmt[0])
    # fp16 weight rounding only: 2^-11 per product, far less in the sum
    assert rel_err(y[np.ix_(rows, cols)], O.gemm(O.pack(q, fmt[0]), s, fmt[0], x[rows])) <= 2e-3


@pytest.mark.parametrize("fmt", FORMATS, ids=lambda f: str(f[1]))
@pytest.mark.parametrize("m,n,k,tile", [(300, 1000, 512, (32, 1, 2)), (700, 4090, 928, (64, 1, 2)),
                                        (500, 3000, 2080, (64, 2, 2)), (2040, 2040, 96, (64, 4, 1)),
                                        (1000, 4001, 2080, (64, 4, 2)), (2000, 8000, 96, (128, 4, 1))])
def test_gemm_tile_integers_exact(fmt, m, n, k, tile):
    """Integer weights at scale 1 (F16, BF16: up to 64) times small integers:
    products and sums below 2^24 are exact."""
    rng = np.random.default_rng(m + n)
    qm = O.QMAX.get(fmt[0], 64)
    w = rng.integers(-qm, qm + 1, size=(n, k)).astype(np.float32)
    w[:, ::32] = qm
    x = rng.integers(-4, 5, size=(m, k)).astype(np.float16)
    y = _run(w, x, fmt, tile)
    cols = _cols(n)
    q, s = O.quantise(w[cols], fmt[0])
    assert np.array_equal(y[:, cols].astype(np.float64), O.gemm(O.pack(q, fmt[0]), s, fmt[0], x))


@pytest.mark.parametrize("fmt", FORMATS, ids=lambda f: str(f[1]))
@pytest.mark.parametrize("m,n,tile", [(300, 1000, (32, 1, 1)), (2048, 1990, (64, 4, 1)), (2000, 8000, (128, 4, 1))])
def test_gemm_tile_uses_fp16_rounded_weights(fmt, m, n, tile):
    """Identity rows over and over: every output is the fp16 operand of its weight."""
    k = 64
    w, x = inputs.weights_np(m, (n, k)), np.tile(np.eye(k, dtype=np.float16), (m // k + 1, 1))[:m]
    y = _run(w, x, fmt, tile)
    cols = _cols(n)
    q, s = O.quantise(w[cols], fmt[0])
    tile_values = O.fp16_value(O.dequantise_f16_tile_value(O.pack(q, fmt[0]), s, fmt[0])).astype(np.float64)
    assert np.array_equal(y[:, cols].astype(np.float64), tile_values[:, np.arange(m) % k].T)
