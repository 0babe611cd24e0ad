"""An infinite activation among the last ones of K gives infinities of the
weight's sign, in its own row alone, on every kind of tile: K a multiple of
64 or not, K slices of unequal length."""

import numpy as np
import pytest
import torch

from oracle import qmatmul_oracle as O
from paper_2607_00501_amd import binding as B
from paper_2607_00501_amd import inputs
from tests.helpers import fewrow_plan, gemm_plan

pytestmark = pytest.mark.gpu


def _weight(seed, shape, fmt):
    w = inputs.weights_np(seed, shape)
    last = O.quantise(w.reshape(-1, shape[-1])[:, -32:], fmt[0])[0][:, -1]
    dev = B.qm_repack(B.qm_quantise(torch.from_numpy(w).cuda(), fmt[1]), B.LAYOUT_DEVICE)
    sign = np.sign(last.astype(np.float64)) if fmt[0] not in O.FLOATS else np.sign(w.reshape(-1, shape[-1])[:, -1])
    return dev, sign


def _check_row(y, row, sign):
    nz = sign != 0
    assert nz.any() and np.isfinite(np.delete(y, row, 0)).all()
    assert np.array_equal(y[row, nz], sign[nz] * np.inf)


@pytest.mark.parametrize("fmt", [(O.Q4, B.Q4_G32), (O.Q8, B.Q8_G32), (O.Q6, B.Q6_G32), (O.F16, B.F16)],
                         ids=["q4", "q8", "q6", "f16"])
@pytest.mark.parametrize("m,n,k,tile", [
    (1000, 4001, 2112, (64, 4, 2)), (1000, 4001, 2080, (64, 4, 2)),     # 33 steps, the last one whole / half
    (500, 3000, 2112, (64, 2, 2)), (500, 3000, 2080, (64, 2, 2)),
    (700, 4096, 960, (64, 1, 2)), (700, 4096, 928, (64, 1, 2)),
    (300, 1024, 1088, (32, 1, 4)), (200, 1024, 8224, (32, 1, 8)),       # empty steps in several slices
    (1100, 2048, 96, (32, 1, 1)), (2048, 2048, 96, (64, 4, 1)), (2000, 8000, 96, (128, 4, 1)),
])
def test_gemm_infinite_activation(fmt, m, n, k, tile):
    assert fewrow_plan(fmt[1], m, n, k) is None and gemm_plan(m, n, k) == tile
    w, sign = _weight(m + n + k, (n, k), fmt)
    x = inputs.activations_np(k, (m, k))
    x[m - 2, k - 1] = np.inf
    _check_row(B.qmatmul_gemm(w, torch.from_numpy(x).cuda()).cpu().numpy(), m - 2, sign)


@pytest.mark.parametrize("fmt", [(O.Q4, B.Q4_G32), (O.Q8, B.Q8_G32)], ids=["q4", "q8"])
@pytest.mark.parametrize("inter", [64, 96, 192])      # one whole K step, two with a half, three: two slices
def test_moe_infinite_hidden_activation(fmt, inter):
    """h overflows fp16 in its last column for one token; 61 tokens on five
    experts take the 2-panel tiles, whose down product splits K in two."""
    m, e, hidden = 61, 5, 1056
    wd, sign = _weight(inter, (e, hidden, inter), fmt)
    wg, wu = (inputs.weights_np(i, (e, inter, hidden)) for i in (1, 2))
    wg[:, -1, 0] = wu[:, -1, 0] = 40.0
    x = inputs.activations_np(3, (m, hidden))
    x[:, 0] = 0
    x[7, 0] = 1000
    dev = [B.qm_repack(B.qm_quantise(torch.from_numpy(w).cuda(), fmt[1]), B.LAYOUT_DEVICE) for w in (wg, wu)]
    r = B.qmoe_route(torch.from_numpy(inputs.logits_np(5, (m, e))).cuda(), 1)
    y = B.qmoe_grouped_gemm(*dev, wd, torch.from_numpy(x).cuda(), r).cpu().numpy()
    expert = int(r.ids.cpu().numpy()[7, 0])
    _check_row(y, 7, sign.reshape(e, hidden)[expert])
