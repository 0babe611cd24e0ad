"""GPU parity of the MoE path for a few tokens: the one-launch routing and
bucketing, and the expert layer on the few-row kernel."""

import numpy as np
import pytest
import torch

from oracle import qmatmul_oracle as O
from paper_2607_00501_amd import binding as B
from paper_2607_00501_amd import inputs
from tests.helpers import MFMA_TOL, rel_err
from tests.test_gpu_moe import _experts, _route_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("e,k", [(1, 1), (5, 5), (64, 6), (65, 8), (128, 8), (128, 16), (200, 13), (256, 8)])
@pytest.mark.parametrize("m", [1, 2, 3, 8, 10, 11, 16, 17])
def test_small_route_bit_exact(m, e, k):
    _route_check(inputs.logits_np(31 * m + e, (m, e)), k)


def test_small_route_ties_signed_zeros_infinities():
    rng = np.random.default_rng(4)
    for m, e, k in [(1, 128, 8), (9, 128, 8), (3, 7, 4), (16, 64, 6)]:
        _route_check(np.zeros((m, e), np.float32), k)
        logits = rng.integers(-1, 2, size=(m, e)).astype(np.float32)
        logits[logits == 0] *= rng.choice([-1.0, 1.0], size=(logits == 0).sum()).astype(np.float32)
        logits[:, 1] = -np.inf
        _route_check(logits, k)


def test_small_route_leaves_nans_unselected():
    m, e, k = 4, 96, 8
    logits = inputs.logits_np(8, (m, e))
    logits[:, ::3] = np.nan
    r = B.qmoe_route(torch.from_numpy(logits).cuda(), k)
    ids, gates = O.moe_route(np.where(np.isnan(logits), np.float32(-1e30), logits), k)
    assert np.array_equal(r.ids.cpu().numpy(), ids)
    assert np.abs(r.gates.cpu().numpy() - gates).max() <= 1e-6


@pytest.mark.parametrize("fmts", [(O.Q4, B.Q4_G32), (O.Q2, B.Q2_G32), (O.Q3, B.Q3_G32), (O.Q5, B.Q5_G32),
                                  (O.Q6, B.Q6_G32), (O.Q8, B.Q8_G32)], ids=["q4", "q2", "q3", "q5", "q6", "q8"])
@pytest.mark.parametrize("m,e,k,hidden,inter", [
    (1, 8, 2, 64, 96),          # K shorter than a step; a half-filled panel
    (3, 16, 4, 1056, 160),      # K with a partial last step in both products
    (24, 32, 2, 160, 1088),     # 1.5 rows per expert: the last size of the rule
    (16, 128, 8, 288, 64),
])
def test_few_row_layer_parity(fmts, m, e, k, hidden, inter):
    (wg, wu, wd), ora = _experts(3000 + m, e, hidden, inter, fmts)
    x = inputs.activations_np(40 + m, (m, hidden))
    logits = inputs.logits_np(50 + m, (m, e))
    r = _route_check(logits, k)
    y = B.qmoe_grouped_gemm(wg, wu, wd, torch.from_numpy(x).cuda(), r).cpu().numpy()
    ref, *_ = O.moe_layer(x, logits, k, *ora, fmt=fmts[0])
    assert rel_err(y, ref) <= MFMA_TOL


def test_few_row_layer_with_all_tokens_on_the_same_experts():
    """Every token picks experts 5 and 6: 20 rows each, three 8-row blocks, the
    last one ragged; the same bits twice."""
    m, e, k, hidden, inter = 20, 64, 2, 128, 96
    (wg, wu, wd), ora = _experts(91, e, hidden, inter)
    x = inputs.activations_np(92, (m, hidden))
    logits = np.zeros((m, e), np.float32)
    logits[:, 5:7] = (2.0, 1.0)
    r = _route_check(logits, k)
    xt = torch.from_numpy(x).cuda()
    y1, y2 = (B.qmoe_grouped_gemm(wg, wu, wd, xt, r) for _ in range(2))
    assert torch.equal(y1, y2)
    ref, *_ = O.moe_layer(x, logits, k, *ora)
    assert rel_err(y1.cpu().numpy(), ref) <= MFMA_TOL
