"""GPU parity of the expert layer on 32-row bucket tiles at the line between
2-panel tiles with 2-way split-K (few column blocks) and 4-panel tiles."""

import numpy as np
import pytest
import torch

from oracle import qmatmul_oracle as O
from paper_2607_00501_amd import binding as B
from paper_2607_00501_amd import inputs
from tests.helpers import MFMA_TOL, rel_err
from tests.test_gpu_moe import _experts, _route_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmts", [(O.Q4, B.Q4_G32), (O.Q2, B.Q2_G32), (O.Q3, B.Q3_G32), (O.Q5, B.Q5_G32),
                                  (O.Q6, B.Q6_G32), (O.Q8, B.Q8_G32)], ids=["q4", "q2", "q3", "q5", "q6", "q8"])
@pytest.mark.parametrize("m,e,k,hidden,inter", [
    (40, 6, 2, 96, 160),         # second K slice a step short, half-filled panels, buckets of one row tile
    (61, 5, 1, 1056, 32),        # one step in the down product: an empty slice
    (97, 8, 2, 64, 1088),        # 24 rows per expert, some buckets over 32 rows
    (30, 64, 4, 64, 992),        # 256 column blocks: the 4-panel tiles
])
def test_narrow_layer_parity(fmts, m, e, k, hidden, inter):
    (wg, wu, wd), ora = _experts(7000 + m, e, hidden, inter, fmts)
    x = inputs.activations_np(60 + m, (m, hidden))
    logits = inputs.logits_np(70 + m, (m, e))
    r = _route_check(logits, k)
    xt = torch.from_numpy(x).cuda()
    y1, y2 = (B.qmoe_grouped_gemm(wg, wu, wd, xt, r) for _ in range(2))
    assert torch.equal(y1, y2)
    ref, *_ = O.moe_layer(x, logits, k, *ora, fmt=fmts[0])
    assert rel_err(y1.cpu().numpy(), ref) <= MFMA_TOL


@pytest.mark.parametrize("m,e,k,hidden,inter", [(40, 128, 8, 288, 288),    # both products on 4-panel tiles
                                                 (60, 100, 6, 544, 64)])    # gate/up on 2, down on 4
def test_wide_and_mixed_layer_parity(m, e, k, hidden, inter):
    (wg, wu, wd), ora = _experts(8000 + m, e, hidden, inter)
    x = inputs.activations_np(80 + m, (m, hidden))
    logits = inputs.logits_np(90 + m, (m, e))
    r = _route_check(logits, k)
    y = B.qmoe_grouped_gemm(wg, wu, wd, torch.from_numpy(x).cuda(), r).cpu().numpy()
    ref, *_ = O.moe_layer(x, logits, k, *ora)
    assert rel_err(y, ref) <= MFMA_TOL
