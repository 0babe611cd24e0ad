"""Limits of the launch plans at sizes no test allocates (host functions, no GPU
needed)."""

import pytest

from paper_2607_00501_amd import binding as B
from tests.helpers import fewrow_plan, fewrow_swiglu_plan, moe_few_rows


# The few-row kernel addresses activations in 16-byte units of 32 bits: the last
# size that fits has rows x k / 8 = 2^32.
@pytest.mark.parametrize("m,k", [(32, 1 << 30), (16, (1 << 31) - 32), (1024, 1 << 25)])
def test_fewrow_addresses_its_activations(m, k):
    assert m * k // 8 <= 1 << 32 < (m + 1) * (k + 32) // 8
    for fmt in (B.Q4_G32, B.Q8_G32, B.F16):
        assert fewrow_plan(fmt, m, 64, k) and fewrow_swiglu_plan(fmt, min(m, 256), 64, k)
        for rows in (m + m // 16 + 1, 2 * m):
            assert fewrow_plan(fmt, rows, 64, k) is None
            assert fewrow_swiglu_plan(fmt, rows, 64, k) is None


def test_moe_few_rows_addresses_its_activations():
    assert moe_few_rows(16, 8, 128, 2048, 768) and not moe_few_rows(25, 8, 128, 2048, 768)
    assert moe_few_rows(16, 1, 64, (1 << 31) - 32, 64) and not moe_few_rows(17, 1, 64, (1 << 31) - 32, 64)
    # the down product reads a row per assignment
    assert moe_few_rows(4, 4, 64, 64, (1 << 31) - 32) and not moe_few_rows(5, 4, 64, 64, (1 << 31) - 32)
