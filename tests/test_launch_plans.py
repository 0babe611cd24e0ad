"""Limits of the launch plans at sizes no test allocates (host functions, no GPU
needed)."""

import pytest

from paper_2607_00501_amd import binding as B
from tests.helpers import (attn_decode_slices, fewrow_plan, fewrow_swiglu_plan, gemm_tile_name, moe_few_rows,
                           moe_tile_name)


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
    for m, top_k, experts, hidden, inter in [(1024, 1, 1024, 1 << 25, 64), (16, 4, 128, 64, 1 << 29)]:
        assert m * top_k * max(hidden, inter) // 8 >= 1 << 32
        assert not moe_few_rows(B.Q4_G32, m, top_k, experts, hidden, inter)


@pytest.mark.parametrize("fmt,few,many", [(B.Q4_G32, 9, 40), (B.Q8_G32, 8, 24), (B.Q3_G32, 8, 24)])
def test_moe_few_rows_leaves_many_short_products_to_the_tiles(fmt, few, many):
    """256 and 1,024 small experts: a few tokens only; large matrices up to 1.5
    rows per expert."""
    assert moe_few_rows(fmt, few, 8, 256, 1024, 512) and not moe_few_rows(fmt, many, 8, 256, 1024, 512)
    assert moe_few_rows(fmt, 4, 16, 1024, 512, 256) and not moe_few_rows(fmt, many, 16, 1024, 512, 256)
    assert moe_few_rows(fmt, 24, 8, 128, 4096, 1536) and not moe_few_rows(fmt, 25, 8, 128, 4096, 1536)


# 512 threads per workgroup, fewer than 2^32 per grid dimension: 2^23 workgroups
# are too many.
def test_fewrow_grids_can_be_launched():
    for m, k in ((2, 32), (16, 32), (32, 1024)):
        assert fewrow_plan(B.Q4_G32, m, 64 * ((1 << 23) - 1), k) == (4, max(2, m // 4), 1)
        for n in (64 << 23, (64 << 23) - 63, 1 << 30):
            assert fewrow_plan(B.Q4_G32, m, n, k) is None
    # gate/up: two sub-panels of every panel and assignment; down: one
    large = lambda hidden, inter: moe_few_rows(B.Q4_G32, 1, 8, 1024, hidden, inter)
    assert large(1024, 16 << 20) and not large(1024, 32 << 20)
    assert large((64 << 20) - 640, 1024) and not large(64 << 20, 1024)


def test_fewrow_swiglu_grids_can_be_launched():
    for m in (2, 16, 32):
        assert fewrow_swiglu_plan(B.Q4_G32, m, 64 * ((1 << 22) - 1), 32) == (2, 4 if m <= 16 else 8, 1)
        assert fewrow_swiglu_plan(B.Q4_G32, m, 64 << 22, 32) is None
    assert fewrow_swiglu_plan(B.Q6_G32, 2, 64 * ((1 << 21) - 1), 32) == (1, 4, 1)
    assert fewrow_swiglu_plan(B.Q6_G32, 2, 64 << 21, 32) is None


def test_fewrow_leaves_short_k_on_wide_matrices_to_the_tiles():
    """More panels than CUs: up to 16 rows at any K, up to 32 from K = 1024."""
    for fmt in (B.Q4_G32, B.Q8_G32, B.F16):
        for n in (16448, 151936):
            assert fewrow_plan(fmt, 16, n, 512) == (4, 4, 1) and fewrow_plan(fmt, 17, n, 992) is None
            assert fewrow_plan(fmt, 32, n, 1024) == (4, 8, 1) and fewrow_plan(fmt, 33, n, 1024) is None


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group", range(1, 9))
def test_decode_attention_of_short_caches_is_one_launch(d, group):
    one = max(128, 65536 // (group * d))
    for hkv in (1, 8, 128):
        for length in (1, 64, 128, one):
            assert attn_decode_slices(hkv, group, d, length) == (length, 1)
        assert attn_decode_slices(hkv, group, d, one + 1)[1] > 1


def test_tile_names_follow_the_plans():
    assert gemm_tile_name(B.Q4_G32, 8, 2048, 2048) == "few-row, 8 rows x 16"
    assert gemm_tile_name(B.Q4_G32, 512, 2048, 2048) == "BM64 x 64, 4-way split-K"
    assert gemm_tile_name(B.Q8_G32, 2048, 2048, 8192) == "BM64 x 256, 2-way split-K"
    layer = lambda fmt, m, experts=128: moe_tile_name(fmt, m, 8, experts, 2048, 768)
    assert layer(B.Q4_G32, 1) == "few-row, 8 rows x 32 and 64"
    assert layer(B.Q4_G32, 128) == "32-row bucket tiles x 4 and 4 panels"
    assert moe_tile_name(B.Q4_G32, 48, 4, 32, 1024, 512) == "32-row bucket tiles x 2 and 2 panels"
    assert layer(B.Q4_G32, 2048) == "64- and 64-row bucket tiles x 4 panels"
    assert layer(B.Q8_G32, 2048) == "32- and 64-row bucket tiles x 4 panels"
