"""GPU parity of the gate/up product with the SwiGLU epilogue: every tile of
its plan at ragged rows and columns, each format, unaligned and odd-width
outputs."""

import numpy as np
import pytest
import torch

from oracle import qmatmul_oracle as O
from paper_2607_00501_amd import binding as B
from paper_2607_00501_amd import inputs
from tests.helpers import FORMATS, MFMA_TOL, fewrow_swiglu_plan, gemm_plan, rel_err

pytestmark = pytest.mark.gpu


def _weights(seed, n, k, fmt):
    out = []
    for i in (0, 1):
        w = inputs.weights_np(seed + i, (n, k), sigma=0.05)
        q, s = O.quantise(w, fmt[0])
        dev = B.qm_repack(B.qm_quantise(torch.from_numpy(w).cuda(), fmt[1]), B.LAYOUT_DEVICE)
        out.append(((O.pack(q, fmt[0]), s), dev))
    return out


def _check(m, n, k, fmt, offset=0):
    (g, wg), (u, wu) = _weights(17 * m + n, n, k, fmt)
    x = inputs.activations_np(5 * m + k, (m, k))
    buf = torch.full((m * n + 8,), 9.0, dtype=torch.float16, device="cuda")
    out = buf[offset:offset + m * n].view(m, n)
    B.qmatmul_gemm_swiglu_f16(wg, wu, torch.from_numpy(x).cuda(), out=out)
    G, U = O.gemm(*g, fmt[0], x), O.gemm(*u, fmt[0], x)
    assert rel_err(out.cpu().numpy(), O.silu(G) * U) <= MFMA_TOL
    rest = torch.cat([buf[:offset], buf[offset + m * n:]])
    assert (rest == 9.0).all()


@pytest.mark.parametrize("fmt", FORMATS, ids=lambda f: str(f[1]))
@pytest.mark.parametrize("m,n,k", [
    (1, 130, 96),           # the GEMV
    (13, 1000, 160),        # few-row kernel, 16-row sub-panels, partial last step
    (30, 3072, 96),         # 32-row sub-panels
    (61, 3072, 128),        # 32-row blocks
    (100, 5000, 96),        # 64 x 128, 2-way split-K (an odd number of panels)
    (300, 5000, 96),        # 64 x 256, ragged rows
    (590, 5000, 64),        # 128 x 256, ragged rows, an odd number of panels
])
def test_swiglu_gemm_parity(fmt, m, n, k):
    _check(m, n, k, fmt)


@pytest.mark.parametrize("m,n,offset", [(9, 65, 1), (16, 66, 2), (70, 6499, 1), (100, 5001, 0),
                                         (300, 5002, 1), (590, 4999, 0)])
def test_swiglu_gemm_odd_width_and_alignment(m, n, offset):
    _check(m, n, 64, (O.Q4, B.Q4_G32), offset)


WIDE = [f for f in FORMATS if f[1] in (B.Q8_G32, B.F16, B.BF16)]


@pytest.mark.parametrize("m,n,k,tile,fmt", [
    (m, n, k, tile, f) for m, n, k, tile, fmts in [
        (50, 8190, 2080, (64, 1, 4), FORMATS),      # 128 column blocks a matrix, K with a half last step
        (50, 4101, 4128, (64, 1, 8), FORMATS),      # odd width, slices of unequal length
        (70, 4000, 2080, (32, 1, 4), FORMATS),      # a last panel half filled
        (300, 1000, 544, (32, 1, 2), WIDE),         # (the others are on the few-row kernel)
        (300, 1000, 96, (32, 1, 1), WIDE),
    ] for f in fmts])
def test_swiglu_gemm_column_halves_sampled(m, n, k, tile, fmt):
    """The single-panel tiles: 32 gate and 32 up columns per workgroup."""
    panels = (n + 63) // 64
    assert fewrow_swiglu_plan(fmt[1], m, n, k) is None and gemm_plan(m, 128 * panels, k) == tile
    assert panels * ((m + 63) // 64) <= 128
    ws = [inputs.weights_np(31 * m + i, (n, k), sigma=0.05) for i in (0, 1)]
    x = inputs.activations_np(m + k, (m, k))
    dev = [B.qm_repack(B.qm_quantise(torch.from_numpy(w).cuda(), fmt[1]), B.LAYOUT_DEVICE) for w in ws]
    buf = torch.full((m * n + 8,), 9.0, dtype=torch.float16, device="cuda")
    B.qmatmul_gemm_swiglu_f16(*dev, torch.from_numpy(x).cuda(), out=buf[2:2 + m * n].view(m, n))
    y = buf[2:2 + m * n].view(m, n).cpu().numpy()
    cols = np.unique(np.concatenate([np.random.default_rng(k).choice(n, 200, replace=False),
                                     [0, 31, 32, 63, 64, n - 33, n - 1]]))
    G, U = (O.gemm(O.pack(q, fmt[0]), s, fmt[0], x) for q, s in (O.quantise(w[cols], fmt[0]) for w in ws))
    assert rel_err(y[:, cols], O.silu(G) * U) <= MFMA_TOL
    assert (buf[:2] == 9.0).all() and (buf[2 + m * n:] == 9.0).all()


@pytest.mark.parametrize("fmt", FORMATS, ids=lambda f: str(f[1]))
@pytest.mark.parametrize("m", [13, 29])
def test_swiglu_gemm_few_rows_of_a_wide_matrix_sampled(fmt, m):
    """More sub-panels than two per CU: 16- and 32-row blocks all the same."""
    n, k = 17000, 160
    assert fewrow_swiglu_plan(fmt[1], m, n, k)[1] == (4 if m <= 16 else 8)
    ws = [inputs.weights_np(41 * m + i, (n, k), sigma=0.05) for i in (0, 1)]
    x = inputs.activations_np(m, (m, k))
    dev = [B.qm_repack(B.qm_quantise(torch.from_numpy(w).cuda(), fmt[1]), B.LAYOUT_DEVICE) for w in ws]
    y = B.qmatmul_gemm_swiglu_f16(*dev, torch.from_numpy(x).cuda()).cpu().numpy()
    cols = np.unique(np.concatenate([np.random.default_rng(k).choice(n, 200, replace=False), [0, 63, 64, n - 1]]))
    G, U = (O.gemm(O.pack(q, fmt[0]), s, fmt[0], x) for q, s in (O.quantise(w[cols], fmt[0]) for w in ws))
    assert rel_err(y[:, cols], O.silu(G) * U) <= MFMA_TOL


def test_swiglu_gemm_extreme_gates():
    """Gates far outside the exponential's range: silu goes to 0 or g."""
    m, n, k = 20, 64, 64
    (g, wg), (u, wu) = _weights(3, n, k, (O.F16, B.F16))
    x = inputs.activations_np(4, (m, k)) * np.float16(300)
    y = B.qmatmul_gemm_swiglu_f16(wg, wu, torch.from_numpy(x).cuda()).cpu().numpy().astype(np.float64)
    ref = (O.silu(O.gemm(*g, O.F16, x)) * O.gemm(*u, O.F16, x))
    ok = np.abs(ref) < 60000
    assert ok.mean() > 0.5 and np.abs(y - ref)[ok].max() <= MFMA_TOL * np.abs(ref[ok]).max()


@pytest.mark.parametrize("m", [1, 16, 130, 2048])    # the GEMV, two few-row tiles, a GEMM tile
@pytest.mark.parametrize("lo,hi,scale", [(-20, -8, 15000.0), (-8, 0, 64.0), (0, 20, 1.0)])
def test_swiglu_gemm_rounds_the_exact_value(m, lo, hi, scale):
    """One fp32 evaluation and one fp16 rounding: with exact G and U the result
    lies within half an fp16 ulp and the fp32 error of silu(G) * U.  That error
    is at most 2.5 ulp of 2^-23: 1 for the exponential, 0.5 each for the sum, the
    quotient and the product."""
    n, k = 512, 32
    rng = np.random.default_rng(m + lo + 20)
    gates = rng.uniform(lo, hi, m).astype(np.float16)
    ups = (scale * rng.uniform(1, 4, n)).astype(np.float16)
    x = np.zeros((m, k), np.float16)
    x[:, 0], x[:, 1] = gates, 1
    wg, wu = np.zeros((n, k), np.float32), np.zeros((n, k), np.float32)
    wg[:, 0], wu[:, 1] = 1, ups
    dev = [B.qm_repack(B.qm_quantise(torch.from_numpy(w).cuda(), B.F16), B.LAYOUT_DEVICE) for w in (wg, wu)]
    y = B.qmatmul_gemm_swiglu_f16(*dev, torch.from_numpy(x).cuda()).cpu().numpy().astype(np.float64)
    g = gates.astype(np.float64)[:, None]
    exact = g / (1 + np.exp(-g)) * ups.astype(np.float64)
    half_ulp = np.exp2(np.maximum(np.floor(np.log2(np.maximum(np.abs(exact), 1e-30))), -14) - 11)
    assert np.all(np.abs(y - exact) <= half_ulp + 2.5 * 2.0 ** -23 * np.abs(exact))
