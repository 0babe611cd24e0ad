"""qdec_rope_append_rows on its two kernels (the wide one takes a table and
aligned buffers): the same bits, with and without the per-head norm, and nothing
written outside the chunk."""

import pytest
import torch

from paper_2607_00501_amd import binding as B

pytestmark = pytest.mark.gpu


# Threads per token that fill no workgroup, one token, and a last workgroup in part.
@pytest.mark.parametrize("hq,hkv,d,m,p0", [(1, 1, 64, 1, 0), (3, 1, 64, 7, 5), (32, 8, 64, 33, 100), (16, 8, 128, 9, 3),
                                           (5, 2, 128, 50, 0)])
@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("interleaved", [False, True])
def test_wide_kernel_matches(hq, hkv, d, m, p0, norm, interleaved):
    g = torch.Generator(device="cuda")
    g.manual_seed(hq + d + m)
    max_len = p0 + m + 3
    rows = lambda heads: torch.randn(m * heads * d + 1, generator=g, device="cuda")
    flat = [rows(hq), rows(hkv), rows(hkv)]
    gains = [(1 + 0.1 * torch.randn(d, generator=g, device="cuda")).half() if norm else None for _ in range(2)]
    tab = B.qdec_rope_table(max_len, d, 1e4)
    got = []
    for off in (0, 1):               # 4 bytes off: the kernel of one pair per thread
        q, k, v = (t[:t.numel() - 1] if off == 0 else torch.cat([t[:1], t[:-1]])[1:] for t in flat)
        q, k, v = q.view(m, hq * d), k.view(m, hkv * d), v.view(m, hkv * d)
        assert q.data_ptr() % 16 == 4 * off
        kc = torch.full((hkv, max_len, d), 7.0, dtype=torch.float16, device="cuda")
        vc = kc.clone()
        qo = B.qdec_rope_append_rows(q, k, v, p0, 1e4, kc, vc, interleaved=interleaved, q_norm=gains[0],
                                     k_norm=gains[1], eps=1e-6, table=tab)
        got.append((qo, kc, vc))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    kc, vc = got[0][1:]
    assert torch.all(kc[:, :p0] == 7) and torch.all(kc[:, p0 + m:] == 7)
    assert torch.all(vc[:, :p0] == 7) and torch.all(vc[:, p0 + m:] == 7)
    assert torch.equal(vc[:, p0:p0 + m].transpose(0, 1).reshape(m, hkv * d), flat[2][:-1].view(m, hkv * d).half())
