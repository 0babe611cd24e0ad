"""GPU parity of decode attention at the edges of its plan: one slice or
several, partial steps of a wavefront, every group size, and caches long enough
for slices of many steps."""

import numpy as np
import pytest

from tests.helpers import rel_err
from tests.test_gpu_attention import ATTN_TOL, _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("edge", [-1, 0, 1])
def test_one_slice_limit(d, group, edge):
    length = 65536 // (group * d) + edge
    o, ref = _case(2 * group, 2, d, length, length + 5, seed=100 * group + d + edge)
    assert np.all(np.isfinite(o)) and rel_err(o, ref) <= ATTN_TOL


@pytest.mark.parametrize("hq,hkv,d,length", [
    (2, 2, 64, 1), (16, 2, 128, 15), (8, 2, 64, 31), (4, 2, 128, 65),     # fewer rows than a step
    (48, 8, 128, 97), (64, 8, 128, 128), (64, 8, 128, 129),               # one slice up to 128 rows at any group
    (8, 4, 128, 64 * 128), (8, 4, 128, 64 * 128 + 1),                     # whole slices, then one row more
    (6, 2, 64, 256 * 64 + 3), (16, 2, 128, 40000),                        # the largest number of slices
])
def test_slices(hq, hkv, d, length):
    o, ref = _case(hq, hkv, d, length, length, seed=length)
    assert np.all(np.isfinite(o)) and rel_err(o, ref) <= ATTN_TOL


def test_scores_far_apart_and_negative_scale():
    for scale, seed in ((2.0, 3), (-1.0, 4)):
        o, ref = _case(8, 2, 128, 1500, 1600, seed=seed, scale=scale)
        assert rel_err(o, ref) <= ATTN_TOL
