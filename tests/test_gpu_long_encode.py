"""Elias encode of buckets above 8192 values: one to many groups of segments, one to many buckets, a
last bucket of a few values, strings whose segments share words (hardly any records, none at all)
and fill them (Code'_s), more segments than one trip of the scan takes, and messages that end one word
short.  Bar: message words equal to the oracle's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device, compare_encode  # noqa: E402


def gradient(kind, n):
    g = torch.randn(n, generator=torch.Generator().manual_seed(n))
    if kind == "zeros":
        g.zero_()
    elif kind == "ends":          # records in the first and the last segment of a bucket only
        g[100:-100] = 0.0
    return g


@pytest.mark.parametrize("kind", ["normal", "ends", "zeros"])
@pytest.mark.parametrize("code,norm", [(q.CODE_SPARSE, q.NORM_L2), (q.CODE_SPARSE, q.NORM_MAX),
                                       (q.CODE_DENSE, q.NORM_L2)])
@pytest.mark.parametrize("d,s,n", [
    (8193, 1, 8193), (8193, 3, 3 * 8193 + 1), (16_384, 2, 40_000), (32_768, 1, 70_000),
    (32_769, 100, 65_538), (34_817, 4, 5 * 34_817 - 2048), (10_001, 30, 200_003),
    (8200, 2, 300 * 8200 + 5), (3_000_001, 1, 3_000_001), (9_000_000, 2, 9_000_000),
])
def test_long_buckets(kind, code, norm, d, s, n):
    P = q.Params(n=n, s=s, d=d, code=code, norm=norm, seed=9, stream_id=3)
    g = gradient(kind, n)
    status, words, _ = Device(P).encode(g.cuda())
    assert status == 0
    assert compare_encode(P, g.numpy(), words) == 0


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
@pytest.mark.parametrize("d,n", [(50_000, 50_000), (9000, 100_000)])
def test_message_one_word_short(code, d, n):
    P = q.Params(n=n, s=4, d=d, code=code, seed=9)
    g = gradient("normal", n).cuda()
    status, words, _ = Device(P).encode(g)
    assert status == 0
    size = 4 * words.size
    status, again, _ = Device(P, capacity=(size + 15) // 16 * 16).encode(g)
    assert status == 0 and np.array_equal(again, words)
    status, need, _ = Device(P, capacity=size - 4).encode(g)
    assert status == -2 and need == size
