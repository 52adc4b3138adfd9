"""The encoder in which every lane codes its own values, where it changes course: bucket sizes
around the number of lanes times the run length, gaps and levels at the reach of its code word
table (64, 32) and beyond, runs of more than 64 bits, few and many buckets.  Bar: the message is
the oracle's, word for word."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device, compare_encode  # noqa: E402


def gradient(n, kind, seed):
    gen = torch.Generator().manual_seed(seed)
    sign = torch.where(torch.rand(n, generator=gen) < 0.5, -1.0, 1.0)
    if kind == "even":                     # with the largest value as scale: all levels up to s
        return sign * (0.02 + torch.rand(n, generator=gen))
    g = torch.zeros(n)
    if kind == "gaps":                     # first gaps of a run around the table's last row
        at, i = -1, 0
        for gap in [1, 2, 8, 9, 56, 57, 63, 64, 65, 71, 72, 100, 255, 256, 700] * (n // 1500 + 1):
            at += gap
            if at < n:
                g[at] = 0.5 + (i % 7) / 7
            i += 1
    else:                                  # one value holds nearly all of a bucket's norm
        g = torch.randn(n, generator=gen) * 1e-3
        g[::97] = 1.0
    return g * sign


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
@pytest.mark.parametrize("norm", [q.NORM_L2, q.NORM_MAX])
@pytest.mark.parametrize("d", [4, 60, 64, 68, 128, 132, 256, 260, 512, 516, 768, 772, 1024, 1028,
                               1536, 1540, 2048])
def test_bucket_sizes(code, norm, d):
    for s, kind in [(1, "gaps"), (4, "gaps"), (16, "even"), (31, "even"), (32, "spike"), (63, "even"),
                    (65535, "even")]:
        n = d * 9 + d // 2 + 1
        P = q.Params(n=n, s=s, d=d, code=code, norm=norm, seed=9, stream_id=3)
        g = gradient(n, kind, d + s)
        status, words, _ = Device(P).encode(g.cuda())
        assert status == 0
        assert compare_encode(P, g.numpy(), words) == 0


@pytest.mark.parametrize("d,nb", [(128, 5000), (256, 4097), (512, 9000)])
@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
def test_many_buckets(d, nb, code):
    n = d * nb - 40
    P = q.Params(n=n, s=5, d=d, code=code, seed=2)
    g = torch.randn(n, generator=torch.Generator().manual_seed(d))
    status, words, _ = Device(P).encode(g.cuda())
    assert status == 0
    assert compare_encode(P, g.numpy(), words) == 0
