"""Levels that the encoder's table of code words does not hold: around the four-value (63, 126)
and two-value code word paths' ends, mixed with small levels, long gaps and few large values, for
bucket sizes of every shape.  Bar: the oracle's words."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device, compare_encode  # noqa: E402


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
@pytest.mark.parametrize("s", [33, 64, 126, 127, 128, 255, 4096, 65535])
@pytest.mark.parametrize("d", [64, 128, 256, 443, 512, 900, 1536, 2047, 2048, 2052])
def test_levels_beyond_the_table(code, s, d):
    n = d * 21 - d // 3
    gen = torch.Generator().manual_seed(s + d)
    mag = torch.exp(-12.0 * torch.rand(n, generator=gen))      # levels spread over their logarithm
    mag[torch.rand(n, generator=gen) < 0.3] = 0.0              # and gaps
    mag[(n // 2) // d * d:][: 3 * d] *= (torch.rand(mag[(n // 2) // d * d:][: 3 * d].numel(),
                                                    generator=gen) < 0.01)    # long ones
    g = torch.where(torch.rand(n, generator=gen) < 0.5, -mag, mag)
    for norm in (q.NORM_L2, q.NORM_MAX):
        P = q.Params(n=n, s=s, d=d, code=code, norm=norm, seed=4, stream_id=1)
        status, words, _ = Device(P).encode(g.cuda())
        assert status == 0
        assert compare_encode(P, g.numpy(), words) == 0
