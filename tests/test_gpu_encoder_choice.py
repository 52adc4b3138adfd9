"""Code_s strings of 2048 < d <= 8192 on both sides of the lines between the encoder with a team of
wavefronts per bucket and the one in which every lane codes its own values: the share of nonzero levels,
d, and the number of buckets choose.  Bar: message words equal to the oracle's; a slice of a few buckets
(another encoder) gives the strings of the whole vector's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device, compare_encode  # noqa: E402


@pytest.mark.parametrize("outliers", [0, 1000])
@pytest.mark.parametrize("d,s", [(2052, 2), (2052, 3), (2500, 5), (4096, 3), (4096, 4), (4100, 8), (7168, 7), (7172, 7)])
def test_either_side(d, s, outliers):
    few = 40
    n = d * 1030 + 3
    g = torch.randn(n, generator=torch.Generator().manual_seed(d + s))
    if outliers:
        g[::outliers] *= 100.0
    P = q.Params(n=n, s=s, d=d, code=q.CODE_SPARSE, seed=8, stream_id=1)
    status, words, _ = Device(P).encode(g.cuda())
    assert status == 0
    assert compare_encode(P, g.numpy(), words) == 0
    at = 500 * d
    Ps = q.Params(n=few * d, s=s, d=d, code=q.CODE_SPARSE, seed=8, stream_id=1)
    msg = torch.zeros(q.qsgd_max_encoded_bytes(Ps) // 4, dtype=torch.int32, device="cuda")
    ws = torch.zeros(q.qsgd_workspace_bytes(Ps, 1) // 4, dtype=torch.int32, device="cuda")
    q.qsgd_encode_slice(Ps, at, g[at:at + few * d].cuda(), msg, ws)
    part = msg.cpu().numpy().view(np.uint32)
    pay, pay_s = 16 + (1031 + 1 + 3) // 4 * 4, 16 + (few + 1 + 3) // 4 * 4
    lo, hi = int(words[16 + 500]), int(words[16 + 500 + few])
    assert int(part[16 + few]) == hi - lo
    assert np.array_equal(words[pay + lo:pay + hi], part[pay_s:pay_s + hi - lo])
