"""Fixed width at bucket sizes no vector load fits and above 8192 values: every field width, tails of a
few values, escapes (level s = 2^B under the L2 scale), fields above s in a message, up to 64 peers.
Bar: messages equal to the oracle's, x bit-identical."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device, check_step, compare_encode  # noqa: E402


@pytest.mark.parametrize("s,norm", [(3, q.NORM_MAX), (4, q.NORM_L2), (15, q.NORM_MAX), (16, q.NORM_L2),
                                    (255, q.NORM_MAX), (256, q.NORM_L2), (1000, q.NORM_L2), (65535, q.NORM_MAX)])
@pytest.mark.parametrize("d,n,K", [
    (1, 70, 1), (3, 1000, 2), (33, 8001, 3), (61, 61 * 40, 5), (65, 700, 4), (127, 127 * 9 + 5, 64),
    (255, 3000, 2), (257, 2571, 6), (511, 511, 1), (513, 10_000, 4), (1021, 50_001, 3), (1023, 1030, 9),
    (1025, 20_000, 2), (8191, 30_000, 3), (8193, 8193, 2), (9000, 27_001, 17), (100_000, 99_999, 4),
])
def test_fixed_width(d, n, K, s, norm):
    dev, host = [], []
    for k in range(K):
        P = q.Params(n=n, s=s, d=d, code=q.CODE_FIXED, norm=norm, seed=2, stream_id=k)
        g = torch.randn(n, generator=torch.Generator().manual_seed(n + k))
        g[d // 2::d] *= 1e4          # one value has the bucket to itself: level s
        status, words, msg = Device(P).encode(g.cuda())
        assert status == 0
        assert compare_encode(P, g.numpy(), words) == 0
        dev.append(msg)
        host.append(words)
    P0 = q.Params(n=n, s=s, d=d, code=q.CODE_FIXED, norm=norm, seed=2)
    assert check_step(P0, dev, host, 0.1, np.linspace(-1, 1, n, dtype=np.float32), K) == 0


@pytest.mark.parametrize("d,n", [(33, 330), (9001, 18_002)])
def test_field_above_s(d, n):
    """s = 9 in fields of 4 bits: 10 to 15 are refused."""
    P = q.Params(n=n, s=9, d=d, code=q.CODE_FIXED, norm=q.NORM_MAX, seed=2)
    _, words, msg = Device(P).encode(torch.zeros(n, device="cuda"))
    ws = torch.zeros(max(q.qsgd_workspace_bytes(P, 1), 256) // 4, dtype=torch.int32, device="cuda")
    x = torch.zeros(n + 64, device="cuda")
    q.qsgd_decode_accumulate(P, [msg[: words.size].clone()], x[:n], ws)
    assert q.qsgd_workspace_status(ws) == 0
    bad = msg[: words.size].clone()
    bad[16 + 2] = 0xA                # the first value's field
    q.qsgd_decode_accumulate(P, [bad], x[:n], ws)
    assert q.qsgd_workspace_status(ws) == -3
    assert not x[n:].any()
