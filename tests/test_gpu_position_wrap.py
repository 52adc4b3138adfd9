"""Strings whose gaps add up to 2^32 and a little more: the position they claim to end at is inside
the bucket again when it is counted in 32 bits.  They name coordinates that do not exist and must
be refused, whichever decoder reads them."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402


def omega(k):
    bits = "0"
    while k > 1:
        b = format(k, "b")
        bits = b + bits
        k = len(b) - 1
    return bits


def message(n, d, gaps, entries=None):
    """A Code_s message (s = 1) of one bucket: `gaps` with level 1 each."""
    bits = "".join(omega(g) + "0" + "0" for g in gaps) + "1"
    bits += "0" * (-len(bits) % 32)
    string = [int(np.array(1.0, np.float32).view(np.uint32))]
    string += [int(bits[i:i + 32], 2) for i in range(0, len(bits), 32)]
    if entries is not None:
        string += list(entries) + [len(entries) // 2]
    P = q.Params(n=n, s=1, d=d, code=q.CODE_SPARSE, seed=3)
    small = q.Params(n=8, s=1, d=d, code=q.CODE_SPARSE, seed=3)     # a header to start from
    ws = torch.zeros(q.qsgd_workspace_bytes(small, 1) // 4, dtype=torch.int32, device="cuda")
    head = torch.zeros(q.qsgd_max_encoded_bytes(small) // 4, dtype=torch.int32, device="cuda")
    q.qsgd_encode(small, torch.ones(8, device="cuda"), head, ws)
    h = head.cpu().numpy().view(np.uint32)[:16].copy()
    h[6], h[7], h[8], h[9] = min(d, n) & 0xFFFFFFFF, min(d, n) >> 32, n & 0xFFFFFFFF, n >> 32
    h[10], h[11], h[12], h[13] = 1, 0, len(string), 0
    words = np.concatenate([h, np.array([0, len(string), 0, 0], np.uint32), np.array(string, np.uint32)])
    return P, torch.from_numpy(words.view(np.int32)).cuda()


def step(P, msg):
    ws = torch.zeros(q.qsgd_workspace_bytes(P, 1) // 4, dtype=torch.int32, device="cuda")
    x = torch.zeros(P.n, device="cuda")
    q.qsgd_sgd_step(P, [msg], -1.0, x, ws)
    return q.qsgd_workspace_status(ws), x


@pytest.mark.parametrize("d", [8192, 8191])
def test_short_bucket(d):
    P, msg = message(d, d, [65535] * 3)
    assert step(P, msg)[0] == -3
    P, msg = message(d, d, [65535] * 65537 + [6])       # 65535 * 65537 = 2^32 - 1
    assert step(P, msg)[0] == -3
    P, msg = message(d, d, [5, 100])                    # (and what is sound is read)
    status, x = step(P, msg)
    assert status == 0 and x.nonzero().flatten().tolist() == [4, 104]


def test_long_bucket_of_more_than_2_31_values():
    n = (1 << 31) + 2000
    P, msg = message(n, n, [(1 << 31) + 1000, 1 << 31], entries=())
    status, x = step(P, msg)
    assert status == -3
    assert not bool(x[:4096].any()) and not bool(x[1 << 31:].any())
    P, msg = message(n, n, [7, (1 << 31) + 1000], entries=())
    status, x = step(P, msg)
    assert status == 0
    assert float(x[6]) == 1.0 and float(x[(1 << 31) + 1006]) == 1.0 and int(x[:1 << 20].count_nonzero()) == 1


@pytest.mark.parametrize("n", [(1 << 32) - 1, (1 << 32) - 31])
def test_the_longest_buckets(n):
    """Buckets whose length plus 31 does not fit 32 bits: bitmaps, lists and x keep apart."""
    at = [3, 41, 42, 300, 70_000, (1 << 31) + 5, n]
    P, msg = message(n, n, [b - a for a, b in zip([0] + at, at)], entries=())
    status, x = step(P, msg)
    assert status == 0
    assert [float(x[i - 1]) for i in at] == [1.0] * len(at)
    assert int(x[:1 << 20].count_nonzero()) == 5 and int(x[-(1 << 20):].count_nonzero()) == 1
