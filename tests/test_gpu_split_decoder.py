"""The decoder that gives every word of a string a lane, and bucket sizes that no vector load
fits in the decoders of short buckets: strings of less than a word up to many turns of a
workgroup, rows that do not fit LDS at once, up to 64 peers, tails of a few values, scales that
are not finite, damaged strings.  Bar: x bit-identical to the oracle's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device, check_step, compare_encode  # noqa: E402


def messages(P0, n, K, scale=None):
    dev, host = [], []
    for k in range(K):
        P = q.Params(n=n, s=P0.s, d=P0.d, code=P0.code, norm=P0.norm, seed=5, stream_id=k)
        g = torch.randn(n, generator=torch.Generator().manual_seed(31 * k + n))
        g[n // 2:] *= 1e-3     # a second half that is mostly zeros: short strings, long gaps
        status, words, msg = Device(P).encode(g.cuda())
        assert status == 0
        if scale is None:
            assert compare_encode(P, g.numpy(), words) == 0
        dev.append(msg)
        host.append(words)
    return dev, host


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
@pytest.mark.parametrize("d,s,K,n", [
    (8192, 60, 3, 20_000), (8192, 127, 16, 8192), (8188, 4, 2, 30_000), (4100, 32, 64, 9000),
    (2124, 23, 5, 50_001), (512, 16, 2, 20_004), (512, 1, 1, 515),          # few strings
    (523, 3, 8, 10_001), (37, 5, 3, 1003), (1, 1, 2, 100), (3, 127, 33, 1000), (8191, 40, 4, 8191),
    (443, 2, 33, 400_000), (129, 11, 2, 2_000_003),                         # odd sizes, many strings
])
def test_words_of_a_string_in_parallel(code, d, s, K, n):
    norm = q.NORM_MAX if d % 3 == 0 else q.NORM_L2
    P0 = q.Params(n=n, s=s, d=d, code=code, norm=norm, seed=5)
    dev, host = messages(P0, n, K)
    assert check_step(P0, dev, host, 0.1, np.linspace(-1, 1, n, dtype=np.float32), K) == 0


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
@pytest.mark.parametrize("d,n", [(501, 5000), (131, 300_000)])
def test_scale_that_is_not_finite(code, d, n):
    """A coordinate without a record keeps its value whatever the bucket's scale."""
    P = q.Params(n=n, s=8, d=d, code=code, seed=5)
    dev, _ = messages(P, n, 2, scale=np.inf)
    zero = Device(P).encode(torch.zeros(n, device="cuda"))[2]
    table = (((n + d - 1) // d + 1) + 3) & ~3
    zero[16 + table] = int(np.array(np.inf, np.float32).view(np.int32))   # bucket 0's scale
    ws = torch.zeros(q.qsgd_workspace_bytes(P, 3) // 4, dtype=torch.int32, device="cuda")
    x = torch.linspace(-1, 1, n).cuda()
    want = x.clone()
    q.qsgd_decode_accumulate(P, [dev[0], dev[1]], want, ws)
    q.qsgd_decode_accumulate(P, [dev[0], zero, dev[1]], x, ws)
    assert q.qsgd_workspace_status(ws) == 0
    assert torch.equal(x, want)


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
@pytest.mark.parametrize("d,n", [(8192, 16_000), (501, 5000)])
def test_damaged_strings_are_flagged(code, d, n):
    P = q.Params(n=n, s=20, d=d, code=code, seed=5)
    dev, _ = messages(P, n, 1)
    ws = torch.zeros(q.qsgd_workspace_bytes(P, 1) // 4, dtype=torch.int32, device="cuda")
    table = (((n + d - 1) // d + 1) + 3) & ~3
    for word, value in ((16 + table + 3, -1), (17, 2), (17, 0)):   # a string, the offset table
        msg = dev[0].clone()
        msg[word] = value
        x = torch.zeros(n + 64, device="cuda")
        q.qsgd_decode_accumulate(P, [msg], x[:n], ws)
        assert q.qsgd_workspace_status(ws) != 0
        assert not x[n:].any()


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
@pytest.mark.parametrize("d,s,K,n", [
    (8193, 40, 3, 8193), (10_000, 127, 40, 25_001), (8200, 5, 64, 20_000), (37_906, 103, 2, 37_906),
    (100_000, 2, 16, 350_003), (70_001, 30, 5, 140_002),
])
def test_segments_of_long_buckets(code, d, s, K, n):
    P0 = q.Params(n=n, s=s, d=d, code=code, norm=q.NORM_MAX if K == 5 else q.NORM_L2, seed=5)
    dev, host = messages(P0, n, K)
    assert check_step(P0, dev, host, 0.1, np.linspace(-1, 1, n, dtype=np.float32), K) == 0


def test_gaps_beyond_16_bits():
    """Values at both ends of a long bucket only; too many records for the sparse path's estimate."""
    n, K = 300_000, 16
    dev, host = [], []
    for k in range(K):
        P = q.Params(n=n, s=4, d=n, code=q.CODE_SPARSE, seed=5, stream_id=k)
        g = torch.zeros(n)
        ends = torch.randn(400, generator=torch.Generator().manual_seed(k))
        g[:200], g[-200:] = ends[:200], ends[200:]
        g[140_000 + k] = 3.0
        status, words, msg = Device(P).encode(g.cuda())
        assert status == 0
        assert compare_encode(P, g.numpy(), words) == 0
        dev.append(msg)
        host.append(words)
    P0 = q.Params(n=n, s=4, d=n, code=q.CODE_SPARSE, seed=5)
    assert check_step(P0, dev, host, 0.1, np.linspace(-1, 1, n, dtype=np.float32), K) == 0


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
def test_damaged_entry_lists_leave_x_alone(code):
    n, K = 60_000, 8
    P = q.Params(n=n, s=60, d=n, code=code, seed=5)
    dev, host = messages(P, n, K)
    nw, ents = host[0].size, int(host[0][-1])
    assert ents >= 6
    lst = nw - 1 - 2 * ents
    ws = torch.zeros(q.qsgd_workspace_bytes(P, K) // 4, dtype=torch.int32, device="cuda")
    x0 = torch.linspace(-1, 1, n).cuda()
    for index, value in [
            (nw - 1, ents + 1), (nw - 1, ents - 1), (nw - 1, nw), (lst, 31), (lst + 2, 32 * nw),
            (lst + 4, int(host[0][lst + 4]) + 1), (lst + 5, int(host[0][lst + 5]) + 1),
            (lst + 5, int(host[0][lst + 3])), (lst + 1, n), (lst + 2 * ents - 1, n + 5), (lst, int(host[0][lst + 2]))]:
        if code == q.CODE_DENSE and (index, value) == (nw - 1, ents - 1):
            continue   # a sound list without its first entry, whose words read as padding
        bad = dev[0][:nw].clone()
        bad[index] = value
        x = x0.clone()
        q.qsgd_sgd_step(P, [bad] + dev[1:], 0.1, x, ws)
        assert q.qsgd_workspace_status(ws) == -3, (index - lst, value)
        assert torch.equal(x, x0)
