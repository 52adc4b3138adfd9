"""Long buckets of sparse Code_s messages, the path that touches only the coordinates with records:
stretches of many turns (a run of nonzero levels in one segment), gaps of 2^16 and more, levels of 16
bits, records across words, no record at all, one to many stretches and buckets; and entry lists and
strings with one word changed.  Bar: x bit-identical to the oracle's; damaged messages leave x alone."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device, check_step  # noqa: E402
from oracle import qsgd_oracle as qo  # noqa: E402


def gradient(kind, n, k):
    gen = torch.Generator().manual_seed(100 * n + k)
    g = torch.randn(n, generator=gen)
    if kind == "run":            # 3000 levels in a row, a few elsewhere
        out = torch.zeros(n)
        out[5000 + 100 * k:8000 + 100 * k] = torch.sign(g[:3000])
        out[::40_009] = 1.0
        return out
    if kind == "rare":           # gaps far beyond 2^16, levels all over the range
        out = torch.zeros(n)
        at = torch.randperm(n, generator=gen)[:40]
        out[at] = g[:40] ** 5
        return out
    if kind == "zeros":
        return torch.zeros(n)
    return g


def made(kind, n, d, s, norm, K):
    dev, host = [], []
    for k in range(K):
        P = q.Params(n=n, s=s, d=d, code=q.CODE_SPARSE, norm=norm, seed=6, stream_id=k)
        status, words, msg = Device(P).encode(gradient(kind, n, k).cuda())
        assert status == 0
        dev.append(msg[: words.size].clone())
        host.append(words)
    return q.Params(n=n, s=s, d=d, code=q.CODE_SPARSE, norm=norm, seed=6), dev, host


@pytest.mark.parametrize("kind,n,d,s,norm,K", [
    ("normal", 300_000, 300_000, 1, q.NORM_L2, 3), ("normal", 4_000_000, 4_000_000, 2, q.NORM_L2, 2),
    ("normal", 200_000, 9000, 1, q.NORM_L2, 4), ("normal", 77_188, 28_725, 1, q.NORM_L2, 2),
    ("normal", 1_000_000, 8193, 1, q.NORM_L2, 5), ("run", 4_000_000, 4_000_000, 1, q.NORM_MAX, 2),
    ("run", 2_500_000, 1_300_000, 1, q.NORM_MAX, 3), ("rare", 4_000_000, 4_000_000, 60_000, q.NORM_MAX, 16),
    ("rare", 20_000_000, 20_000_000, 3, q.NORM_MAX, 2), ("zeros", 100_000, 50_000, 1, q.NORM_L2, 2),
])
def test_lists(kind, n, d, s, norm, K):
    P, dev, host = made(kind, n, d, s, norm, K)
    x = np.linspace(-1, 1, n, dtype=np.float32)
    x[::5] = -0.0        # a step leaves it where no record is, a sum of +0 does not
    assert check_step(P, dev, host, 0.1, x, K) == 0


def sign_of_first_record(w, first):
    """Word and bit of the sign behind the gap's recursive Elias code, which starts at word `first`."""
    at = 32 * first
    bits = lambda count: int("".join(str(int(w[(at + i) // 32]) >> (31 - (at + i) % 32) & 1) for i in range(count)), 2)
    value = 1
    while bits(1):
        value, at = bits(value + 1), at + value + 1
    at += 1
    return at // 32, np.uint32(31 - at % 32)


@pytest.mark.parametrize("kind,n", [("normal", 400_000), ("run", 4_000_000)])
def test_changed_words(kind, n):
    norm = q.NORM_L2 if kind == "normal" else q.NORM_MAX
    P, dev, host = made(kind, n, n, 1, norm, 2)
    ents = int(host[0][-1])
    assert ents >= 2
    first, last = 16 + 4 + 1, host[0].size - 2 * ents - 1     # the string's words behind its scale
    ws = torch.zeros(q.qsgd_workspace_bytes(P, 2) // 4, dtype=torch.int32, device="cuda")
    x0 = np.linspace(-1, 1, n, dtype=np.float32)
    rng = np.random.default_rng(n)
    read = refused = 0
    for i in range(31):
        w = host[0].copy()
        if i == 30:          # a sign: as sound a message as before
            at, bit = sign_of_first_record(w, first)
            w[at] ^= np.uint32(1) << bit
        elif i % 5 == 4:       # an entry point, or their count
            w[int(rng.integers(last, host[0].size))] += np.uint32(rng.integers(1, 40))
        else:
            w[int(rng.integers(first, last))] ^= np.uint32(1) << np.uint32(rng.integers(32))
        x = torch.cat([torch.from_numpy(x0), torch.full((64,), 7.0)]).cuda()
        q.qsgd_sgd_step(P, [torch.from_numpy(w.view(np.int32)).cuda(), dev[1]], 0.1, x[:n], ws)
        status = q.qsgd_workspace_status(ws)
        assert bool((x[n:] == 7.0).all())
        try:
            want = qo.sgd_step([w, host[1]], 0.1, x0)
        except qo.OracleError:
            assert status == -3
            assert np.array_equal(x[:n].cpu().numpy(), x0)
            refused += 1
            continue
        assert status == 0
        assert np.array_equal(x[:n].cpu().numpy(), want)
        read += 1
    assert read and refused
