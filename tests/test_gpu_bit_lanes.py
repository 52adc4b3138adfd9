"""The split decoder's reader with a lane for every bit of a string: strings of less than a unit,
of several units and of several turns (data that codes longer than the estimate the plan goes by),
one to many buckets per compute unit, gaps of 2^16 and more, and strings with one word changed,
which the oracle either refuses or reads as the same values.  Bar: x bit-identical to the oracle's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device, check_step  # noqa: E402
from oracle import qsgd_oracle as qo  # noqa: E402


def encoded(P0, gradients):
    dev, host = [], []
    for k, g in enumerate(gradients):
        P = q.Params(n=P0.n, s=P0.s, d=P0.d, code=P0.code, norm=P0.norm, seed=5, stream_id=k)
        status, words, msg = Device(P).encode(g.cuda())
        assert status == 0
        dev.append(msg)
        host.append(words)
    return dev, host


@pytest.mark.parametrize("kind", ["normal", "flat"])
@pytest.mark.parametrize("d,s,K,n,norm", [
    (512, 4, 2, 20_004, q.NORM_L2), (512, 3, 8, 6000, q.NORM_L2), (96, 1, 3, 5001, q.NORM_L2),
    (512, 1, 8, 10_000, q.NORM_MAX), (1024, 8, 4, 400_000, q.NORM_L2), (2048, 6, 8, 9000, q.NORM_L2),
    (4096, 12, 4, 16_000, q.NORM_L2), (8192, 16, 2, 40_000, q.NORM_L2), (501, 3, 5, 200_003, q.NORM_L2),
    (8192, 1, 1, 8192, q.NORM_L2), (512, 4, 2, 1 << 20, q.NORM_L2),
    (10_000, 30, 3, 50_000, q.NORM_L2), (9001, 20, 5, 45_000, q.NORM_L2),      # segments
])
def test_every_bit_a_lane(kind, d, s, K, n, norm):
    P0 = q.Params(n=n, s=s, d=d, code=q.CODE_SPARSE, norm=norm, seed=5)
    gs = []
    for k in range(K):
        g = torch.randn(n, generator=torch.Generator().manual_seed(n + k))
        gs.append(torch.sign(g) if kind == "flat" else g)
    dev, host = encoded(P0, gs)
    assert check_step(P0, dev, host, 0.1, np.linspace(-1, 1, n, dtype=np.float32), K) == 0


def test_far_gaps():
    n, K = 300_000, 8
    gs = []
    for k in range(K):
        g = torch.zeros(n)
        ends = torch.randn(400, generator=torch.Generator().manual_seed(k))
        g[:200], g[-200:] = ends[:200], ends[200:]
        g[140_000 + k] = 3.0
        gs.append(g)
    P0 = q.Params(n=n, s=4, d=n, code=q.CODE_SPARSE, seed=5)
    dev, host = encoded(P0, gs)
    assert check_step(P0, dev, host, 0.1, np.linspace(-1, 1, n, dtype=np.float32), K) == 0


@pytest.mark.parametrize("d,s,n", [(512, 4, 2000), (2048, 6, 4000)])
def test_changed_words(d, s, n):
    """Status and values as the oracle has them for the same damaged message."""
    P0 = q.Params(n=n, s=s, d=d, code=q.CODE_SPARSE, seed=5)
    gs = [torch.randn(n, generator=torch.Generator().manual_seed(k)) for k in range(2)]
    dev, host = encoded(P0, gs)
    nb = (n + d - 1) // d
    pay = 16 + (nb + 1 + 3) // 4 * 4
    rng = np.random.default_rng(d)
    ws = torch.zeros(q.qsgd_workspace_bytes(P0, 2) // 4, dtype=torch.int32, device="cuda")
    x0 = np.linspace(-1, 1, n, dtype=np.float32)
    read = refused = 0
    for _ in range(60):
        w = host[0].copy()
        b = int(rng.integers(nb))
        at = pay + int(rng.integers(int(w[16 + b]) + 1, int(w[16 + b + 1])))   # (not the scale)
        w[at] ^= np.uint32(1) << np.uint32(rng.integers(32))
        x = torch.cat([torch.from_numpy(x0), torch.full((64,), 7.0)]).cuda()
        q.qsgd_sgd_step(P0, [torch.from_numpy(w.view(np.int32)).cuda(), dev[1]], 0.1, x[:n], ws)
        status = q.qsgd_workspace_status(ws)
        assert bool((x[n:] == 7.0).all())
        try:
            want = qo.sgd_step([w, host[1]], 0.1, x0)
        except qo.OracleError:
            assert status == -3
            refused += 1
            continue
        assert status == 0
        assert np.array_equal(x[:n].cpu().numpy(), want)
        read += 1
    assert read and refused
