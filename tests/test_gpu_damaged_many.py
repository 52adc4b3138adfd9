"""Damaged strings all over a message, in launches of many workgroups that find them at different
times: the status says so, nothing outside x is touched, and the buffers serve a sound call next."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device  # noqa: E402
from oracle import qsgd_oracle as qo  # noqa: E402


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
@pytest.mark.parametrize("d,s,K,n", [
    (64, 5, 8, 64 * 20_000),        # tile decoder, several groups of buckets per wavefront
    (8192, 60, 3, 8192 * 400),      # split decoder, more buckets than workgroups
    (441, 9, 2, 441 * 600),         # split decoder, bucket sizes off 4
    (20_000, 40, 4, 20_000 * 40),   # segments of long buckets
])
def test_damage_in_many_buckets(code, d, s, K, n):
    gen = torch.Generator().manual_seed(d)
    dev, host = [], []
    for k in range(K):
        P = q.Params(n=n, s=s, d=d, code=code, seed=5, stream_id=k)
        status, words, msg = Device(P).encode(torch.randn(n, generator=gen).cuda())
        assert status == 0
        dev.append(msg[: words.size].clone())
        host.append(words)
    rng = np.random.default_rng(d)
    nb = (n + d - 1) // d
    pay = 16 + (nb + 1 + 3) // 4 * 4
    bad = []
    for w in host:
        w = w.copy()
        for b in range(int(rng.integers(5)), nb, 5):
            lo, hi = int(w[16 + b]), int(w[16 + b + 1])
            at = pay + lo + 1 + int(rng.integers(max(1, hi - lo - 1)))
            w[at:pay + hi] = 0xFFFFFFFF if b % 2 else 0
        bad.append(torch.from_numpy(w.view(np.int32)).cuda())
    ws = torch.zeros(q.qsgd_workspace_bytes(P, K) // 4, dtype=torch.int32, device="cuda")
    x0 = torch.linspace(-1, 1, n)
    for msgs in (bad, [bad[0]] + dev[1:]):
        x = torch.cat([x0, torch.full((256,), 7.0)]).cuda()
        q.qsgd_sgd_step(P, msgs, 0.1, x[:n], ws)
        assert q.qsgd_workspace_status(ws) == -3
        assert bool((x[n:] == 7.0).all())
    x = x0.cuda()
    q.qsgd_sgd_step(P, dev, 0.1, x, ws)
    assert q.qsgd_workspace_status(ws) == 0
    assert np.array_equal(x.cpu().numpy(), qo.sgd_step(host, 0.1, x0.numpy()))
