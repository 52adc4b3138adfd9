"""The decoder of dense strings at the places where it changes course: windows of 128
positions and what is decided past their end, code words at and beyond the table's reach
(gaps and levels around 16 and 32), buckets that end inside a word or a window, more groups
of buckets than wavefronts, few and many peers.  Bar: x bit-identical to the oracle's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device, check_step, compare_encode  # noqa: E402


def gradient(n, d, s, kind, seed):
    """Values whose levels are known to be spread: `kind` picks the gaps."""
    gen = torch.Generator().manual_seed(seed)
    g = torch.zeros(n)
    if kind == "full":                       # every level of 1 .. s about equally often
        g = torch.rand(n, generator=gen) * 2 - 1
    elif kind == "gaps":                     # gaps of 1, 2, 3, 4, 15, 16, 17, 31, 32, 33, 127 ...
        gaps = [1, 1, 2, 3, 4, 5, 7, 8, 15, 16, 17, 31, 32, 33, 63, 64, 127, 128, 129]
        at, i = -1, seed
        while True:
            at += gaps[(i * 7 + i // 5) % len(gaps)]
            i += 1
            if at >= n:
                break
            g[at] = float(torch.rand((), generator=gen)) + 0.5
    else:                                    # few values near the top level, the rest small
        g = torch.randn(n, generator=gen) * 0.3 / s
        g[torch.randint(0, n, (max(1, n // 100),), generator=gen)] = 1.0
    sign = torch.where(torch.rand(n, generator=gen) < 0.5, -1.0, 1.0)
    return g * sign


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
@pytest.mark.parametrize("d,s,K,nb", [
    (128, 7, 8, 40), (132, 16, 5, 40), (256, 15, 3, 33), (124, 31, 1, 70), (512, 32, 2, 40),
    (516, 127, 16, 21), (1020, 127, 33, 5), (4, 3, 9, 90), (8192, 100, 4, 3),
    (64, 5, 8, 30_000),                      # several groups per wavefront
])
@pytest.mark.parametrize("kind", ["full", "gaps", "top"])
def test_dense_strings(code, d, s, K, nb, kind):
    n = nb * d - d // 3
    norm = q.NORM_MAX if kind == "full" else q.NORM_L2
    msgs_dev, msgs_host = [], []
    for k in range(K):
        P = q.Params(n=n, s=s, d=d, code=code, norm=norm, seed=11, stream_id=k)
        g = gradient(n, d, s, kind, 100 * k + d) if nb < 1000 else \
            torch.randn(n, generator=torch.Generator().manual_seed(k))
        status, words, msg = Device(P).encode(g.cuda())
        assert status == 0
        assert compare_encode(P, g.numpy(), words) == 0
        msgs_dev.append(msg)
        msgs_host.append(words)
    P0 = q.Params(n=n, s=s, d=d, code=code, norm=norm, seed=11)
    assert check_step(P0, msgs_dev, msgs_host, 0.1, np.linspace(-1, 1, n, dtype=np.float32), K) == 0
