"""The encoder in which every lane codes its own values, at the sizes it took over: buckets that
are no multiple of 4 (they start anywhere in a Philox block) and buckets of 2049 to 8192 values,
with levels around 31, 63 and 126 and runs of more than 64 bits.  Bar: the oracle's words."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402
from gpu_harness import Device, compare_encode, oracle_params  # noqa: E402
from oracle import qsgd_oracle as qo  # noqa: E402


def gradient(n, kind, seed):
    gen = torch.Generator().manual_seed(seed)
    if kind == "full":                    # levels of 1 .. s about equally often
        return torch.rand(n, generator=gen) * 2 - 1
    g = torch.randn(n, generator=gen)
    if kind == "spikes":                  # long gaps, top levels behind leading zeros
        g *= 1e-4
        g[torch.randint(0, n, (max(1, n // 97),), generator=gen)] = 1.0
    return g


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
@pytest.mark.parametrize("d,s,n", [
    (1, 1, 50), (3, 5, 100), (63, 7, 5001), (65, 31, 5000), (127, 32, 40_003), (255, 63, 9999),
    (257, 64, 9998), (511, 126, 10_001), (513, 127, 10_003), (1023, 200, 20_002), (2047, 40, 20_471),
    (2049, 45, 30_001), (4097, 300, 12_345), (8191, 90, 40_000), (101, 2, 1_500_001),
    (2052, 45, 2052 * 2100 + 7), (4096, 63, 4096 * 600), (3000, 64, 3000 * 530 + 1),
    (8192, 90, 8192 * 1030 + 5),
])
@pytest.mark.parametrize("kind", ["full", "normal", "spikes"])
def test_sizes(code, d, s, n, kind):
    if n > 3_000_000 and (kind == "spikes" or (code == q.CODE_DENSE and d > 4096)):
        pytest.skip("the large sizes run once per code word path")
    norm = q.NORM_L2 if kind == "normal" else q.NORM_MAX
    P = q.Params(n=n, s=s, d=d, code=code, norm=norm, seed=3 + (1 << 40), stream_id=2)
    g = gradient(n, kind, d)
    status, words, _ = Device(P).encode(g.cuda())
    assert status == 0
    assert compare_encode(P, g.numpy(), words) == 0


@pytest.mark.parametrize("code", [q.CODE_SPARSE, q.CODE_DENSE])
def test_odd_buckets_small_message(code):
    """A message buffer that is too small ends with the size needed, nothing written past it."""
    n, d = 30_001, 445
    P = q.Params(n=n, s=9, d=d, code=code, seed=3)
    g = gradient(n, "normal", 1).cuda()
    _, words, _ = Device(P).encode(g)
    status, need, _ = Device(P, capacity=words.nbytes - 16).encode(g)
    assert status == -2 and need == words.nbytes


def test_odd_buckets_of_a_slice():
    """Draws are indexed by the position in the whole vector, also past 2^34."""
    d, n = 203, 203 * 40
    base = (1 << 34) - 203 * 20 // 4 * 4
    for b in (0, 203 * 4 * 7, base):
        P = q.Params(n=n, s=11, d=d, code=q.CODE_SPARSE, seed=9)
        g = gradient(n, "normal", 2)
        dev = Device(P)
        msg = torch.zeros(dev.cap // 4, dtype=torch.int32, device="cuda")
        q.qsgd_encode_slice(P, b, g.cuda(), msg, dev.ws)
        status, total = q.qsgd_message_status(msg)
        assert status == 0
        want = qo.encode_slice(oracle_params(P), g.numpy(), b)
        assert np.array_equal(msg.cpu().numpy().view(np.uint32)[: total // 4], want)
