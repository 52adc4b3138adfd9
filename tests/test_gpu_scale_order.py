"""A bucket's scale does not depend on the other buckets of the call: the same buckets encoded in
a call of many and in calls of few (which other kernel shapes take) give the same words, and the
double-buffered pass leaves the x of one flat step.  The buckets are built so that the square root
of the sum of squares lies halfway between two 32-bit values, to some 1e-17: sums that are rounded
in another order come out as another scale."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1610_02132_amd as q  # noqa: E402


def halfway(nb, d, seed):
    """nb buckets of d values whose norm is halfway between two floats."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((nb, d)).astype(np.float32)
    x[:, -2:] = 0
    rest = (x.astype(np.longdouble) ** 2).sum(axis=1)
    f = np.sqrt(rest).astype(np.float32)
    f = np.where(f.astype(np.longdouble) ** 2 < rest, np.nextafter(f, np.float32(np.inf)), f)
    mid = (f.astype(np.longdouble) + np.nextafter(f, np.float32(np.inf))) / 2
    for j in (d - 2, d - 1):          # the second value makes up for the first one's rounding
        missing = mid * mid - (x.astype(np.longdouble) ** 2).sum(axis=1)
        assert (missing > 0).all()
        e = np.sqrt(missing).astype(np.float32)
        x[:, j] = np.nextafter(e, np.float32(0)) if j == d - 2 else e
    norm = np.sqrt((x.astype(np.longdouble) ** 2).sum(axis=1))
    assert (np.abs(norm / mid - 1) < 1e-16).all()
    return x.reshape(-1)


def strings(P, g, base):
    ws = torch.zeros(q.qsgd_workspace_bytes(P, 1) // 4, dtype=torch.int32, device="cuda")
    msg = torch.zeros(q.qsgd_max_encoded_bytes(P) // 4, dtype=torch.int32, device="cuda")
    q.qsgd_encode_slice(P, base, g, msg, ws)
    status, total = q.qsgd_message_status(msg)
    assert status == 0
    words = msg[: total // 4].cpu().numpy()
    nb = P.n // P.d
    return np.split(words[16 + (nb + 1 + 3) // 4 * 4:], words[17:16 + nb])


@pytest.mark.parametrize("code,d,s,nb,few", [
    (q.CODE_SPARSE, 128, 5, 4500, 4000), (q.CODE_DENSE, 100, 7, 4500, 900),
    (q.CODE_SPARSE, 256, 5, 4500, 4000), (q.CODE_DENSE, 132, 7, 4500, 4096),
    (q.CODE_SPARSE, 4096, 9, 600, 500), (q.CODE_SPARSE, 2500, 9, 600, 300),
    (q.CODE_DENSE, 2052, 9, 2100, 700), (q.CODE_SPARSE, 8192, 33, 1100, 1000),
    (q.CODE_SPARSE, 5000, 11, 1100, 550),
])
def test_few_and_many_buckets_give_the_same_words(code, d, s, nb, few):
    g = torch.from_numpy(halfway(nb, d, d)).cuda()
    P = q.Params(n=nb * d, s=s, d=d, code=code, seed=3)
    many = strings(P, g, 0)
    other = 0
    for b in range(0, nb, few):
        part = g[b * d:(b + few) * d]
        Pf = q.Params(n=part.numel(), s=s, d=d, code=code, seed=3)
        for i, w in enumerate(strings(Pf, part, b * d)):
            other += not np.array_equal(w, many[b + i])
    assert other == 0, f"{other} of {nb} buckets differ"


def test_pipeline_leaves_the_x_of_the_flat_step():
    K, d, nb = 2, 128, 4500
    n = nb * d
    P = q.Params(n=n, s=5, d=d, seed=3)
    grads = [torch.from_numpy(halfway(nb, d, k)).cuda() for k in range(K)]
    ws = [torch.zeros(q.qsgd_workspace_bytes(P, K) // 4, dtype=torch.int32, device="cuda") for _ in range(2)]
    flat = []
    for k in range(K):
        msg = torch.zeros(q.qsgd_max_encoded_bytes(P) // 4, dtype=torch.int32, device="cuda")
        q.qsgd_encode(q.Params(n=n, s=5, d=d, seed=3, stream_id=k), grads[k], msg, ws[0])
        flat.append(msg)
    want = torch.linspace(-1, 1, n).cuda()
    x = want.clone()
    q.qsgd_sgd_step(P, flat, 0.1, want, ws[0])
    msgs = [torch.zeros_like(flat[0]) for _ in range(2 * K)]
    q.qsgd_pipeline_step(q.Pipeline(), P, 1000 * d, grads, 0.1, x, msgs, ws[0], ws[1])
    assert torch.equal(x, want)
