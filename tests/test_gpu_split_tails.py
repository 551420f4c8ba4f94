"""Two tail workgroups per solver: what they add to and gather from the private vector is ordered, so that a job repeats to the
rounding of sums in another order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K", [(1100, 1), (24000, 5)])
def test_jobs_repeat_to_rounding(n, K):
    """Popular columns in the head, the rest in the tails; blocks in both parities, a last block alone in its iteration."""
    import torch
    import paper_1909_04885_amd as chicle
    assert torch.cuda.is_available()
    print("\ncase tails n=%d K=%d" % (n, K), flush=True)
    g = np.random.default_rng(3)
    d, m = 60000, 40
    popular = g.choice(2000, (n, m // 2)) * 30
    col = np.sort(np.concatenate([popular, g.integers(0, d, (n, m - m // 2))], axis=1), axis=1)
    keep = np.ones((n, m), dtype=bool)
    keep[:, 1:] = col[:, 1:] != col[:, :-1]
    rp = np.concatenate([[0], np.cumsum(keep.sum(axis=1))]).astype(np.int64)
    col = col[keep].astype(np.int32)
    val = (g.standard_normal(col.size) / np.sqrt(m)).astype(np.float32)
    y = np.where(g.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    orders = [[g.permutation(n // K) for _ in range(K)] for _ in range(4)]
    assert n % K == 0
    got = []
    for _ in range(3):
        r = chicle.ChicleRound("hinge", n, d, 1.0 / n, K, K, False, int(rp[-1]))
        for k in range(K):
            a, b = k * (n // K), (k + 1) * (n // K)
            r.load_chunk_csr(k, rp[a:b + 1] - rp[a], col[rp[a]:rp[b]], val[rp[a]:rp[b]], y[a:b])
        r.assign(K, np.arange(K, dtype=np.int32))
        assert r.debug_solver()[:2] == ("batched", 3)
        for perms in orders:
            r.local_epoch(r.upload_perm(perms))
            r.aggregate()
        got.append(r.get_w().astype(np.float64))
        r.close()
    for w in got[1:]:
        # a column's adds in another order differ by roundings of 2^-24 of partial sums, a few of them per column and round
        assert np.linalg.norm(w - got[0]) <= 8 * 2.0 ** -24 * np.linalg.norm(got[0])
