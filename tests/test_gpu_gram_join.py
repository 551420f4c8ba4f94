"""Gram tiles of short sparse rows against x_i . x_j in double: columns of the dense product only, with slots of their own,
sharing slots; runs of tiles that pass from one solver to the next, short ones and ones in which the tables, the places of the
rows and the lookups ahead are used over and over; solvers of less than a block; empty rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = {
    # name: (rows, columns, shortest and longest row, Zipf columns, solvers)
    "dense_product_only": (300, 60, 1, 40, False, 2),
    "slots_of_their_own": (700, 1000, 0, 48, False, 3),
    "shared_slots": (2000, 60000, 30, 48, False, 2),
    "zipf": (3000, 20000, 48, 48, True, 2),
    "runs_over_solvers": (40000, 3000, 4, 10, True, 37),
    "long_runs": (150000, 3000, 4, 10, True, 37),
    "long_runs_shared_slots": (140000, 200000, 0, 8, False, 300),
    "less_than_a_block": (150, 200, 0, 20, False, 7),
    "one_row": (1, 50, 7, 7, False, 1),
}


@pytest.mark.parametrize("name,loss", [(n, "hinge") for n in CASES] + [("zipf", "squared"), ("zipf", "logistic")])
def test_gram_tiles(name, loss):
    import scipy.sparse as sp
    import torch
    import paper_1909_04885_amd as chicle
    assert torch.cuda.is_available()
    n, d, low, high, zipf, K = CASES[name]
    g = np.random.default_rng(7)
    lens = g.integers(low, high + 1, n)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    p = (np.arange(d) + 1.0) ** -1.1
    ids = g.permutation(d)
    rank = np.cumsum(p / p.sum())
    rows = []
    for m in lens:
        if not zipf:
            c = g.choice(d, m, replace=False)
        else:
            c = np.empty(0, dtype=np.int64)
            while c.size < m:
                c = np.unique(np.concatenate([c, ids[np.minimum(np.searchsorted(rank, g.random(m - c.size)), d - 1)]]))
        rows.append(np.sort(c))
    col = np.concatenate(rows).astype(np.int32)
    val = g.uniform(0.1, 1.0, col.size).astype(np.float32)
    y = np.where(g.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    chunk = max(1, n // (4 * K))
    bounds = list(range(0, n, chunk)) + [n]
    lam = 1e-2
    r = chicle.ChicleRound(loss, n, d, lam, len(bounds) - 1, K, False, int(rp[-1]))
    for i, (a, b) in enumerate(zip(bounds, bounds[1:])):
        r.load_chunk_csr(i, rp[a:b + 1] - rp[a], col[rp[a]:rp[b]], val[rp[a]:rp[b]], y[a:b])
    table = chicle.balance(np.diff(rp[bounds]), K)
    r.assign(K, table)
    perms = [g.permutation(m) for m in r.solver_rows()]
    tiles = r.debug_gram(r.upload_perm(perms))
    if name.startswith("long_runs"):     # (a workgroup per compute unit takes as many tiles in turn)
        assert tiles.shape[0] >= 8 * torch.cuda.get_device_properties(0).multi_processor_count
    X = sp.csr_matrix((val.astype(np.float64), col, rp), shape=(n, d))
    q = np.asarray(X.multiply(X).sum(axis=1)).ravel()
    c = lam * n / K
    scale = np.zeros(n)
    scale[q > 0] = -1.0 / q[q > 0] if loss == "hinge" else -1.0 / (c + q[q > 0]) if loss == "squared" else -1.0 / c
    s = np.ones(n) if loss == "squared" else y.astype(np.float64)
    t = 0
    for k in range(K):
        own = np.concatenate([np.arange(bounds[i], bounds[i + 1]) for i in np.nonzero(table == k)[0]]) if np.any(table == k) else np.empty(0, int)
        order = own[perms[k]]
        for b in range(0, order.size, 64):
            cur, prev = order[b:b + 64], order[max(b - 64, 0):b]
            window = np.concatenate([prev, cur])
            G = (X[window] @ X[cur].T).toarray()                       # [jp, i]; values are positive
            G[prev.size:] = np.triu(G[prev.size:], k=1)
            want, got = np.zeros((128, 64)), tiles[t].astype(np.float64)
            at = np.r_[np.arange(prev.size), 64 + np.arange(cur.size)]
            want[at[:, None], np.arange(cur.size)] = G * scale[cur] * s[cur] * s[window][:, None]
            # fp32 products, those of up to 64 columns summed in fp32, the others in double; scaled by two more products
            # with a rounded scale: at most 64 + 6 roundings of the sum, all of whose terms have one sign
            assert np.all(np.abs(got - want) <= 70 * 2.0 ** -24 * np.abs(want) + 1e-30), (k, b)
            t += 1
    assert t == tiles.shape[0]
    r.close()
