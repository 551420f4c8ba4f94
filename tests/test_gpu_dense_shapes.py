"""The dense solver at the edges of the shapes it chooses from (lanes per row, columns per lane, rows per block),
against the oracle: every loss, ragged chunks, a block of one row, an empty row, a solver without rows."""
import numpy as np
import pytest

from harness import run_lockstep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("loss", ["hinge", "squared", "logistic"])
@pytest.mark.parametrize("d,n", [(1, 130), (3, 65), (32, 333), (33, 200), (64, 129), (65, 333), (128, 97), (129, 200),
                                 (256, 333), (257, 160), (512, 200), (513, 130), (768, 97), (769, 130), (1021, 200),
                                 (1024, 97), (1025, 130), (1280, 97), (1281, 130), (1536, 97), (1537, 70)])
def test_dense_widths(oracle_mod, loss, d, n):
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    g = np.random.default_rng(d)
    X = (g.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    X[5] = 0
    y = g.standard_normal(n).astype(np.float32) if loss == "squared" else np.where(g.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    bounds = np.array([0, 1, 40, 64, n], dtype=np.int64)
    p = Problem("width", loss, n, d, 0.02, y, bounds, X=X)
    K = 4
    table = np.array([0, 1, 1, 3], dtype=np.int32)             # one row; 63 rows; none; the rest
    print("\ncase dense n=%d d=%d %s" % (n, d, loss), flush=True)
    # In one to three dimensions ridge is solved after two rounds: the third's update is a difference of the solvers' parts
    # thousands of times its own size.
    run_lockstep({"seed": 3, "rounds": 3, "schedule": [(0, K)], "K": K}, p, oracle_mod, binding, check_alpha_every=1,
                 cancelling=loss == "squared" and d <= 3, ahead=d % 2 == 0, tables=lambda r, Kp, tp: (K, table, table.copy()) if r == 0 else None, max_solvers=K)


@pytest.mark.parametrize("d,rows,K,runs", [(48, 1, 4, "dense"), (49, 8, 4, "rowwise"), (49, 9, 4, "dense"), (400, 8, 4, "rowwise"),
                                           (400, 9, 4, "dense"), (1536, 8, 4, "rowwise"), (1536, 9, 4, "dense"), (1537, 9, 4, "rowwise"),
                                           (100, 10, 512, "rowwise"), (100, 11, 512, "dense"), (100, 20, 1024, "rowwise"), (100, 21, 1024, "dense")])
def test_solvers_of_few_dense_rows_go_row_by_row(oracle_mod, d, rows, K, runs):
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    print("\ncase dense choice d=%d rows=%d K=%d" % (d, rows, K), flush=True)
    g = np.random.default_rng(d)
    n = K * rows
    X = (g.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    y = np.where(g.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    p = Problem("choice", "hinge", n, d, 0.5 / n, y, np.arange(0, n + 1, rows, dtype=np.int64), X=X)
    table = np.arange(K, dtype=np.int32)
    c = binding.ChicleRound.from_problem(p, max_solvers=K)
    c.assign(K, table)
    assert c.debug_solver()[0] == runs
    c.set_solver("rowwise")
    assert c.debug_solver()[0] == "rowwise"
    if d <= 320:
        c.set_solver("batched")
        assert c.debug_solver()[0] == "dense"
    c.close()
    if K <= 4:
        run_lockstep({"seed": 3, "rounds": 2, "schedule": [(0, K)], "K": K}, p, oracle_mod, binding, check_alpha_every=1, ahead=True,
                     tables=lambda r, Kp, tp: (K, table, table.copy()) if r == 0 else None, max_solvers=K)


@pytest.mark.parametrize("d,rows,runs", [(512, 12, "rowwise"), (512, 13, "dense"), (513, 8, "rowwise"), (513, 9, "dense"), (1000, 12, "dense")])
def test_few_dense_rows_logistic(oracle_mod, d, rows, runs):
    """A step row by row takes longer the wider the row is, and a block hardly does."""
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    print("\ncase dense choice logistic d=%d rows=%d" % (d, rows), flush=True)
    g = np.random.default_rng(d + rows)
    n, K = 4 * rows, 4
    X = (g.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    p = Problem("choice", "logistic", n, d, 0.5 / n, np.where(g.random(n) < 0.5, 1.0, -1.0).astype(np.float32), np.arange(0, n + 1, rows, dtype=np.int64), X=X)
    table = np.arange(K, dtype=np.int32)
    c = binding.ChicleRound.from_problem(p, max_solvers=K)
    c.assign(K, table)
    assert c.debug_solver()[0] == runs
    c.close()
    run_lockstep({"seed": 3, "rounds": 2, "schedule": [(0, K)], "K": K}, p, oracle_mod, binding, check_alpha_every=1, ahead=True,
                 tables=lambda r, Kp, tp: (K, table, table.copy()) if r == 0 else None, max_solvers=K)


@pytest.mark.parametrize("ahead,n", [(False, 2500), (True, 1250)])
@pytest.mark.parametrize("d", [1, 28, 32, 33, 64, 65, 200, 511, 700, 1001, 1200, 1500])
def test_squared_loss_with_solved_tiles(oracle_mod, d, ahead, n):
    """Long passes of one solver, ragged last block: tiles hold the squared loss's recurrence solved, in the first pass
    (2500 rows, orders not announced) or from the second on (1250 rows, announced)."""
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    print("\ncase solved tiles n=%d d=%d ahead=%s" % (n, d, ahead), flush=True)
    g = np.random.default_rng(d)
    X = g.standard_normal((n, d)).astype(np.float32)
    X[n // 3] = 0
    y = (X @ g.standard_normal(d) / np.sqrt(d) + 0.1 * g.standard_normal(n)).astype(np.float32)
    p = Problem("solved", "squared", n, d, 0.02, y, np.array([0, 1001, n], dtype=np.int64), X=X)
    table = np.zeros(2, dtype=np.int32)
    run_lockstep({"seed": 5, "rounds": 3, "schedule": [(0, 1)], "K": 1}, p, oracle_mod, binding, check_alpha_every=1, ahead=ahead,
                 tables=lambda r, Kp, tp: (1, table, table.copy()) if r == 0 else None, max_solvers=1)


@pytest.mark.parametrize("loss,n,solved", [("hinge", 333, False), ("squared", 333, False), ("squared", 2400, True), ("logistic", 333, False)])
@pytest.mark.parametrize("d", [1, 7, 16, 33, 48])
def test_dense_tiles_match_their_definition(loss, d, n, solved):
    """What the tile kernel of dense rows writes against x_i . x_j in double: ragged last block, an empty row."""
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    print("\ncase dense tiles n=%d d=%d %s" % (n, d, loss), flush=True)
    g = np.random.default_rng(d)
    X = (g.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    X[5] = 0
    y = np.where(g.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    lam, K = 0.02, 1
    r = binding.ChicleRound(loss, n, d, lam, 1, K, True, n * d)
    r.load_chunk_dense(0, X, y)
    r.assign(K, np.zeros(1, dtype=np.int32))
    perm = g.permutation(n).astype(np.int32)
    tiles = r.debug_gram(r.upload_perm([perm]))
    assert tiles.shape[0] == (n + 63) // 64
    Xd, yd = X.astype(np.float64)[perm], y.astype(np.float64)[perm]
    q, c = (Xd ** 2).sum(1), lam * n / K
    scale = {"hinge": -1.0 / np.where(q > 0, q, np.inf), "squared": np.where(q > 0, -1.0 / (c + q), 0.0),
             "logistic": np.where(q > 0, -1.0 / c, 0.0)}[loss]
    sgn = np.ones(n) if loss == "squared" else yd
    eps = 2.0 ** -24
    for b in range(tiles.shape[0]):
        cur = np.arange(b * 64, min(n, b * 64 + 64))
        for part, rows in ((0, np.arange(b * 64 - 64, b * 64) if b else cur[:0]), (64, cur)):
            want, bound = np.zeros((64, 64)), np.zeros((64, 64))
            if rows.size:
                norm = np.sqrt(q[rows])[:, None] * np.sqrt(q[cur])[None, :] * np.abs(scale[cur])[None, :]
                want[:rows.size, :cur.size] = (Xd[rows] @ Xd[cur].T) * sgn[rows][:, None] * sgn[cur][None, :] * scale[cur][None, :]
                # d products and d - 1 sums in fp32, then three more roundings
                bound[:rows.size, :cur.size] = (2 * d + 4) * eps * norm
            if part:
                want, bound = np.triu(want, 1), np.triu(bound, 1)
                if solved:
                    # the tile holds N = (1 - T)^-1 from 64-term sums in fp32; T is read back from it in double:
                    # dT = M dN M with M = 1 - T, and |dN| <= |N| (bound of T + 64 eps |T|) |N| + eps |N|
                    M = np.eye(64) - want
                    N = np.linalg.inv(M)
                    dN = np.abs(N) @ (bound + 64 * eps * np.abs(want)) @ np.abs(N) + eps * np.abs(N)
                    bound = np.triu(np.abs(M) @ dN @ np.abs(M), 1) + eps * np.abs(want)
            got = tiles[b][part:part + 64].astype(np.float64)
            assert (np.abs(got - want) <= bound + 1e-30).all(), (b, part, np.max(np.abs(got - want) - bound))
    r.close()
