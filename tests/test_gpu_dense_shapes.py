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
    # An update is a sum of up to n steps' terms in fp32: its error is bounded by about n 2^-24 of the terms' sizes.
    # In one to three dimensions ridge is solved after two rounds and the third's update, a difference of the
    # solvers' parts thousands of times its own size, is below that bound relative to itself.
    rounds = 2 if d <= 3 else 3
    run_lockstep({"seed": 3, "rounds": rounds, "schedule": [(0, K)], "K": K}, p, oracle_mod, binding, check_alpha_every=1,
                 ahead=d % 2 == 0, tables=lambda r, Kp, tp: (K, table, table.copy()) if r == 0 else None, max_solvers=K)


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
