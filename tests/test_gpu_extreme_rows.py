"""Rows whose squared norm a float can hardly hold, in every solver a data set may be given: as small as its smallest values
(against the oracle), and beyond its largest (no step, as row by row)."""
import numpy as np
import pytest

from harness import run_lockstep

pytestmark = pytest.mark.gpu


def _problem(kind, loss, scales):
    """300 rows, some of them scaled."""
    from workloads.generate import Problem
    g = np.random.default_rng(3)
    n = 300
    factor = np.ones(n)
    factor[g.choice(n, 40, replace=False)] = np.resize(scales, 40)
    y = np.where(g.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    bounds = np.array([0, 70, 150, n], dtype=np.int64)
    if isinstance(kind, int):
        X = g.standard_normal((n, kind)) / np.sqrt(kind) * factor[:, None]
        return Problem("extreme", loss, n, kind, 0.02, y, bounds, X=X.astype(np.float32))
    d, m = 400, 60
    col = np.concatenate([np.sort(g.choice(d, m, replace=False)) for _ in range(n)]).astype(np.int32)
    val = (g.standard_normal(n * m) / np.sqrt(m) * np.repeat(factor, m)).astype(np.float32)
    return Problem("extreme", loss, n, d, 0.02, y, bounds, row_ptr=np.arange(n + 1, dtype=np.int64) * m, col=col, val=val)


@pytest.mark.parametrize("kind", [100, 400, 1100, "sparse"])
def test_rows_of_tiny_norm(oracle_mod, kind):
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    p = _problem(kind, "hinge", [1e-20, 3e-20, 1e-19, 1e-10])
    print("\ncase tiny rows %s" % kind, flush=True)
    table = np.array([0, 1, 0], dtype=np.int32)
    run_lockstep({"seed": 3, "rounds": 3, "schedule": [(0, 2)], "K": 2}, p, oracle_mod, binding, check_alpha_every=1,
                 tables=lambda r, Kp, tp: (2, table, table.copy()) if r == 0 else None, max_solvers=2)


@pytest.mark.parametrize("loss", ["hinge", "squared", "logistic"])
@pytest.mark.parametrize("kind", [100, 400, 1100, "sparse"])
def test_rows_of_huge_norm_take_no_step(kind, loss):
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    p = _problem(kind, loss, [1e20, 1e22])
    print("\ncase huge rows %s %s" % (kind, loss), flush=True)
    table = np.array([0, 1, 0], dtype=np.int32)
    got = []
    for solver in ("auto", "rowwise"):
        g = binding.ChicleRound.from_problem(p, max_solvers=2)
        g.assign(2, table)
        g.set_solver(solver)
        order = np.random.default_rng(9)
        g.local_epoch(g.upload_perm([order.permutation(int(m)).astype(np.int32) for m in g.solver_rows()]))
        g.aggregate()
        got.append((np.concatenate([g.get_alpha(c) for c in range(3)]), g.get_w()))
        g.close()
    norm = np.array([float(np.sum(x.astype(np.float64) ** 2)) for x in (p.X if p.X is not None else p.val.reshape(300, -1))])
    huge = norm > 3.5e38
    assert huge.sum() == 40
    (alpha, w), (alpha_rows, w_rows) = got
    assert np.isfinite(alpha).all() and np.isfinite(w).all()
    assert (alpha[huge] == 0).all()
    if loss != "logistic":       # (row by row the logistic step has no meaning for such a row)
        assert np.max(np.abs(alpha - alpha_rows)) <= 5e-4          # the oracle tests' bound for alpha
        assert np.linalg.norm(w - w_rows) <= 1e-4 * np.linalg.norm(w_rows)


@pytest.mark.parametrize("loss", ["hinge", "squared"])
def test_huge_rows_that_share_a_column_blocks_apart(loss):
    """Short sparse rows, unpopular columns that two rows two and three blocks apart hold, both of them huge: what does not fit a
    float is their product alone (the tiles hold products of rows of one block and the next, of which none are huge here)."""
    import torch
    import paper_1909_04885_amd as binding
    from harness import tail_pairs
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    print("\ncase huge rows blocks apart %s" % loss, flush=True)
    g = np.random.default_rng(13)
    n, popular, m = 1280, 8768, 36                       # every popular column 4 or 5 times
    common = np.arange(n * 30).reshape(n, 30) % popular
    pairs = [(64 * a + i, 64 * b + j) for a, b in ((1, 3), (5, 8), (10, 12), (14, 17)) for i, j in ((3, 60), (40, 40))]
    own = np.empty((n, 6), dtype=np.int64)               # unpopular columns of two rows each
    for q in range(6):
        partner = g.permutation(n)
        own[partner, q] = popular + q * (n // 2) + np.arange(n) // 2
    d = popular + 6 * (n // 2) + len(pairs)
    for s, (a, b) in enumerate(pairs):
        own[a, 5] = own[b, 5] = popular + 6 * (n // 2) + s
    huge = np.unique(pairs)
    col = np.sort(np.concatenate([common, own], axis=1), axis=1)
    factor = np.ones(n)
    factor[huge] = np.resize([1e20, 1e25], huge.size)
    val = (g.standard_normal((n, m)) / np.sqrt(m) * factor[:, None]).astype(np.float32)
    y = np.where(g.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    p = Problem("extreme", loss, n, d, 1.0 / n, y, np.array([0, n], dtype=np.int64), row_ptr=m * np.arange(n + 1, dtype=np.int64),
                col=col.reshape(-1).astype(np.int32), val=val.reshape(-1))
    order = np.arange(n)
    assert sum(tail_pairs(p, [order], [order], n_hot=popular)[0][0]) >= len(pairs)
    got = []
    for solver in ("auto", "rowwise"):
        r = binding.ChicleRound.from_problem(p, max_solvers=1)
        r.assign(1, np.zeros(1, dtype=np.int32))
        r.set_solver(solver)
        assert solver == "rowwise" or r.debug_solver()[:2] == ("batched", 3)
        for announced in (False, True):          # (pairs are always listed with the tiles of announced orders here)
            r.local_epoch_ahead(None if announced else r.upload_perm([order]), r.upload_perm([order]))
            r.aggregate()
        got.append((r.get_alpha(0), r.get_w()))
        r.close()
    (alpha, w), (alpha_rows, w_rows) = got
    assert np.isfinite(alpha).all() and np.isfinite(w).all()
    assert (alpha[huge] == 0).all()
    assert np.max(np.abs(alpha - alpha_rows)) <= 5e-4              # the oracle tests' bound for alpha
    assert np.linalg.norm(w - w_rows) <= 1e-4 * np.linalg.norm(w_rows)
