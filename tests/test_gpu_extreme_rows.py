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
