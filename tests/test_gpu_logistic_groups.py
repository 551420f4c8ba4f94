"""Logistic loss in blocks: steps are taken in groups from series that are renewed only where rows have moved.  Strongly coupled
rows leave their series inside a group, a run that settles goes from short groups to long ones, and last blocks are partial."""
import numpy as np
import pytest

from harness import TOL_DW, dw_floor, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,lam_n", [("dense24", 200, 0.05), ("dense24", 65, 3.0), ("dense600", 97, 0.02), ("dense1100", 49, 0.3),
                                          ("dense1100", 300, 0.01), ("sparse40", 257, 0.05), ("sparse40", 640, 3.0), ("sparse70", 193, 0.05)])
def test_groups_of_steps(oracle_mod, kind, n, lam_n):
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    print("\ncase logistic groups %s n=%d lam_n=%g" % (kind, n, lam_n), flush=True)
    g = np.random.default_rng(n)
    y = np.where(g.random(n) < 0.5, -1, 1).astype(np.float32)
    bounds = np.array([0, n])
    if kind.startswith("dense"):
        d = int(kind[5:])
        X = (g.standard_normal((n, d)) + 0.5).astype(np.float32)
        X /= np.linalg.norm(X, axis=1, keepdims=True)
        p = Problem("groups", "logistic", n, d, lam_n / n, y, bounds, X=X)
    else:
        m, d = int(kind[6:]), 900                     # (rows share a good part of their columns)
        col = np.concatenate([np.sort(g.choice(d, m, replace=False)) for _ in range(n)]).astype(np.int32)
        val = (g.random(n * m) / np.sqrt(m / 3.0)).astype(np.float32)
        p = Problem("groups", "logistic", n, d, lam_n / n, y, bounds, row_ptr=np.arange(n + 1, dtype=np.int64) * m, col=col, val=val)
    r = binding.ChicleRound.from_problem(p, max_solvers=1)
    o = oracle_mod.OracleCoCoA.from_problem(p)
    table = np.zeros(1, dtype=np.int32)
    r.assign(1, table)
    o.assign(1, table)
    assert r.debug_solver()[0] != "rowwise"
    for k in range(6):
        perm = [g.permutation(n).astype(np.int32)]
        r.local_epoch(r.upload_perm(perm))
        dw = o.local_epoch(perm)[0]
        err = rel_l2(r.get_delta_w(0), dw, dw_floor(float(np.linalg.norm(o.w))))
        # (a row's state is fp32 on the device: where its change is far below the value, the change carries the value's rounding)
        print("round %d error %.2e" % (k, err), flush=True)
        assert err <= TOL_DW
        o.aggregate()
        r.aggregate()
        r.gap()
    # Every step rounds its alpha once and is itself off by a few 2^-24 of values up to 1; sqrt(n) of them add up over six rounds.
    err = np.abs(r.get_alpha(0) - o.alpha).max()
    print("alpha off by %.2e" % err, flush=True)
    assert err <= 6 * 16 * 2.0 ** -24 * max(1.0, 1.0 / lam_n) ** 0.5
    r.close()
