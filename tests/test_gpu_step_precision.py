"""The dual steps of the block solvers are as precise as a row-wise step: the influence of a block's other steps on a row is
summed apart from the row's own value, not added to it one by one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n", [(100, 640), (400, 640), (1100, 640), ("sparse", 640), (100, 2560)])
def test_ridge_steps_carry_few_roundings(oracle_mod, kind, n):
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    print("\ncase precision %s n=%d" % (kind, n), flush=True)
    g = np.random.default_rng(4)
    y = g.standard_normal(n).astype(np.float32)
    lam = 100.0 / n                               # weakly coupled rows: the steps are of the size of y
    if kind == "sparse":
        d, m = 12000, 250
        col = np.concatenate([np.sort(g.choice(d, m, replace=False)) for _ in range(n)]).astype(np.int32)
        val = (g.standard_normal(n * m) / np.sqrt(m)).astype(np.float32)
        p = Problem("precision", "squared", n, d, lam, y, np.array([0, n]), row_ptr=np.arange(n + 1, dtype=np.int64) * m, col=col, val=val)
    else:
        X = (g.standard_normal((n, kind)) / np.sqrt(kind)).astype(np.float32)
        p = Problem("precision", "squared", n, kind, lam, y, np.array([0, n]), X=X)
    r = binding.ChicleRound.from_problem(p, max_solvers=1)
    o = oracle_mod.OracleCoCoA.from_problem(p)
    table = np.zeros(1, dtype=np.int32)
    r.assign(1, table)
    o.assign(1, table)
    assert r.debug_solver()[0] == ("blocks" if kind == "sparse" else "dense")
    perm = [g.permutation(n).astype(np.int32)]
    r.local_epoch(r.upload_perm(perm))
    o.local_epoch(perm)
    error = np.linalg.norm(r.get_alpha(0) - o.alpha) / np.linalg.norm(o.alpha)
    # A step is rounded where it is multiplied, where the others' influence is added, and once more in between: three roundings
    # of 2^-24 at most, 0.29 of 2^-23 of the value's binade and so about 4.5e-8 together in the mean square.  Twice that is
    # allowed for the influence's own error.  (63 additions to the value itself came to 1.3e-7 to 1.7e-7.)
    print("relative error of alpha %.2e" % error)
    assert error <= 9e-8
    r.close()
