"""Long passes over narrow dense rows, squared loss: the pass as affine maps of runs of rows, at the edges of its row widths,
run lengths and number of solvers, against the oracle; the rows' order and the update as precise as the shorter passes'."""
import numpy as np
import pytest

from harness import run_lockstep

pytestmark = pytest.mark.gpu

# 47 blocks of 64 rows are solved block by block, 48 to 255 go in runs of 64 rows, more in runs of 128
CASES = [(1, 3073, 1), (3, 3008, 1), (4, 3100, 1), (5, 4160, 1), (8, 3073, 2), (9, 6200, 3), (16, 3200, 1), (17, 4097, 1),
         (21, 5000, 2), (24, 3073, 1), (28, 16321, 1), (29, 16320, 1), (32, 16449, 1), (32, 3136, 4), (13, 40000, 2)]


@pytest.mark.parametrize("d,n,K", CASES)
def test_affine_runs(oracle_mod, d, n, K):
    """n: rows of the longest solver; the others have a quarter, and one of them none."""
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    print("\ncase affine runs n=%d d=%d K=%d" % (n, d, K), flush=True)
    g = np.random.default_rng(100 * d + K)
    sizes = [n // 3, n - n // 3] + [n // 4] * (K - 1 if K < 4 else K - 2)
    bounds = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    total = int(bounds[-1])
    X = (g.standard_normal((total, d)) / np.sqrt(d)).astype(np.float32)
    X[7] = 0                                       # rows that take no step
    X[n - 1] = 0
    y = (X @ g.standard_normal(d) + g.standard_normal(total)).astype(np.float32)
    p = Problem("affine", "squared", total, d, 20.0 / total, y, bounds, X=X)
    table = np.concatenate([[0, 0], np.arange(1, len(sizes) - 1)]).astype(np.int32)
    run_lockstep({"seed": 11, "rounds": 3, "schedule": [(0, K)], "K": K}, p, oracle_mod, binding, check_alpha_every=1, ahead=d % 2 == 0,
                 cancelling=d <= 5, tables=lambda r, Kp, tp: (K, table, table.copy()) if r == 0 else None, max_solvers=K)


def test_order_entry_out_of_range_is_reported():
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    g = np.random.default_rng(3)
    n, d = 3200, 8
    X = g.standard_normal((n, d)).astype(np.float32)
    p = Problem("range", "squared", n, d, 0.01, X[:, 0].copy(), np.array([0, n]), X=X)
    r = binding.ChicleRound.from_problem(p, max_solvers=1)
    r.assign(1, np.zeros(1, dtype=np.int32))
    perm = np.arange(n, dtype=np.int32)
    perm[100], perm[3000] = -1, n
    r.local_epoch(r.upload_perm([perm]))
    r.aggregate()
    with pytest.raises(binding.ChicleError):
        r.gap()
    r.close()
